"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs.  Tolerances (those of the benchmark definition): H within 1e-5 relative Frobenius error;
layer objective within 1e-3 relative; at most 0.1 % of plane bits differing; packing bit-exact.
"""
import numpy as np
import pytest
import torch

from oracle import bpdq_oracle as orc
from paper_2602_04163_amd import binding as bq
from paper_2602_04163_amd import workloads as wk
from tests import parity_tools as pt

pytestmark = pytest.mark.gpu

H_TOL = 1e-5
OBJ_TOL = 1e-3
PLANE_TOL = 1e-3


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    bq.load()
    return torch.device("cuda:0")


def _relfro(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _problem(name, d_out, d_in, n_tok, **kw):
    wl = wk.WORKLOADS[name].scaled(d_out=d_out, d_in=d_in, n_tok=n_tok, chunk=n_tok, **kw)
    W = wk.make_weight(wl)
    s = wk.channel_scales(wl)
    X = wk.make_activation_chunk(wl, 0, s)
    return wl, W, X


# ------------------------------------------------------------------ step 1: Hessian
# the three kernels: fp32 matrix cores, three bf16 pieces per value, two fp16 halves per scaled value
HESSIAN_CALLS = {"f32": bq.bpdq_hessian_accumulate_f32, "bf16x3": bq.bpdq_hessian_accumulate_bf16x3,
                 "f16x2": bq.bpdq_hessian_accumulate}


@pytest.fixture(params=["f32", "bf16x3", "f16x2"])
def hess(request):
    return HESSIAN_CALLS[request.param]


@pytest.mark.parametrize("n_tok,d_in", [(1, 20), (8, 256), (511, 260), (513, 20), (1024, 516), (1025, 260),
                                        (2049, 20), (4095, 260), (4096, 516), (4097, 260)])
def test_hessian_small_call_paths(dev, n_tok, d_in):
    """Token counts at the edges of the one-launch pre-pass (512, 1024, 2048, 4096 tokens) with strided rows, and
    the mirror image written by the reduction: symmetric bit for bit, its upper half that of a plain call."""
    print(f"hessian small call n_tok={n_tok} d_in={d_in}", flush=True)
    g = torch.Generator().manual_seed(n_tok + d_in)
    X = torch.randn((n_tok, d_in + 8), generator=g) * torch.exp(2.0 * torch.randn(d_in + 8, generator=g))
    Xd = X.to(dev)[:, 4:4 + d_in]
    H0 = torch.randn((d_in, d_in), generator=g).to(dev)
    Hs, Hp = H0.clone(), H0.clone()
    bq.bpdq_hessian_accumulate(Xd, Hs, 2.0, True)
    bq.bpdq_hessian_accumulate(Xd, Hp, 2.0, False)
    assert torch.equal(Hs, Hs.t())
    assert torch.equal(Hs.triu(), Hp.triu())
    x = X[:, 4:4 + d_in].numpy().astype(np.float64)
    want = np.triu(H0.cpu().numpy().astype(np.float64) + 2.0 * x.T @ x)
    # halves: 2^-21 of a product; fp32 sums: 2^-24 per addition along a chain, and the rounding of H itself
    scale = np.sqrt(np.outer((x * x).sum(0), (x * x).sum(0))) * 2.0 + np.abs(H0.cpu().numpy())
    assert np.all(np.abs(Hs.triu().cpu().numpy() - want) <= 5e-6 * scale)


@pytest.mark.parametrize("n_tok,d_in", [(1, 4), (3, 516), (64, 512), (64, 3072), (65, 388), (64, 3076), (256, 384),
                                        (255, 2044), (257, 260), (256, 2052), (512, 256), (400, 508), (512, 1024),
                                        (513, 36), (512, 1028), (1024, 512), (1000, 516), (1025, 100), (2048, 384),
                                        (2047, 388), (2049, 256), (65, 1728), (70, 1732), (191, 1792), (192, 1792),
                                        (65, 1852), (65, 1856), (257, 704), (512, 704), (512, 708), (1025, 320),
                                        (2048, 320), (2048, 324)])
def test_hessian_one_launch_calls(dev, n_tok, d_in):
    """Both sides of the lines between one launch and three, at the edges of the tiles and of the tokens a lane
    holds: strided rows, channels far apart in magnitude, a scale, a start that is not zero; the blocks of 32 x 32 on
    the diagonal come whole and nothing below them is touched unless H is symmetrized."""
    print(f"hessian one launch n_tok={n_tok} d_in={d_in}", flush=True)
    g = torch.Generator().manual_seed(7 * n_tok + d_in)
    X = torch.randn((n_tok, d_in + 4), generator=g) * torch.pow(10.0, torch.randint(-15, 16, (d_in + 4,), generator=g).float())
    Xd = X.to(dev)[:, :d_in]
    x = Xd.double()
    h0 = torch.linalg.vector_norm(x, dim=0)
    H0 = (torch.randn((d_in, d_in), generator=g).to(dev).double() * h0[:, None] * h0[None, :]).float()
    Hp = bq.bpdq_hessian_accumulate(Xd, H0.clone(), 0.5, False)
    Hs = bq.bpdq_hessian_accumulate(Xd, H0.clone(), 0.5, True)
    i = torch.arange(d_in, device=dev) // 32
    whole = i[:, None] <= i[None, :]
    want = H0.double() + 0.5 * (x.t().contiguous() @ x)
    # 2^-21 of a product of halves, 2^-24 for each addition of a chain (at most 8192 tokens between roundings, and
    # about the square root of that in practice), and the rounding of H itself
    bound = 5e-6 * (0.5 * h0[:, None] * h0[None, :] + H0.double().abs())
    assert bool(((Hp.double() - want).abs()[whole] <= bound[whole]).all())
    assert torch.equal(Hp[~whole], H0[~whole])
    assert torch.equal(Hs, Hs.t()) and torch.equal(Hs.triu(), Hp.triu())


def _hessian_takes_one_launch(X):
    """Whether the call leaves its workspace alone, as the one launch does (the three write their planes into it)."""
    d_in = X.shape[1]
    ws = torch.full((bq.bpdq_hessian_workspace_bytes(*X.shape),), 0xA5, dtype=torch.uint8, device=X.device)
    bq.bpdq_hessian_accumulate(X, torch.zeros((d_in, d_in), device=X.device), 2.0, True, ws)
    return bool((ws == 0xA5).all())


@pytest.mark.parametrize("n_tok,d_in,one", [(64, 3072, True), (65, 1728, True), (65, 2044, True), (192, 2048, True),
                                            (257, 704, True), (512, 704, True), (513, 512, True), (1025, 320, True),
                                            (2048, 320, True), (64, 3076, False), (65, 1792, False), (128, 1820, False),
                                            (160, 2048, False), (257, 768, False), (400, 1024, False), (512, 708, False),
                                            (512, 1024, False), (1025, 352, False), (2048, 384, False), (2049, 256, False)])
def test_hessian_one_launch_only_where_it_is_quicker(dev, n_tok, d_in, one):
    """Calls whose tiles fill the chip more than once, or whose channels fill 256 x 256 tiles, keep to the three
    launches: on activations not read before one launch took up to half as long again (512 x 1024: 36 us against 24)."""
    print(f"hessian one launch or three n_tok={n_tok} d_in={d_in}", flush=True)
    X = torch.randn((n_tok, d_in), generator=torch.Generator().manual_seed(n_tok)).to(dev)
    took = _hessian_takes_one_launch(X)
    assert took == one


@pytest.mark.parametrize("n_tok,d_in", [(100, 2052), (300, 772), (1100, 516), (4096, 260), (5000, 260)])
def test_hessian_of_activations_that_are_not_finite(dev, n_tok, d_in):
    """An infinity or NaN makes its channel's row and column NaN and touches nothing else, through either pre-pass."""
    print(f"hessian not finite n_tok={n_tok} d_in={d_in}", flush=True)
    X = torch.randn((n_tok, d_in), generator=torch.Generator().manual_seed(n_tok)).to(dev)
    assert not _hessian_takes_one_launch(X)
    clean = bq.bpdq_hessian_accumulate(X, torch.zeros((d_in, d_in), device=dev), 2.0, True)
    X[7, 3], X[n_tok - 1, d_in - 1], X[11, 100] = float("inf"), -float("inf"), float("nan")
    H = bq.bpdq_hessian_accumulate(X, torch.zeros((d_in, d_in), device=dev), 2.0, True)
    bad = torch.zeros(d_in, dtype=torch.bool, device=dev)
    bad[[3, 100, d_in - 1]] = True
    nan = bad[:, None] | bad[None, :]
    assert torch.equal(torch.isnan(H), nan)
    assert torch.equal(H[~nan], clean[~nan])


@pytest.mark.parametrize("n_tok,d_in", [(13, 260), (64, 1028), (100, 260), (256, 1028), (300, 260), (300, 516),
                                        (512, 700), (700, 100), (1500, 260)])
def test_hessian_one_launch_of_activations_that_are_not_finite(dev, n_tok, d_in):
    """Every form of the one launch: a channel with an infinity, a NaN (first, last, and followed by larger and smaller
    values, so that the channel's maximum meets it in every place) or both is NaN, and nothing else changes."""
    print(f"hessian one launch not finite n_tok={n_tok} d_in={d_in}", flush=True)
    X = torch.randn((n_tok, d_in), generator=torch.Generator().manual_seed(n_tok + d_in)).to(dev)
    assert _hessian_takes_one_launch(X)
    clean = bq.bpdq_hessian_accumulate(X, torch.zeros((d_in, d_in), device=dev), 2.0, True)
    X[0, 3], X[n_tok - 1, d_in - 1], X[11, 40] = float("inf"), -float("inf"), float("nan")
    X[0, 60], X[n_tok - 1, 33], X[5, 17], X[6, 17] = float("nan"), float("nan"), 1e30, float("nan")
    X[2, 90], X[9, 90] = float("inf"), float("nan")
    X[3, 70], X[8, 70] = float("nan"), -float("inf")
    H = bq.bpdq_hessian_accumulate(X, torch.zeros((d_in, d_in), device=dev), 2.0, True)
    bad = torch.zeros(d_in, dtype=torch.bool, device=dev)
    bad[[3, 17, 33, 40, 60, 70, 90, d_in - 1]] = True
    nan = bad[:, None] | bad[None, :]
    assert torch.equal(torch.isnan(H), nan)
    assert torch.equal(H[~nan], clean[~nan])


@pytest.mark.parametrize("n_tok,d_in,n_sized,one", [(256, 512, 300, True), (256, 768, 300, True), (400, 1024, 512, False),
                                                    (300, 1280, 344, False), (512, 1536, 556, False),
                                                    (1024, 768, 1136, False), (2100, 324, 2401, False)])
def test_hessian_workspace_of_another_call(dev, n_tok, d_in, n_sized, one):
    """A short call on a workspace sized for a longer one, where its own finest plan would want more than that:
    it runs on coarser slices, to the same tolerance, and their sums are rounded in other places, so that the bits
    tell which plan ran; a workspace too small for those is refused.  A call that takes one launch writes into neither
    workspace, but asks for the same sizes."""
    print(f"hessian n_tok={n_tok} d_in={d_in} on the workspace of {n_sized} tokens", flush=True)
    have, own = bq.bpdq_hessian_workspace_bytes(n_sized, d_in), bq.bpdq_hessian_workspace_bytes(n_tok, d_in)
    assert have < own
    g = torch.Generator().manual_seed(n_tok + d_in)
    X = torch.randn((n_tok, d_in), generator=g)
    want = 2.0 * X.double().t() @ X.double()
    results = []
    for nbytes in (own, own + 4096, have, have):
        H = torch.zeros((d_in, d_in), device=dev)
        bq.bpdq_hessian_accumulate(X.to(dev), H, 2.0, True, torch.empty(nbytes, dtype=torch.uint8, device=dev))
        assert _relfro(H.cpu().numpy(), want.numpy()) < 2e-6
        results.append(H)
    assert torch.equal(results[0], results[1]) and torch.equal(results[2], results[3])
    assert _hessian_takes_one_launch(X.to(dev)) == one and torch.equal(results[0], results[2]) == one
    planes_only = 4 * ((n_tok + 31) // 32 * 32) * ((d_in + 255) // 256 * 256)
    with pytest.raises(bq.BpdqError):
        bq.bpdq_hessian_accumulate(X.to(dev), torch.zeros((d_in, d_in), device=dev), 2.0, False,
                                   torch.empty(planes_only - 256, dtype=torch.uint8, device=dev))


def test_stream_handle_without_the_private_name(dev, monkeypatch):
    """The current stream's handle comes from a private function of torch where it exists, else by way of a Stream."""
    print("stream handle", flush=True)
    for s in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            fast = bq._stream().value
            with monkeypatch.context() as m:
                m.setattr(bq, "_raw_stream", None)
                assert bq._stream().value == fast == (s.cuda_stream or None)


def test_hessian_with_a_workspace_asks_for_no_size(dev, monkeypatch):
    """The size query plans all three kernels; a call that brings its workspace does not make it."""
    print("hessian with a workspace", flush=True)
    X = torch.randn((300, 64), generator=torch.Generator().manual_seed(3)).to(dev)
    ws = torch.empty(bq.bpdq_hessian_workspace_bytes(300, 64), dtype=torch.uint8, device=dev)
    want = bq.bpdq_hessian_accumulate(X, torch.zeros((64, 64), device=dev))

    class NoQuery:
        def __getattr__(self, name):
            assert name != "bpdq_hessian_workspace_bytes"
            return getattr(lib, name)

    lib = bq.load()
    monkeypatch.setattr(bq, "_lib", NoQuery())
    assert torch.equal(bq.bpdq_hessian_accumulate(X, torch.zeros((64, 64), device=dev), ws=ws), want)


@pytest.mark.parametrize("n_tok,d_in", [(100, 96), (512, 256), (1000, 640), (5000, 776), (37, 4), (16, 260),
                                        (17, 516), (20000, 264)])
def test_hessian_matches_oracle(dev, hess, n_tok, d_in):
    print(f"hessian {hess.__name__} n_tok={n_tok} d_in={d_in}", flush=True)
    g = torch.Generator().manual_seed(n_tok * 1000 + d_in)
    X = torch.randn((n_tok, d_in), generator=g) * torch.exp(torch.randn(d_in, generator=g))
    Href = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), Href)
    H = torch.zeros((d_in, d_in), device=dev)
    hess(X.to(dev), H, symmetrize=True)
    Hg = H.cpu().numpy().astype(np.float64)
    assert _relfro(Hg, Href) < H_TOL
    assert np.array_equal(Hg, Hg.T)
    # element-wise too: every entry within a few fp32 ulps of the row/column scale
    scale = np.sqrt(np.outer(np.diag(Href), np.diag(Href)))
    worst = float(np.max(np.abs(Hg - Href) / scale))
    print(f"   relFro {_relfro(Hg, Href):.2e}, worst entry / sqrt(H_ii H_jj) {worst:.2e}", flush=True)
    assert worst < 2e-5


def test_hessian_chunks_strided_and_deterministic(dev, hess):
    print(f"hessian chunked {hess.__name__}", flush=True)
    n_tok, d_in = 3000, 520
    g = torch.Generator().manual_seed(7)
    Xfull = torch.randn((n_tok, d_in + 8), generator=g)
    Xd = Xfull.to(dev)[:, :d_in]                  # row stride d_in + 8
    Href = np.zeros((d_in, d_in))
    orc.hessian_accumulate(Xfull[:, :d_in].numpy(), Href)
    outs = []
    for rep in range(2):
        H = torch.zeros((d_in, d_in), device=dev)
        edges = [0, 1000, 1016, 2500, 3000]
        for a, b in zip(edges[:-1], edges[1:]):
            hess(Xd[a:b], H, symmetrize=(b == n_tok))
        outs.append(H.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])       # no float atomics: bit-reproducible
    assert _relfro(outs[0].astype(np.float64), Href) < H_TOL
    # empty chunk is a no-op
    H0 = torch.ones((d_in, d_in), device=dev)
    hess(Xd[:0], H0)
    assert bool((H0 == 1).all())


def test_hessian_exact_on_short_values(dev):
    """Values with at most 8 significant bits are their own first piece (the power-of-two channel
    scale of the fp16 path changes no significand), and small integers make every partial sum
    exact in fp32: all three kernels must then return the exact H, bit for bit."""
    print("hessian exact integers", flush=True)
    n_tok, d_in = 3000, 520
    g = torch.Generator().manual_seed(11)
    X = torch.randint(-15, 16, (n_tok, d_in), generator=g).float()
    Href = 2.0 * (X.double().T @ X.double())
    for name, fn in HESSIAN_CALLS.items():
        H = torch.zeros((d_in, d_in), device=dev)
        fn(X.to(dev), H, symmetrize=True)
        assert torch.equal(H.cpu().double(), Href), name


SPLIT_CALLS = {"bf16x3": bq.bpdq_hessian_accumulate_bf16x3, "f16x2": bq.bpdq_hessian_accumulate}


@pytest.mark.parametrize("kernel", sorted(SPLIT_CALLS))
def test_hessian_split_long_accumulation(dev, kernel):
    """More tokens than one accumulation chain of a split kernel holds (8192), on a ragged
    two-tile width: slices and their fixed-order sum, checked entry by entry."""
    print(f"hessian {kernel} long", flush=True)
    n_tok, d_in = 40000, 300
    g = torch.Generator().manual_seed(12)
    X = torch.randn((n_tok, d_in), generator=g) * torch.exp(1.5 * torch.randn(d_in, generator=g))
    Href = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), Href)
    H = torch.zeros((d_in, d_in), device=dev)
    SPLIT_CALLS[kernel](X.to(dev), H, symmetrize=True)
    Hg = H.cpu().numpy().astype(np.float64)
    assert _relfro(Hg, Href) < H_TOL
    scale = np.sqrt(np.outer(np.diag(Href), np.diag(Href)))
    assert np.max(np.abs(Hg - Href) / scale) < 2e-5


@pytest.mark.parametrize("kernel", sorted(HESSIAN_CALLS))
def test_hessian_host_split_launches(dev, kernel):
    """Every kernel bounds its accumulation chains (8192 tokens for the split kernels, 16384 for the
    fp32 one).  Two host-side cases: a layer wide enough to add straight into H (>= 1024 tiles)
    is cut into launches of one chain each, and a call with more tokens than 64 slices of a chain
    cover is cut as well."""
    print(f"hessian {kernel} wide layer, 20000 tokens in one call", flush=True)
    accumulate = HESSIAN_CALLS[kernel]
    d_in, n_tok = 11520, 20000
    g = torch.Generator(device=dev).manual_seed(13)
    X = torch.randn((n_tok, d_in), generator=g, device=dev)
    idx = torch.randperm(d_in, generator=torch.Generator().manual_seed(5))[:96].sort().values.to(dev)
    H = torch.zeros((d_in, d_in), device=dev)
    accumulate(X, H, symmetrize=True)
    Hsub = np.zeros((96, 96))
    orc.hessian_accumulate(X[:, idx].cpu().numpy(), Hsub)
    Hg = H[idx][:, idx].cpu().numpy().astype(np.float64)
    assert _relfro(Hg, Hsub) < H_TOL
    assert torch.equal(H, H.T)
    # every 256 x 256 tile of the result (the launch walks the triangle in an order of its own: a
    # tile left out or taken twice would pass a sampled check with some probability), against
    # the definition evaluated in fp64 by torch on 4096 of the tokens
    H.zero_()
    accumulate(X[:4096], H, symmetrize=True)
    Xd = X[:4096].double()
    Hd = 2.0 * (Xd.T @ Xd)
    del Xd
    err = (H.double() - Hd).square_()
    nt = d_in // 256
    tile_err = err.view(nt, 256, nt, 256).sum(dim=(1, 3))
    tile_ref = Hd.square_().view(nt, 256, nt, 256).sum(dim=(1, 3))
    # an off-diagonal tile of uncorrelated channels is pure noise (entries ~ sqrt(N)), so its own
    # rounding error is set against the size of the diagonal entries that bound it
    scale = torch.sqrt(tile_ref.diagonal()[:, None] * tile_ref.diagonal()[None, :])
    assert float((tile_err / scale).max()) < H_TOL ** 2
    assert float(torch.sqrt(tile_err.sum() / tile_ref.sum())) < H_TOL
    del X, H, Hd, err
    n_tok = 530000 if kernel != "f32" else 1060000
    print(f"hessian {kernel} {n_tok} tokens", flush=True)
    d_in = 8
    X = torch.randn((n_tok, d_in), generator=g, device=dev) * 3.0
    H = torch.zeros((d_in, d_in), device=dev)
    accumulate(X, H, symmetrize=True)
    Href = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.cpu().numpy(), Href)
    assert _relfro(H.cpu().numpy().astype(np.float64), Href) < H_TOL


def test_hessian_f16_path_channel_scaling(dev):
    """The fp16 path scales every channel by a power of two before cutting it into halves: channels
    whose magnitudes lie far outside the fp16 range (1e-20 .. 1e+15), an all-zero channel, and a
    channel with one value dwarfing the rest must come out as accurately as on the fp32 path."""
    print("hessian f16x2 channel scaling", flush=True)
    n_tok, d_in = 4096, 264
    g = torch.Generator().manual_seed(21)
    X = torch.randn((n_tok, d_in), generator=g)
    mags = torch.logspace(-20, 15, d_in)
    X = X * mags[torch.randperm(d_in, generator=g)]
    X[:, 5] = 0.0                                   # dead channel
    X[7, 9] = X[:, 9].abs().max() * 3.0e4           # one outlier 30000 times the rest of its channel
    Href = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), Href)
    H = torch.zeros((d_in, d_in), device=dev)
    bq.bpdq_hessian_accumulate(X.to(dev), H, symmetrize=True)
    Hg = H.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(Hg))
    assert np.all(Hg[5] == 0) and np.all(Hg[:, 5] == 0)
    scale = np.sqrt(np.outer(np.diag(Href), np.diag(Href)))
    scale[5, :] = scale[:, 5] = 1.0
    ok = scale > 1e-37                               # entries the fp32 result can hold at all
    assert np.max((np.abs(Hg - Href) / scale)[ok]) < 2e-5


# ------------------------------------------------------------------ step 2: prepare
@pytest.mark.parametrize("n_tok,d_in", [(131077, 1024), (44740, 3000)])
@pytest.mark.parametrize("kind", ["plain", "missed", "not_finite"])
def test_hessian_scales_from_a_sample(dev, n_tok, d_in, kind):
    """Calls of 2^27 values and more take a channel's scale from every 16th token.  A channel whose sample is all zeros, or
    small against an outlier that it missed (first, middle, last token), is split again with all tokens; so is one
    with an infinity or a NaN, whose row and column of H alone are not finite."""
    print(f"sampled scales {n_tok}x{d_in} {kind}", flush=True)
    assert n_tok * d_in >= 1 << 27
    g = torch.Generator(device=dev)
    g.manual_seed(n_tok)
    X = torch.randn((n_tok, d_in), generator=g, device=dev)
    X *= torch.exp(2 * torch.randn(d_in, generator=g, device=dev))
    X[:, 17] = 0.0
    X[:, 33] *= 1e-30
    X[:, 34] *= 1e15 / X[:, 34].abs().max()                   # (its H entry, below 2 n_tok 1e30, is in fp32's range)
    if kind != "plain":
        X[::8, 300] = 0.0                                    # the whole sample
        X[1, 301], X[n_tok // 2 | 1, 302] = 3e4 * X[1, 301], 1e6
        X[n_tok - 1 if (n_tok - 1) % 8 else n_tok - 2, 999] = -1e5
    bad = [] if kind != "not_finite" else [40, 600]
    if bad:
        X[5, 40], X[70001 % n_tok | 1, 600] = float("inf"), float("nan")
    H = torch.zeros((d_in, d_in), device=dev)
    bq.bpdq_hessian_accumulate(X, H, 2.0, True)
    good = [c for c in range(d_in) if c not in bad]
    ref = torch.zeros((len(good), len(good)), dtype=torch.float64, device=dev)
    for a in range(0, n_tok, 16384):
        x = X[a:a + 16384, good].double()
        ref.addmm_(x.t().contiguous(), x, alpha=2.0)
    got = H[good][:, good].double()
    for c in bad:
        assert not torch.isfinite(H[c, c])
    root = ref.diagonal().sqrt().clamp_min(1e-300)
    scaled, want = got / root[:, None] / root[None, :], ref / root[:, None] / root[None, :]
    tiny = root < 1e-18                                       # squares below fp32's range
    scaled[tiny], want[tiny] = 0.0, 0.0
    scaled[:, tiny], want[:, tiny] = 0.0, 0.0
    assert torch.isfinite(scaled).all()
    assert float((scaled - want).abs().max()) < 2e-5           # the bar of every entry
    assert float((scaled - want).norm() / want.norm()) < H_TOL
    assert torch.equal(H[good][:, good], H[good][:, good].t())
    again = torch.zeros_like(H)
    bq.bpdq_hessian_accumulate(X, again, 2.0, True)
    assert torch.equal(torch.nan_to_num(H), torch.nan_to_num(again))


def test_hessian_scales_from_a_sample_with_loud_tokens_in_it(dev):
    """A value's halves are no coarser where its channel's scale comes from a sample: tokens 2^15 to 2^16 times the rest, at places
    that the sample holds (the first of every 2048).  An entry of H is a single product of such a value and 1, so nothing but
    the halves is rounded: the value scaled is at least 2^-3 and keeps an absolute error of 2^-25."""
    n_tok, d_in = 131072, 1024
    print(f"sampled scales, loud tokens, {n_tok}x{d_in}", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    c = 1.0 + torch.rand(d_in // 2, generator=g, device=dev)
    X = torch.zeros((n_tok, d_in), device=dev)
    X[::2048, 0::2], X[64::2048, 1::2] = 2.0 ** 16, 1.0
    X[777, 0::2], X[777, 1::2] = c, 1.0
    H = torch.zeros((d_in, d_in), device=dev)
    bq.bpdq_hessian_accumulate(X, H, 2.0, True)
    assert float((H[0::2, 1::2].double() / (2.0 * c.double())[:, None] - 1.0).abs().max()) <= 2.0 ** -22


@pytest.mark.parametrize("n_tok,d_in,first", [(10000, 16640, 8192), (600000, 256, 524288)])
def test_hessian_scales_from_a_sample_in_the_first_of_two_launches(dev, n_tok, d_in, first):
    """A launch of 2^27 values or more, whose scales come from a sample, and one of fewer behind it in the same workspace;
    16640 channels add their tiles straight into H.  Values that the sample misses in one block of 256 channels, in both
    launches' tokens."""
    print(f"sampled scales in the first launch {n_tok}x{d_in}", flush=True)
    assert first * d_in >= 1 << 27 > (n_tok - first) * d_in
    g = torch.Generator(device=dev)
    g.manual_seed(d_in)
    X = torch.randn((n_tok, d_in), generator=g, device=dev)
    X *= torch.exp(torch.randn(d_in, generator=g, device=dev))
    loud = d_in - 200
    X[first - 1, loud], X[n_tok - 1, loud], X[1, loud + 70] = 3e3, -2e4, 1e5
    H = torch.zeros((d_in, d_in), device=dev)
    bq.bpdq_hessian_accumulate(X, H, 2.0, False)
    c = torch.arange(1, d_in, max(1, d_in // 300), device=dev)
    c = torch.unique(torch.cat([c, torch.tensor([loud, loud + 1, loud + 70], device=dev)]))
    ref = torch.zeros((len(c), len(c)), dtype=torch.float64, device=dev)
    for a in range(0, n_tok, 16384):
        x = X[a:a + 16384, c].double()
        ref.addmm_(x.t().contiguous(), x, alpha=2.0)
    root = ref.diagonal().sqrt()
    off = ((H[c][:, c].double() - ref) / root[:, None] / root[None, :]).triu()
    assert float(off.abs().max()) < 2e-5
    assert float(off.norm() / (ref / root[:, None] / root[None, :]).triu().norm()) < H_TOL
    again = torch.zeros_like(H)
    bq.bpdq_hessian_accumulate(X, again, 2.0, False)
    assert torch.equal(H, again)


@pytest.mark.parametrize("d_in,sigma", [(96, 1.0), (200, 1.0), (640, 1.5), (1288, 1.0)])
def test_prepare_matches_oracle(dev, d_in, sigma):
    print(f"prepare d_in={d_in}", flush=True)
    wl, W, X = _problem("cfg1_tiny", 8, d_in, 3 * d_in, x_sigma=sigma)
    Href = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), Href)
    H32 = Href.astype(np.float32)
    Uref, dead_ref, info_ref = orc.prepare(H32.astype(np.float64), wl.damp)
    U, dead, info = bq.bpdq_prepare(torch.from_numpy(H32).to(dev), wl.damp)
    assert int(info.item()) == 0 and info_ref == 0
    Ug = U.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.tril(Ug, -1), np.zeros_like(Ug))
    assert not dead.cpu().numpy().any()
    assert _relfro(Ug, Uref) < 1e-6
    # row-relative: every row of U within fp32 rounding of the oracle's row
    rown = np.linalg.norm(Uref, axis=1)
    assert np.max(np.linalg.norm(Ug - Uref, axis=1) / rown) < 1e-6


def test_prepare_dead_channel_aliasing_and_failure(dev):
    print("prepare edge cases", flush=True)
    d_in = 160
    wl, W, X = _problem("cfg1_tiny", 8, d_in, 500)
    X[:, 17] = 0.0
    Href = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), Href)
    H32 = Href.astype(np.float32)
    Uref, dead_ref, _ = orc.prepare(H32.astype(np.float64), wl.damp)
    Hd = torch.from_numpy(H32).to(dev)
    U, dead, info = bq.bpdq_prepare(Hd, wl.damp, U=Hd)        # U aliases H
    assert int(info.item()) == 0
    assert np.array_equal(dead.cpu().numpy().astype(bool), dead_ref)
    assert dead_ref[17] and dead_ref.sum() == 1
    assert _relfro(U.cpu().numpy().astype(np.float64), Uref) < 1e-6
    # indefinite input: reported through info, no hang, no exception
    Hbad = torch.eye(d_in, device=dev)
    Hbad[3, 100] = 5.0
    _, _, info = bq.bpdq_prepare(Hbad, 0.0)
    assert int(info.item()) > 0


# ------------------------------------------------------------------ steps 3-4: the sweep
def _run_both(dev, wl, W, U32, dead, bits, group, block, iters, coef_fp16=False):
    """Stage-isolated: both sides get the same fp32 U."""
    ref = orc.quantize_layer(W.numpy(), U32.astype(np.float64), dead, bits, group, block, iters,
                             alpha=float(np.float32(wl.alpha)),
                             coef_dtype=np.float16 if coef_fp16 else None)
    p = bq.make_params(bits, group, block, iters, wl.alpha, coef_fp16=coef_fp16)
    dead_t = None if dead is None else torch.from_numpy(dead.astype(np.uint8)).to(dev)
    out = bq.bpdq_quantize_layer(W.to(dev), torch.from_numpy(U32).to(dev), dead_t, p)
    torch.cuda.synchronize()
    return ref, out


def _teacher_forced(ref, out, W, U32, bits, group, iters, alpha, coef_fp16=False, uniform=False):
    """Every group of the layer against the oracle started from the GPU's own group-start block
    (tests/parity_tools.py), then the end-to-end statement that holds at any layer size: rows may
    differ from the free-running oracle only where a decision was a near-tie."""
    code = orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), W.shape[1])
    U64 = U32.astype(np.float64)
    Wn = W.numpy().astype(np.float64)
    What = out["W_hat"].cpu().numpy().astype(np.float64)
    st = pt.teacher_forced(Wn, U64, code, out["coefs"].cpu().numpy(), out["grp_iter"].cpu().numpy(),
                           bits, group, iters, float(np.float32(alpha)), What=What,
                           coef_dtype=np.float16 if coef_fp16 else None, uniform=uniform)
    print("   " + pt.describe(st), flush=True)
    assert st["mismatch_clear_rows"] == 0          # identical planes wherever no decision was a near-tie
    assert st["selection_gap"] < 1e-4              # another kept iterate only if the two scores tie
    assert st["rounding_flip_rows"] <= max(2, 0.02 * st["rows"])
    assert st["coef_dev"] < 2e-3 and st["clear_score_rel"] < OBJ_TOL
    n_diff, n_allowed = pt.end_to_end_rows(Wn, U64, code, What, ref, st, OBJ_TOL)
    print(f"   end to end: {n_diff} of {code.shape[0]} rows differ from the free-running oracle "
          f"({n_allowed} rows have a near-tie decision)", flush=True)
    return st


def _check_layer(ref, out, W, Ht, bits, group):
    planes = out["planes"].cpu().numpy().view(np.uint32)
    code = orc.unpack_planes(planes, W.shape[1])
    n_bits_diff = sum(int(np.sum(((code >> i) & 1) != ((ref["code"] >> i) & 1))) for i in range(bits))
    frac = n_bits_diff / (bits * code.size)
    What = out["W_hat"].cpu().numpy().astype(np.float64)
    coefs = out["coefs"].cpu().numpy()
    # neutral scorer, applied identically to both sides
    Wn = W.numpy().astype(np.float64)
    obj_g = orc.layer_objective(Wn, What, Ht)
    obj_r = orc.layer_objective(Wn, ref["What"], Ht)
    rel = abs(obj_g - obj_r) / obj_r
    print(f"   plane bits differing {frac:.2e}, objective rel diff {rel:.2e}", flush=True)
    assert frac <= PLANE_TOL
    assert rel <= OBJ_TOL
    # the pass's own objective (sum of group errors) is the same number (App. B.2)
    err_sum = float(out["grp_err"].cpu().numpy().sum())
    assert abs(err_sum - obj_g) / obj_g < 1e-3
    # W_hat is exactly the dequantised storage format
    Wd = bq.bpdq_dequant(out["planes"], out["coefs"], group)
    assert torch.equal(Wd, out["W_hat"])
    # fp32 level sums vs the exact sums: a few fp32 ulps of the largest coefficient
    assert np.allclose(What, orc.dequant(planes, coefs.astype(np.float64), group), rtol=0,
                       atol=4e-7 * float(np.abs(coefs).max()))
    # coefficients agree wherever a (row, group) has identical planes
    same = (code == ref["code"]).reshape(code.shape[0], -1, group).all(axis=2)
    same &= (out["grp_iter"].cpu().numpy() == ref["grp_iter"])[None, :]
    cg = coefs.transpose(1, 2, 0)[same]
    cr = ref["coef"].transpose(1, 2, 0)[same]
    scale = np.abs(cr).max(axis=1, keepdims=True) + 1e-30
    assert same.mean() > 0.98
    assert np.max(np.abs(cg - cr) / scale) < 2e-3
    assert np.median(np.abs(cg - cr) / scale) < 1e-5
    return frac, rel


@pytest.mark.parametrize("bits,group,block,iters,d_out,d_in", [
    (2, 64, 128, 3, 256, 256),      # the tiny configuration's knobs
    (2, 128, 128, 5, 200, 384),     # ragged rows (200 = 12 work-groups + 8 rows)
    (3, 128, 128, 5, 64, 256),
    (2, 64, 128, 8, 50, 320),       # g < B with a ragged last block
    (4, 32, 64, 2, 33, 128),
    (3, 64, 64, 0, 40, 128),        # T = 0: initialisation + one fit
    (1, 32, 32, 4, 48, 96),
    (4, 128, 128, 3, 32, 256),
])
def test_quantize_layer_stage_isolated(dev, bits, group, block, iters, d_out, d_in):
    print(f"quantize k={bits} g={group} B={block} T={iters} {d_out}x{d_in}", flush=True)
    wl, W, X = _problem("cfg1_tiny", d_out, d_in, 4 * d_in)
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, info = orc.prepare(H, wl.damp)
    U32 = Uref.astype(np.float32)
    Ht = np.linalg.inv(U32.astype(np.float64).T @ U32.astype(np.float64))
    ref, out = _run_both(dev, wl, W, U32, dead, bits, group, block, iters)
    _check_layer(ref, out, W, Ht, bits, group)
    _teacher_forced(ref, out, W, U32, bits, group, iters, wl.alpha)
    it_g = out["grp_iter"].cpu().numpy()
    assert np.mean(it_g == ref["grp_iter"]) >= 0.9
    assert np.all(it_g >= 0) and np.all(it_g <= iters)


@pytest.mark.parametrize("bits,group,block,d_out,d_in", [
    (2, 256, 128, 96, 512),        # g = 256 (the paper's W2-G256 setting), block widened to g
    (3, 256, 256, 40, 256),
    (1, 256, 256, 24, 512),
])
def test_quantize_layer_group_256(dev, bits, group, block, d_out, d_in):
    print(f"quantize k={bits} g={group} {d_out}x{d_in}", flush=True)
    wl, W, X = _problem("cfg1_tiny", d_out, d_in, 4 * d_in)
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, info = orc.prepare(H, wl.damp)
    U32 = Uref.astype(np.float32)
    Ht = np.linalg.inv(U32.astype(np.float64).T @ U32.astype(np.float64))
    ref, out = _run_both(dev, wl, W, U32, dead, bits, group, block, 4)
    _check_layer(ref, out, W, Ht, bits, group)
    _teacher_forced(ref, out, W, U32, bits, group, 4, wl.alpha)


@pytest.mark.parametrize("bits,group,block,iters,d_out,d_in", [
    (2, 128, 128, 5, 200, 384),
    (3, 64, 128, 4, 72, 320),
    (4, 32, 64, 2, 33, 128),
    (2, 256, 256, 3, 40, 512),
])
def test_quantize_layer_fp16_coefficient_storage(dev, bits, group, block, iters, d_out, d_in):
    """coef_fp16 = 1: coefficients rounded to half right after every fit (the storage precision
    Table 1 counts).  Same parity bar as the fp32 path, against the oracle with the same reading;
    the stored format (packed planes + halves) must reproduce W_hat bit for bit, and its size is
    the closed form k + 16 (k+1) / g bits per weight."""
    print(f"fp16 storage k={bits} g={group} B={block} T={iters} {d_out}x{d_in}", flush=True)
    wl, W, X = _problem("cfg1_tiny", d_out, d_in, 4 * d_in)
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, info = orc.prepare(H, wl.damp)
    U32 = Uref.astype(np.float32)
    Ht = np.linalg.inv(U32.astype(np.float64).T @ U32.astype(np.float64))
    ref, out = _run_both(dev, wl, W, U32, dead, bits, group, block, iters, coef_fp16=True)
    _check_layer(ref, out, W, Ht, bits, group)
    _teacher_forced(ref, out, W, U32, bits, group, iters, wl.alpha, coef_fp16=True)
    coefs = out["coefs"]
    ch = bq.bpdq_coefs_to_fp16(coefs)
    assert torch.equal(ch.float(), coefs)                      # every coefficient is a half
    assert np.array_equal(ch.cpu().numpy(), coefs.cpu().numpy().astype(np.float16))
    Wd = bq.bpdq_dequant_fp16(out["planes"], ch, group)
    assert torch.equal(Wd, out["W_hat"])                       # stored format == W_hat
    stored_bits = 8 * (out["planes"].numel() * 4 + ch.numel() * 2)
    assert stored_bits / (d_out * d_in) == orc.bits_per_weight(bits, group)
    # objective re-measured after rounding: rounding in the pass vs rounding afterwards vs fp32
    Wn = W.numpy().astype(np.float64)
    p32 = bq.make_params(bits, group, block, iters, wl.alpha)
    out32 = bq.bpdq_quantize_layer(W.to(dev), torch.from_numpy(U32).to(dev), None, p32)
    post = bq.bpdq_dequant_fp16(out32["planes"], bq.bpdq_coefs_to_fp16(out32["coefs"]), group)
    o32 = orc.layer_objective(Wn, out32["W_hat"].cpu().numpy(), Ht)
    o16 = orc.layer_objective(Wn, out["W_hat"].cpu().numpy(), Ht)
    opost = orc.layer_objective(Wn, post.cpu().numpy(), Ht)
    print(f"   objective fp32 {o32:.6e}; fp16 in the pass {o16 / o32:.5f}x; "
          f"fp16 afterwards {opost / o32:.5f}x", flush=True)
    assert abs(o16 / o32 - 1) < 2e-2 and abs(opost / o32 - 1) < 2e-2
    # the pass's own scores describe the stored layer (App. B.2) only when it rounds itself
    assert abs(float(out["grp_err"].sum().item()) - o16) / o16 < 1e-3


def test_coefs_to_fp16_rounding_and_errors(dev):
    print("coefs_to_fp16 rounding", flush=True)
    rng = np.random.default_rng(11)
    x = np.concatenate([rng.standard_normal(5000).astype(np.float32) * 0.05,
                        np.float32([0.0, -0.0, 1.0 + 2.0 ** -11, 1.0 + 3 * 2.0 ** -11, 65504.0,
                                    6e-8, 3e-8, -2.5e-5, 1e-7])])
    got = bq.bpdq_coefs_to_fp16(torch.from_numpy(x).to(dev)).cpu().numpy()
    assert np.array_equal(got.view(np.uint16), x.astype(np.float16).view(np.uint16))
    empty = bq.bpdq_coefs_to_fp16(torch.empty(0, dtype=torch.float32, device=dev))
    assert empty.numel() == 0


@pytest.mark.parametrize("bits,group,block,d_out,d_in", [
    (2, 64, 128, 200, 384), (3, 128, 128, 64, 256), (4, 32, 64, 33, 128), (2, 256, 256, 48, 512),
])
def test_uniform_grid_comparator(dev, bits, group, block, d_out, d_in):
    """BPDQ_GRID_UNIFORM: the fixed-uniform-grid sweep (GPTQ on the min/max grid, App. A)
    against the oracle's statement of it, both given the same fp32 U."""
    print(f"uniform grid k={bits} g={group} {d_out}x{d_in}", flush=True)
    wl, W, X = _problem("cfg2_qwen7b_attn", d_out, d_in, 4 * d_in)
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, info = orc.prepare(H, wl.damp)
    U32 = Uref.astype(np.float32)
    U64 = U32.astype(np.float64)
    Ht = np.linalg.inv(U64.T @ U64)
    ref = orc.quantize_layer(W.numpy(), U64, dead, bits, group, block, 0,
                             group_fn=lambda T, UL: orc.uniform_frozen_group(T, UL, bits))
    p = bq.make_params(bits, group, block, 5, wl.alpha, grid=bq.GRID_UNIFORM)
    out = bq.bpdq_quantize_layer(W.to(dev), torch.from_numpy(U32).to(dev), None, p)
    torch.cuda.synchronize()
    code = orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), d_in)
    assert np.mean(code != ref["code"]) <= PLANE_TOL
    Wn = W.numpy().astype(np.float64)
    og = orc.layer_objective(Wn, out["W_hat"].cpu().numpy(), Ht)
    orf = orc.layer_objective(Wn, ref["What"], Ht)
    print(f"   codes differing {np.mean(code != ref['code']):.2e}, objective rel {abs(og - orf) / orf:.2e}", flush=True)
    assert abs(og - orf) / orf <= OBJ_TOL
    assert abs(float(out["grp_err"].sum().item()) - og) / og < 1e-3
    assert bool((out["grp_iter"] == 0).all())
    # coefficients are the uniform grid (lo, s, 2s, ...) and What is on that grid
    cf = out["coefs"].cpu().numpy()
    for i in range(2, bits + 1):
        assert np.array_equal(cf[i], 2 * cf[i - 1])
    assert np.allclose(cf[0], ref["coef"][0], rtol=1e-6, atol=1e-9)
    # the paper's claim at layer level: the variable grid does better on the same inputs
    pv = bq.make_params(bits, group, block, 5, wl.alpha)
    outv = bq.bpdq_quantize_layer(W.to(dev), torch.from_numpy(U32).to(dev), None, pv)
    ov = orc.layer_objective(Wn, outv["W_hat"].cpu().numpy(), Ht)
    print(f"   objective variable grid / uniform grid = {ov / og:.3f}", flush=True)
    assert ov < og


def test_quantize_layer_heavy_tails_and_dead_channel(dev):
    print("quantize student-t + dead channel", flush=True)
    wl, W, X = _problem("cfg5_qwen72b_down", 96, 256, 1024)
    X[:, 70] = 0.0
    H = np.zeros((256, 256))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, info = orc.prepare(H, wl.damp)
    assert dead[70]
    U32 = Uref.astype(np.float32)
    Ht = np.linalg.inv(U32.astype(np.float64).T @ U32.astype(np.float64))
    ref, out = _run_both(dev, wl, W, U32, dead, 2, 64, 128, 8)
    Wz = W.clone()
    Wz[:, 70] = 0.0
    _check_layer(ref, out, Wz, Ht, 2, 64)


def test_identity_hessian_on_gpu(dev):
    # H = I: U = I, no propagation; every group is an independent plain fit
    print("quantize identity hessian", flush=True)
    d_out, d_in = 64, 128
    g = torch.Generator().manual_seed(3)
    W = torch.randn((d_out, d_in), generator=g) * 0.02
    U32 = np.eye(d_in, dtype=np.float32)
    ref = orc.quantize_layer(W.numpy(), U32.astype(np.float64), None, 2, 32, 64, 4,
                             alpha=float(np.float32(1e-4)))
    out = bq.bpdq_quantize_layer(W.to(dev), torch.from_numpy(U32).to(dev), None,
                                 bq.make_params(2, 32, 64, 4, 1e-4))
    code = orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), d_in)
    assert np.mean(code != ref["code"]) <= PLANE_TOL
    assert abs(out["grp_err"].cpu().numpy().sum() - ref["objective"]) / ref["objective"] < OBJ_TOL


# ------------------------------------------------------------------ step 4: lazy block update
@pytest.mark.parametrize("d_out,lde,Kd,k0,c0,c1,d_in", [
    (200, 256, 128, 128, 256, 1000, 1024),      # ragged rows and a ragged last column tile
    (128, 128, 64, 0, 64, 192, 192),            # one tile, short K
    (515, 576, 1024, 0, 1024, 1536, 1536),      # deep K (the far-tail form)
    (64, 64, 128, 256, 384, 384, 512),          # empty column range: nothing to do
])
def test_block_update_matches_definition(dev, d_out, lde, Kd, k0, c0, c1, d_in):
    """W'[:, c0:c1] -= E_blk U[blk, c0:c1] (Eq. 4 for a whole block; App. B.3 tail form) against
    the same product in fp64; columns outside [c0, c1) must not change."""
    print(f"block update {d_out}x[{c0},{c1}) K={Kd}", flush=True)
    g = torch.Generator().manual_seed(d_out + Kd)
    Et = torch.randn((Kd, lde), generator=g) * 0.01
    U = torch.triu(torch.randn((d_in, d_in), generator=g)) * 0.1
    Wp = torch.randn((d_out, d_in), generator=g) * 0.02
    want = Wp.double().clone()
    want[:, c0:c1] -= Et[:, :d_out].double().T @ U[k0:k0 + Kd, c0:c1].double()
    got = bq.bpdq_block_update(Et.to(dev), U.to(dev), k0, Wp.to(dev), c0, c1).cpu().double()
    bound = 4e-6 * (Et[:, :d_out].double().abs().T @ U[k0:k0 + Kd].double().abs()) + 2e-7 * Wp.double().abs()
    assert bool(((got - want).abs() <= bound + 1e-12).all())
    keep = torch.ones(d_in, dtype=torch.bool)
    keep[c0:c1] = False
    assert torch.equal(got[:, keep], Wp.double()[:, keep])


# ------------------------------------------------------------------ whole pass, tiny config
def test_whole_pass_tiny_config(dev):
    print("whole pass cfg1", flush=True)
    wl = wk.WORKLOADS["cfg1_tiny"]
    W = wk.make_weight(wl)
    s = wk.channel_scales(wl)
    X = wk.make_activation_chunk(wl, 0, s)
    # oracle
    Href = np.zeros((wl.d_in, wl.d_in))
    orc.hessian_accumulate(X.numpy(), Href)
    Uref, dead_ref, info = orc.prepare(Href, wl.damp)
    ref = orc.quantize_layer(W.numpy(), Uref, dead_ref, wl.bits, wl.group, wl.block,
                             wl.refine_iters, alpha=float(np.float32(wl.alpha)))
    # GPU, every step in the library
    H = torch.zeros((wl.d_in, wl.d_in), device=dev)
    bq.bpdq_hessian_accumulate(X.to(dev), H, symmetrize=True)
    U, dead, info_g = bq.bpdq_prepare(H, wl.damp)
    out = bq.bpdq_quantize_layer(W.to(dev), U, dead, bq.make_params(
        wl.bits, wl.group, wl.block, wl.refine_iters, wl.alpha))
    torch.cuda.synchronize()
    assert int(info_g.item()) == 0
    assert _relfro(H.cpu().numpy().astype(np.float64), Href) < H_TOL
    Wn = W.numpy().astype(np.float64)
    # the paper's layer objective ||WX - What X||^2 / ||WX||^2 through H (undamped)
    den = orc.layer_objective(Wn, np.zeros_like(Wn), Href)
    o_g = orc.layer_objective(Wn, out["W_hat"].cpu().numpy(), Href) / den
    o_r = orc.layer_objective(Wn, ref["What"], Href) / den
    print(f"   relative output error: gpu {o_g:.6e} oracle {o_r:.6e}", flush=True)
    assert abs(o_g - o_r) / o_r < OBJ_TOL
    code = orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), wl.d_in)
    nd = sum(int(np.sum(((code >> i) & 1) != ((ref["code"] >> i) & 1))) for i in range(wl.bits))
    print(f"   plane bits differing {nd / (wl.bits * code.size):.2e}", flush=True)
    assert nd / (wl.bits * code.size) <= PLANE_TOL


@pytest.mark.parametrize("bits,group,block,iters,d_out,d_in", [
    (2, 32, 32, 3, 1, 32),          # one row, one group, one plane word
    (2, 128, 4096, 2, 17, 256),     # lazy block wider than the layer: no block update at all
    (3, 32, 32, 63, 16, 64),        # the largest iteration count the library accepts
    (2, 64, 64, 2, 16, 64),         # exactly one work-group, one group
])
def test_quantize_layer_degenerate_shapes(dev, bits, group, block, iters, d_out, d_in):
    print(f"degenerate k={bits} g={group} B={block} T={iters} {d_out}x{d_in}", flush=True)
    wl, W, X = _problem("cfg1_tiny", d_out, d_in, 4 * d_in)
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, info = orc.prepare(H, wl.damp)
    U32 = Uref.astype(np.float32)
    Ht = np.linalg.inv(U32.astype(np.float64).T @ U32.astype(np.float64))
    ref, out = _run_both(dev, wl, W, U32, dead, bits, group, block, iters)
    planes = out["planes"].cpu().numpy().view(np.uint32)
    code = orc.unpack_planes(planes, d_in)
    # tiny layers: a fraction of differing bits means little (one flipped near-tie is a visible
    # share of the layer), so the comparison is the one that holds at any size: group by group
    # from the GPU's own group-start blocks the planes are identical wherever no decision was a
    # near-tie, and end to end only rows with such a decision may differ from the oracle
    _teacher_forced(ref, out, W, U32, bits, group, iters, wl.alpha)
    Wn = W.numpy().astype(np.float64)
    og = orc.layer_objective(Wn, out["W_hat"].cpu().numpy(), Ht)
    assert abs(float(out["grp_err"].sum().item()) - og) / og < 1e-3
    assert torch.equal(bq.bpdq_dequant(out["planes"], out["coefs"], group), out["W_hat"])
    assert int(code.max()) < (1 << bits)
    it = out["grp_iter"].cpu().numpy()
    assert np.all(it >= 0) and np.all(it <= iters)


def test_constant_rows_and_zero_weights(dev):
    """Degenerate inputs of the method: a row that is constant inside a group (flat: hi == lo, all
    codes 0 at initialisation) and an all-zero layer must give finite results and What == W."""
    print("constant rows / zero weights", flush=True)
    d_out, d_in, g = 32, 128, 64
    wl, W, X = _problem("cfg1_tiny", d_out, d_in, 4 * d_in)
    W[3, :] = 0.125                              # constant row
    W[5, :64] = -0.5                             # constant inside the first group only
    W[7, :] = 0.0
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, info = orc.prepare(H, wl.damp)
    U32 = Uref.astype(np.float32)
    ref, out = _run_both(dev, wl, W, U32, dead, 2, g, 64, 3)
    What = out["W_hat"].cpu().numpy()
    assert np.all(np.isfinite(What)) and np.all(np.isfinite(out["coefs"].cpu().numpy()))
    # the relative ridge of the fit (alpha tr(G)/(k+1) with only the bias column active) shrinks
    # the constant by alpha/(k+1): 1 / (1 + 1e-4 / 3)
    shrink = 1.0 / (1.0 + wl.alpha / 3.0)
    assert np.allclose(What[3], 0.125 * shrink, rtol=1e-6) and np.allclose(What[7], 0.0, atol=1e-9)
    assert np.allclose(What[5, :64], -0.5 * shrink, rtol=1e-6)
    assert np.allclose(What[[3, 5, 7]], ref["What"][[3, 5, 7]], rtol=1e-5, atol=1e-9)
    Ht = np.linalg.inv(U32.astype(np.float64).T @ U32.astype(np.float64))
    Wn = W.numpy().astype(np.float64)
    og = orc.layer_objective(Wn, What, Ht)
    orf = orc.layer_objective(Wn, ref["What"], Ht)
    assert abs(og - orf) / orf <= OBJ_TOL
    # an all-zero layer
    Z = torch.zeros(16, d_in)
    p = bq.make_params(2, g, 64, 2, wl.alpha)
    outz = bq.bpdq_quantize_layer(Z.to(dev), torch.from_numpy(U32).to(dev), None, p)
    assert float(outz["W_hat"].abs().max().item()) == 0.0
    assert float(outz["grp_err"].abs().max().item()) == 0.0


def test_pass_is_bit_reproducible(dev):
    """No floating-point atomics anywhere: two runs of the whole pass on the same inputs (fresh
    outputs and workspaces, a layer with several blocks, a ragged row tile and tail updates) give
    bit-identical H, U, planes, coefficients, W_hat, group errors and kept iterates."""
    print("two runs, bit-identical", flush=True)
    wl, W, X = _problem("cfg2_qwen7b_attn", 328, 640, 5000)
    runs = []
    for rep in range(2):
        H = torch.zeros((640, 640), device=dev)
        bq.bpdq_hessian_accumulate(X.to(dev), H, symmetrize=True)
        U, dead, info = bq.bpdq_prepare(H, wl.damp)
        out = bq.bpdq_quantize_layer(W.to(dev), U, dead, bq.make_params(2, 64, 128, 4, wl.alpha))
        torch.cuda.synchronize()
        runs.append((H, U, out))
        if rep == 0:          # disturb the allocator between the runs
            junk = torch.randn(1 << 22, device=dev)
            del junk
    (H0, U0, o0), (H1, U1, o1) = runs
    assert torch.equal(H0, H1) and torch.equal(U0, U1)
    for key in ("planes", "coefs", "W_hat", "grp_err", "grp_iter"):
        assert torch.equal(o0[key], o1[key]), key


def test_stacked_layers_equal_separate_calls(dev):
    """q/k/v-style layers that share one U, stacked by rows in one call: every output must equal
    the separate calls bit for bit, the kept iterate being chosen per layer."""
    print("stacked layers sharing U", flush=True)
    d_in = 384
    rows = [112, 48, 40]                     # the last one is ragged (not a multiple of 16)
    wl, W, X = _problem("cfg2_qwen7b_attn", sum(rows), d_in, 4 * d_in)
    W[rows[0]:rows[0] + rows[1]] *= 7.0      # different scales: different iterates win per layer
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, info = orc.prepare(H, wl.damp)
    U = torch.from_numpy(Uref.astype(np.float32)).to(dev)
    p = bq.make_params(2, 128, 128, 5, wl.alpha)
    Wd = W.to(dev)
    ends = np.cumsum(rows).tolist()
    both = bq.bpdq_quantize_layers(Wd, ends, U, None, p)
    r0 = 0
    for s, r1 in enumerate(ends):
        one = bq.bpdq_quantize_layer(Wd[r0:r1].contiguous(), U, None, p)
        assert torch.equal(both["planes"][:, r0:r1], one["planes"])
        assert torch.equal(both["coefs"][:, r0:r1], one["coefs"])
        assert torch.equal(both["W_hat"][r0:r1], one["W_hat"])
        assert torch.equal(both["grp_iter"][s], one["grp_iter"])
        assert torch.equal(both["grp_err"][s], one["grp_err"])
        r0 = r1
    it = both["grp_iter"].cpu().numpy()
    print(f"   kept iterates per layer: {it.tolist()}", flush=True)
    # argument checks: boundaries must ascend, end at d_out, and be multiples of 16 inside
    for bad in ([100, 200], [112, 150, 200], [112, 112, 200], [200, 112]):
        with pytest.raises(bq.BpdqError):
            bq.bpdq_quantize_layers(Wd, bad, U, None, p)


@pytest.mark.parametrize("rows,bits,group,iters", [
    ([16, 16, 16, 1], 2, 64, 9),             # a boundary inside every 32 rows that are committed together; more iterates than wavefronts
    ([80, 49], 4, 32, 0),                    # one iterate, 16 levels, a ragged end
    ([48, 544], 1, 128, 7),                  # more row blocks than a lane takes scores
    ([33], 3, 256, 8),                       # one row past a work-group
])
def test_commit_of_stacked_and_unaligned_layers(dev, rows, bits, group, iters):
    """Two row blocks are committed together: they may belong to two layers, and W_hat may lie anywhere.  Every output
    equals that of the layers by themselves bit for bit, and W_hat the matrix that the stored format gives."""
    print(f"commit rows={rows} k={bits} g={group} T={iters}", flush=True)
    d_in = 512
    wl, W, X = _problem("cfg2_qwen7b_attn", sum(rows), d_in, 2 * d_in)
    W[rows[0]:] *= 7.0
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    U = torch.from_numpy(orc.prepare(H, wl.damp)[0].astype(np.float32)).to(dev)
    p = bq.make_params(bits, group, max(128, group), iters, wl.alpha)
    Wd, n_grp = W.to(dev), d_in // group
    both = bq.bpdq_quantize_layers(Wd, np.cumsum(rows).tolist(), U, None, p)
    r0 = 0
    for s, n in enumerate(rows):
        r1 = r0 + n
        for shift in (0, 1, 2, 3):
            flat = torch.full((n * d_in + shift + 4,), 3.0, device=dev)
            out = dict(planes=torch.empty((bits, n, d_in // 32), dtype=torch.int32, device=dev),
                       coefs=torch.empty((bits + 1, n, n_grp), device=dev),
                       W_hat=flat[shift:shift + n * d_in],
                       grp_err=torch.empty(n_grp, dtype=torch.float64, device=dev),
                       grp_iter=torch.empty(n_grp, dtype=torch.int32, device=dev))
            bq.bpdq_quantize_layer(Wd[r0:r1].contiguous(), U, None, p, out=out)
            assert torch.equal(both["planes"][:, r0:r1], out["planes"])
            assert torch.equal(both["coefs"][:, r0:r1], out["coefs"])
            assert torch.equal(both["W_hat"][r0:r1].reshape(-1), out["W_hat"])
            assert bool((flat[:shift] == 3.0).all()) and bool((flat[shift + n * d_in:] == 3.0).all())
            assert torch.equal(both["grp_iter"][s], out["grp_iter"])
            assert torch.equal(both["grp_err"][s], out["grp_err"])
        r0 = r1
    assert torch.equal(both["W_hat"], bq.bpdq_dequant(both["planes"], both["coefs"], group))


# ------------------------------------------------------------------ serving side
@pytest.mark.parametrize("bits,group,d_out,d_in", [
    (2, 128, 200, 384), (3, 64, 37, 320), (4, 32, 64, 2080), (1, 256, 19, 512), (2, 128, 515, 3584),
])
def test_gemv_from_stored_format(dev, bits, group, d_out, d_in):
    """y = What x from packed planes + half coefficients against the oracle's Eq. 1 + matvec."""
    print(f"gemv k={bits} g={group} {d_out}x{d_in}", flush=True)
    rng = np.random.default_rng(bits * 1000 + d_in)
    code = rng.integers(0, 1 << bits, size=(d_out, d_in)).astype(np.uint8)
    coef = (rng.standard_normal((bits + 1, d_out, d_in // group)) * 0.02).astype(np.float16)
    x = rng.standard_normal(d_in).astype(np.float32)
    planes_np = orc.pack_planes(code, bits)
    planes = torch.from_numpy(planes_np.view(np.int32)).to(dev)
    y = bq.bpdq_gemv(planes, torch.from_numpy(coef).to(dev), group, torch.from_numpy(x).to(dev))
    want = orc.gemv(planes_np, coef, group, x)
    # fp32 accumulation: bound relative to sum |C_0| |x| + sum_i |C_i| b_i |x|
    A = np.repeat(np.abs(coef[0].astype(np.float64)), group, axis=1)
    for i in range(1, bits + 1):
        A = A + np.repeat(np.abs(coef[i].astype(np.float64)), group, axis=1) * ((code >> (i - 1)) & 1)
    bound = 1e-5 * (A @ np.abs(x.astype(np.float64))) + 1e-12
    err = np.abs(y.cpu().numpy().astype(np.float64) - want)
    print(f"   max err / bound = {np.max(err / bound):.3f}", flush=True)
    assert np.all(err <= bound)


@pytest.mark.parametrize("bits,group,d_out,d_in,shift", [
    (1, 32, 1, 32, 0), (2, 64, 17, 2048, 0), (2, 32, 33, 2080, 0),          # one word; all 64 lanes of one word; two words
    (3, 64, 40, 4096, 0), (3, 96, 40, 2400, 0),                             # two words per lane: full, odd word count
    (4, 64, 4100, 4160, 0), (2, 128, 4130, 8448, 0), (2, 64, 70, 16512, 1),  # four words, two rows, chunks, unaligned planes
    (3, 32, 4097, 4224, 0), (1, 256, 8200, 512, 0),                         # one row of three planes; several passes
    (2, 128, 8230, 8448, 0),                                                # passes times chunks
    (4, 32, 33, 2112, 0), (3, 96, 50, 3072, 0), (1, 32, 20, 4032, 1),       # two words: group per word, group of three words, unaligned
    (4, 32, 35, 8192, 0), (3, 32, 4099, 8192, 0), (2, 64, 41, 8192, 0),     # four words: four and two groups to a lane
    (2, 32, 4100, 8224, 0), (4, 64, 33, 8320, 0), (3, 128, 8195, 12416, 0),  # strided: 257 words, 260 and 388 for the idle lanes
    (2, 192, 18, 6144, 0), (1, 160, 4100, 20480, 2),                        # strided: groups that no lane holds whole
])
def test_gemv_tile_edges(dev, bits, group, d_out, d_in, shift):
    """Every words-per-lane, groups-per-lane, lane-order and rows-per-wavefront variant at its edges against Eq. 1 in
    fp64; a second time with the coefficients two bytes off, where they no longer come as one load."""
    print(f"gemv edges k={bits} g={group} {d_out}x{d_in} shift={shift}", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(d_in + bits)
    n = bits * d_out * (d_in // 32)
    buf = torch.randint(-(1 << 31), 1 << 31, (n + 4,), generator=g, device=dev, dtype=torch.int64).to(torch.int32)
    planes = buf[shift:shift + n].reshape(bits, d_out, d_in // 32)
    coef = (torch.randn((bits + 1, d_out, d_in // group), generator=g, device=dev) * 0.02).half()
    x = torch.randn(d_in, generator=g, device=dev)
    y = torch.full((d_out + 3,), float("nan"), device=dev)
    bq.bpdq_gemv(planes, coef, group, x, y[:d_out])
    off = torch.empty(coef.numel() + 1, dtype=torch.float16, device=dev)[1:].view_as(coef).copy_(coef)
    y2 = bq.bpdq_gemv(planes, off, group, x)
    bit = torch.arange(32, device=dev, dtype=torch.int32)
    W = coef[0].double().repeat_interleave(group, 1)
    A = W.abs()
    for i in range(bits):
        b = ((planes[i][:, :, None] >> bit) & 1).reshape(d_out, d_in).double()
        c = coef[i + 1].double().repeat_interleave(group, 1)
        W, A = W + b * c, A + b * c.abs()
    want, bound = W @ x.double(), 1e-5 * (A @ x.double().abs()) + 1e-12
    for got in (y[:d_out], y2):
        assert bool(((got.double() - want).abs() <= bound).all())
    assert bool(torch.isnan(y[d_out:]).all())


@pytest.mark.parametrize("bits,group,d_in", [(2, 32, 32 * 65), (2, 32, 32 * 129), (2, 64, 32 * 130), (1, 96, 96 * 25),
                                             (4, 32, 32 * 257), (2, 32, 32 * 64), (2, 128, 32 * 132)])
def test_gemv_infinite_coefficient(dev, bits, group, d_in):
    """A coefficient beyond the half range is stored as an infinity and shows as one: the idle lanes and words past a
    row's end contribute nothing, not zero times it."""
    print(f"gemv infinite coefficient k={bits} g={group} d_in={d_in}", flush=True)
    d_out = 5
    planes = torch.full((bits, d_out, d_in // 32), -1, dtype=torch.int32, device=dev)
    coef = torch.zeros((bits + 1, d_out, d_in // group), device=dev).half()
    coef[0] = 0.5
    coef[0, 2, -1] = float("inf")
    coef[bits, 4, 0] = float("-inf")
    y = bq.bpdq_gemv(planes, coef, group, torch.ones(d_in, device=dev))
    assert y.tolist() == [d_in / 2, d_in / 2, float("inf"), d_in / 2, float("-inf")]


def test_gemv_of_a_quantized_layer(dev):
    print("gemv of a quantized layer (fp16 storage) + timing", flush=True)
    wl, W, X = _problem("cfg2_qwen7b_attn", 512, 3584, 4096)
    H = torch.zeros(3584, 3584, device=dev)
    bq.bpdq_hessian_accumulate(X.to(dev), H, 2.0, True)
    U, dead, info = bq.bpdq_prepare(H, wl.damp)
    p = bq.make_params(2, 128, 128, 2, wl.alpha, coef_fp16=True)
    out = bq.bpdq_quantize_layer(W.to(dev), U, dead, p)
    ch = bq.bpdq_coefs_to_fp16(out["coefs"])
    x = X[7].contiguous().to(dev)
    y = bq.bpdq_gemv(out["planes"], ch, 128, x)
    want = out["W_hat"].double() @ x.double()
    scale = (out["W_hat"].double().abs() @ x.double().abs())
    assert bool(((y.double() - want).abs() <= 2e-5 * scale + 1e-9).all())
    # rejected sizes
    with pytest.raises(bq.BpdqError):
        bq.bpdq_gemv(out["planes"], ch, 48, x)


# ------------------------------------------------------------------ channel ordering
@pytest.mark.parametrize("d_in,group_size", [(96, 1), (1000, 1), (384, 128), (2048, 64), (29568, 1)])
def test_channel_order_matches_oracle(dev, d_in, group_size):
    print(f"channel order d={d_in} gs={group_size}", flush=True)
    rng = np.random.default_rng(d_in + group_size)
    diag = (rng.random(d_in).astype(np.float32) * 10).round(1)      # rounded: plenty of ties
    if d_in <= 2048:
        H = torch.zeros(d_in, d_in)
        H.diagonal().copy_(torch.from_numpy(diag))
        Hd = H.to(dev)
    else:                                   # only the diagonal is read: a strided view will do
        Hd = torch.zeros(d_in * d_in, device=dev)
        Hd[:: d_in + 1] = torch.from_numpy(diag).to(dev)
        Hd = Hd.view(d_in, d_in)
    perm = bq.bpdq_channel_order(Hd, group_size).cpu().numpy()
    want = orc.channel_order(np.diag(diag.astype(np.float64)), group_size)
    assert np.array_equal(perm, want)


def test_gather_scatter_bit_exact_and_ordered_pass(dev):
    """Columns in and out of the permuted order are exact copies; the pass run in descending
    order of diag(H) gives a valid layer whose objective (under the original metric) equals its
    own sum of scores, compared against the oracle run on the same permuted inputs."""
    print("gather / scatter / ordered pass", flush=True)
    d_out, d_in = 72, 256
    wl, W, X = _problem("cfg3a_qwen7b_up", d_out, d_in, 4 * d_in)      # lognormal channel scales
    Hd = torch.zeros(d_in, d_in, device=dev)
    bq.bpdq_hessian_accumulate(X.to(dev), Hd, 2.0, True)
    perm = bq.bpdq_channel_order(Hd)
    pn = perm.cpu().numpy()
    Hn = Hd.cpu().numpy()
    assert np.array_equal(pn, orc.channel_order(Hn.astype(np.float64)))
    Wp = bq.bpdq_gather_columns(W.to(dev), perm)
    Hp = bq.bpdq_gather_symmetric(Hd, perm)
    assert np.array_equal(Wp.cpu().numpy(), W.numpy()[:, pn])
    assert np.array_equal(Hp.cpu().numpy(), Hn[np.ix_(pn, pn)])
    assert torch.equal(bq.bpdq_scatter_columns(Wp, perm), W.to(dev))
    U, dead, info = bq.bpdq_prepare(Hp, wl.damp)
    assert int(info.item()) == 0
    p = bq.make_params(3, 64, 128, 4, wl.alpha)
    out = bq.bpdq_quantize_layer(Wp, U, dead, p)
    What = bq.bpdq_scatter_columns(out["W_hat"], perm).cpu().numpy().astype(np.float64)
    # oracle on the same permuted inputs and the same fp32 U
    U64 = U.cpu().numpy().astype(np.float64)
    ref = orc.quantize_layer(Wp.cpu().numpy(), U64, dead.cpu().numpy().astype(bool), 3, 64, 128, 4,
                             alpha=float(np.float32(wl.alpha)))
    code = orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), d_in)
    assert np.mean(code != ref["code"]) <= PLANE_TOL
    Htp = np.linalg.inv(U64.T @ U64)                                  # damped metric, permuted order
    inv = np.argsort(pn)
    Ht = Htp[np.ix_(inv, inv)]                                        # ... back in the original order
    Wn = W.numpy().astype(np.float64)
    og = orc.layer_objective(Wn, What, Ht)
    Wr = np.empty_like(ref["What"])
    Wr[:, pn] = ref["What"]
    orf = orc.layer_objective(Wn, Wr, Ht)
    assert abs(og - orf) / orf <= OBJ_TOL
    assert abs(float(out["grp_err"].sum().item()) - og) / og < 1e-3
    # for reference: the natural order on the same layer
    U0, dead0, _ = bq.bpdq_prepare(Hd, wl.damp)
    out0 = bq.bpdq_quantize_layer(W.to(dev), U0, dead0, p)
    o0 = orc.layer_objective(Wn, out0["W_hat"].cpu().numpy(), Ht)
    print(f"   objective descending-diagonal order / natural order = {og / o0:.3f}", flush=True)


@pytest.mark.parametrize("bits,group", [(k, g) for k in (1, 2, 3, 4) for g in (32, 64, 128, 256) if (k, g) != (4, 256)])
def test_nearest_level_ties_take_the_lowest_code(dev, bits, group):
    """With U = I nothing propagates, and the fixed grid over [0, 2^k - 1] has the integers as levels: every
    half-way weight must take the lower code, whatever column it is in, and every other the nearest."""
    print(f"ties k={bits} g={group}", flush=True)
    rng = np.random.default_rng(bits * 100 + group)
    top = (1 << bits) - 1
    d_out = 21
    W = rng.integers(0, 4 * top + 1, size=(d_out, group)).astype(np.float32) / 4      # quarters: exact distances
    W[:, 0], W[:, -1] = 0.0, float(top)
    W[1] = np.minimum(np.arange(group) % (top + 1) + 0.5, top)                        # a row of half-way weights
    W[1, 0], W[1, -1] = 0.0, float(top)
    U = torch.eye(group, device=dev)
    p = bq.make_params(bits, group, group, 0, grid=bq.GRID_UNIFORM)
    out = bq.bpdq_quantize_layer(torch.from_numpy(W).to(dev), U, None, p)
    code = orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), group)
    want = np.ceil(W - 0.5).astype(np.int64)
    assert np.array_equal(code, want)
    assert np.array_equal(out["W_hat"].cpu().numpy(), want.astype(np.float32))
    assert float(out["grp_err"][0]) == float(((W - want).astype(np.float64) ** 2).sum())


@pytest.mark.parametrize("group", [32, 64, 128, 256])
def test_ties_between_descending_levels(dev, group):
    """Code 1 fitted above code 2, and a weight half-way between the two (114 between 115.75 and 112.25): the lower code
    wins, not the lower level.  U = I and no ridge: every number of the first refinement is exact."""
    print(f"descending tie g={group}", flush=True)
    t = np.repeat([0, 114, 142, 255, 202, 17, 118], np.array([10, 1, 1, 1, 3, 2, 14]) * (group // 32)).astype(np.float32)
    W = np.tile(t, (19, 1))
    W[7] = np.roll(t, 5)
    W[11] = np.linspace(-1, 1, group)
    ref = orc.quantize_layer(W.astype(np.float64), np.eye(group), None, 2, group, group, 1, alpha=0.0)
    assert ref["grp_iter"][0] == 1 and np.all(ref["code"][0][t == 114] == 1)
    out = bq.bpdq_quantize_layer(torch.from_numpy(W).to(dev), torch.eye(group, device=dev), None,
                                 bq.make_params(2, group, group, 1, 0.0))
    assert int(out["grp_iter"][0]) == 1
    assert np.array_equal(orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), group), ref["code"])


@pytest.mark.parametrize("bits,group", [(1, 64), (2, 128), (3, 32), (3, 256), (4, 128)])
@pytest.mark.parametrize("exponent", [-70, -64, 0, 64])
def test_sweep_is_its_definition_where_squares_leave_fp32(dev, bits, group, exponent):
    """A decision is the smallest squared distance in fp32, the lowest code of several, also where the squares are
    denormal, zero or infinite and more and more levels tie.  Fixed grid, one group; the sweep column by column in
    fp32: e = (w - level) (1 / U_ll), and a fused multiply-add (a product of two fp32 is exact in 64 bits) per later column."""
    print(f"sweep by definition k={bits} g={group} 2^{exponent}", flush=True)
    rng = np.random.default_rng(100 * bits + group)
    f = np.float32
    W = np.ldexp(rng.standard_normal((37, group)).astype(f), exponent)
    U = (np.eye(group) * (1 + 0.2 * rng.random(group)) + np.triu(rng.standard_normal((group, group)), 1) * 0.3 / group ** 0.5).astype(f)
    lo, hi = W.min(1), W.max(1)
    step = (hi - lo) / f((1 << bits) - 1)
    levels = np.empty((37, 1 << bits), f)
    for c in range(1 << bits):
        levels[:, c] = lo
        for i in range(bits):
            if c >> i & 1:
                levels[:, c] += step * f(1 << i)
    w, want, inv = W.copy(), np.empty((37, group), np.int64), f(1) / U.diagonal()
    with np.errstate(over="ignore", under="ignore"):
        for j in range(group):
            d = w[:, j:j + 1] - levels
            want[:, j] = np.argmin(d * d, 1)
            e = d[np.arange(37), want[:, j]] * inv[j]
            w[:, j + 1:] = (w[:, j + 1:].astype(np.float64) - e[:, None].astype(np.float64) * U[j, j + 1:]).astype(f)
    out = bq.bpdq_quantize_layer(torch.from_numpy(W).to(dev), torch.from_numpy(U).to(dev), None,
                                 bq.make_params(bits, group, group, 0, grid=bq.GRID_UNIFORM))
    assert np.array_equal(orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), group), want)


def _fma32(a, b, c):
    """Fused multiply-add of fp32 arrays, rounded once: the product is exact in 64 bits, the sum is rounded to odd there
    and then to fp32."""
    p, c = a.astype(np.float64) * b.astype(np.float64), c.astype(np.float64)
    s = p + c
    back = s - p
    lost = (p - (s - back)) + (c - back)
    odd = np.nextafter(s, np.where(lost > 0, np.inf, -np.inf))
    return np.where((lost != 0) & (s.view(np.int64) & 1 == 0), odd, s).astype(np.float32)


def _solve_chain(v, b, U, fused=True):
    """z U = v + b by the ascending recurrence in fp32: z_l = (b_l + v_l) (1 / U_ll), v_j = v_j - z_l U_lj."""
    f, inv = np.float32, np.float32(1) / U.diagonal()
    v, z = v.copy(), np.empty_like(v)
    for l in range(U.shape[0]):
        z[:, l] = (v[:, l] if b is None else b[:, l] + v[:, l]) * inv[l]
        if fused:
            v[:, l + 1:] = _fma32(z[:, l:l + 1], -U[l:l + 1, l + 1:], v[:, l + 1:])
        else:
            v[:, l + 1:] = (z[:, l:l + 1] * -U[l:l + 1, l + 1:]).astype(f) + v[:, l + 1:]
    return z


@pytest.mark.parametrize("bits,group", [(k, g) for k in (1, 2, 3, 4) for g in (32, 64, 128, 256) if (k, g) != (4, 256)])
@pytest.mark.parametrize("iters,exponent", [(0, 0), (3, 0), (3, -66)])
def test_solves_are_an_ascending_chain_of_fused_multiply_adds(dev, bits, group, iters, exponent):
    """tau and the planes' solves, whose products to later blocks go through the matrix cores, are the ascending recurrence in
    fp32 with one rounding per multiply-add, bit for bit.  Seen through a group's error, the sum of E'^2 in 64 bits over one
    row block: E' from the recurrence emulated with the returned planes and coefficients.  Off-diagonals of the factor over
    12 binary orders of magnitude, so that products meet larger and smaller sums.  iters = 0: tau beside the planes (alone
    first where there are four); 3: a kept iterate's planes by themselves, one plane of a large group with the sweep unless
    its decisions were taken again, as they are at 2^-66, where squared distances underflow and tie."""
    print(f"solves k={bits} g={group} T={iters} 2^{exponent}", flush=True)
    rng = np.random.default_rng(1000 * bits + group + iters)
    f, d_out = np.float32, 16
    W = rng.standard_normal((d_out, group)).astype(f)
    W *= np.exp2(exponent + rng.integers(-3, 4, size=(d_out, 1))).astype(f)
    off = rng.standard_normal((group, group)) * np.exp2(rng.uniform(-10, 2, (group, group)))
    U = (np.diag(1 + 0.3 * rng.random(group)) + 0.3 / group ** 0.5 * np.triu(off, 1)).astype(f)
    out = bq.bpdq_quantize_layer(torch.from_numpy(W).to(dev), torch.from_numpy(U).to(dev), None,
                                 bq.make_params(bits, group, group, iters, 1e-4))
    assert (int(out["grp_iter"][0]) > 0) == (iters > 0)
    code = orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), group)
    coef = out["coefs"].cpu().numpy()[:, :, 0]

    def group_error(fused):
        e = _fma32(-coef[0][:, None], _solve_chain(np.ones((1, group), f), None, U), _solve_chain(W, None, U, fused))
        for i in range(bits):
            e = _fma32(-coef[i + 1][:, None], _solve_chain(np.zeros_like(W), (code >> i & 1).astype(f), U, fused), e)
        lanes = np.zeros((d_out, 16))
        for m in range(group // 16):                       # a lane's columns in order, then the butterfly, then the rows
            lanes += e[:, 16 * m:16 * m + 16].astype(np.float64) ** 2
        for x in (1, 2, 4, 8):
            lanes = lanes + lanes[:, np.arange(16) ^ x]
        total = 0.0
        for r in range(d_out):
            total += lanes[r, 0]
        return total

    assert float(out["grp_err"][0]) == group_error(True)
    assert float(out["grp_err"][0]) != group_error(False)


@pytest.mark.parametrize("bits,group", [(1, 64), (2, 32), (2, 128), (3, 256), (4, 64)])
def test_levels_that_are_not_finite_never_win(dev, bits, group):
    """The nearest level is the one that a scan from code 0 with a strict `<` keeps: an infinite or NaN distance never
    replaces code 0, whatever the bit patterns of its NaN.  U = I, fixed grid."""
    print(f"levels not finite k={bits} g={group}", flush=True)
    rng = np.random.default_rng(bits + group)
    U = torch.eye(group, device=dev)
    W = rng.standard_normal((24, group)).astype(np.float32)
    W[:, 0], W[:, 1] = -4.0, 4.0                       # the row's grid, so that one weight does not move it

    def run(w, fp16):
        out = bq.bpdq_quantize_layer(torch.from_numpy(w).to(dev), U, None, bq.make_params(bits, group, group, 0,
                                                                                      grid=bq.GRID_UNIFORM, coef_fp16=fp16))
        return orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), group), out

    clean, _ = run(W, False)
    bad = W.copy()
    bad[3, 7] = np.nan                                 # from here on the row's weights are NaN: code 0
    bad[5, 9] = np.inf                                 # step infinite, C_0 finite
    bad[7, 11] = -np.inf                               # C_0 infinite: every level is
    bad[9] *= 1e6                                      # (beyond the half range below)
    code, out = run(bad, False)
    want = clean.copy()
    want[3, 7:] = 0
    want[5] = want[7] = 0
    assert np.array_equal(code, want)
    assert np.all(out["W_hat"].cpu().numpy()[7] == -np.inf)
    code, out = run(bad, True)
    keep = [r for r in range(24) if r not in (3, 5, 7, 9)]
    assert np.array_equal(code[keep], run(W, True)[0][keep])
    assert not code[[5, 7, 9]].any() and not code[3, 7:].any()
    assert np.all(out["W_hat"].cpu().numpy()[[7, 9]] == -np.inf)
    # with propagation an infinite C_0 meets infinite weights too: NaN distances of different origin
    U = torch.eye(group, device=dev) + 0.1 * torch.randn((group, group), device=dev).triu(1)
    for fp16, rows in ((False, [7]), (True, [7, 9])):
        code, out = run(bad, fp16)
        assert not code[rows].any() and np.all(out["W_hat"].cpu().numpy()[rows] == -np.inf)


def test_levels_beyond_the_half_range(dev):
    """A plane step above 65504 is stored as an infinity; its levels are never the nearest."""
    print("levels beyond the half range", flush=True)
    rng = np.random.default_rng(5)
    g, d_out = 64, 20
    W = 5000.0 * rng.integers(0, 29, size=(d_out, g)).astype(np.float32)
    W[:, 0], W[:, -1] = 0.0, 140000.0                  # lo 0, step 20000: coefficients 0, 20000, 40000, infinite
    p = bq.make_params(3, g, g, 0, grid=bq.GRID_UNIFORM, coef_fp16=True)
    out = bq.bpdq_quantize_layer(torch.from_numpy(W).to(dev), torch.eye(g, device=dev), None, p)
    want = np.minimum(np.ceil(W / 20000.0 - 0.5), 3).astype(np.int64)
    assert np.array_equal(orc.unpack_planes(out["planes"].cpu().numpy().view(np.uint32), g), want)
    assert bool(torch.isinf(out["coefs"][3]).all()) and np.array_equal(out["W_hat"].cpu().numpy(), 20000.0 * want)
    assert float(out["grp_err"][0]) == float(((W - 20000.0 * want).astype(np.float64) ** 2).sum())


def test_half_coefficients_are_rounded_once(dev):
    """The fitted fp64 coefficient goes to a half in one step: values a little off a midpoint of two halves, which
    rounding to fp32 first would put on it."""
    print("half rounding", flush=True)
    g = 32
    up, down = np.float32(1 + 2.0 ** -11), np.float32(1 + 3 * 2.0 ** -11)      # midpoints of neighbouring halves
    W = np.full((2, g), 3.0, dtype=np.float32)
    W[0, :16], W[0, 0] = up, np.nextafter(up, np.float32(2))
    W[1, :16], W[1, 0] = down, np.nextafter(down, np.float32(0))
    mean = W[:, :16].astype(np.float64).mean(axis=1)                           # midpoint +- 2^-27
    p = bq.make_params(1, g, g, 0, alpha=0.0, coef_fp16=True)
    out = bq.bpdq_quantize_layer(torch.from_numpy(W).to(dev), torch.eye(g, device=dev), None, p)
    got = out["coefs"][0, :, 0].cpu().numpy()
    assert got.tolist() == [1 + 2.0 ** -10, 1 + 2.0 ** -10]
    assert np.array_equal(got, orc.round_coefficients(mean[:, None], np.float16)[:, 0])


@pytest.mark.parametrize("bits,group,d_out,d_in", [(2, 32, 40, 128), (2, 128, 33, 256), (1, 64, 20, 192)])
def test_most_iterations(dev, bits, group, d_out, d_in):
    """refine_iters = 63: the row scores of all 64 iterates, kept where the pending tile was, and their sums."""
    print(f"63 iterations k={bits} g={group} {d_out}x{d_in}", flush=True)
    wl, W, X = _problem("cfg1_tiny", d_out, d_in, 4 * d_in)
    H = np.zeros((d_in, d_in))
    orc.hessian_accumulate(X.numpy(), H)
    Uref, dead, _ = orc.prepare(H, wl.damp)
    U32 = Uref.astype(np.float32)
    ref, out = _run_both(dev, wl, W, U32, dead, bits, group, group, 63)
    assert int(out["grp_iter"].max()) <= 63
    _teacher_forced(ref, out, W, U32, bits, group, 63, wl.alpha)


# ------------------------------------------------------------------ storage helpers
@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_pack_and_dequant_bit_exact(dev, bits):
    print(f"pack/dequant k={bits}", flush=True)
    rng = np.random.default_rng(bits)
    d_out, d_in, group = 37, 320, 64
    code = rng.integers(0, 1 << bits, size=(d_out, d_in)).astype(np.uint8)
    planes = bq.bpdq_pack_planes(torch.from_numpy(code).to(dev), bits)
    pg = planes.cpu().numpy().view(np.uint32)
    assert np.array_equal(pg, orc.pack_planes(code, bits))
    coef = rng.standard_normal((bits + 1, d_out, d_in // group)).astype(np.float32)
    Wg = bq.bpdq_dequant(planes, torch.from_numpy(coef).to(dev), group).cpu().numpy()
    # fp32 evaluation order ((c0 + b1 c1) + b2 c2) + ... reproduced on the host
    want = np.repeat(coef[0], group, axis=1)
    for i in range(1, bits + 1):
        b = ((code >> (i - 1)) & 1).astype(bool)
        want = np.where(b, (want + np.repeat(coef[i], group, axis=1)).astype(np.float32), want)
    assert np.array_equal(Wg, want)
    assert np.allclose(Wg, orc.dequant(pg, coef, group), rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("d_out,d_in,group,shift", [
    (1, 32, 32, 0), (3, 1056, 32, 0), (5, 2080, 4, 0),      # vector stores: one row, columns past a work-group's 1024
    (4, 1024, 2, 0), (7, 96, 3, 0), (6, 64, 64, 1),         # groups that four columns straddle, W_hat off 16 bytes
    (33, 32, 32, 0), (130, 96, 32, 0),                      # several row blocks to a work-group, the last one part full
    (4099, 256, 64, 0), (1025, 1056, 32, 0),                # several rows per thread: narrow, wide
    (1027, 1056, 3, 0), (8201, 128, 64, 1),                 # ... with scalar stores
    (16369, 1024, 32, 0), (16387, 1056, 96, 0),             # tiles through LDS: one column tile, rows past the last tile's
    (8177, 3584, 256, 0), (4097, 7456, 32, 0),              # ... several, the last one part full
])
def test_dequant_tile_edges(dev, half, d_out, d_in, group, shift):
    """Both store widths of the dequant kernel at the edges of its tiles, bit for bit."""
    _check_dequant(dev, half, 3, d_out, d_in, group, shift)


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("bits,d_out,d_in,group", [
    (1, 16369, 1024, 128), (2, 16369, 1024, 32), (4, 16369, 1024, 64), (4, 8177, 3616, 32),      # tiles through LDS
    (4, 32753, 1024, 32), (4, 32737, 1024, 32),            # where 32-bit coefficients begin to go by them, and one tile fewer
])
def test_dequant_tiles_of_every_plane_count(dev, half, bits, d_out, d_in, group):
    _check_dequant(dev, half, bits, d_out, d_in, group, 0)


def _check_dequant(dev, half, bits, d_out, d_in, group, shift):
    print(f"dequant k={bits} d_out={d_out} d_in={d_in} g={group} shift={shift} half={half}", flush=True)
    rng = np.random.default_rng(d_in + group)
    code = rng.integers(0, 1 << bits, size=(d_out, d_in)).astype(np.uint8)
    planes = torch.from_numpy(orc.pack_planes(code, bits).view(np.int32)).to(dev)
    coef = rng.standard_normal((bits + 1, d_out, d_in // group)).astype(np.float16 if half else np.float32)
    coef_d = torch.from_numpy(coef).to(dev)
    buf = torch.full((d_out * d_in + 8,), np.nan, device=dev)
    lib = bq.load()
    fn = lib.bpdq_dequant_fp16 if half else lib.bpdq_dequant
    W = buf[shift:]
    assert fn(planes.data_ptr(), coef_d.data_ptr(), d_out, d_in, bits, group, W.data_ptr(), bq._stream()) == 0
    torch.cuda.synchronize()
    c32 = coef.astype(np.float32)
    want = np.repeat(c32[0], group, axis=1)
    for i in range(1, bits + 1):
        b = ((code >> (i - 1)) & 1).astype(bool)
        want = np.where(b, (want + np.repeat(c32[i], group, axis=1)).astype(np.float32), want)
    got = buf.cpu().numpy()
    assert np.array_equal(got[shift:shift + d_out * d_in].reshape(d_out, d_in), want)
    assert np.isnan(got[:shift]).all() and np.isnan(got[shift + d_out * d_in:]).all()


@pytest.mark.parametrize("d,bad", [
    (64, (20, 25)), (64, (0, 15)), (192, (1, 2)),                   # one block; an odd single panel at the left edge
    (128, (3, 9)), (128, (3, 70)), (256, (17, 30)), (256, (200, 201, 207)),   # first and second block of a pair
    (130, (70, 75)), (100, (97, 98)), (640, (40, 600)), (65, (64,)),          # ragged last block; two outer blocks
])
def test_prepare_info_names_the_first_bad_pivot(dev, d, bad):
    """The factorisation runs from the last column to the first, so the first pivot that is not positive is the last
    of the negative entries of a diagonal H, wherever it lies among the panels."""
    print(f"prepare info d={d} bad={bad}", flush=True)
    h = torch.full((d,), 101.0)
    h[list(bad)] = -50.0
    _, _, info = bq.bpdq_prepare(torch.diag(h).to(dev), 0.0)
    assert int(info.item()) == max(bad) + 1


def test_prepare_many_panels_defining_property(dev):
    """A width whose panel launches have more work-groups than the chip holds at once
    (18944 = 296 panels): checked through the defining property U^T U (H + lambda I) = I on
    sampled columns, evaluated in fp64 by torch (neither side's code)."""
    print("prepare d_in=18944 (property check)", flush=True)
    d, ntok = 18944, 4096
    g = torch.Generator(device=dev)
    g.manual_seed(11)
    X = torch.randn((ntok, d), device=dev, generator=g)
    H = torch.zeros((d, d), device=dev)
    bq.bpdq_hessian_accumulate(X, H, symmetrize=True)
    H.diagonal().add_(float(H.diagonal().mean()))        # well conditioned although N < d
    U, dead, info = bq.bpdq_prepare(H, 0.01)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    idx = torch.arange(0, d, d // 48, device=dev)[:48]
    Ht = H.double()
    Ht.diagonal().add_(0.01 * float(H.diagonal().mean()))
    R = U.double().T @ (U.double() @ Ht[:, idx])
    R[idx, torch.arange(len(idx), device=dev)] -= 1.0
    assert float(R.abs().max()) < 1e-5


@pytest.mark.parametrize("d", [64, 128, 192, 576, 642, 1217, 1216, 1600, 1604])
def test_prepare_tile64_paths(dev, d):
    """U of the same fp32 H against a 64-bit factor, at widths around the 64-column blocks and the 512-column
    outer blocks: one block, odd and even block counts, odd and ragged widths (which leave the LDS-DMA tiles
    for the register-staged ones in the trailing update, the inversion, or both).  Only the rounding of U to
    fp32 separates the two sides: 2^-24 relative per entry."""
    print(f"prepare d_in={d} (64-tile paths)", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(91 + d)
    X = torch.randn((2 * d + 64, d), device=dev, generator=g, dtype=torch.float64)
    X *= torch.logspace(-1.0, 1.0, d, device=dev, dtype=torch.float64)[None, :]
    H = (X.t().contiguous() @ X).float()
    U, dead, info = bq.bpdq_prepare(H, 0.01)
    assert int(info.item()) == 0
    Hn = H.double().cpu().numpy()
    Hn = np.triu(Hn) + np.triu(Hn, 1).T
    Uref, _, _ = orc.prepare(Hn, float(np.float32(0.01)))
    Un = U.cpu().numpy().astype(np.float64)
    assert np.count_nonzero(np.tril(Un, -1)) == 0
    assert np.linalg.norm(Un - Uref) / np.linalg.norm(Uref) < 1e-7


@pytest.mark.parametrize("d", [65, 127, 128, 129, 191, 256, 257, 383, 385, 640, 1001])
def test_prepare_by_pairs_is_prepare_by_panels(dev, d):
    """Widths around the 128-column pairs, and 65, the smallest that is done by pairs.  With a workspace that is too small
    for the padded matrix of the pairs, the panels of 64 columns do the same, odd and ragged widths included.  Both are
    64-bit computations of the same U, whose rounding to fp32 may fall either way in a few entries (d 2^-53 times the
    condition, 1e4 here, against 2^-24); the workspaces hold NaN, H is overwritten, and the same pivot is reported."""
    print(f"prepare d_in={d} (pairs and panels)", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(57 + d)
    X = torch.randn((2 * d + 64, d), device=dev, generator=g, dtype=torch.float64)
    X *= torch.logspace(-1.0, 1.0, d, device=dev, dtype=torch.float64)[None, :]
    X[:, d // 3] = 0.0
    H = (X.t().contiguous() @ X).float()
    bad = H.clone()
    bad[d // 2, d // 2] = -1.0
    lib, blocks = bq.load(), -(-d // 64)
    align = lambda n: -(-n // 256) * 256
    panels = (align(8 * d * d) + align(8 * d * 64 * ((blocks + 1) // 2)) + 2 * align(8 * blocks * 64 * 64)
              + align(4 * blocks) + 256)
    full = lib.bpdq_prepare_workspace_bytes(d)
    assert panels < full
    got = []
    for size in (full, full - 256, panels):
        for h in (H, bad):
            U, dead = h.clone(), torch.full((d,), 7, dtype=torch.uint8, device=dev)
            info = torch.full((1,), -7, dtype=torch.int32, device=dev)
            ws = torch.full((size // 8,), float("nan"), dtype=torch.float64, device=dev)
            assert lib.bpdq_prepare(U.data_ptr(), d, 0.01, U.data_ptr(), dead.data_ptr(), info.data_ptr(), ws.data_ptr(),
                                    size, bq._stream()) == 0
            got.append((U.cpu().numpy(), dead.cpu().numpy(), int(info.item())))
    assert lib.bpdq_prepare(H.data_ptr(), d, 0.01, U.data_ptr(), None, info.data_ptr(), ws.data_ptr(), panels - 256,
                            bq._stream()) == -8
    Hn = np.triu(H.double().cpu().numpy())
    Uref, _, _ = orc.prepare(Hn + np.triu(Hn, 1).T, float(np.float32(0.01)))
    for i in (0, 2, 4):
        U, dead, info = got[i]
        assert info == 0 and got[i + 1][2] == got[1][2] > 0
        assert dead[d // 3] == 1 and dead.sum() == 1 and np.array_equal(dead, got[i + 1][1])
        assert np.count_nonzero(np.tril(U, -1)) == 0
        assert np.linalg.norm(U - Uref) / np.linalg.norm(Uref) < 1e-7
        assert np.linalg.norm(U - got[4][0]) / np.linalg.norm(Uref) < 1e-9


@pytest.mark.parametrize("d", [4608, 4609, 6272, 6273, 6400, 8191, 8192, 12288, 12289, 12416])
def test_prepare_where_the_pairs_change(dev, d):
    """The widths where a tile begins to wait for two pairs and for three, the widest matrix that is done by pairs and the
    narrowest that are not, one ragged and one with an odd number of pairs: U on sampled columns through
    U^T U (H + lambda I) = I."""
    print(f"prepare d_in={d} (pairs to panels)", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(d)
    X = torch.randn((2 * d, d), device=dev, generator=g)
    H = (X.t().contiguous() @ X).triu()
    H += H.triu(1).t()
    U, dead, info = bq.bpdq_prepare(H, 0.01)
    assert int(info.item()) == 0 and int(dead.sum().item()) == 0
    assert float(torch.tril(U, diagonal=-1).abs().max()) == 0.0
    idx = torch.cat([torch.arange(0, d, 97, device=dev), torch.arange(d - 140, d, device=dev)])
    Ht = H.double()
    Ht.diagonal().add_(0.01 * float(H.diagonal().mean()))
    R = U.double().T @ (U.double() @ Ht[:, idx])
    R[idx, torch.arange(len(idx), device=dev)] -= 1.0
    assert float(R.abs().max()) < 1e-5


@pytest.mark.parametrize("d", [4672, 8256, 1088, 4700])
def test_prepare_wide_tile_paths_defining_property(dev, d):
    """Widths around the switches to the 128 x 128 tile kernels: the factorisation takes them from
    4096 columns on, the inversion for tree levels with at least 512 such tiles.  73 and 129 blocks
    of 64 columns are odd at several levels of the inversion tree, so half-empty tiles occur
    (8256 has them in both kernels); 17 blocks stay on the 64-tile kernels; 4700 is ragged (its last
    block has 28 columns), so the rightmost outer block is updated by the 64-tile kernel and the
    others by the 128-tile one.  Checked: the whole of
    U^T U (H + lambda I) - I in fp64 by torch, and U upper triangular."""
    print(f"prepare d_in={d} (wide-tile paths, property check)", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(17 + d)
    X = torch.randn((2 * d, d), device=dev, generator=g)
    X *= torch.logspace(-1.0, 1.0, d, device=dev)[None, :]       # channel scales over two decades
    H = torch.zeros((d, d), device=dev)
    bq.bpdq_hessian_accumulate(X, H, symmetrize=True)
    U, dead, info = bq.bpdq_prepare(H, 0.01)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    assert int(dead.sum().item()) == 0
    assert float(torch.tril(U, diagonal=-1).abs().max()) == 0.0
    Ht = H.double()
    Ht.diagonal().add_(0.01 * float(H.diagonal().mean()))
    Ud = U.double()
    R = Ud.T @ (Ud @ Ht)
    R.diagonal().sub_(1.0)
    # U is stored in fp32: the residual is its rounding (6e-8 relative) times the condition of the product
    scale = torch.sqrt(Ht.diagonal())
    assert float((R / scale[:, None] * scale[None, :]).abs().max()) < 2e-4
    assert float(R.abs().max()) < 2e-3
