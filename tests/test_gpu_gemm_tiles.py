"""The fp32 products at the edges of their tiles, against 64-bit products.

The kernel splits every fp32 operand exactly into three bf16 values and sums
six of their nine products per K step of 32 from zero, adding the step's sum
to the running one. The terms left out are below 2^-23 |ab| with either sign,
and the running sum is rounded once per 32 products, so the normwise error is
of the order of (1 + sqrt(K / 32)) 2^-24: the bound below is eight times that.
"""
import numpy as np
import pytest

from paper_2001_02498_amd import synth
from tests.gpu_helpers import GraphCase, dev, empty, need_gpu, say, torch

pytestmark = pytest.mark.gpu


def _case(n, seed=1):
    wl = synth.small_workload(n, 6, 2, 4, 4, 2, synth.SOFTMAX_CE, (seed,))
    inp = synth.make_inputs(wl)
    return GraphCase(n, inp.src, inp.dst, rounds=0)


def _close(got, ref, K):
    err = (got.double() - ref).norm() / ref.norm()
    assert err < 8 * (1 + (K / 32) ** 0.5) * 2.0 ** -24, (float(err), K)


def _randn(*shape, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + sum(shape))
    return torch.randn(*shape, device="cuda", generator=g)


# the planned shapes of the forward product: 160 x 128 (n 10,001), 128 x 128
# (8,065), 128 x 64 (6,785), 64 x 64 (to 17), 64 x 64 with two buffers (the
# rest: six, eight and eight K steps, the last one whole or not; the input
# gradients' operands concatenated on a step and off it); the rows, columns and
# K end one past a tile, one short of one, and on one
@pytest.mark.parametrize("n,F,h", [(10001, 33, 512), (8065, 64, 512), (6785, 97, 256),
                                   (65, 1, 4), (63, 31, 20), (128, 32, 64), (17, 130, 68),
                                   (300, 192, 96), (257, 225, 100), (1000, 250, 132)])
@pytest.mark.parametrize("bias", [False, True])
def test_layer_products(n, F, h, bias):
    need_gpu()
    say("tiles", n, F, h, bias)
    case = _case(n)
    gcn = case.gcn
    ws = gcn.alloc_ws(gcn.scratch_bytes(case.dg, max(F, 2 * h)))
    H = empty(n, F, (F + 3) // 4 * 4)
    H.copy_(_randn(n, F))
    Ws, Wn = _randn(F, h, seed=1) * 0.1, _randn(F, h, seed=2) * 0.1
    b = _randn(2 * h, seed=3) if bias else None
    AH, out = empty(n, F, (F + 3) // 4 * 4), empty(n, 2 * h)
    gcn.layer_fwd(case.dg, H, Ws, Wn, b, AH, out, ws)
    d = lambda t: t.double()  # noqa: E731
    Z = torch.cat([d(H) @ d(Ws), d(AH) @ d(Wn)], 1)
    _close(out, (Z + d(b) if bias else Z).clamp(min=0), F)
    G = empty(n, 2 * h)
    G.copy_(_randn(n, 2 * h, seed=4) * 1e-5)
    Gin = empty(n, F, (F + 3) // 4 * 4)
    dWs, dWn = torch.empty_like(Ws), torch.empty_like(Wn)
    db = torch.empty_like(b) if bias else None
    Ws0, Wn0 = d(Ws), d(Wn)
    T = empty(n, h)
    gcn.aggregate(case.dg, gcn.AGG_TRANSPOSED, G[:, h:], T, ws)
    gcn.layer_bwd(case.dg, G, H, AH, Ws, Wn, b, 0.5, Gin, dWs, dWn, db, ws)
    _close(Gin, (d(G[:, :h]) @ Ws0.T + d(T) @ Wn0.T) * (H > 0), 2 * h)
    _close(dWs, d(H).T @ d(G[:, :h]), n)
    _close(dWn, d(AH).T @ d(G[:, h:]), n)
    if bias:
        _close(db, d(G).sum(0), n)
    torch.cuda.synchronize()


# unaligned rows of W_cls (C % 4 != 0), one column tile and two, with and
# without K slices, one buffer and two (n 16,000)
@pytest.mark.parametrize("n,K,C", [(1000, 256, 7), (129, 1024, 41), (4097, 512, 121),
                                   (2000, 64, 130), (33, 36, 1), (16000, 228, 41)])
def test_classifier_products(n, K, C):
    need_gpu()
    say("cls tiles", n, K, C)
    from paper_2001_02498_amd import gcn
    ws = gcn.alloc_ws(gcn.scratch_bytes(None, max(K, C), n))
    H, W, b = _randn(n, K), _randn(K, C, seed=1) * 0.1, _randn(C, seed=2)
    Z, dZ, G = empty(n, C, (C + 3) // 4 * 4), empty(n, C, (C + 3) // 4 * 4), empty(n, K)
    gcn.classifier_fwd(H, K, W, b, Z, ws)
    d = lambda t: t.double()  # noqa: E731
    _close(Z, d(H) @ d(W) + d(b), K)
    dZ.copy_(_randn(n, C, seed=3) * 1e-6)
    dW, db, W0 = torch.empty_like(W), torch.empty_like(b), d(W)
    gcn.classifier_bwd(dZ, C, H, K, W, b, 0.5, G, dW, db, ws)
    _close(G, (d(dZ) @ W0.T) * (H > 0), C)
    _close(dW, d(H).T @ d(dZ), n)
    _close(db, d(dZ).sum(0), n)
    torch.cuda.synchronize()


# sums of a few terms (one or two are fp32 products, more are split): a product of one term is the rounded product, and
# K terms are rounded K times at most at the size of their sum of magnitudes
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("n,C", [(1000, 30), (129, 130)])
def test_short_sums(K, n, C):
    need_gpu()
    say("short sums", K, n, C)
    from paper_2001_02498_amd import gcn
    ws = gcn.alloc_ws(gcn.scratch_bytes(None, max(n, C), max(n, C)))
    d = lambda t: t.double()  # noqa: E731
    one = K == 1

    def check(got, A, B):
        ref = d(A) @ d(B)
        if one:
            assert torch.equal(got, ref.float())
        assert ((d(got) - ref).abs() <= K * 2.0 ** -24 * (d(A).abs() @ d(B).abs())).all()

    H, W = empty(n, K, 8), _randn(K, C, seed=1)
    H.copy_(_randn(n, K).abs() + 0.01)
    Z = empty(n, C, (C + 3) // 4 * 4)
    gcn.classifier_fwd(H, K, W, None, Z, ws)
    check(Z, H, W)
    # the input gradient sums over the K classes, the weight gradient over the K rows
    W, dZ, G = _randn(n, K, seed=3), empty(C, K, 8), empty(C, n, (n + 3) // 4 * 4)
    H = empty(C, n, (n + 3) // 4 * 4)
    H.fill_(1.0)
    dZ.copy_(_randn(C, K, seed=4))
    W0 = W.clone()
    gcn.classifier_bwd(dZ, K, H, n, W, None, 0.0, G, None, None, ws)
    check(G, dZ, W0.T)
    H, dZ = empty(K, n, (n + 3) // 4 * 4), empty(K, C, (C + 3) // 4 * 4)
    H.copy_(_randn(K, n, seed=5))
    dZ.copy_(_randn(K, C, seed=6))
    W, b = torch.zeros(n, C, device="cuda"), torch.zeros(C, device="cuda")
    dW, db = torch.empty_like(W), torch.empty_like(b)
    gcn.classifier_bwd(dZ, C, H, n, W, b, 0.0, None, dW, db, ws)
    check(dW, H.T, dZ)
    check(db[None], torch.ones(1, K, device="cuda"), dZ)
    torch.cuda.synchronize()


def _powers(n, width, e, seed):
    """+-[1, 2) x 2^e, exact in float32 down to its last subnormal bit."""
    x = (torch.rand(n, width, generator=torch.Generator().manual_seed(seed),
                    dtype=torch.float64) * 2 - 1)
    return torch.copysign(1 + x.abs(), x).mul(2.0 ** e).float().cuda()


# operands down to the smallest subnormals times large ones: the split keeps
# every bit of any finite value
@pytest.mark.parametrize("e", [-100, -112, -118, -126, -130, -140])
@pytest.mark.parametrize("n,K,C", [(300, 40, 24), (65, 130, 7)])
def test_tiny_operands(e, n, K, C):
    need_gpu()
    say("tiny operands", e, n, K, C)
    from paper_2001_02498_amd import gcn
    ws = gcn.alloc_ws(gcn.scratch_bytes(None, max(K, C), n))
    f = min(-e, 110)
    d = lambda t: t.double()  # noqa: E731
    for a, b in ((e, f), (f, e)):
        H, W = empty(n, K, (K + 3) // 4 * 4), _powers(K, C, b, 2)
        H.copy_(_powers(n, K, a, 1).abs())
        Z, dZ, G = empty(n, C, (C + 3) // 4 * 4), empty(n, C, (C + 3) // 4 * 4), empty(
            n, K, (K + 3) // 4 * 4)
        gcn.classifier_fwd(H, K, W, None, Z, ws)
        _close(Z, d(H) @ d(W), K)
        dZ.copy_(_powers(n, C, a, 3))
        dW, W0 = torch.empty_like(W), d(W)
        gcn.classifier_bwd(dZ, C, H, K, W.clone(), None, 0.0, G, dW, None, ws)
        _close(G, d(dZ) @ W0.T, C)
        dZ.copy_(_powers(n, C, b, 4))
        gcn.classifier_bwd(dZ, C, H, K, W, None, 0.0, None, dW, None, ws)
        _close(dW, d(H).T @ d(dZ), n)
    torch.cuda.synchronize()


# sums that overflow only by the split's scale are fp32 products: K of them are
# rounded K times at most at the size of their sum of magnitudes
@pytest.mark.parametrize("a,b", [(47, 49), (60, 60), (113, -20), (126, -126), (-130, 126)])
@pytest.mark.parametrize("n,K,C", [(300, 40, 24), (65, 130, 7)])
def test_large_operands(a, b, n, K, C):
    need_gpu()
    say("large operands", a, b, n, K, C)
    from paper_2001_02498_amd import gcn
    ws = gcn.alloc_ws(gcn.scratch_bytes(None, max(K, C), n))
    H, W, Z = empty(n, K, (K + 3) // 4 * 4), _powers(K, C, b, 2), empty(n, C, (C + 3) // 4 * 4)
    H.copy_(_powers(n, K, a, 1))
    gcn.classifier_fwd(H, K, W, None, Z, ws)
    ref, size = H.double() @ W.double(), H.double().abs() @ W.double().abs()
    assert ((Z.double() - ref).abs() <= K * 2.0 ** -24 * size).all()
    torch.cuda.synchronize()


# products below the smallest normal value: one rounding to a multiple of
# 2^-149 per K step (and one per K slice) and nothing else at that size
@pytest.mark.parametrize("e", [-64, -68, -72])
def test_tiny_products(e):
    need_gpu()
    say("tiny products", e)
    from paper_2001_02498_amd import gcn
    n, K, C = 300, 32, 24
    ws = gcn.alloc_ws(gcn.scratch_bytes(None, K, n))
    H, W, Z = _powers(n, K, e, 1), _powers(K, C, e, 2), empty(n, C)
    gcn.classifier_fwd(H, K, W, None, Z, ws)
    ref = H.double() @ W.double()
    bound = 0.5 * 2.0 ** -149 + 8 * 2.0 ** -24 * (H.double().abs() @ W.double().abs())
    assert ((Z.double() - ref).abs() <= bound).all()
    torch.cuda.synchronize()


# a bf16 part of an infinity, a NaN or a value above the largest bf16 is not
# finite: the outputs it enters are recomputed as fp32 products, the others
# stay bit for bit what they are without it
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("n,K,C", [(300, 100, 24), (8100, 40, 512)])
def test_non_finite(bad, n, K, C):
    need_gpu()
    say("non-finite", bad, n, K, C)
    from paper_2001_02498_amd import gcn
    ws = gcn.alloc_ws(gcn.scratch_bytes(None, max(K, C), n))
    H, W = _randn(n, K), _randn(K, C, seed=1) * 1e-3
    W[7, 3] = 0.0
    Z, ref = empty(n, C), empty(n, C)
    gcn.classifier_fwd(H, K, W, None, ref, ws)
    H[70, 7] = bad
    gcn.classifier_fwd(H, K, W, None, Z, ws)
    others = torch.arange(n, device="cuda") != 70
    want = H[70].double() @ W.double()
    if np.isfinite(bad):
        assert torch.isfinite(Z[70]).all()
        _close(Z[70], want, K)
    else:
        assert torch.equal(torch.isnan(Z[70]).cpu(), torch.isnan(want).cpu())
        fin = ~torch.isnan(want)
        assert torch.equal(Z[70][fin].double(), want[fin])
    assert torch.equal(Z[others], ref[others])
    torch.cuda.synchronize()


def _redone(got, want, with_inf, clean, bad, K):
    """`want` (64 bits) holds a bad operand's outputs, `with_inf` those of an
    infinity in its place (non-finite where it enters), `clean` the call
    without it."""
    if np.isfinite(bad):
        assert torch.isfinite(got).all()
        _close(got, want, K)
    else:
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        inf = torch.isinf(want)
        assert torch.equal(got[inf].double(), want[inf])
    other = torch.isfinite(with_inf)
    assert not other.all()
    assert torch.equal(got[other], clean[other])


# the same in the backward products: K-major operands with the row of ones and
# K slices (the gradients), K-concatenated operands with the weights as [n][k]
# (the input gradient); in the classifier's the weight rows are not aligned
@pytest.mark.parametrize("bad", [np.inf, np.nan, 3e38])
@pytest.mark.parametrize("n,F,h", [(300, 33, 20), (8100, 97, 128)])
@pytest.mark.parametrize("where", ["H", "G", "W"])
def test_non_finite_layer_bwd(bad, n, F, h, where):
    need_gpu()
    say("non-finite layer_bwd", bad, n, F, h, where)
    case = _case(n)
    gcn = case.gcn
    ws = gcn.alloc_ws(gcn.scratch_bytes(case.dg, max(F, 2 * h)))
    H, AH = empty(n, F, (F + 3) // 4 * 4), empty(n, F, (F + 3) // 4 * 4)
    H.copy_(_randn(n, F) * 0.1)      # 3e38 times them is finite
    AH.copy_(_randn(n, F, seed=1) * 0.1)
    W0 = [_randn(F, h, seed=2 + i) * 1e-3 for i in range(2)]
    G, T = empty(n, 2 * h), empty(n, h)
    G.copy_(_randn(n, 2 * h, seed=4) * 1e-5)
    row, col = n - 17, h + 3

    def call():
        W = [w.clone() for w in W0]
        out = [empty(n, F, (F + 3) // 4 * 4)] + [torch.empty(F, h, device="cuda") for _ in
                                                 range(2)] + [torch.empty(2 * h, device="cuda")]
        gcn.aggregate(case.dg, gcn.AGG_TRANSPOSED, G[:, h:], T, ws)
        gcn.layer_bwd(case.dg, G, H, AH, *W, torch.zeros(2 * h, device="cuda"), 0.0, *out, ws)
        return out

    def spoil(x):
        t, i, j = {"H": (H, row, 5), "G": (G, row, col), "W": (W0[1], 5, 3)}[where]
        t[i, j] = x

    def exact():
        d = lambda t: t.double()  # noqa: E731
        gin = d(G[:, :h]) @ d(W0[0]).T + d(T) @ d(W0[1]).T
        return [torch.where(H > 0, gin, 0.0), d(H).T @ d(G[:, :h]), d(AH).T @ d(G[:, h:]),
                d(G).sum(0)]

    clean = call()
    spoil(np.inf)
    call()     # (T)
    with_inf = exact()
    spoil(bad)
    got = call()
    want = exact()
    entered = {"H": [1], "G": [0, 2, 3], "W": [0]}[where]
    for i, K in enumerate((2 * h, n, n, n)):
        if i in entered:
            _redone(got[i], want[i], with_inf[i], clean[i], bad, K)
        elif i:
            assert torch.equal(got[i], clean[i])
    torch.cuda.synchronize()


@pytest.mark.parametrize("bad", [np.inf, np.nan, 3e38])
@pytest.mark.parametrize("n,K,C", [(300, 100, 7), (8100, 260, 41)])
def test_non_finite_classifier_bwd(bad, n, K, C):
    need_gpu()
    say("non-finite classifier_bwd", bad, n, K, C)
    from paper_2001_02498_amd import gcn
    ws = gcn.alloc_ws(gcn.scratch_bytes(None, max(K, C), n))
    H, dZ = empty(n, K), empty(n, C, (C + 3) // 4 * 4)
    H.copy_(_randn(n, K).abs() * 0.1)
    dZ.copy_(_randn(n, C, seed=1) * 1e-5)
    W0 = _randn(K, C, seed=2) * 1e-3

    def call():
        out = [empty(n, K), torch.empty(K, C, device="cuda"), torch.empty(C, device="cuda")]
        gcn.classifier_bwd(dZ, C, H, K, W0.clone(), torch.zeros(C, device="cuda"), 0.0, *out, ws)
        return out

    def exact():
        d = lambda t: t.double()  # noqa: E731
        return [d(dZ) @ d(W0).T, d(H).T @ d(dZ), d(dZ).sum(0)]

    clean = call()
    dZ[n - 17, 3] = np.inf
    with_inf = exact()
    dZ[n - 17, 3] = bad
    for got, want, wi, c, k in zip(call(), exact(), with_inf, clean, (C, n, n)):
        _redone(got, want, wi, c, bad, k)
    torch.cuda.synchronize()


# the update takes four weights per thread in launches of 2^19 weights or more
# where every pointer allows 16-byte accesses, one otherwise: the same sums
# either way
@pytest.mark.parametrize("K,C", [(68, 24), (68, 25), (1024, 512), (1024, 513), (1022, 512)])
@pytest.mark.parametrize("shift", [0, 1])
def test_update_alignment(K, C, shift):
    need_gpu()
    say("update", K, C, shift)
    from paper_2001_02498_amd import gcn
    n = 513
    ws = gcn.alloc_ws(gcn.scratch_bytes(None, max(K, C), n))
    H, dZ = empty(n, K), empty(n, C, (C + 3) // 4 * 4)
    H.copy_(_randn(n, K))
    dZ.copy_(_randn(n, C, seed=3))
    W0, b0 = _randn(K, C, seed=1), _randn(C, seed=2)
    W = torch.zeros(K * C + shift, device="cuda")[shift:].view(K, C)
    b = torch.zeros(C + shift, device="cuda")[shift:]
    W.copy_(W0)
    b.copy_(b0)
    dW, db = torch.empty_like(W0), torch.empty_like(b0)
    gcn.classifier_bwd(dZ, C, H, K, W, b, 0.25, None, dW, db, ws)
    _close(dW, H.double().T @ dZ.double(), n)
    # one fused multiply-add each
    ulp = 2.0 ** -23
    assert ((W.double() - (W0.double() - 0.25 * dW.double())).abs() <= ulp * W0.abs().clamp(
        min=1) * (1 + dW.abs())).all()
    assert ((b.double() - (b0.double() - 0.25 * db.double())).abs() <= ulp * b0.abs().clamp(
        min=1) * (1 + db.abs())).all()
    torch.cuda.synchronize()
