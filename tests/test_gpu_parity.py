"""GPU parity: every entry point of libobc.so, called through the C ABI, against the CPU oracle on
the same seeded inputs.  Tolerances are stated in tests/parity.py."""
import numpy as np
import pytest
import torch

import obc_inputs
from tests.parity import FP32_ORDER_GAP, RowParity, check_block_row, check_row

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def obc():
    import paper_2208_11580_amd as pkg

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ctx = pkg.Context()
    yield ctx
    ctx.close()


def _np(t):
    return t.detach().cpu().numpy()


def _layer(name, **kw):
    W, X, spec = obc_inputs.make_layer(name, device="cuda", **kw)
    return W, X


def _hinv(obc, X, damp=0.01):
    H = obc.obc_hessian(X, damp_rel=damp)
    obc.obc_invert(H)
    return H


# ------------------------------------------------------------------------------ Hessian
@pytest.mark.parametrize("d,N,pad", [(32, 256, 0), (200, 3001, 3), (131, 777, 0), (576, 20000, 0)])
def test_hessian_matches_oracle(obc, orc, d, N, pad):
    torch.manual_seed(d)
    Xfull = torch.randn(d, N + pad, device="cuda")
    X = Xfull[:, :N]
    H = obc.obc_hessian(X, damp_rel=0.01)
    Href = orc.hessian(_np(X))
    Hg = _np(H).astype(np.float64)
    assert np.array_equal(Hg, Hg.T)
    rel = np.linalg.norm(Hg - Href) / np.linalg.norm(Href)
    assert rel < 2e-6, rel
    assert np.allclose(Hg, Href, rtol=0, atol=3e-6 * np.abs(Href).max())
    # undamped, then accumulated in two batches
    H0 = obc.obc_hessian(X, damp_rel=-1.0)
    h = N // 2
    Hacc = obc.obc_hessian(Xfull[:, :h], damp_rel=-1.0)
    Hacc = obc.obc_hessian(Xfull[:, h:N], damp_rel=-1.0, H=Hacc, accumulate=True)
    ref0 = orc.hessian(_np(X), damp_rel=-1)
    assert np.linalg.norm(_np(H0) - ref0) / np.linalg.norm(ref0) < 2e-6
    assert np.linalg.norm(_np(Hacc) - ref0) / np.linalg.norm(ref0) < 2e-6


@pytest.mark.parametrize("d", [1, 5, 24, 31, 32, 33, 100])
def test_hessian_dampening_with_the_last_batch(obc, d):
    """Up to 32 columns the launch that sums the slices dampens too, above a launch of its own: lambda is the stated
    share of the mean diagonal, formed in fp64 and rounded, added with one rounding; nothing else changes, in one batch
    and with the last of two."""
    gen = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn(d, 300, generator=gen, device="cuda") + 0.5
    A, B = X[:, :130].contiguous(), X[:, 130:].contiguous()

    def two(damp):
        H = obc.obc_hessian(A, damp_rel=-1.0)
        return obc.obc_hessian(B, damp_rel=damp, H=H, accumulate=True)

    for solve in (lambda damp: obc.obc_hessian(X, damp_rel=damp), two):
        plain, damped = solve(-1.0).cpu(), solve(0.01).cpu()
        h = plain.diagonal().double()
        lam = float(np.float32(0.01)) * h.mean()
        err = (damped.diagonal().double() - (h + lam)).abs()
        assert bool((err <= 2.0 ** -24 * (h + lam) + 1.01 * 2.0 ** -24 * lam).all()), float(err.max())
        off = ~torch.eye(d, dtype=torch.bool)
        assert torch.equal(damped[off], plain[off])


@pytest.mark.parametrize("d,N,off,pad", [(1, 1, 0, 0), (5, 15, 1, 1), (127, 16, 0, 1), (128, 17, 2, 2), (129, 33, 3, 0),
                                         (256, 64, 0, 3), (1153, 1000, 1, 0), (2049, 49, 0, 1)])
def test_second_moments_at_tile_edges(obc, d, N, off, pad):
    """Edges of the 128 / 256 tiles and of the 16-sample slabs, rows at any float's address; values
    over many binades, so that every one of the split's terms counts.  Both sums of N products
    (obc_cross shares the kernel).  Bound: a product loses at most 3 * 2^-24 to the split, a sum of
    N / 16 slabs half a unit per slab, everything relative to the sum of the magnitudes."""
    gen = torch.Generator(device="cuda").manual_seed(d + N)
    buf = torch.randn(d * (N + pad) + off, generator=gen, device="cuda")
    buf *= torch.exp2(torch.randint(-12, 13, buf.shape, generator=gen, device="cuda").float())
    X = buf[off:].view(d, N + pad)[:, :N]
    r = min(d, 130)
    Y = torch.randn(r, N + pad, generator=gen, device="cuda")[:, :N]
    H, C = obc.obc_hessian(X, damp_rel=-1.0), obc.obc_cross(X, Y)
    assert torch.equal(H, H.T)
    eps = 3 * 2.0 ** -24 + 2.0 ** -24 * (N / 16 + 8)
    Xd, Yd = X.cpu().double(), Y.cpu().double()
    for got, a in ((H, Xd), (C, Yd)):
        err = (got.cpu().double() - 2 * a @ Xd.T).abs()
        assert bool((err <= eps * 2 * (a.abs() @ Xd.abs().T)).all()), float(err.max())


def test_second_moments_of_values_beyond_the_split(obc):
    """Infinities, NaN and values that round to infinity in bf16 come out as fp32 arithmetic has them."""
    X = torch.rand(140, 40, device="cuda") + 0.5
    X[3, 7] = float("inf")
    X[9, 0], X[9, 5] = float("inf"), float("-inf")
    X[70, 39] = float("nan")
    X[135, 11] = 3.4e38
    X[:, 11][:130] *= 1e-38
    H, C = obc.obc_hessian(X, damp_rel=-1.0), obc.obc_cross(X, X[:20].contiguous())
    ref = (2 * X.cpu().double() @ X.cpu().double().T)
    ref = torch.where(ref.abs() > 3.4028234e38, ref.sign() * float("inf"), ref)
    for got, want in ((H.cpu().double(), ref), (C.cpu().double(), ref[:20])):
        assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
        ok = want.isfinite()
        assert torch.allclose(got[ok], want[ok], rtol=1e-5)
        assert torch.equal(got[want.isinf()] > 0, want[want.isinf()] > 0)


@pytest.mark.parametrize("e", [-100, -109, -112, -118, -126, -135, -142])
def test_second_moments_of_values_below_the_split(obc, e):
    """Values whose third bf16 plane would fall under the smallest bf16, alone in their rows or met by a
    partner that is zero everywhere else: fp32 arithmetic holds them.  Bound: half a unit per fp32 addition,
    N of them, relative to the sum of the magnitudes, and half of the smallest fp32 each where they underflow."""
    gen = torch.Generator(device="cuda").manual_seed(-e)
    N = 333
    X = torch.randn(150, N, generator=gen, device="cuda")
    Y = torch.randn(40, N, generator=gen, device="cuda")
    Y[:30] = (Y[:30].double() * 2.0 ** e).float()
    Y[30:, 200] = (Y[30:, 200].double() * 2.0 ** e).float()
    X[140:] = 0.0
    X[140:, 200] = 1.0
    Z = torch.cat([Y, X])
    Z[:30, :5] *= 2.0 ** 60
    Xd, Yd, Zd = (t.cpu().double() for t in (X, Y, Z))
    H, C = obc.obc_hessian(Z, damp_rel=-1.0), obc.obc_cross(X, Y)
    assert torch.equal(H, H.T)
    for got, a, b in ((C, Yd, Xd), (H, Zd, Zd)):
        err = (got.cpu().double() - 2 * a @ b.T).abs()
        bound = 2.0 ** -24 * N * 2 * (a.abs() @ b.abs().T) + 2.0 ** -150 * 2 * N
        assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("N", [1, 2])
def test_second_moments_of_one_or_two_samples(obc, N):
    """One fp32 rounding per product: N half units relative to the sum of the magnitudes."""
    gen = torch.Generator(device="cuda").manual_seed(N)
    X, Y = torch.randn(700, N, generator=gen, device="cuda"), torch.randn(90, N, generator=gen, device="cuda")
    H, C = obc.obc_hessian(X, damp_rel=-1.0), obc.obc_cross(X, Y)
    Xd, Yd = X.cpu().double(), Y.cpu().double()
    for got, a in ((H, Xd), (C, Yd)):
        err = (got.cpu().double() - 2 * a @ Xd.T).abs()
        assert bool((err <= N * 2.0 ** -24 * 2 * (a.abs() @ Xd.abs().T)).all())


def test_hessian_on_correlated_relu_inputs(obc, orc):
    W, X = _layer("conv64x576", n_samples=10000)
    H = obc.obc_hessian(X)
    Href = orc.hessian(_np(X))
    assert np.linalg.norm(_np(H) - Href) / np.linalg.norm(Href) < 2e-6


# ------------------------------------------------------------------------------ inverse
@pytest.mark.parametrize("d", [1, 32, 100, 257, 576])
def test_invert_matches_oracle(obc, orc, d):
    W, X = _layer("conv64x576", d_col=d, d_row=2, n_samples=4 * d + 50)
    H = obc.obc_hessian(X)
    H64 = _np(H).astype(np.float64)
    A = _np(obc.obc_invert(H.clone())).astype(np.float64)
    assert np.array_equal(A, A.T)
    Aref = orc.invert(H64)
    assert np.linalg.norm(A - Aref) / np.linalg.norm(Aref) < 3e-7
    assert np.linalg.norm(A @ H64 - np.eye(d)) / np.sqrt(d) < 1e-4


@pytest.mark.parametrize("d", [2, 15, 16, 17, 31, 33, 47, 48, 49, 63, 64, 65, 79, 81, 112, 113, 127, 129])
def test_invert_at_sub_block_edges(obc, d):
    """Last blocks of every number of 16-column sub-blocks, with and without padding.  A fp64 inverse rounded to fp32
    is off by half a unit, 6e-8 of an entry; the condition number, about 10, leaves the fp64 part of it below that."""
    gen = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn(d, 10 * d + 50, generator=gen, device="cuda")
    H = obc.obc_hessian(X)
    ref = torch.linalg.inv(H.double().cpu())
    A = obc.obc_invert(H)
    assert torch.equal(A, A.T)
    assert float((A.double().cpu() - ref).norm() / ref.norm()) < 1e-7


def test_invert_reports_non_spd(obc):
    import paper_2208_11580_amd as pkg

    H = torch.eye(70, device="cuda")
    H[65, 65] = -1.0
    with pytest.raises(pkg.ObcError) as e:
        obc.obc_invert(H)
    assert e.value.code == pkg.OBC_ERR_NOT_SPD
    obc.obc_check()  # latch is cleared


# ------------------------------------------------------------------------------ sequential re-fit
@pytest.mark.parametrize("d_col,d_row,N,pad", [(32, 16, 256, 0), (200, 77, 3001, 3), (131, 300, 777, 1),
                                               (576, 64, 20000, 0)])
def test_cross_matches_oracle(obc, orc, d_col, d_row, N, pad):
    torch.manual_seed(d_col + d_row)
    Xf = torch.randn(d_col, N + pad, device="cuda")
    Yf = torch.randn(d_row, N + 2 * pad, device="cuda") + 0.3 * Xf[:1, :N].mean()
    X, Y = Xf[:, :N], Yf[:, :N]
    C = obc.obc_cross(X, Y)
    ref = orc.cross(_np(X), _np(Y))
    assert C.shape == (d_row, d_col)
    assert np.linalg.norm(_np(C) - ref) / np.linalg.norm(ref) < 2e-6
    assert np.allclose(_np(C), ref, rtol=0, atol=3e-6 * np.abs(ref).max())
    # accumulated in two batches
    h = N // 2
    Cacc = obc.obc_cross(Xf[:, :h], Yf[:, :h])
    Cacc = obc.obc_cross(Xf[:, h:N], Yf[:, h:N], C=Cacc, accumulate=True)
    assert np.linalg.norm(_np(Cacc) - ref) / np.linalg.norm(ref) < 2e-6


@pytest.mark.parametrize("d_col,d_row", [(32, 16), (203, 70), (576, 64), (257, 1)])
def test_refit_matches_oracle(obc, orc, d_col, d_row):
    # appendix "Sequential Quantization with OBQ": inputs of the compressed model (here the dense
    # inputs plus a perturbation), outputs of the dense layer
    W, X = _layer("conv64x576", d_col=d_col, d_row=d_row, n_samples=4 * d_col + 50)
    torch.manual_seed(3)
    Xc = (X + 0.1 * X.std() * torch.randn_like(X)).contiguous()
    Y = (W.double() @ X.double()).float()
    H = obc.obc_hessian(Xc)
    C = obc.obc_cross(Xc, Y)
    H0 = H.clone()
    Wr = obc.obc_refit(H, C)
    assert torch.equal(H, H0)                     # H is left alone
    ref = orc.refit(_np(H).astype(np.float64), _np(C).astype(np.float64))
    err = np.linalg.norm(_np(Wr) - ref) / np.linalg.norm(ref)
    assert err < 1e-6, err
    # sharing the factorisation: same weights, and H becomes what obc_invert gives
    Wr2 = obc.obc_refit(H, C, invert_in_place=True)
    assert torch.equal(Wr, Wr2)
    assert torch.equal(H, obc.obc_invert(H0.clone()))
    # the re-fitted weights have (up to the fp32 rounding of H, C and W) zero gradient under the
    # new inputs, the gradient being written out from the data in fp64
    Wn, Xn, Yn = _np(Wr).astype(np.float64), _np(Xc).astype(np.float64), _np(Y).astype(np.float64)
    lam = 0.01 * np.mean(2.0 * np.sum(Xn * Xn, axis=1))
    grad = 2.0 * (Wn @ Xn - Yn) @ Xn.T + lam * Wn
    scale = np.linalg.norm(2.0 * Yn @ Xn.T)
    assert np.linalg.norm(grad) < 5e-4 * scale


def test_sequential_obq_flow(obc, orc):
    # re-fit, then OBQ on the re-fitted weights with the same Hessian, as the appendix describes;
    # each stage is compared with the oracle fed the GPU's previous stage
    W, X = _layer("conv64x576", d_col=260, d_row=6, n_samples=3000)
    torch.manual_seed(4)
    Xc = (X + 0.2 * X.std() * torch.randn_like(X)).contiguous()
    Y = (W.double() @ X.double()).float()
    H = obc.obc_hessian(Xc)
    C = obc.obc_cross(Xc, Y)
    Wr = obc.obc_refit(H, C, invert_in_place=True)      # H now holds the inverse
    _check_quant(obc, orc, Wr, H, 3, 0)


# ------------------------------------------------------------------------------ pruning rows
def _check_prune(obc, orc, W, Hinv, k_steps, nm, strategy, rows=None, want_trace=False):
    res = obc.obc_prune_rows(W, Hinv, k_steps=k_steps, nm=nm, strategy=strategy, want_trace=want_trace)
    obc.obc_check()
    A = _np(Hinv)
    Wn = _np(W)
    st = RowParity()
    order, loss, Wo = _np(res["order"]), _np(res["loss"]), _np(res["W"])
    tr = _np(res["trace"]) if want_trace else None
    for i in (range(W.shape[0]) if rows is None else rows):
        check_row(orc, st, "prune", A, Wn[i], order[i], loss[i], Wo[i], order.shape[1], nm=nm,
                  g_trace=None if tr is None else tr[i])
    print(st)
    st.assert_order_rule()
    return res, st


@pytest.mark.parametrize("strategy", [1, 2])
def test_prune_rows_tiny_layer_full_trace(obc, orc, strategy):
    W, X = _layer("lin16x32")
    Hinv = _hinv(obc, X)
    _check_prune(obc, orc, W, Hinv, 32, (0, 0), strategy, want_trace=True)


@pytest.mark.parametrize("strategy", [1, 2])
@pytest.mark.parametrize("d,R,k", [(203, 5, 203), (320, 6, 320), (576, 4, 576), (1100, 3, 300)])
def test_prune_rows_streamed_sizes(obc, orc, strategy, d, R, k):
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=3 * d)
    Hinv = _hinv(obc, X)
    _check_prune(obc, orc, W, Hinv, k, (0, 0), strategy, want_trace=(d <= 320))


@pytest.mark.parametrize("d", [1, 4, 63, 64, 65, 128, 129, 190, 193])
def test_small_widths_take_the_blocked_solver(obc, orc, d):
    """Rows of one panel (up to 64 columns, no workspace), and widths that also fit the rank-1 solver's
    LDS: pruning with its trace, stop counts, OBQ dense and on survivors, blocks of four."""
    W, X = _layer("conv64x576", d_col=d, d_row=5, n_samples=max(200, 4 * d))
    Hinv = _hinv(obc, X)
    full, _ = _check_prune(obc, orc, W, Hinv, d, (0, 0), 0, want_trace=True)
    stop = torch.tensor([0, 1, d // 2, d, d + 3], dtype=torch.int32, device="cuda")
    cut = obc.obc_prune_rows(W, Hinv, stop_counts=stop, want_trace=True)
    for i, n in enumerate(stop.clamp(max=d).tolist()):
        assert torch.equal(cut["order"][i, :n], full["order"][i, :n]) and bool((cut["order"][i, n:] == -1).all())
        assert torch.equal(cut["trace"][i, :n], full["trace"][i, :n]) and not bool(cut["trace"][i, n:].any())
        assert torch.equal(cut["W"][i], full["trace"][i, n - 1] if n else W[i])
    _check_quant(obc, orc, W, Hinv, 4, 0)
    live = (torch.arange(5 * d, device="cuda").view(5, d) % 3 != 0).to(torch.uint8)
    live[4] = 0
    q, _ = _check_quant(obc, orc, W, Hinv, 3, 0, live=live, rows=range(4) if d > 1 else [])
    assert bool((q["codes"][live == 0] == -1).all()) and not bool(q["W"][live == 0].any())
    if d % 4 == 0:
        _check_blocks(obc, orc, W, Hinv, 4, d // 4, 0, want_trace=True)


def test_small_widths_without_a_workspace(obc, orc):
    """A call that brings less than the blocked solver's workspace is served by the rank-1 solver."""
    import paper_2208_11580_amd as pkg
    W, X = _layer("conv64x576", d_col=150, d_row=4, n_samples=800)
    Hinv = _hinv(obc, X)
    ctx = pkg.Context()
    ctx.rows_workspace_bytes = lambda *a: 256
    a, b = ctx.obc_prune_rows(W, Hinv), obc.obc_prune_rows(W, Hinv, strategy=pkg.STRATEGY_RANK1)
    assert all(torch.equal(a[k], b[k]) for k in ("order", "loss", "W"))
    with pytest.raises(pkg.ObcError):
        ctx.obc_prune_rows(W, Hinv, strategy=pkg.STRATEGY_BLOCKED)
    ctx.close()


@pytest.mark.parametrize("run", [1, 2, 3, 5, 8, 9, 13, 64])
def test_flush_closes_up_runs_of_eliminated_rows(obc, orc, run):
    """The flush takes a tile's rows from whole groups of four rows of the old matrix and closes them up.  Zero weights
    are pruned first, in index order: the first panel's 64 at the row's start, the second's in runs of `run` that begin
    at every residue of 4 (a row's place moves them), up to more than a tile's rows can reach over."""
    d, R = 602, 4
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=4 * d)
    Hinv = _hinv(obc, X)
    for r in range(R):
        W[r, :64] = 0.0
        left, at = 64, 70 + r
        while left:
            n = min(run, left)
            W[r, at:at + n] = 0.0
            left, at = left - n, at + n + 7 - n % 2
    _check_prune(obc, orc, W, Hinv, 330, (0, 0), 2)


@pytest.mark.parametrize("left", [31, 32, 33, 63, 65, 127, 129, 383, 384, 385, 447, 513])
def test_flush_at_tile_edges(obc, orc, left):
    """`left` live columns after two flushes of 64: ends of the tiles of 32 x 64, of the strips of 128 rows, and the
    live size from which whole groups of rows are read (384)."""
    d = left + 128
    W, X = _layer("conv64x576", d_col=d, d_row=3, n_samples=4 * d)
    _check_prune(obc, orc, W, _hinv(obc, X), d, (0, 0), 2)


@pytest.mark.parametrize("mode,d,R,few,k", [
    ("prune", 2096, 128, 2, 100), ("prune", 2097, 128, 2, 100), ("quant", 2225, 110, 2, 2225), ("prune", 2303, 100, 2, 100),
    ("blocks", 2304, 100, 2, 100), ("prune", 1999, 140, 2, 120), ("prune", 1283, 360, 2, 150), ("prune", 1000, 600, 2, 130),
    ("prune", 768, 1024, 768, 100), ("prune", 512, 3072, 768, 200), ("prune", 2801, 96, 2, 170), ("blocks", 2904, 64, 2, 100),
    ("prune", 4000, 40, 2, 180), ("blocks", 3996, 40, 2, 180), ("prune", 4608, 96, 2, 200), ("prune", 4600, 64, 2, 150),
    ("prune", 4601, 25, 2, 100), ("dead", 2304, 101, 2, 40)])
def test_first_flush_by_strips_and_by_tiles(obc, orc, mode, d, R, few, k):
    """Five hundred million entries in all rows' matrices send the first flush to strips of 128 or 256 rows; the same rows
    in a smaller call go by tiles, bit for bit the same.  Every number of vectors and of panels that share the flush,
    ends at, before and behind the strips' and their tiles' edges, then past a second flush; one row against the oracle."""
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=d + 500)
    Hinv = _hinv(obc, X)
    gen = torch.Generator(device="cuda").manual_seed(d)
    live = torch.ones(R, d, dtype=torch.uint8, device="cuda")
    if mode == "dead":                       # one bulk elimination of 64 in every row, and 6 one by one
        live.scatter_(1, torch.rand(R, d, generator=gen, device="cuda").topk(70, dim=1).indices, 0)

    def solve(n):
        w = W[:n].contiguous()
        if mode == "blocks":
            r = obc.obc_prune_blocks(w, Hinv, 4, k_blocks=k // 4)
            return r["order"], r["loss"], r["W"]
        if mode == "quant":
            delta, offset, maxq = obc.obc_minmax_grid(w, 4)
            r = obc.obc_quant_rows(w, Hinv, delta, offset, maxq)
            return r["order"], r["loss"], r["W"], r["codes"]
        r = obc.obc_prune_rows(w, Hinv, k_steps=k, live=live[:n].contiguous() if mode == "dead" else None)
        return r["order"], r["loss"], r["W"]

    many, less = solve(R), solve(few)
    for a, b in zip(many, less):
        assert torch.equal(a[:few], b)
    if mode == "prune":
        st = RowParity()
        check_row(orc, st, "prune", _np(Hinv), _np(W[R - 1]), _np(many[0][R - 1]), _np(many[1][R - 1]), _np(many[2][R - 1]), k)
        st.assert_order_rule()


@pytest.mark.parametrize("d,k,R", [(2305, 90, 2), (2344, 100, 2), (3073, 100, 2), (3200, 130, 2), (4097, 60, 2), (4608, 130, 2),
                                   (2900, 130, 96), (3073, 130, 96), (4097, 60, 96), (4608, 130, 3), (4608, 130, 64),
                                   (4608, 130, 96)])
def test_panels_that_share_a_flush(obc, orc, d, k, R):
    """Widths above 2304: a flush after each panel or after several, as width and rows have it (24 steps a panel: none
    shared with two rows, two with 3, three with 64, four with 96; 28: three; 40: two with 96), the group cut short
    where the live size changes the variant, the last step inside a group."""
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=2 * d)
    _check_prune(obc, orc, W, _hinv(obc, X), k, (0, 0), 2, rows=[1])


def test_panel_account_counts_the_vectors_read_again(obc):
    """Three panels of 28 steps that share a flush: a step reads a matrix row and every vector since the last
    flush, 4 bytes per column each."""
    W, X = _layer("conv64x576", d_col=3200, d_row=2, n_samples=6400)
    Hinv = _hinv(obc, X)
    obc.obc_profile_begin()
    obc.obc_prune_rows(W, Hinv, k_steps=84, strategy=2)
    stat = obc.obc_profile_end()["panel"]
    assert stat["launches"] == 3 and stat["bytes"] == 2 * 28 * 4 * 3200 * (1 + (1 + 28) + (1 + 56))


@pytest.mark.parametrize("d,k,R", [(3200, 130, 2), (4200, 150, 2), (4200, 150, 96)])
def test_wide_quantization_and_n_m_first_steps(obc, orc, d, k, R):
    """OBQ and the N:M rule on panels that share a flush, past one group of three (28 steps a panel, any rows) or
    four (24 steps, 96 rows), and on panels of 24 that do not (two rows): the first steps of a row against the
    oracle (OBQ follows the GPU's order; a pick may be above the least score by no more than fp32 storage explains)."""
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=2 * d)
    Hinv = _hinv(obc, X)
    _check_prune(obc, orc, W, Hinv, k, (2, 4), 2, rows=[1])
    delta, offset, maxq = obc.obc_minmax_grid(W, 4)
    res = obc.obc_quant_rows(W, Hinv, delta, offset, maxq)
    obc.obc_check()
    order, loss, codes = _np(res["order"][1]), _np(res["loss"][1])[:k], _np(res["codes"][1])
    ref = orc.quant_row(_np(Hinv).astype(np.float64), _np(W[1]).astype(np.float64),
                        (float(delta[1]), float(offset[1]), maxq), k_steps=k, forced=order[:k].astype(np.int32))
    gap = np.abs(ref.pick_score - ref.min_score)
    assert np.all(gap <= FP32_ORDER_GAP * ref.min_score + 1e-12 * ref.min_score.max())
    assert abs(loss.sum() - ref.loss.sum()) <= 1e-3 * ref.loss.sum()
    assert np.array_equal(codes[order[:k]], ref.codes[order[:k]])
    assert sorted(order.tolist()) == list(range(d))


@pytest.mark.parametrize("mode", ["prune", "n_m", "quant"])
def test_shared_flushes_leave_no_trace(obc, mode):
    """From 96 rows on two panels of 2416 .. 2815 columns share a flush, with fewer each has its own: the
    results are the same bit for bit."""
    W, X = _layer("conv64x576", d_col=2600, d_row=96, n_samples=6000)
    Hinv = _hinv(obc, X)

    def solve(rows):
        if mode == "quant":
            delta, offset, maxq = obc.obc_minmax_grid(rows, 4)
            r = obc.obc_quant_rows(rows, Hinv, delta, offset, maxq)
            return r["order"], r["loss"], r["W"], r["codes"]
        r = obc.obc_prune_rows(rows, Hinv, k_steps=300, nm=(2, 4) if mode == "n_m" else (0, 0))
        return r["order"], r["loss"], r["W"]

    for many, few in zip(solve(W), solve(W[:8].contiguous())):
        assert torch.equal(many[:8], few)


@pytest.mark.parametrize("mode", ["prune", "n_m", "quant", "blocks"])
@pytest.mark.parametrize("d,R", [(2900, 96), (4200, 96), (4200, 64), (4200, 3)])
def test_the_panels_that_share_a_flush_follow_the_rows(obc, d, R, mode):
    """How many panels of 24 or 40 steps share a flush (four, three, two, none) depends on the rows; a row's results
    do not.  Past a whole group and the change to panels of 28 steps."""
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=d + 500)
    Hinv = _hinv(obc, X)

    def solve(rows):
        if mode == "quant":
            delta, offset, maxq = obc.obc_minmax_grid(rows, 4)
            r = obc.obc_quant_rows(rows, Hinv, delta, offset, maxq, strategy=2)
        elif mode == "blocks":
            r = obc.obc_prune_blocks(rows, Hinv, 4, k_blocks=38)
        else:
            r = obc.obc_prune_rows(rows, Hinv, k_steps=150, nm=(2, 4) if mode == "n_m" else (0, 0), strategy=2)
        return [r[name] for name in ("order", "loss", "W", "codes") if r.get(name) is not None]

    many, few = solve(W), solve(W[:2].contiguous())
    assert len(many) == (4 if mode == "quant" else 3)
    for a, b in zip(many, few):
        assert torch.equal(a[:2], b)


@pytest.mark.parametrize("strategy", [1, 2])
@pytest.mark.parametrize("nm", [(2, 4), (4, 8)])
def test_prune_rows_n_m(obc, orc, strategy, nm):
    d = 264
    W, X = _layer("conv64x576", d_col=d, d_row=4, n_samples=2000)
    Hinv = _hinv(obc, X)
    k = d // nm[1] * (nm[1] - nm[0])
    res, _ = _check_prune(obc, orc, W, Hinv, k, nm, strategy)
    zeros = (_np(res["W"]) == 0).reshape(4, -1, nm[1]).sum(axis=2)
    assert np.all(zeros == nm[1] - nm[0])


@pytest.mark.parametrize("d,nm", [(32, (2, 4)), (64, (3, 8)), (64, (10, 64)), (240, (20, 60)), (250, (50, 250)),
                                  (264, (2, 4)), (765, (100, 255)), (1275, (215, 255)), (2310, (225, 231)),
                                  (4590, (251, 255))])
def test_n_m_counts_and_trace(obc, orc, d, nm):
    """N:M in rows of one panel (which load no counters) and of several, whose counts travel from panel to
    panel; M up to the largest.  The trace is written at the indices that the counts share a word with."""
    W, X = _layer("conv64x576", d_col=d, d_row=3, n_samples=4 * d)
    Hinv = _hinv(obc, X)
    k = d // nm[1] * (nm[1] - nm[0])
    res, _ = _check_prune(obc, orc, W, Hinv, k, nm, 2, want_trace=True)
    zeros = (res["W"] == 0).reshape(3, d // nm[1], nm[1]).sum(dim=2)
    assert bool((zeros == nm[1] - nm[0]).all())


@pytest.mark.parametrize("strategy", [1, 2])
def test_prune_rows_zero_weights_and_ties(obc, orc, strategy):
    d = 96
    W, X = _layer("conv64x576", d_col=d, d_row=3, n_samples=1000)
    W[0, 5] = 0.0
    W[0, 50] = 0.0
    W[1, :] = 0.0
    Hinv = _hinv(obc, X)
    res, _ = _check_prune(obc, orc, W, Hinv, d, (0, 0), strategy)
    assert _np(res["order"])[0, :2].tolist() == [5, 50]
    assert _np(res["order"])[1].tolist() == list(range(d))  # all scores equal: index order


@pytest.mark.parametrize("R,d", [(768, 320), (768, 600), (2, 1100), (2, 1700), (2, 2200), (2, 2500), (96, 2500),
                                 (2, 3400), (2, 4400), (96, 4400)])
def test_ties_among_several_owned_indices(obc, R, d):
    """Exact ties go to the least index, also where a thread owns several: of a wave's candidates the least
    may sit on a higher lane than another one, of the waves' candidates in a later wave.  Every variant with
    more than one index a thread, with panels that share a flush among them."""
    k, kz = 136, 40
    gen = torch.Generator(device="cuda").manual_seed(d)
    Hinv = _hinv(obc, torch.randn(d, 2 * d, generator=gen, device="cuda"))
    W = torch.randn(R, d, generator=gen, device="cuda")
    W[0] = 0.0
    zero = torch.sort(torch.randperm(d, generator=gen, device="cuda")[:kz]).values
    W[1, zero] = 0.0
    first = torch.arange(k, device="cuda", dtype=torch.int32)
    res = obc.obc_prune_rows(W, Hinv, k_steps=k, strategy=2)
    assert torch.equal(res["order"][0], first)
    assert torch.equal(res["order"][1, :kz], zero.to(torch.int32))
    assert not res["W"][0].any() and not res["loss"][0].any() and not res["loss"][1, :kz].any()
    # weights that lie on the grid: no error, nothing changes
    codes = torch.randint(0, 16, (R, d), generator=gen, device="cuda")
    Wq = (codes - 8).float() * 0.125
    q = obc.obc_quant_rows(Wq, Hinv, torch.full((R,), 0.125, device="cuda"), torch.full((R,), -1.0, device="cuda"), 15,
                           strategy=2)
    assert torch.equal(q["order"], torch.arange(d, device="cuda", dtype=torch.int32).expand(R, d))
    assert torch.equal(q["codes"], codes.to(torch.int32)) and torch.equal(q["W"], Wq)
    b = obc.obc_prune_blocks(W, Hinv, 4, k_blocks=k // 4, strategy=2)
    assert torch.equal(b["order"][0], first[:k // 4])
    obc.obc_check()


@pytest.mark.parametrize("strategy", [1, 2])
def test_prune_rows_is_deterministic(obc, strategy):
    W, X = _layer("conv64x576", d_col=300, d_row=8, n_samples=2000)
    Hinv = _hinv(obc, X)
    a = obc.obc_prune_rows(W, Hinv, strategy=strategy)
    b = obc.obc_prune_rows(W, Hinv, strategy=strategy)
    torch.cuda.synchronize()
    for key in ("order", "loss", "W"):
        assert torch.equal(a[key], b[key])


def test_strategies_agree_on_order(obc):
    W, X = _layer("conv64x576", d_col=448, d_row=6, n_samples=3000)
    Hinv = _hinv(obc, X)
    a = obc.obc_prune_rows(W, Hinv, strategy=1)
    b = obc.obc_prune_rows(W, Hinv, strategy=2)
    assert (a["order"] != b["order"]).float().mean().item() < 0.01
    assert torch.allclose(a["loss"], b["loss"], rtol=1e-3, atol=1e-9)


# ------------------------------------------------------------------------------ block pruning
def _check_blocks(obc, orc, W, Hinv, c, k_blocks, strategy, want_trace=False):
    res = obc.obc_prune_blocks(W, Hinv, c, k_blocks=k_blocks, want_trace=want_trace, strategy=strategy)
    obc.obc_check()
    A, Wn = _np(Hinv), _np(W)
    order, loss, Wo = _np(res["order"]), _np(res["loss"]), _np(res["W"])
    swaps = 0
    for i in range(W.shape[0]):
        swaps += check_block_row(orc, A, Wn[i], c, order[i], loss[i], Wo[i], k_blocks,
                                 g_trace=_np(res["trace"])[i] if want_trace else None)
    return res, swaps


@pytest.mark.parametrize("strategy,d,R,c,kb", [
    (1, 32, 16, 4, 8), (1, 32, 16, 2, 16), (1, 200, 4, 8, 20), (1, 576, 4, 4, 100), (1, 260, 3, 4, 65),
    (1, 126, 3, 3, 42),
    (2, 32, 16, 4, 8), (2, 200, 4, 4, 50), (2, 576, 4, 4, 100), (2, 260, 3, 4, 65), (2, 576, 3, 4, 144),
    (2, 768, 2, 4, 192)])
def test_prune_blocks_matches_oracle(obc, orc, strategy, d, R, c, kb):
    name = "lin16x32" if d == 32 else ("attn768x768" if d == 768 else "conv64x576")
    W, X = _layer(name, d_col=d, d_row=R, n_samples=max(256, 3 * d))
    Hinv = _hinv(obc, X)
    _check_blocks(obc, orc, W, Hinv, c, kb, strategy, want_trace=(d <= 200))


def test_block_strategies_agree(obc):
    W, X = _layer("conv64x576", d_col=576, d_row=8, n_samples=3000)
    Hinv = _hinv(obc, X)
    a = obc.obc_prune_blocks(W, Hinv, 4, strategy=1)
    b = obc.obc_prune_blocks(W, Hinv, 4, strategy=2)
    obc.obc_check()
    same = (a["order"] == b["order"]).float().mean().item()
    assert same > 0.98, same
    assert torch.allclose(a["loss"].sum(dim=1), b["loss"].sum(dim=1), rtol=1e-4)
    import paper_2208_11580_amd as pkg
    with pytest.raises(pkg.ObcError):
        obc.obc_prune_blocks(W, Hinv, 2, strategy=2)     # the deferred-update solver does blocks of 4


@pytest.mark.parametrize("strategy", [1])
def test_prune_blocks_of_one_is_prune_rows(obc, strategy):
    W, X = _layer("conv64x576", d_col=260, d_row=4, n_samples=2000)
    Hinv = _hinv(obc, X)
    a = obc.obc_prune_rows(W, Hinv, k_steps=100, strategy=strategy)
    b = obc.obc_prune_blocks(W, Hinv, 1, k_blocks=100, strategy=strategy)
    obc.obc_check()
    assert torch.equal(a["order"], b["order"])
    assert torch.allclose(a["loss"], b["loss"], rtol=1e-6, atol=0)
    assert torch.allclose(a["W"], b["W"], rtol=1e-6, atol=1e-9)


@pytest.mark.parametrize("d", [128, 320])
def test_block_traces_feed_the_global_step(obc, orc, d):
    # Alg. 2 on the block loss traces, then the weights of the chosen per-row block counts both by
    # replay (stop_counts) and from the stored trace (d = 128: LDS-resident solver, 320: deferred)
    W, X = _layer("conv64x576", d_col=d, d_row=12, n_samples=1000)
    Hinv = _hinv(obc, X)
    c = 4
    full = obc.obc_prune_blocks(W, Hinv, c, want_trace=True)
    k = (12 * (d // 4)) // 2
    counts, block_mask = obc.obc_global_select(full["loss"], full["order"], k)
    ref = orc.global_select(_np(full["loss"]).astype(np.float64), k)
    assert np.array_equal(_np(counts), ref)
    assert int(block_mask.sum()) == k
    replay = obc.obc_prune_blocks(W, Hinv, c, stop_counts=counts)
    gathered = obc.obc_gather_trace(W, full["trace"], counts)
    obc.obc_check()
    assert torch.equal(replay["W"], gathered)
    zeros = (gathered == 0).sum(dim=1)
    assert torch.equal(zeros.to(torch.int32), counts * c)


# ------------------------------------------------------------------------------ OBQ rows
def _check_quant(obc, orc, W, Hinv, bits, strategy, live=None, rows=None, grid=None, outliers=False):
    if grid is None:
        delta, offset, maxq = obc.obc_minmax_grid(W, bits, live=live)
    else:
        delta, offset, maxq = grid
    res = obc.obc_quant_rows(W, Hinv, delta, offset, maxq, live=live, strategy=strategy, outliers=outliers)
    obc.obc_check()
    A, Wn = _np(Hinv), _np(W)
    dl, of = _np(delta), _np(offset)
    lv = None if live is None else _np(live)
    st = RowParity()
    order, loss, Wo, codes = _np(res["order"]), _np(res["loss"]), _np(res["W"]), _np(res["codes"])
    for i in (range(W.shape[0]) if rows is None else rows):
        wl = Wn[i] if lv is None else Wn[i][lv[i] != 0]
        if grid is None:
            # the grid the GPU computed is the oracle's min-max grid of the same fp32 weights
            g = orc.minmax_grid(wl.astype(np.float64), bits)
            assert np.float32(g[1]) == of[i] and np.isclose(g[0], dl[i], rtol=1e-6)
        k = len(wl)
        check_row(orc, st, "quant", A, Wn[i], order[i], loss[i], Wo[i], k,
                  grid=(float(dl[i]), float(of[i]), maxq), g_codes=codes[i],
                  live=None if lv is None else lv[i], outlier=outliers)
    print(st)
    st.assert_order_rule()
    return res, st


@pytest.mark.parametrize("strategy", [1, 2])
@pytest.mark.parametrize("d,R,bits", [(32, 16, 4), (203, 4, 3), (576, 4, 4), (768, 3, 2)])
def test_quant_rows_matches_oracle(obc, orc, strategy, d, R, bits):
    name = "lin16x32" if d == 32 else ("attn768x768" if d == 768 else "conv64x576")
    W, X = _layer(name, d_col=d, d_row=R, n_samples=max(256, 3 * d))
    Hinv = _hinv(obc, X)
    _check_quant(obc, orc, W, Hinv, bits, strategy)


@pytest.mark.parametrize("strategy", [1, 2])
@pytest.mark.parametrize("d", [64, 320])
def test_quant_rows_at_rounding_boundaries(obc, orc, strategy, d):
    """Weights exactly on a half step of the grid, and one fp32 ulp to either side: the code written
    is the code the candidate was scored with (round half to even), and both equal the oracle's.
    The inverse Hessian is diagonal, so OBQ is plain rounding and every weight keeps its value
    until it is chosen."""
    delta, offset, maxq = 0.25, -1.0, 7          # the grid -1, -0.75, ..., 0.75; exact in fp32
    base = np.float32(offset) + np.float32(delta) * (np.arange(d, dtype=np.float32) % 7 + np.float32(0.5))
    rows = np.stack([base, np.nextafter(base, np.float32(-4), dtype=np.float32),
                     np.nextafter(base, np.float32(4), dtype=np.float32)]).astype(np.float32)
    rng = np.random.default_rng(5)
    diag = rng.uniform(0.5, 2.0, d).astype(np.float32)
    W = torch.tensor(rows, device="cuda")
    Hinv = torch.diag(torch.tensor(diag, device="cuda")).contiguous()
    dl = torch.full((3,), delta, device="cuda")
    of = torch.full((3,), offset, device="cuda")
    q = obc.obc_quant_rows(W, Hinv, dl, of, maxq, strategy=strategy)
    obc.obc_check()
    codes = _np(q["codes"])
    for i in range(3):
        want = np.array([orc.quant_code(float(rows[i, j]), delta, offset, maxq) for j in range(d)])
        assert np.array_equal(codes[i], want), (i, np.flatnonzero(codes[i] != want)[:5])
        ro = orc.quant_row(np.diag(diag.astype(np.float64)), rows[i].astype(np.float64), (delta, offset, maxq))
        assert np.array_equal(codes[i], ro.codes)
        # the recorded loss is the one of the written code
        step_of = np.empty(d, np.int64)
        step_of[_np(q["order"][i])] = np.arange(d)
        err = (offset + delta * codes[i].astype(np.float64)) - rows[i].astype(np.float64)
        assert np.allclose(_np(q["loss"][i])[step_of], err * err / (2.0 * diag.astype(np.float64)), rtol=1e-5, atol=1e-12)
    # exactly on the half step the even code wins: 0.5 -> 0, 1.5 -> 2, 2.5 -> 2, ...
    half = (np.arange(d) % 7) + 0.5
    assert np.array_equal(codes[0], np.minimum(np.round(half), maxq).astype(np.int32))
    deq = (of[:, None].double() + dl[:, None].double() * q["codes"].double()).float()
    assert torch.equal(q["W"], deq)


def _narrow_grid(W, bits, shrink):
    """A min-max grid shrunk about its centre: the weights beyond it start as outliers."""
    maxq = (1 << bits) - 1
    lo, hi = W.min(dim=1).values, W.max(dim=1).values
    mid, half = 0.5 * (lo + hi), 0.5 * (hi - lo) * shrink
    return (2.0 * half / maxq).contiguous(), (mid - half).contiguous(), maxq


@pytest.mark.parametrize("strategy", [1, 2])
@pytest.mark.parametrize("d,R,bits,shrink", [(32, 16, 3, 0.5), (203, 4, 3, 0.6), (576, 4, 4, 0.7), (768, 3, 2, 0.5)])
def test_quant_rows_outlier_heuristic_matches_oracle(obc, orc, strategy, d, R, bits, shrink):
    # Sec. 5, outlier heuristic: on a grid narrower than the weight range several weights start
    # beyond half a step from the grid, and compensation pushes more of them out on the way
    name = "lin16x32" if d == 32 else ("attn768x768" if d == 768 else "conv64x576")
    W, X = _layer(name, d_col=d, d_row=R, n_samples=max(256, 3 * d))
    Hinv = _hinv(obc, X)
    grid = _narrow_grid(W, bits, shrink)
    res, st = _check_quant(obc, orc, W, Hinv, bits, strategy, grid=grid, outliers=True)
    # the heuristic changed the outcome (else the case does not test it)
    plain = obc.obc_quant_rows(W, Hinv, *grid, strategy=strategy)
    assert not torch.equal(plain["order"], res["order"])


@pytest.mark.parametrize("strategy", [1, 2])
def test_outlier_heuristic_is_inactive_on_a_covering_grid(obc, strategy):
    # on the min-max grid no weight starts as an outlier; the flag only matters once compensation
    # has pushed a weight out, so with a very wide grid both runs are bit-identical
    W, X = _layer("conv64x576", d_col=260, d_row=4, n_samples=2000)
    Hinv = _hinv(obc, X)
    delta, offset, maxq = obc.obc_minmax_grid(W, 8)
    wide = (delta * 4, offset - delta * 4 * 384, 1023)
    a = obc.obc_quant_rows(W, Hinv, *wide, strategy=strategy)
    b = obc.obc_quant_rows(W, Hinv, *wide, strategy=strategy, outliers=True)
    for k in ("order", "loss", "codes", "W"):
        assert torch.equal(a[k], b[k])


def test_symmetric_grid_matches_oracle(obc, orc):
    W, _ = _layer("conv64x576", d_col=203, d_row=8, n_samples=256)
    W[3] = 0.0                       # empty range
    live = (torch.rand_like(W) > 0.3).to(torch.uint8)
    live[5] = 0                      # no live weight
    for lv in (None, live):
        delta, offset, maxq = obc.obc_minmax_grid(W, 4, live=lv, symmetric=True)
        Wn = _np(W)
        for i in range(W.shape[0]):
            wl = Wn[i] if lv is None else Wn[i][_np(lv)[i] != 0]
            if wl.size == 0:
                assert delta[i].item() == 1.0 and offset[i].item() == 0.0
                continue
            g = orc.symmetric_grid(wl.astype(np.float64), 4)
            assert np.float32(g[1]) == offset[i].item()
            assert np.isclose(g[0], delta[i].item(), rtol=1e-6)
            assert maxq == g[2]


@pytest.mark.parametrize("strategy", [1, 2])
def test_quant_with_single_point_grid_is_pruning(obc, strategy):
    # quant(.) == 0 turns OBQ into ExactOBS (Sec. 5): bit-identical on the GPU too
    W, X = _layer("conv64x576", d_col=260, d_row=4, n_samples=2000)
    Hinv = _hinv(obc, X)
    p = obc.obc_prune_rows(W, Hinv, strategy=strategy)
    delta = torch.ones(4, device="cuda")
    offset = torch.zeros(4, device="cuda")
    q = obc.obc_quant_rows(W, Hinv, delta, offset, 0, strategy=strategy)
    obc.obc_check()
    assert torch.equal(p["order"], q["order"])
    assert torch.equal(p["loss"], q["loss"])
    assert torch.equal(q["W"], torch.zeros_like(q["W"]))
    assert torch.all(q["codes"] == 0)


@pytest.mark.parametrize("strategy", [1, 2])
def test_quant_rows_on_survivors_of_2_4(obc, orc, strategy):
    d = 256
    W, X = _layer("conv64x576", d_col=d, d_row=4, n_samples=2000)
    Hinv = _hinv(obc, X)
    p = obc.obc_prune_rows(W, Hinv, nm=(2, 4), strategy=strategy)
    live = (p["W"] != 0).to(torch.uint8)
    _check_quant(obc, orc, p["W"], Hinv, 4, strategy, live=live)


# ------------------------------------------------------------------------------ global step
def _check_global(obc, orc, loss, order, k):
    counts, mask = obc.obc_global_select(loss, order, k)
    torch.cuda.synchronize()
    ref = orc.global_select(_np(loss).astype(np.float64), k)
    assert np.array_equal(_np(counts), ref)
    assert np.array_equal(_np(mask), orc.mask_from_counts(_np(order), ref, loss.shape[1]))
    return counts, mask


def test_global_select_matches_algorithm_2(obc, orc):
    W, X = _layer("lin16x32")
    Hinv = _hinv(obc, X)
    res = obc.obc_prune_rows(W, Hinv)
    for k in (0, 1, 100, 256, 511, 512):
        _check_global(obc, orc, res["loss"], res["order"], k)
    W, X = _layer("conv64x576", d_col=300, d_row=37, n_samples=2000)
    Hinv = _hinv(obc, X)
    res = obc.obc_prune_rows(W, Hinv)
    for k in (1, 37 * 300 // 2, int(0.6 * 37 * 300), 37 * 300 - 1):
        _check_global(obc, orc, res["loss"], res["order"], k)


@pytest.mark.parametrize("R,d", [(1, 1), (1, 65), (3, 7), (128, 128), (1024, 16), (1025, 15), (129, 128), (17, 1000)])
def test_global_select_sizes(obc, orc, R, d):
    """Both sides of the one-workgroup form (16384 keys, 1024 rows), ties and a NaN among the losses."""
    gen = torch.Generator(device="cuda").manual_seed(R * d)
    loss = torch.randint(0, 40, (R, d), generator=gen, device="cuda").float() / 8
    if d > 4:
        loss[R // 2, 4] = float("nan")
    order = torch.argsort(torch.rand(R, d, generator=gen, device="cuda"), dim=1).to(torch.int32)
    ref = torch.nan_to_num(loss, nan=float("inf"))
    for k in sorted({1, R * d // 3, R * d // 2 + 1, R * d} - {0}):
        counts, mask = obc.obc_global_select(loss, order, k)
        want = orc.global_select(_np(ref).astype(np.float64), k)
        assert np.array_equal(_np(counts), want), k
        assert np.array_equal(_np(mask), orc.mask_from_counts(_np(order), want, d))


def test_global_select_beyond_32_bit_sums(obc):
    """More than 2^32 weights, each bucket of the selection below that: the ranks need 64 bits, and the mask's
    memory, which held something else before, is cleared to its end."""
    R, d = 65537, 65536
    used = torch.full((R, d), 7, dtype=torch.uint8, device="cuda")
    loss = torch.ones(R, d, device="cuda")
    loss[:, d // 2:] = 2.0
    order = torch.arange(d, dtype=torch.int32, device="cuda").expand(R, d).contiguous()
    del used
    counts, mask = obc.obc_global_select(loss, order, R * d - 10)
    want = torch.full((R,), d, dtype=torch.int32, device="cuda")
    want[-1] = d - 10                       # ties go to the rows in index order
    assert torch.equal(counts, want)
    assert bool(mask[:-1].all()) and bool(mask[-1, :d - 10].all()) and not bool(mask[-1, d - 10:].any())
    del loss, order, counts, mask
    obc.release_workspace()
    torch.cuda.empty_cache()


def test_global_select_non_monotone_and_tied_traces(obc, orc):
    rng = np.random.default_rng(0)
    R, d = 1100, 24   # more rows than one scan chunk
    L = rng.integers(0, 6, size=(R, d)).astype(np.float32)   # many exact ties, non-monotone rows
    loss = torch.tensor(L, device="cuda")
    order = torch.stack([torch.randperm(d, device="cuda") for _ in range(R)]).to(torch.int32)
    for k in (1, 5, 1234, R * d // 2, R * d):
        _check_global(obc, orc, loss, order, k)


def test_end_to_end_tiny_layer(obc, orc):
    """configs[0]: 16 x 32, prune to 50 % with the global step; whole path GPU vs whole path oracle."""
    W, X = _layer("lin16x32")
    Hinv = _hinv(obc, X)
    res = obc.obc_prune_rows(W, Hinv, want_trace=True)
    k = obc_inputs.target_count(0.5, 16, 32)
    counts, mask = obc.obc_global_select(res["loss"], res["order"], k)
    What = obc.obc_gather_trace(W, res["trace"], counts)
    replay = obc.obc_prune_rows(W, Hinv, stop_counts=counts)
    obc.obc_check()
    assert torch.equal(replay["W"], What)
    Xn, Wn = _np(X), _np(W)
    Ao = orc.invert(orc.hessian(Xn))
    ro = orc.prune_rows(Ao, Wn.astype(np.float64))
    co = orc.global_select(ro["loss"], k)
    Wo = orc.reconstruct(Ao, Wn.astype(np.float64), co)
    assert np.array_equal(_np(counts), co)
    assert np.array_equal(_np(mask), orc.mask_from_counts(ro["order"], co, 32))
    e_gpu = orc.layer_error(Wn, _np(What), Xn)
    e_orc = orc.layer_error(Wn, Wo, Xn)
    assert abs(e_gpu - e_orc) <= 1e-3 * e_orc
    assert np.linalg.norm(_np(What) - Wo) <= 1e-4 * np.linalg.norm(Wo)


@pytest.mark.parametrize("strategy", [1, 2])
def test_prune_rows_on_an_already_sparse_matrix(obc, orc, strategy):
    """Sec. 4 "Implementation Details": an already sparse matrix is pruned further on the dense
    sub-problem of its non-zeros.  The oracle works on that sub-problem directly (inverse of the
    sub-Hessian); the GPU reaches it by eliminating the zeros from H^-1 first."""
    d, k1, k2 = 260, 100, 60
    W, X = _layer("conv64x576", d_col=d, d_row=4, n_samples=2000)
    Hinv = _hinv(obc, X)
    first = obc.obc_prune_rows(W, Hinv, k_steps=k1, strategy=strategy)
    live = (first["W"] != 0).to(torch.uint8)
    assert int(live.sum()) == 4 * (d - k1)
    second = obc.obc_prune_rows(first["W"], Hinv, k_steps=k2, live=live, strategy=strategy, want_trace=True)
    obc.obc_check()
    A, W1 = _np(Hinv), _np(first["W"])
    st = RowParity()
    for i in range(4):
        check_row(orc, st, "prune", A, W1[i], _np(second["order"][i]), _np(second["loss"][i]),
                  _np(second["W"][i]), k2, live=_np(live[i]), g_trace=_np(second["trace"][i]))
    print(st)
    st.assert_order_rule()
    assert int((second["W"] == 0).sum()) == 4 * (k1 + k2)
    # continuing from the reduced inverse is continuing the same greedy run: the one-pass run over
    # k1 + k2 steps takes (up to near ties) the same weights next
    one = obc.obc_prune_rows(W, Hinv, k_steps=k1 + k2, strategy=strategy)
    same = (one["order"][:, k1:] == second["order"]).float().mean().item()
    assert same > 0.9, same
    assert torch.allclose(one["W"], second["W"], rtol=1e-3, atol=1e-5)
    # a row with fewer survivors than k_steps stops when none is left
    live2 = live.clone()
    live2[1, 5:] = 0
    W2 = first["W"] * live2
    few = obc.obc_prune_rows(W2, Hinv, k_steps=k2, live=live2, strategy=strategy)
    obc.obc_check()
    assert torch.all(few["W"][1] == 0)
    n1 = int(live2[1].sum())
    assert torch.all(few["order"][1, n1:] == -1) and torch.all(few["order"][1, :n1] >= 0)
    # not combined with N:M
    import paper_2208_11580_amd as pkg
    with pytest.raises(pkg.ObcError):
        obc.obc_prune_rows(W[:, :256].contiguous(), Hinv[:256, :256].contiguous(), nm=(2, 4),
                           live=live[:, :256].contiguous(), strategy=strategy)


def test_many_sparsity_levels_from_one_trace(obc, orc):
    """The paper's database of sparsity levels s_i = 1 - (1 - delta)^i (Sec. 6) comes from ONE run of
    the row solver: every level is a global step over the same loss traces and a gather from the
    same weight trace.  Each level is checked against the oracle's replay of its own traces."""
    W, X = _layer("conv64x576", d_col=96, d_row=24, n_samples=800)
    Hinv = _hinv(obc, X)
    res = obc.obc_prune_rows(W, Hinv, want_trace=True)
    obc.obc_check()
    R, d = W.shape
    A, Wn = _np(Hinv).astype(np.float64), _np(W).astype(np.float64)
    ro = orc.prune_rows(A, Wn)
    assert np.array_equal(ro["order"], _np(res["order"]))       # no near ties in this layer
    levels = [1.0 - 0.9 ** i for i in range(1, 31, 3)]
    prev = -1
    for sp in levels:
        k = obc_inputs.target_count(sp, R, d)
        assert k > prev
        prev = k
        counts, mask = obc.obc_global_select(res["loss"], res["order"], k)
        What = obc.obc_gather_trace(W, res["trace"], counts)
        # Alg. 2 on the GPU's own (fp32) traces: the counts are then an exact integer comparison
        co = orc.global_select(_np(res["loss"]).astype(np.float64), k)
        assert np.array_equal(_np(counts), co), sp
        assert int(mask.sum()) == k and int((What == 0).sum()) >= k
        Wo = orc.reconstruct(A, Wn, co)
        assert np.linalg.norm(_np(What) - Wo) <= 1e-4 * np.linalg.norm(Wo), sp


@pytest.mark.parametrize("strategy", [1, 2])
def test_rows_that_do_no_step_keep_their_weights(obc, strategy):
    W, X = _layer("conv64x576", d_col=280, d_row=5, n_samples=1500)
    Hinv = _hinv(obc, X)
    full = obc.obc_prune_rows(W, Hinv, strategy=strategy, want_trace=True)
    counts = torch.tensor([0, 1, 70, 0, 280], dtype=torch.int32, device="cuda")
    rep = obc.obc_prune_rows(W, Hinv, stop_counts=counts, strategy=strategy)
    obc.obc_check()
    assert torch.equal(rep["W"], obc.obc_gather_trace(W, full["trace"], counts))
    assert torch.equal(rep["W"][0], W[0]) and torch.equal(rep["W"][3], W[3])
    none = obc.obc_prune_rows(W, Hinv, k_steps=0, strategy=strategy)
    assert torch.equal(none["W"], W)


@pytest.mark.parametrize("strategy", [1, 2])
def test_trace_beyond_a_rows_last_step_is_zero(obc, strategy):
    """Trace entries of the steps a row does not take (per-row step limits, fewer survivors than
    steps) are zero in both solvers, whatever the buffer held before."""
    W, X = _layer("conv64x576", d_col=264, d_row=4, n_samples=1500)
    Hinv = _hinv(obc, X)
    k = 100
    counts = torch.tensor([0, 7, 100, 64], dtype=torch.int32, device="cuda")
    out = dict(trace=torch.full((4, k, 264), float("nan"), device="cuda"))
    res = obc.obc_prune_rows(W, Hinv, k_steps=k, stop_counts=counts, strategy=strategy, out=out)
    full = obc.obc_prune_rows(W, Hinv, k_steps=k, strategy=strategy, want_trace=True)
    obc.obc_check()
    for i, c in enumerate(counts.tolist()):
        assert torch.equal(res["trace"][i, :c], full["trace"][i, :c])
        assert torch.all(res["trace"][i, c:] == 0)
    # an already sparse row runs out of survivors before k steps
    live = torch.ones(4, 264, dtype=torch.uint8, device="cuda")
    live[1, 40:] = 0                                           # 40 survivors
    out = dict(trace=torch.full((4, k, 264), float("nan"), device="cuda"))
    sp = obc.obc_prune_rows(W * live, Hinv, k_steps=k, live=live, strategy=strategy, out=out)
    obc.obc_check()
    assert torch.isfinite(sp["trace"]).all()
    assert torch.all(sp["trace"][1, 40:] == 0)
    assert torch.all(sp["trace"][1, 39] == 0) and not torch.all(sp["trace"][1, 38] == 0)


def test_membench_kernels_move_what_they_say(obc):
    """The plain copy kernel copies (both store policies); read and write passes return a time."""
    n = 1 << 22
    src = (torch.arange(n, device="cuda", dtype=torch.int32) * 2).view(torch.uint8)    # low bits clear
    dst = torch.zeros_like(src)
    for streaming in (False, True):
        dst.zero_()
        ms = obc.obc_membench(2, src, dst, src.numel(), reps=2, streaming=streaming)
        assert ms > 0 and torch.equal(dst, src)
    assert obc.obc_membench(0, src, None, src.numel(), reps=2) > 0
    assert obc.obc_membench(1, None, dst, dst.numel(), reps=2, streaming=True) > 0
    import paper_2208_11580_amd as pkg
    with pytest.raises(pkg.ObcError):
        obc.obc_membench(2, src, dst, 24, reps=1)              # not a multiple of 16 bytes


def test_mfmabench_stays_below_the_data_sheet(obc):
    """The loop of independent MFMA instructions runs and reports a rate no matrix core can exceed."""
    f32 = obc.obc_mfmabench(0, iters=2000, reps=2)
    f64 = obc.obc_mfmabench(1, iters=2000, reps=2)
    print("fp32 MFMA %.1f TFLOP/s, fp64 MFMA %.1f TFLOP/s" % (f32, f64))
    assert 10.0 < f32 < 157.3 * 1.05
    assert 5.0 < f64 < 78.6 * 1.05
    import paper_2208_11580_amd as pkg
    with pytest.raises(pkg.ObcError):
        obc.obc_mfmabench(2)


def test_trace_of_an_odd_width_is_fully_written(obc, orc):
    # the trace is cleared by a 16-byte-wide fill before the steps scatter into it: a size that is
    # no multiple of four floats, over memory that held NaNs before
    W, X = _layer("conv64x576", d_col=301, d_row=3, n_samples=1500)
    Hinv = _hinv(obc, X)
    poison = torch.full((3 * 301 * 301 + 64,), float("nan"), device="cuda")
    del poison
    res = obc.obc_prune_rows(W, Hinv, strategy=2, want_trace=True)
    obc.obc_check()
    tr = _np(res["trace"])
    assert np.isfinite(tr).all()
    order = _np(res["order"])
    for i in range(3):
        r = orc.prune_row(_np(Hinv).astype(np.float64), _np(W[i]).astype(np.float64), forced=order[i].astype(np.int32),
                          want_trace=True)
        for t in (0, 1, 150, 299, 300):
            assert np.all(tr[i, t, order[i, :t + 1]] == 0.0)
            assert np.linalg.norm(tr[i, t] - r.trace[t]) <= 1e-4 * np.linalg.norm(r.trace[t]) + 1e-30


# ------------------------------------------------------------------------------ closed-form recovery
@pytest.mark.parametrize("d,R,sparsity", [(32, 16, 0.5), (203, 5, 0.4), (576, 4, 0.6), (1100, 3, 0.5)])
def test_reconstruct_rows_matches_oracle_and_the_trace(obc, orc, d, R, sparsity):
    """Sec. 4 Step 2: the weights of the global step's mask by the group-OBS closed form, against the
    oracle's closed form (same fp32 inputs) and against the weights gathered from the pruning trace."""
    name = "lin16x32" if d == 32 else "conv64x576"
    W, X = _layer(name, d_col=d, d_row=R, n_samples=max(256, 3 * d))
    Hinv = _hinv(obc, X)
    res = obc.obc_prune_rows(W, Hinv, want_trace=True)
    k = obc_inputs.target_count(sparsity, R, d)
    counts, mask = obc.obc_global_select(res["loss"], res["order"], k)
    from_trace = obc.obc_gather_trace(W, res["trace"], counts)
    got = obc.obc_reconstruct_rows(W, Hinv, mask, max_pruned=int(counts.max()))
    obc.obc_check()
    ref = orc.reconstruct_closed_form(_np(Hinv), _np(W), _np(mask))
    g = _np(got).astype(np.float64)
    for i in range(R):
        assert np.linalg.norm(g[i] - ref[i]) <= 1e-6 * np.linalg.norm(ref[i]) + 1e-30, i
        assert np.linalg.norm(g[i] - _np(from_trace[i])) <= 1e-4 * np.linalg.norm(ref[i]) + 1e-30, i
    assert torch.equal(got == 0, mask.bool())
    # the default workspace bound (any count up to d) gives the same weights
    assert torch.equal(obc.obc_reconstruct_rows(W, Hinv, mask), got)


@pytest.mark.parametrize("d", [200, 1400])
def test_reconstruct_rows_beside_a_non_finite_index(obc, d):
    """An infinite or NaN row of H^-1 that a row of W does not prune reaches that index's own weight alone;
    a row that prunes nothing is W itself."""
    W, X = _layer("conv64x576", d_col=d, d_row=4, n_samples=2 * d)
    Hinv = _hinv(obc, X)
    mask = torch.zeros(4, d, dtype=torch.uint8, device="cuda")
    mask[0, 1::2] = 1
    mask[1, :20] = 1
    mask[3, 101:] = 1
    good = obc.obc_reconstruct_rows(W, Hinv, mask)
    for bad in (float("inf"), float("nan")):
        H = Hinv.clone()
        H[100, :] = bad
        H[:, 100] = bad
        got = obc.obc_reconstruct_rows(W, H, mask)
        keep = torch.arange(d, device="cuda") != 100
        assert torch.equal(got[:, keep], good[:, keep])
        assert torch.equal(got[2], W[2]) and not bool(got[[0, 1, 3], 100].isfinite().any())


def test_reconstruct_rows_edge_cases(obc, orc):
    import paper_2208_11580_amd as pkg

    d, R = 200, 6
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=900)
    Hinv = _hinv(obc, X)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    mask = (torch.rand(R, d, generator=g, device="cuda") < 0.45).to(torch.uint8)
    mask[0] = 0                                    # nothing pruned
    mask[1] = 1                                    # everything pruned
    mask[2] = 0
    mask[2, 77] = 1                                # a single weight
    mask[3, :65] = 1                               # one more than a block of 64 among others
    got = obc.obc_reconstruct_rows(W, Hinv, mask)
    obc.obc_check()
    ref = orc.reconstruct_closed_form(_np(Hinv), _np(W), _np(mask))
    assert torch.equal(got[0], W[0]) and int(got[1].abs().sum()) == 0
    assert np.linalg.norm(_np(got) - ref) <= 1e-6 * np.linalg.norm(ref)
    assert torch.equal(got == 0, mask.bool())
    # the single-weight row is the OBS update of eq. (3): w - H^-1[:, p] w_p / [H^-1]_pp
    A = _np(Hinv).astype(np.float64)
    w2 = _np(W[2]).astype(np.float64)
    one = w2 - A[:, 77] * w2[77] / A[77, 77]
    one[77] = 0.0
    assert np.allclose(_np(got[2]), one, rtol=1e-6, atol=1e-9)
    # a workspace bound below a row's count: that row comes back unchanged and the call is flagged
    small = obc.obc_reconstruct_rows(W, Hinv, mask, max_pruned=70)
    with pytest.raises(pkg.ObcError) as e:
        obc.obc_check()
    assert e.value.code == pkg.OBC_ERR_WORKSPACE
    many = mask.sum(dim=1) > 70
    assert bool(many.any()) and torch.equal(small[many], W[many])
    assert torch.equal(small[~many], got[~many])
    # argument errors
    with pytest.raises(pkg.ObcError):
        obc.obc_reconstruct_rows(W, Hinv, mask, max_pruned=d + 1)


def test_reconstruct_rows_on_both_sides_of_the_product(obc, orc):
    """The bound from which the closing product runs over all columns (640): the same weights, bit for bit,
    from both sides of it, and a row beyond its bound unchanged on both."""
    import paper_2208_11580_amd as pkg

    d = 1000
    W, X = _layer("conv64x576", d_col=d, d_row=6, n_samples=2 * d)
    Hinv = _hinv(obc, X)
    mask = torch.zeros(6, d, dtype=torch.uint8, device="cuda")
    for i, c in enumerate((0, 1, 64, 65, 600, 639)):
        mask[i, torch.randperm(d, generator=torch.Generator().manual_seed(i))[:c].cuda()] = 1
    got = [obc.obc_reconstruct_rows(W, Hinv, mask, max_pruned=m) for m in (639, 640, d)]
    obc.obc_check()
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    ref = orc.reconstruct_closed_form(_np(Hinv), _np(W), _np(mask))
    assert np.linalg.norm(_np(got[0]) - ref) <= 1e-6 * np.linalg.norm(ref)
    mask[5] = 1
    for m in (60, 639, 640):
        cut = obc.obc_reconstruct_rows(W, Hinv, mask, max_pruned=m)
        with pytest.raises(pkg.ObcError):
            obc.obc_check()
        over = mask.sum(dim=1) > m
        assert torch.equal(cut[over], W[over]) and torch.equal(cut[~over], got[0][~over])


@pytest.mark.parametrize("d,keep", [(19904, 5), (20032, 70)])
def test_reconstruct_rows_at_the_edge_of_lds(obc, d, keep):
    """The longest row whose solve fits LDS and one beyond it.  H^-1 = I + u u^T: the closed form is
    w_S - u_S (u_P . w_P) / (1 + u_P . u_P) by Sherman-Morrison.  H^-1 is rounded to fp32 (2^-24 of entries
    of at most u_i u_j), which moves the result by a few units of that."""
    gen = torch.Generator(device="cuda").manual_seed(d)
    u = torch.randn(d, generator=gen, device="cuda") / 32
    Hinv = torch.outer(u, u)
    Hinv.diagonal().add_(1.0)
    W = torch.randn(1, d, generator=gen, device="cuda")
    mask = torch.ones(1, d, dtype=torch.uint8, device="cuda")
    at = torch.randperm(d, generator=gen, device="cuda")[:keep]
    mask[0, at] = 0
    got = obc.obc_reconstruct_rows(W, Hinv, mask)
    obc.obc_check()
    P = mask[0].bool()
    ud, wd = u.double(), W[0].double()
    want = wd - ud * (ud[P] @ wd[P]) / (1.0 + ud[P] @ ud[P])
    assert not bool(got[0, P].any())
    assert float((got[0, ~P].double() - want[~P]).norm() / want[~P].norm()) < 1e-5
    del Hinv
    obc.release_workspace()
    torch.cuda.empty_cache()


# ------------------------------------------------------------------------------ boundary errors
def test_argument_errors(obc):
    import paper_2208_11580_amd as pkg

    W = torch.randn(4, 30, device="cuda")
    Hinv = torch.eye(30, device="cuda")
    with pytest.raises(pkg.ObcError) as e:
        obc.obc_prune_rows(W, Hinv, k_steps=31)
    assert e.value.code == pkg.OBC_ERR_BAD_SHAPE
    with pytest.raises(pkg.ObcError) as e:
        obc.obc_prune_rows(W, Hinv, nm=(2, 4), k_steps=10)   # 30 % 4 != 0
    assert e.value.code == pkg.OBC_ERR_BAD_SHAPE
    with pytest.raises(pkg.ObcError) as e:
        obc.obc_global_select(torch.zeros(4, 30, device="cuda"), torch.zeros(4, 30, dtype=torch.int32, device="cuda"), 121)
    assert e.value.code == pkg.OBC_ERR_BAD_SHAPE
    # a non-positive pivot is latched by the kernel and reported by obc_check
    bad = torch.eye(30, device="cuda")
    bad[3, 3] = -1.0
    obc.obc_prune_rows(W, bad)
    with pytest.raises(pkg.ObcError) as e:
        obc.obc_check()
    assert e.value.code == pkg.OBC_ERR_NUMERIC
    obc.obc_check()
    # empty inputs are fine
    out = obc.obc_prune_rows(W[:0], Hinv)
    assert out["order"].shape == (0, 30)


@pytest.mark.parametrize("d", [420, 600])
def test_rows_many_more_rows_than_cus(obc, orc, d):
    """Several times more rows than CUs at a mid-size width: the solver switches to the panel variants
    of which three workgroups share a CU (two owned indices a thread up to 512 columns, three above);
    sampled rows against the oracle, all rows against invariants."""
    R = 1030
    W, X = _layer("attn768x768", d_col=d, d_row=R, n_samples=2000)
    Hinv = _hinv(obc, X)
    rows = [0, 515, 1029]
    res, _ = _check_prune(obc, orc, W, Hinv, d, (0, 0), 2, rows=rows)
    srt = torch.sort(res["order"], dim=1).values
    assert torch.equal(srt, torch.arange(d, device="cuda", dtype=torch.int32).expand(R, d))
    assert torch.all(res["W"] == 0)
    q, _ = _check_quant(obc, orc, W, Hinv, 4, 2, rows=rows)
    srt = torch.sort(q["order"], dim=1).values
    assert torch.equal(srt, torch.arange(d, device="cuda", dtype=torch.int32).expand(R, d))
    assert bool(((q["codes"] >= 0) & (q["codes"] <= 15)).all())
    # block pruning: one owned index a thread
    kb = d // 4
    blk = obc.obc_prune_blocks(W, Hinv, 4, strategy=2)
    obc.obc_check()
    A, Wn = _np(Hinv), _np(W)
    for i in rows:
        check_block_row(orc, A, Wn[i], 4, _np(blk["order"][i]), _np(blk["loss"][i]), _np(blk["W"][i]), kb)
    srt = torch.sort(blk["order"], dim=1).values
    assert torch.equal(srt, torch.arange(kb, device="cuda", dtype=torch.int32).expand(R, kb))
    assert torch.all(blk["W"] == 0)


@pytest.mark.parametrize("R,d,k", [(768, 257, 257), (769, 512, 170), (768, 600, 260), (2, 1025, 150), (3, 1536, 150),
                                   (768, 272, 136), (768, 273, 273), (768, 304, 150), (768, 305, 305), (770, 336, 130),
                                   (768, 337, 337), (768, 352, 170), (768, 353, 353)])
def test_panels_of_72_and_80_steps(obc, orc, R, d, k):
    """The ends of the variants whose flush applies 72 vectors at once or 80 as two groups: both sides of the
    change to the next smaller one and of the widths at which 48 steps take the place of 80, the last step inside
    a group; the N:M counts carried from panel to panel."""
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=2 * d)
    Hinv = _hinv(obc, X)
    rows = [0, R - 1]
    _check_prune(obc, orc, W, Hinv, k, (0, 0), 2, rows=rows)
    if d % 4 == 0:
        _check_prune(obc, orc, W, Hinv, k, (2, 4), 2, rows=rows)
    if d <= 600:
        _check_quant(obc, orc, W, Hinv, 4, 2, rows=rows)


@pytest.mark.parametrize("R,d,k", [(512, 353, 120), (513, 257, 60), (513, 352, 120), (513, 353, 120), (640, 600, 270)])
def test_three_rows_per_cu_past_512_rows(obc, orc, R, d, k):
    """Both sides of the row count from which three workgroups share a CU, and of the widths from which OBQ and pruning do."""
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=2 * d)
    Hinv = _hinv(obc, X)
    _check_prune(obc, orc, W, Hinv, k, (0, 0), 2, rows=[0, R - 1])
    _check_quant(obc, orc, W, Hinv, 4, 2, rows=[0, R - 1])


@pytest.mark.parametrize("R,d,k,nm,panels", [(513, 520, 56, (0, 0), 1), (640, 768, 64, (0, 0), 1), (767, 768, 49, (0, 0), 1),
                                             (600, 600, 60, (2, 4), 1), (700, 768, 100, (0, 0), 2), (700, 768, 48, (0, 0), 1),
                                             (640, 600, 65, (0, 0), 2)])
def test_few_steps_past_512_rows_end_without_another_flush(obc, orc, R, d, k, nm, panels):
    """513 .. 767 rows of 513 .. 768 columns: 49 to 64 steps that are left are one panel, not one of 48 and a rest."""
    W, X = _layer("conv64x576", d_col=d, d_row=R, n_samples=2 * d)
    Hinv = _hinv(obc, X)
    obc.obc_profile_begin()
    obc.obc_prune_rows(W, Hinv, k_steps=k, nm=nm, strategy=2)
    stat = obc.obc_profile_end()
    assert stat["panel"]["launches"] == panels and stat["flush"]["launches"] == panels - 1
    _check_prune(obc, orc, W, Hinv, k, nm, 2, rows=[0, R - 1])


def test_edge_cases_of_the_widened_entry_points(obc, orc):
    """Smallest shapes and degenerate masks: one sample, one column, one block, rows whose weights are
    all pruned already, every row with enough pruned weights for the bulk elimination."""
    ctx = obc
    torch.manual_seed(0)
    for N in (1, 3, 17):
        X = torch.randn(5, N, device="cuda")
        Y = torch.randn(3, N, device="cuda")
        C = ctx.obc_cross(X, Y)
        assert np.allclose(_np(C), orc.cross(_np(X), _np(Y)), rtol=1e-5, atol=1e-6), N
    X = torch.randn(1, 50, device="cuda")
    Y = torch.randn(2, 50, device="cuda")
    H = ctx.obc_hessian(X)
    C = ctx.obc_cross(X, Y)
    assert np.allclose(_np(ctx.obc_refit(H, C)), orc.refit(_np(H), _np(C)), rtol=1e-5)
    # a row that is one block
    X = torch.randn(4, 64, device="cuda")
    W = torch.randn(3, 4, device="cuda")
    Hinv = _hinv(ctx, X)
    for st in (0, 1, 2):
        r = ctx.obc_prune_blocks(W, Hinv, 4, strategy=st)
        ctx.obc_check()
        assert torch.all(r["W"] == 0) and torch.all(r["order"] == 0)
        ro = orc.block_prune_row(_np(Hinv).astype(np.float64), _np(W[0]).astype(np.float64), 4)
        assert abs(r["loss"][0, 0].item() - ro.loss[0]) <= 1e-4 * ro.loss[0]
    # live masks on both solvers
    d = 260
    X = torch.randn(d, 1000, device="cuda")
    W = torch.randn(3, d, device="cuda") * 0.1
    Hinv = _hinv(ctx, X)
    for st in (1, 2):
        live = torch.ones(3, d, dtype=torch.uint8, device="cuda")
        live[1] = 0                                  # a row with nothing left
        Wl = W * live
        delta, offset, maxq = ctx.obc_minmax_grid(Wl, 4, live=live)
        q = ctx.obc_quant_rows(Wl, Hinv, delta, offset, maxq, live=live, strategy=st)
        ctx.obc_check()
        assert torch.all(q["W"][1] == 0) and torch.all(q["codes"][1] == -1)
        q0 = ctx.obc_quant_rows(W, Hinv, *ctx.obc_minmax_grid(W, 4)[:2], 15, strategy=st)
        assert torch.equal(q["W"][0], q0["W"][0]) and torch.equal(q["order"][2], q0["order"][2])
        p = ctx.obc_prune_rows(Wl, Hinv, k_steps=10, live=live, strategy=st)
        ctx.obc_check()
        assert torch.all(p["W"][1] == 0) and torch.all(p["order"][1] == -1)
        # every row has at least 64 pruned weights (bulk elimination), one row has no survivor
        live2 = torch.ones(3, d, dtype=torch.uint8, device="cuda")
        live2[:, :130] = 0
        live2[2, :] = 0
        W2 = W * live2
        p2 = ctx.obc_prune_rows(W2, Hinv, k_steps=20, live=live2, strategy=st)
        ctx.obc_check()
        Hfull = np.linalg.inv(_np(Hinv).astype(np.float64))
        ref = orc.prune_row(orc.invert(Hfull[130:, 130:]), _np(W2[0, 130:]).astype(np.float64), k_steps=20)
        assert np.array_equal(_np(p2["order"][0]) - 130, ref.order)
        assert np.allclose(_np(p2["W"][0, 130:]), ref.w, rtol=1e-3, atol=1e-6)
        assert torch.all(p2["W"][2] == 0)
    # the outlier flag with a single-point grid: everything is an outlier until it sits at zero
    a = ctx.obc_quant_rows(W, Hinv, torch.ones(3, device="cuda"), torch.zeros(3, device="cuda"), 0, outliers=True)
    ctx.obc_check()
    assert torch.all(a["W"] == 0)
