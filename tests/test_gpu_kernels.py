"""GPU kernels at the edges of their tiles and of the rules that choose between them,
against NumPy in FP64.  Every test prints its case before touching the GPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1609_03488_amd")


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _conv_solver(n, k, prec, engine):
    rng = np.random.default_rng(n + k)
    taps = rng.standard_normal(k)
    op = P.Operator(n + k - 1, n).add_conv(0, 0, taps, n, 0.75)
    st = P.Settings.make(precision=prec, normalize=0, conv_mfma=engine)
    return taps, P.Solver(op, n + k - 1, [], st), rng


# one output, less than a wave, tile edges of both forms (FP64: 128 / 256 outputs,
# FP32: 256 / 512), a step of 16 taps with and without remainders, two passes of
# 2048 taps, and both sides of the 512 tiles where the wide form takes over
@pytest.mark.parametrize("n,k", [(1, 1), (60, 3), (128, 16), (257, 17), (500, 20), (513, 36), (2500, 2051),
                                 (131040, 33), (131300, 33), (262100, 45), (262400, 40)])
@pytest.mark.parametrize("prec", [P.FP64, P.FP32], ids=["fp64", "fp32"])
def test_direct_convolution_edges(n, k, prec):
    """|dev - ref| <= (k + 4) u sum_t |w_t||x_t| elementwise: k fused multiply-adds
    and the conversions of the operands, in the working precision."""
    print("[case] direct convolution", n, k, prec, flush=True)
    taps, s, rng = _conv_solver(n, k, prec, 0)
    x, y = rng.standard_normal(n), rng.standard_normal(n + k - 1)
    u = 2.0 ** -53 if prec == P.FP64 else 2.0 ** -24
    a, at = np.abs(taps), 0.75 * taps
    err = np.abs(s.apply(x) - np.convolve(at, x))
    assert np.all(err <= (k + 4) * u * 0.75 * np.convolve(a, np.abs(x)))
    err = np.abs(s.apply(y, transpose=True) - np.correlate(y, at, "valid"))
    assert np.all(err <= (k + 4) * u * 0.75 * np.correlate(np.abs(y), a, "valid"))


def _fft_bound(taps, src):
    """Normwise rounding of the FFT convolution: 12 log2(L) u ||w||_1 sqrt(2) times the
    largest 2-norm of a window of L = 2048 inputs (two windows share a transform)."""
    sq = np.concatenate([[0.0], np.cumsum(src * src)])
    win = np.sqrt(np.max(sq[2048:] - sq[:-2048])) if src.size >= 2048 else np.sqrt(sq[-1])
    return 12 * 11 * 2.0 ** -24 * np.abs(taps).sum() * np.sqrt(2) * win


# the convolution's rows and columns start off the 4-element grid and lie inside vector
# tiles; identity blocks ahead of, across and past them, several to an output, and (70)
# more blocks than a workgroup's list of 64; one window pair, its ragged end, several
@pytest.mark.parametrize("n,k,r0,c0,nid", [(40, 5, 0, 0, 1), (1000, 129, 3, 5, 3), (4061, 34, 1, 2, 3),
                                           (9000, 1536, 7, 1, 70), (5003, 2, 2, 3, 70)])
@pytest.mark.parametrize("engine", [0, 2], ids=["direct", "fft"])
def test_convolution_with_identity_blocks(n, k, r0, c0, nid, engine):
    """A x and A^T y against NumPy; identity terms and the sum rounded in FP64, so the
    FP32 error is the convolution's plus (nid + 4) u of the terms."""
    print("[case] convolution + identity blocks", n, k, r0, c0, nid, engine, flush=True)
    rng = np.random.default_rng(n * k)
    taps = rng.standard_normal(k)
    rows, cols = r0 + n + k - 1 + 9, c0 + n + 6
    op = P.Operator(rows, cols).add_conv(r0, c0, taps, n, -0.5)
    ids = [(0, 0, min(rows, cols), 0.25)]
    for j in range(1, nid):
        ln = int(rng.integers(1, cols // 2))
        ids.append((int(rng.integers(0, rows - ln)), int(rng.integers(0, cols - ln)), ln, float(rng.standard_normal())))
    for b in ids:
        op.add_identity(*b)
    s = P.Solver(op, rows, [], P.Settings.make(precision=P.FP32, normalize=0, conv_mfma=engine))
    u = 2.0 ** -24
    for adj in (False, True):
        v = rng.standard_normal(rows if adj else cols).astype(np.float32).astype(np.float64)
        ref, mag = np.zeros(cols if adj else rows), np.zeros(cols if adj else rows)
        bound = np.zeros_like(ref)
        src = v[r0:r0 + n + k - 1] if adj else v[c0:c0 + n]
        lo, m = (c0, n) if adj else (r0, n + k - 1)
        conv = (lambda a, w: np.correlate(a, w, "valid")) if adj else np.convolve
        ref[lo:lo + m] = -0.5 * conv(src, taps)
        mag[lo:lo + m] = 0.5 * conv(np.abs(src), np.abs(taps))
        bound[lo:lo + m] = 0.5 * _fft_bound(taps, src) if engine == 2 else k * u * mag[lo:lo + m]
        for a0, b0, ln, sc in ids:
            o, i = (b0, a0) if adj else (a0, b0)
            ref[o:o + ln] += sc * v[i:i + ln]
            mag[o:o + ln] += abs(sc) * np.abs(v[i:i + ln])
        err = np.abs(s.apply(v, transpose=adj) - ref)
        assert np.all(err <= bound + (nid + 4) * u * mag)


# sizes at the edges of the fused register form's variants (512 threads times 1, 2, 3, 4
# or 8 outputs), one element past them, and the general form above the last; a waves' worth
# and less; kernels shorter and longer than a step of eight taps
@pytest.mark.parametrize("family,n,k", [("deconv", 20, 3), ("deconv", 482, 31), ("deconv", 483, 31),
                                        ("deconv", 1000, 25), ("deconv", 1001, 25), ("deconv", 1435, 102),
                                        ("deconv", 1436, 102), ("deconv", 2040, 9), ("deconv", 2050, 9),
                                        ("lasso", 500, 13), ("lasso", 505, 13), ("lasso", 1020, 5),
                                        ("lasso", 1100, 40)])
def test_fused_register_form_iterates(family, n, k):
    """FP64, CG to 1e-13: 12 steps (a test inside the launch after 5 and 10) leave the
    oracle's embedding state to 1e-8, as the one-launch-per-kernel path's test asks."""
    import oracle as o
    import workloads as w
    print("[case] fused register form", family, n, k, flush=True)
    if family == "deconv":
        d = w.deconv_instance(n, k, k / 7.0, 0.1, 1e-4, n + k)
        pr, prog = P.deconv_problem(d["c"], d["b"]), o.deconv_program(d["c"], d["b"])
    else:
        d = w.conv_lasso_instance(n, k, k / 5.0, 1e-4, n + k)
        pr = P.conv_lasso_problem(d["c"], d["b"], d["lam"])
        prog = o.conv_lasso_program(d["c"], d["b"], d["lam"])
    st = P.Settings.make(precision=P.FP64, cg_tol=0.0, cg_floor=1e-13, cg_max_iters=60, setup_tol=1e-14,
                         setup_max_iters=2000, eps=1e-300, max_iters=12, check_every=5, fused_lone_max=0)
    s = P.Solver(pr.op, pr.l, pr.q, st)
    s.set_data(0, pr.b, pr.c)
    info = s.solve()[0]
    assert info["iters"] == 12 and info["status"] == P.MAX_ITERS
    ux, uy, tau, vs, kap = s.state(0)
    rux, ruy, rtau, rvs, rkap = o.scs_solve(prog, eps=1e-300, max_iters=12).u
    scale = max(1.0, np.abs(rux).max(), np.abs(ruy).max(), np.abs(rvs).max())
    for a, b in ((ux, rux), (uy, ruy), (vs, rvs)):
        assert np.abs(a - b).max() <= 1e-8 * scale
    assert abs(tau - rtau) <= 1e-8 * max(1, rtau) and abs(kap - rkap) <= 1e-8 * max(1, rkap)


@pytest.mark.parametrize("n,k", [(300, 31), (1500, 151), (3500, 300), (4000, 97)])
def test_fused_register_form_fp32_solves(n, k):
    """FP32 solves in the fused path agree with the one-launch-per-kernel path's, which
    the oracle's tests cover: the natural objectives, FP64 on the host, to 1e-4."""
    import oracle as o
    import workloads as w
    print("[case] fused register form fp32", n, k, flush=True)
    d = w.deconv_instance(n, k, k / 7.0, 0.05, 1e-4, n)
    pr = P.deconv_problem(d["c"], d["b"])
    f = []
    for fused in (0, 65536):
        s = P.Solver(pr.op, pr.l, pr.q, P.Settings.make(eps=1e-4, fused_max=fused, fused_lone_max=0))
        s.set_data(0, pr.b, pr.c)
        assert s.solve()[0]["status"] == P.SOLVED
        f.append(o.deconv_objective(d["c"], d["b"], s.solution(0)[0][:n]))
    assert abs(f[0] - f[1]) <= 1e-4 * f[0]


# CG start tests that always end a step's CG before its first iteration, that do so for
# some steps, and never; one X tile, several, and a batch
@pytest.mark.parametrize("n,k,batch", [(300, 31, 3), (2500, 41, 1)])
@pytest.mark.parametrize("cg_tol", [1e3, 0.3, 1e-9])
def test_steps_without_cg_iterations(n, k, batch, cg_tol):
    """FP64: 12 steps of the launch-by-launch path, whose first update takes the start test,
    against the fused path's, which tests before it iterates: equal counts of CG iterations,
    and the state to 1e-9 of its size (sums differ in order only)."""
    import workloads as w
    print("[case] steps without CG iterations", n, k, batch, cg_tol, flush=True)
    d = w.deconv_instance(n, k, k / 7.0, 0.1, 1e-4, n)
    pr = P.deconv_problem(d["c"], d["b"])
    out = []
    for fused in (0, 65536):
        s = P.Solver(pr.op, pr.l, pr.q, P.Settings.make(precision=P.FP64, cg_tol=cg_tol, cg_floor=1e-12, setup_tol=1e-13,
                                                        cg_max_iters=60, setup_max_iters=2000, fused_max=fused,
                                                        fused_lone_max=0), batch=batch)
        for i in range(batch):
            s.set_data(i, pr.b * (1.0 + i), pr.c)
        s.iterate(0)
        its0 = [r["cg_iters"] for r in s.residuals()]
        s.iterate(12)
        out.append(([r["cg_iters"] - i0 for r, i0 in zip(s.residuals(), its0)], [s.state(i) for i in range(batch)]))
    assert out[0][0] == out[1][0] and (cg_tol < 1e3) == (min(out[0][0]) > 0)
    for x, y in zip(out[0][1], out[1][1]):
        scale = max(1.0, np.abs(y[0]).max(), np.abs(y[1]).max(), np.abs(y[3]).max())
        for j in (0, 1, 3):
            assert np.abs(x[j] - y[j]).max() <= 1e-9 * scale


# one row and column; K that is no whole vector, step or padding; tiles of 128 outputs and
# one past; more instances than a 64-row tile, and identity blocks beside and across the block
@pytest.mark.parametrize("m,n,batch", [(1, 1, 2), (7, 129, 3), (130, 33, 33), (100, 250, 65)])
def test_batched_bf16_iterates(m, n, batch):
    """BF16 products of a batch whose dense block is exact in BF16: the embedding state after
    three steps (CG to 1e-6) agrees with the FP32 solver's, instance by instance.  Products
    differ by rounding, 2^-24 of a sum of n terms; CG stops at 1e-6: 1e-4 bounds both."""
    print("[case] batched bf16", m, n, batch, flush=True)
    rng = np.random.default_rng(m + n)
    A = rng.integers(-4, 5, (m, n)) / 4.0
    r0, c0 = 2, 1
    rows, cols = m + n + 5, n + 3
    op = P.Operator(rows, cols).add_dense(r0, c0, A).add_identity(0, 0, min(rows, cols) - 1, -0.5)
    op.add_identity(rows - cols, 0, cols, 1.0)
    data = [(np.abs(rng.standard_normal(rows)) + 1.0, rng.standard_normal(cols)) for _ in range(batch)]
    out = []
    for prec in (P.BF16, P.FP32):
        s = P.Solver(op, rows, [], P.Settings.make(precision=prec, normalize=0, cg_tol=0.0, cg_floor=1e-6,
                                                   cg_max_iters=200, setup_tol=1e-6, setup_max_iters=2000),
                     batch=batch)
        for i, (b, c) in enumerate(data):
            s.set_data(i, b, c)
        s.iterate(3)
        out.append([s.state(i) for i in range(batch)])
    for x, y in zip(*out):
        scale = max(1.0, np.abs(y[0]).max(), np.abs(y[1]).max(), np.abs(y[3]).max())
        for j in (0, 1, 3):
            assert np.abs(x[j] - y[j]).max() <= 1e-4 * scale


# X vectors of one element a thread up to a whole tile (2048) and past it (launch by
# launch); a limit of 1 and 3 iterations, and one above the single launch's
@pytest.mark.parametrize("n,k,limit", [(20, 3, 2000), (256, 31, 2000), (600, 25, 1), (600, 25, 3), (600, 25, 16384),
                                       (600, 25, 16385), (1000, 101, 2000), (2046, 9, 2000), (2049, 9, 2000)])
def test_setup_solve_in_one_launch(n, k, limit):
    """FP64 setup solve of the fused path against the launch-by-launch one: the same sums,
    so the same number of CG iterations, and a first step (CG to 1e-13) that agrees to 1e-10."""
    import workloads as w
    print("[case] setup solve", n, k, limit, flush=True)
    d = w.deconv_instance(n, k, k / 7.0, 0.1, 1e-4, n + k)
    pr = P.deconv_problem(d["c"], d["b"])
    out = []
    for fused in (0, 65536):
        s = P.Solver(pr.op, pr.l, pr.q, P.Settings.make(
            precision=P.FP64, cg_tol=0.0, cg_floor=1e-13, cg_max_iters=200, setup_tol=1e-12, setup_max_iters=limit,
            fused_max=fused, fused_lone_max=0))
        s.set_data(0, pr.b, pr.c)
        s.iterate(0)
        its = s.residuals()[0]["cg_iters"]
        s.iterate(1)
        out.append((its, s.state(0)))
    assert out[0][0] == out[1][0] and 1 <= out[0][0] <= limit
    scale = max(1.0, *(np.abs(v).max() for v in out[0][1][:2]), np.abs(out[0][1][3]).max())
    for i in (0, 1, 3):
        assert np.abs(out[0][1][i] - out[1][1][i]).max() <= 1e-10 * scale
    assert abs(out[0][1][2] - out[1][1][2]) <= 1e-10 * scale


# columns at the edges of the row-streaming forms (256 threads x 16-byte vectors x 2, 4, ..,
# 12; FP64 1024 columns a pair, FP32 2048) and past the last, with ends that are no whole
# vector; one row, rows that split unevenly over the workgroups, more than 16 per tile;
# the block off the 16-byte grid of the vectors, identity blocks beside and across it
@pytest.mark.parametrize("m,n", [(1, 1), (3, 5), (70, 255), (300, 1023), (1030, 1025), (500, 2049), (17000, 33),
                                 (40, 6145), (33, 12289), (9, 24600)])
@pytest.mark.parametrize("prec", [P.FP64, P.FP32], ids=["fp64", "fp32"])
def test_dense_products_edges(m, n, prec):
    """A x and A^T y against NumPy in FP64: sums accumulate in FP64 and round once, so
    |dev - ref| <= (4 u + cols 2^-52) sum |a||x| with u the working precision's."""
    print("[case] dense products", m, n, prec, flush=True)
    rng = np.random.default_rng(m * 7 + n)
    r0, c0, rows, cols = 3, 1, m + 7, n + 2
    A = rng.standard_normal((m, n)).astype(np.float32).astype(np.float64)
    ln = min(rows, cols) - 1
    op = P.Operator(rows, cols).add_dense(r0, c0, A, 0.5).add_identity(0, 0, ln, -0.25).add_identity(1, 1, ln, 2.0)
    s = P.Solver(op, rows, [], P.Settings.make(precision=prec, normalize=0))
    u = 2.0 ** -53 if prec == P.FP64 else 2.0 ** -24
    for adj in (False, True):
        v = rng.standard_normal(rows if adj else cols).astype(np.float32).astype(np.float64)
        ref, mag = np.zeros(cols if adj else rows), np.zeros(cols if adj else rows)
        for off, sc in ((0, -0.25), (1, 2.0)):
            ref[off:off + ln] += sc * v[off:off + ln]
            mag[off:off + ln] += abs(sc) * np.abs(v[off:off + ln])
        src = v[r0:r0 + m] if adj else v[c0:c0 + n]
        lo, M = (c0, A.T) if adj else (r0, A)
        ref[lo:lo + M.shape[0]] += 0.5 * (M @ src)
        mag[lo:lo + M.shape[0]] += 0.5 * (np.abs(M) @ np.abs(src))
        err = np.abs(s.apply(v, transpose=adj) - ref)
        assert np.all(err <= (4 * u + max(m, n) * 2.0 ** -52) * mag)


# the steps up to the first test beyond 31 bits, as counted over a round, and beyond 30
@pytest.mark.parametrize("check_every", [2 ** 28, 2 ** 30, 2 ** 31 - 1])
@pytest.mark.parametrize("fused", [0, 65536], ids=["multikernel", "fused"])
def test_check_interval_beyond_the_step_limit(check_every, fused):
    """The test runs once, at max_iters: the solve is that of check_every = max_iters, bit for
    bit, though the point passes a test long before."""
    import workloads as w
    print("[case] check interval beyond the limit", check_every, fused, flush=True)
    d = w.deconv_instance(300, 31, 31 / 7.0, 0.1, 1e-4, 300)
    pr = P.deconv_problem(d["c"], d["b"])
    out = []
    for every in (check_every, 400, 10):
        s = P.Solver(pr.op, pr.l, pr.q, P.Settings.make(eps=1e-3, max_iters=400, check_every=every, fused_max=fused))
        s.set_data(0, pr.b, pr.c)
        out.append((s.solve()[0]["iters"],) + s.solution(0))
    assert out[0][0] == out[1][0] == 400 and out[2][0] < 400
    for a, b in zip(out[0][1:], out[1][1:]):
        np.testing.assert_array_equal(a, b)


# dense products (alone, and a batch whose members differ) and a convolution's; CG solves that
# all iterate (None), and a tolerance that early steps meet from the warm start
@pytest.mark.parametrize("family,prec,batch,cg_tol", [("lasso", P.FP64, 1, None), ("lasso", P.FP32, 3, None),
                                                      ("lasso", P.FP64, 1, 3.0), ("lasso", P.FP32, 3, 3.0),
                                                      ("deconv", P.FP64, 2, 3.0)])
def test_start_test_ahead_of_the_products(family, prec, batch, cg_tol):
    """The host moves the CG start test ahead of the first products when it reads that steps
    made no iteration: with a read after every interval it does, with one after 64 intervals
    it cannot, and the solves are the same, bit for bit."""
    import workloads as w
    print("[case] start test ahead of the products", family, prec, batch, cg_tol, flush=True)
    rng = np.random.default_rng(5)
    if family == "lasso":
        A = (rng.standard_normal((300, 900)) / 17).astype(np.float32)
        pr = P.lasso_problem(A, rng.standard_normal(300), 0.3)
        tol = dict(normalize=2)
    else:
        d = w.deconv_instance(3000, 41, 6.0, 0.1, 1e-4, 1)
        pr, tol = P.deconv_problem(d["c"], d["b"]), {}
    if cg_tol is not None:
        tol["cg_tol"] = cg_tol
    out = []
    for intervals in (1, 64):
        s = P.Solver(pr.op, pr.l, pr.q, P.Settings.make(precision=prec, eps=1e-300, max_iters=600, fused_max=0,
                                                        intervals_per_sync=intervals, **tol), batch=batch)
        for i in range(batch):
            s.set_data(i, pr.b * (1.0 + i), pr.c)
        r = s.solve()
        out.append([[(v["iters"], v["cg_iters"]) for v in r]] + [s.state(i) for i in range(batch)])
    assert out[0][0] == out[1][0]
    for x, y in zip(out[0][1:], out[1][1:]):
        for a, b in zip(x, y):
            np.testing.assert_array_equal(a, b)


# both sides of the kernel lengths where a narrow form takes over (padded taps: FP64 128,
# FP32 8), ends of a step of 16 taps, tile edges, a chunk of 1024 taps of the wide form and
# more, and the 512 tiles from which every kernel takes the wide form
@pytest.mark.parametrize("n,k", [(1, 124), (1, 125), (96, 161), (200, 140), (97, 128), (3000, 145), (130900, 160),
                                 (130914, 160), (131000, 1030), (131200, 2060), (300, 8), (300, 7)])
@pytest.mark.parametrize("prec", [P.FP64, P.FP32], ids=["fp64", "fp32"])
def test_direct_convolution_forms(n, k, prec):
    """The bound of test_direct_convolution_edges, at the edges of the rule on kernel lengths."""
    test_direct_convolution_edges(n, k, prec)


@pytest.mark.parametrize("n", [1, 300, 3000, 200000])
@pytest.mark.parametrize("prec", [P.FP64, P.FP32], ids=["fp64", "fp32"])
def test_parts_of_a_solution(n, prec):
    """x, y or s alone, and any two, are the parts of the whole solution, bit for bit: in one
    piece, and (n = 200000: more than 2^20 doubles of data, more than 65536 of a vector) piece by piece."""
    import ctypes as C
    print("[case] parts of a solution", n, prec, flush=True)
    rng = np.random.default_rng(n)
    op = P.Operator(2 * n, n).add_identity(0, 0, n).add_identity(n, 0, n, -0.5)
    s = P.Solver(op, 2 * n, [], P.Settings.make(precision=prec, max_iters=20, fused_max=0))
    s.set_data(0, np.abs(rng.standard_normal(2 * n)), rng.standard_normal(n))
    s.solve()
    whole = s.solution(0)
    for want in range(1, 8):
        out = [np.full(v.size, np.pi) for v in whole]
        rc = P.lib().cgs_solver_get_solution(s._h, 0, *((v.ctypes.data_as(C.POINTER(C.c_double)) if want >> i & 1
                                                         else None) for i, v in enumerate(out)))
        assert rc == 0
        for i in range(3):
            np.testing.assert_array_equal(out[i], whole[i] if want >> i & 1 else np.full(whole[i].size, np.pi))


def _layout(name, rng):
    """Blocks (kind, row0, col0, data) of a 700 x 720 operator; entries exact in BF16."""
    def mat(m, n):
        return rng.integers(-4, 5, (m, n)) / 4.0
    taps = rng.integers(-4, 5, 33) / 4.0
    return {"rows shared": [("dense", 5, 3, mat(300, 200)), ("dense", 100, 210, mat(350, 300))],
            "columns shared": [("dense", 5, 3, mat(200, 300)), ("dense", 210, 100, mat(300, 350))],
            "own ranges": [("dense", 5, 3, mat(300, 200)), ("dense", 310, 207, mat(130, 450)),
                           ("dense", 445, 660, mat(40, 40))],
            "same place": [("dense", 5, 3, mat(200, 300)), ("dense", 5, 3, mat(200, 300))],
            "beside a convolution": [("dense", 5, 3, mat(200, 300)), ("conv", 210, 310, taps)],
            "across a convolution": [("dense", 5, 3, mat(200, 300)), ("conv", 100, 100, taps)]}[name]


# which blocks own their rows or columns, and so which launches write base and identity blocks:
# two dense blocks that share one direction, both or none, several slots, a convolution beside
@pytest.mark.parametrize("name", ["rows shared", "columns shared", "own ranges", "same place", "beside a convolution",
                                  "across a convolution"])
@pytest.mark.parametrize("prec", [P.FP64, P.FP32, P.BF16], ids=["fp64", "fp32", "bf16"])
def test_blocks_that_share_ranges(name, prec):
    """A x and A^T y of two vectors in turn against NumPy.  Dense sums accumulate in FP64 (a
    BF16 batch: in FP32, 720 terms at most), convolutions fuse k multiply-adds in the working
    precision, and every block and identity rounds the output once: within
    (terms + blocks + 4) u sum |a||x|."""
    print("[case] shared ranges", name, prec, flush=True)
    rng = np.random.default_rng(len(name))
    blocks = _layout(name, rng)
    rows, cols, n_in = 700, 720, 400
    op, A = P.Operator(rows, cols), np.zeros((rows, cols))
    mag = np.zeros_like(A)
    for kind, r0, c0, a in blocks:
        if kind == "dense":
            op.add_dense(r0, c0, a, 0.5)
            A[r0:r0 + a.shape[0], c0:c0 + a.shape[1]] += 0.5 * a
            mag[r0:r0 + a.shape[0], c0:c0 + a.shape[1]] += 0.5 * np.abs(a)
        else:
            op.add_conv(r0, c0, a, n_in, 0.5)
            for t in range(a.size):
                i = np.arange(n_in)
                A[r0 + i + t, c0 + i] += 0.5 * a[t]
                mag[r0 + i + t, c0 + i] += 0.5 * abs(a[t])
    for r0, c0, ln, sc in ((0, 0, 690, -0.25), (9, 2, 691, 2.0)):
        op.add_identity(r0, c0, ln, sc)
        A[r0 + np.arange(ln), c0 + np.arange(ln)] += sc
        mag[r0 + np.arange(ln), c0 + np.arange(ln)] += abs(sc)
    s = P.Solver(op, rows, [], P.Settings.make(precision=prec, normalize=0, conv_mfma=0, fused_max=0),
                 batch=3 if prec == P.BF16 else 1)
    u = 2.0 ** -53 if prec == P.FP64 else 2.0 ** -24
    terms = 720 if prec == P.BF16 else 33
    for _ in range(2):
        for adj in (False, True):
            v = rng.standard_normal(rows if adj else cols).astype(np.float32).astype(np.float64)
            M, G = (A.T, mag.T) if adj else (A, mag)
            err = np.abs(s.apply(v, transpose=adj) - M @ v)
            assert np.all(err <= ((terms + len(blocks) + 6) * u + 720 * 2.0 ** -52) * (G @ np.abs(v)))


# one instance, whose pieces ride on the first convolution's launch, and a batch large enough
# that they would outgrow the whole tiles and take a launch of their own
@pytest.mark.parametrize("prec,engine", [(P.FP64, 0), (P.FP32, 0), (P.FP32, 1), (P.FP32, 2)])
def test_many_ranges_inside_a_tile(prec, engine):
    """The same problem alone and as members of a batch of 64: states equal, bit for bit, and
    A x and A^T y against NumPy within the bounds of test_convolution_with_identity_blocks."""
    print("[case] many ranges inside a tile", prec, engine, flush=True)
    rng = np.random.default_rng(11)
    rows, cols, n_in, k = 3663, 900, 150, 31
    taps = [rng.standard_normal(k) for _ in range(4)]
    op = P.Operator(rows, cols).add_identity(0, 0, cols, -1.0)
    for j, t in enumerate(taps):
        op.add_conv(1000 + 600 * j, 30 + 200 * j, t, n_in)
    b, c = np.abs(rng.standard_normal(rows)) + 1.0, rng.standard_normal(cols)
    st = P.Settings.make(precision=prec, conv_mfma=engine, fused_max=0)
    out = []
    for batch in (1, 64):
        s = P.Solver(op, rows, [], st, batch=batch)
        for i in range(batch):
            s.set_data(i, b, c)
        s.iterate(5)
        out.append(s.state(0))
        for x, y in zip(out[0], s.state(batch - 1)):
            np.testing.assert_array_equal(x, y)
    s = P.Solver(op, rows, [], P.Settings.make(precision=prec, conv_mfma=engine, fused_max=0, normalize=0), batch=64)
    u = 2.0 ** -53 if prec == P.FP64 else 2.0 ** -24
    for adj in (False, True):
        v = rng.standard_normal(rows if adj else cols).astype(np.float32).astype(np.float64)
        ref = np.zeros(cols if adj else rows)
        ref[:cols] = -v[:cols]
        mag, bound = np.abs(ref), np.zeros(ref.size)
        for j, t in enumerate(taps):
            src = v[1000 + 600 * j:][:n_in + k - 1] if adj else v[30 + 200 * j:][:n_in]
            lo, m = (30 + 200 * j, n_in) if adj else (1000 + 600 * j, n_in + k - 1)
            conv = (lambda a, w: np.correlate(a, w, "valid")) if adj else np.convolve
            ref[lo:lo + m] += conv(src, t)
            mag[lo:lo + m] += conv(np.abs(src), np.abs(t))
            bound[lo:lo + m] = _fft_bound(t, src) if engine == 2 else k * u * conv(np.abs(src), np.abs(t))
        err = np.abs(s.apply(v, transpose=adj) - ref)
        assert np.all(err <= bound + 5 * u * mag)


# the convolution and its columns off the vectors' starts, the cone's head on, before and
# after the convolution's rows, rows and columns that no block reaches
@pytest.mark.parametrize("n,k,r0,c0,cone", [(100, 7, 3, 5, 40), (470, 31, 17, 1, 300), (900, 64, 1, 130, 500),
                                            (1300, 101, 250, 77, 2), (2000, 33, 5, 40, 0)])
def test_fused_register_form_of_offset_blocks(n, k, r0, c0, cone):
    """FP64, CG to 1e-13: 12 steps of the register form (tests inside the launch after 5 and 10)
    leave the launch-by-launch path's embedding state to 1e-8, as its oracle test asks."""
    print("[case] register form, offset blocks", n, k, r0, c0, cone, flush=True)
    rng = np.random.default_rng(n)
    rows, cols = r0 + n + k - 1 + 23, c0 + n + 9
    op = P.Operator(rows, cols).add_conv(r0, c0, rng.standard_normal(k) / k, n, -1.5)
    op.add_identity(2, 3, min(rows, cols) - 12, -1.0).add_identity(rows - 20, 0, 15, 0.5)
    b, c = rng.standard_normal(rows), rng.standard_normal(cols)
    q = [rows - cone] if cone < rows else []
    out = []
    for fused in (0, 65536):
        s = P.Solver(op, cone if q else rows, q, P.Settings.make(
            precision=P.FP64, cg_tol=0.0, cg_floor=1e-13, cg_max_iters=200, setup_tol=1e-14, setup_max_iters=2000,
            eps=1e-300, max_iters=12, check_every=5, fused_max=fused, fused_lone_max=0))
        s.set_data(0, b, c)
        info = s.solve()[0]
        assert info["iters"] == 12 and info["status"] == P.MAX_ITERS
        out.append(s.state(0))
    scale = max(1.0, *(np.abs(v).max() for v in (out[0][0], out[0][1], out[0][3])))
    for a, b in zip(*out):
        assert np.abs(np.asarray(a) - np.asarray(b)).max() <= 1e-8 * scale


# 20 (one output a thread) to 2000 variables; a certificate inside a launch of many intervals
@pytest.mark.parametrize("n,k", [(20, 3), (600, 5), (1500, 9), (2000, 17)])
@pytest.mark.parametrize("prec", [P.FP64, P.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["infeasible", "unbounded"])
def test_certificates_in_the_register_form(kind, prec, n, k):
    """x >= 1 with w * x <= -1 (w >= 0), and minimise -sum x with x >= 0, -w * x <= 1: the
    certificate meets the header's conditions, recomputed in FP64: -b'y = 1 and ||A'y|| <= eps,
    or -c'x = 1 and ||A x + s|| <= eps, to 10 % for FP32's rounding of the returned point."""
    print("[case] certificate", kind, n, k, prec, flush=True)
    w, rows, eps = np.ones(k) / k, 2 * n + k - 1, 1e-4
    sign = 1.0 if kind == "infeasible" else -1.0
    op = P.Operator(rows, n).add_identity(0, 0, n, -1.0).add_conv(n, 0, w, n, sign)
    b, c = (np.full(rows, -1.0), np.ones(n)) if sign > 0 else (np.ones(rows), np.full(n, -1.0))
    if sign < 0:
        b[:n] = 0.0
    s = P.Solver(op, rows, [], P.Settings.make(precision=prec, eps=eps, max_iters=20000, fused_lone_max=0))
    s.set_data(0, b, c)
    info = s.solve()[0]
    assert info["status"] == (P.INFEASIBLE if sign > 0 else P.UNBOUNDED) and info["iters"] < 20000
    x, y, sl = s.solution(0)
    if sign > 0:
        aty = -y[:n] + np.correlate(y[n:], w, "valid")
        assert np.all(y >= 0) and abs(b @ y + 1.0) <= 1e-5 and np.linalg.norm(aty) <= 1.1 * eps
    else:
        ax = np.concatenate([-x, -np.convolve(x, w)])
        assert np.all(sl >= 0) and abs(c @ x + 1.0) <= 1e-5 and np.linalg.norm(ax + sl) <= 1.1 * eps
