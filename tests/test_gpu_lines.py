"""Faces along lines (tiles of 31 or 32 cells by 16 lines, runs of eight
faces; plain WENO fluxes) at the edges of tiles, runs and line groups: one
right-hand side of a rough admissible state against the oracle, and the same
step through the batch.

Bar: a face value is a few dozen roundings of numbers up to max |U|, and L
divides a difference of two of them by dx on each axis, so with u = 2^-53
(FP32: 2^-24) |dL| <= 128 u max |U| sum 1/dx.  The WENO-Z weights of a rough
state are O(1) functions of the indicators, whose relative rounding they
return undiminished; that is inside the factor.
"""
import numpy as np
import pytest

import oracle as O
from paper_1511_02137_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# edges of a tile (31 | 32 cells), of a run (8 faces), of a line group (16)
SHAPES = [(1, 1, 1), (2, 17, 31), (31, 16, 1), (32, 15, 8), (33, 7, 32), (7, 62, 33), (63, 3, 9), (9, 64, 16),
          (16, 32, 65), (124, 2, 5)]


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")


def H():
    from paper_1511_02137_amd import hydro
    return hydro


def rough_state(n, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nz = n
    U = np.empty((5, nz, ny, nx))
    U[0] = rng.uniform(1.0, 3.0, (nz, ny, nx))
    U[1:4] = U[0] * rng.uniform(-0.4, 0.4, (3, nz, ny, nx))
    U[4] = rng.uniform(0.1, 1.0, (nz, ny, nx))
    return U


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", SHAPES)
def test_rhs_at_tile_edges(n, bc):
    w = W.small_event(1, n=n, with_jet=False)
    for precision, weno, u in (("f64", "z", 2.0 ** -53), ("f64", "z5", 2.0 ** -53), ("f64", "js", 2.0 ** -53),
                               ("f32", "z", 2.0 ** -24)):
        U = rough_state(n, sum(n))
        if precision == "f32":
            U = U.astype(np.float32).astype(np.float64)
        pb = O.Problem(n=w.n, bc=(bc,) * 3, weno=weno)
        Lo, _, _ = O.rhs(pb, U, 1.0, [])
        h = H().from_workload(w, precision=precision, weno=weno, bc=(bc,) * 3)
        L = h.rhs(torch.from_numpy(U).to("cuda", h.dtype), 1.0).double().cpu().numpy()
        bar = 128 * u * np.abs(U).max() * 30.0
        err = np.abs(L - Lo).max()
        print(n, bc, precision, weno, "max |dL| %.2e bar %.2e" % (err, bar), flush=True)
        assert err <= bar
        h.close()


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", SHAPES)
def test_musta_rhs_at_tile_edges(n, bc):
    # MUSTA-FORCE: the flux is a Lipschitz function of the two face values where
    # both are admissible, k = 2 stages of three recoveries each: four times the
    # bar above.  Fluctuations of 0.03 keep every face value admissible (a
    # stencil's weights add up to 64/12 in magnitude).  The marching kernels
    # take one face a time by the same operations: equal bits.
    w = W.small_event(1, n=n, with_jet=False)
    rng = np.random.default_rng(sum(n) + 1)
    shape = (n[2], n[1], n[0])
    U = np.stack([rng.uniform(2.0, 2.06, shape), *rng.uniform(-0.06, 0.06, (3,) + shape),
                  rng.uniform(0.5, 0.515, shape)])
    for precision, weno, u in (("f64", "z", 2.0 ** -53), ("f64", "z5", 2.0 ** -53), ("f32", "z", 2.0 ** -24),
                               ("f32", "z5", 2.0 ** -24)):
        V = U.astype(np.float32).astype(np.float64) if precision == "f32" else U
        pb = O.Problem(n=w.n, bc=(bc,) * 3, weno=weno, flux="musta", musta_k=2)
        Lo, _, _ = O.rhs(pb, V, 1.0, [])
        h = H().from_workload(w, precision=precision, weno=weno, bc=(bc,) * 3, flux="musta", musta_k=2)
        x = torch.from_numpy(V).to("cuda", h.dtype)
        L = h.rhs(x, 1.0).clone()
        h.set_option(H().OPT_YZ_KERNEL, 1)
        M = h.rhs(x, 1.0)
        assert torch.equal(L, M), (n, bc, precision, weno)
        bar = 512 * u * np.abs(V).max() * 30.0
        err = np.abs(L.double().cpu().numpy() - Lo).max()
        print("musta", n, bc, precision, weno, "max |dL| %.2e bar %.2e" % (err, bar), flush=True)
        assert err <= bar
        h.close()


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", SHAPES)
def test_limited_rhs_at_tile_edges_is_bitwise(n, bc):
    # energies over six decades: the limiter acts at many faces.  The marching
    # kernels take one face a time by the same operations: equal bits.
    w = W.small_event(1, n=n, with_jet=False)
    rng = np.random.default_rng(sum(n) + 2)
    U = rough_state(n, sum(n)) * 10.0 ** rng.uniform(-6.0, 0.0, (n[2], n[1], n[0]))
    for precision, weno in (("f64", "z"), ("f64", "z5"), ("f64", "js"), ("f32", "z")):
        out = []
        for limiter, march in (("pp", 0), ("pp", 1), ("none", 0)):
            h = H().from_workload(w, precision=precision, weno=weno, bc=(bc,) * 3, limiter=limiter)
            h.set_option(H().OPT_YZ_KERNEL, march)
            out.append(h.rhs(torch.from_numpy(U).to("cuda", h.dtype), 1.0).clone())
            h.close()
        print("limiter", n, bc, precision, weno, "differs from unlimited:", not torch.equal(out[0], out[2]), flush=True)
        assert torch.equal(out[0], out[1]), (n, bc, precision, weno)
        if n != (1, 1, 1):
            assert not torch.equal(out[0], out[2])


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_batch_of_mixed_tile_lengths_is_bitwise(precision):
    # tile lengths 31 and 32 in one batch (no common one), persistent and not
    ws = [W.small_event(k, n=n) for k, n in enumerate([(31, 64, 20), (32, 31, 33), (5, 40, 62)])]
    single = []
    for w in ws:
        h = H().from_workload(w, precision=precision)
        h.step(2)
        torch.cuda.synchronize()
        single.append(h.U.cpu().numpy())
        h.close()
    b = H().batch_from_workloads(ws, precision=precision)
    b.run(2)
    torch.cuda.synchronize()
    for e, U in enumerate(single):
        assert np.array_equal(b.U[e].cpu().numpy(), U), e


# shorter than the ghosts, a turn's last run full and partly filled, two turns
ADJ_SHAPES = [(1, 3, 7), (8, 9, 2), (63, 4, 5), (5, 64, 6), (6, 5, 72), (71, 3, 4), (4, 103, 3), (2, 7, 128)]


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", ADJ_SHAPES)
def test_line_adjoint_at_run_edges(n, bc):
    """<J^T W, V> against the oracle's forward mode <W, J V> for one step of a
    rough state: both are exact derivatives of the discrete map, so they agree
    to rounding times the step's conditioning, 1e-10 of the sum of |products|;
    any number of lines per workgroup gives the same bits."""
    w = W.small_event(1, n=n, with_jet=False)
    pb = O.Problem(n=w.n, dx=w.dx, t0=w.t0, dt=w.dt, bc=(bc,) * 3)
    U0 = rough_state(n, sum(n))
    rng = np.random.default_rng(sum(n) + 1)
    V, Wt = rng.uniform(-1.0, 1.0, U0.shape), rng.uniform(-1.0, 1.0, U0.shape)
    _, JV = O.jvp(pb, U0, V, 1, [])
    outs = []
    for lines in (0, 1, 4):
        h = H().from_workload(w, bc=(bc,) * 3, adjoint_k=1)
        h.set_option(H().OPT_ADJ_LINES, lines)
        lam = torch.from_numpy(Wt).cuda()
        h.adjoint_step(torch.from_numpy(U0).cuda(), 0, None, 1, lam, None)
        torch.cuda.synchronize()
        outs.append(lam.cpu().numpy())
        h.close()
    rel = abs(np.sum(outs[0] * V) - np.sum(Wt * JV)) / np.sum(np.abs(Wt * JV))
    print(n, bc, "dot product %.2e" % rel, flush=True)
    assert rel <= 1e-10
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


# lengths around which a workgroup takes 8, 4 or 1 lines, and their run lengths
@pytest.mark.parametrize("n", [(77, 3, 2), (90, 2, 3), (100, 3, 2), (128, 3, 3), (200, 2, 2), (310, 2, 3), (3, 83, 2),
                               (2, 100, 3), (3, 2, 128), (2, 310, 3)])
def test_line_adjoint_at_workgroup_edges(n):
    test_line_adjoint_at_run_edges(n, "outflow")


def test_freezeout_range_of_p_t():
    """p_T from 1e-3 to where every exponential is subnormal or zero: rows
    within 1e-12 of their largest value (an exponent x carries x 2^-53, 6e-14
    at 570), a row beyond the range exactly zero with zero harmonics."""
    w = W.small_event(1, n=(21, 18, 13), steps=0)
    h = H().from_workload(w)
    pt = [1e-3, 1.0, 200.0, 1e4]
    spec, harm = h.freezeout(n_phi=48, pt=pt, n_harm=4)
    spec, harm = spec.cpu().numpy(), harm.cpu().numpy()
    pb = O.Problem(n=w.n, dx=w.dx, t0=w.t0, dt=w.dt)
    rs, _, _ = O.freezeout(pb, h.U.cpu().numpy(), n_phi=48, pt=pt, T_min=0.0, dof=1.0, n_harm=4)
    for r in range(4):
        assert np.abs(spec[r] - rs[r]).max() <= 1e-12 * np.abs(rs[r]).max(), r
    assert np.all(rs[4] == 0.0) and np.all(spec[4] == 0.0) and np.all(harm[4] == 0.0)
    h.close()


# axes shorter than a half tile (15 cells), at its edges and at those of runs of two
THIN = [(7, 19, 8), (8, 5, 14), (14, 8, 7), (15, 33, 1), (1, 15, 16), (16, 14, 15), (3, 1, 50)]


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", THIN)
def test_rhs_of_thin_grids(n, bc):
    test_rhs_at_tile_edges(n, bc)
    test_musta_rhs_at_tile_edges(n, bc)
    test_limited_rhs_at_tile_edges_is_bitwise(n, bc)


def kernel_us(n, kernel):
    """Mean time of one launch of a kernel class in a right-hand side, best of five."""
    h = H().from_workload(W.small_event(1, n=n, with_jet=False))
    U = torch.from_numpy(rough_state(n, 1)).cuda()
    best = 1e30
    for _ in range(5):
        h.profile(True)
        for _ in range(10):
            h.rhs(U, 1.0)
        torch.cuda.synchronize()
        ms, launches = h.profile_read()[kernel]
        h.profile(False)
        best = min(best, 1e3 * ms / launches)
    h.close()
    return best


def test_x_faces_of_thin_planes_cost_what_their_rows_do():
    """The same 256 rows of 256 cells as one row of each plane and as one plane:
    the x faces take their rows 16 at a time either way (one at a time: 31 against
    10 us)."""
    thin, flat = kernel_us((256, 1, 256), "xface"), kernel_us((256, 256, 1), "xface")
    print("x faces of 256x1x256 %.1f us, 256x256x1 %.1f us" % (thin, flat), flush=True)
    assert thin <= 2.0 * flat


@pytest.mark.parametrize("axis,kernel", [(0, "xface"), (1, "ymarch"), (2, "zmarch")])
def test_a_thin_axis_does_not_pay_for_a_full_tile(axis, kernel):
    """15 cells along an axis against 31, the same number of tiles: half the face
    rows (all 32 for both: 0.9 of the time)."""
    n = [512, 512, 512]
    times = []
    for m in (15, 31):
        n[axis] = m
        n[(axis + 1) % 3] = 320
        times.append(kernel_us(tuple(n), kernel))
    print("axis %d: 15 cells %.1f us, 31 cells %.1f us" % (axis, *times), flush=True)
    assert times[0] <= 0.75 * times[1]
