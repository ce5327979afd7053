"""The line adjoint where its workgroups differ: 8, 4, 2 or 1 lines by the
length and number of lines, long lines with all five fields, runs and turns of
the other weights and of single precision."""
import numpy as np
import pytest

import oracle as O
from paper_1511_02137_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")


def H():
    from paper_1511_02137_amd import hydro
    return hydro


def rough_state(n, seed):
    rng = np.random.default_rng(seed)
    shape = (n[2], n[1], n[0])
    U = np.empty((5,) + shape)
    U[0] = rng.uniform(1.0, 3.0, shape)
    U[1:4] = U[0] * rng.uniform(-0.4, 0.4, (3,) + shape)
    U[4] = rng.uniform(0.1, 1.0, shape)
    return U


def reverse(w, U, lam, precision, weno="z", bc="outflow", lines=0):
    h = H().from_workload(w, precision=precision, weno=weno, bc=(bc,) * 3, adjoint_k=1)
    h.set_option(H().OPT_ADJ_LINES, lines)
    x = torch.from_numpy(lam).to("cuda", h.dtype)
    h.adjoint_step(torch.from_numpy(U).to("cuda", h.dtype), 0, None, 1, x, None)
    torch.cuda.synchronize()
    out = x.double().cpu().numpy()
    h.close()
    return out


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("weno", ["z", "js", "linear"])
@pytest.mark.parametrize("n", [(72, 3, 4), (4, 72, 3), (130, 2, 3), (3, 130, 2), (2, 3, 130), (20, 18, 33)])
def test_runs_and_turns_of_every_weight(n, weno, bc):
    """<J^T W, V> of one step of a rough state against the oracle's forward mode,
    1e-10 of the sum of |products| (both are exact derivatives of the discrete
    map); the same bits whatever number of lines is asked for."""
    w = W.small_event(1, n=n, with_jet=False)
    pb = O.Problem(n=w.n, dx=w.dx, t0=w.t0, dt=w.dt, bc=(bc,) * 3, weno=weno)
    U0 = rough_state(n, sum(n))
    rng = np.random.default_rng(sum(n) + 1)
    V, Wt = rng.uniform(-1.0, 1.0, U0.shape), rng.uniform(-1.0, 1.0, U0.shape)
    _, JV = O.jvp(pb, U0, V, 1, [])
    outs = [reverse(w, U0, Wt, "f64", weno, bc, lines) for lines in (0, 1, 2, 4)]
    rel = abs(np.sum(outs[0] * V) - np.sum(Wt * JV)) / np.sum(np.abs(Wt * JV))
    print(n, weno, bc, "dot product %.2e" % rel, flush=True)
    assert rel <= 1e-10
    for o in outs[1:]:
        assert np.array_equal(o, outs[0])


@pytest.mark.parametrize("n", [(259, 3, 2), (300, 2, 4), (328, 3, 3), (3, 328, 2), (2, 3, 328)])
def test_long_lines_with_all_five_fields(n):
    """Lines of which four no longer fit a CU's LDS with five fields."""
    test_runs_and_turns_of_every_weight(n, "z", "outflow")


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", [(150, 3, 2), (3, 183, 2), (2, 5, 220), (500, 2, 3), (3, 2, 661), (20, 18, 33)])
def test_single_precision_turns(n, bc):
    """Single precision against double precision on the same state and adjoint,
    with more than one turn of runs along a line.  Bar: the adjoint of a rough
    state returns relative roundings (a few hundred of 2^-24 each, 2e-5) times
    its conditioning, a few: 1e-4 in relative L2; one wrong cell of a line is
    percents.  The same bits whatever number of lines is asked for."""
    w = W.small_event(1, n=n, with_jet=False)
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    U0 = f32(rough_state(n, sum(n)))
    lam = f32(np.random.default_rng(sum(n) + 1).uniform(-1.0, 1.0, U0.shape))
    ref = reverse(w, U0, lam, "f64", bc=bc) if max(n) <= 328 else None
    outs = [reverse(w, U0, lam, "f32", bc=bc, lines=lines) for lines in (0, 1, 2, 4)]
    for o in outs[1:]:
        assert np.array_equal(o, outs[0])
    if ref is None:  # beyond the double-precision limit: the oracle's forward mode
        pb = O.Problem(n=w.n, dx=w.dx, t0=w.t0, dt=w.dt, bc=(bc,) * 3)
        V = np.random.default_rng(sum(n) + 2).uniform(-1.0, 1.0, U0.shape)
        _, JV = O.jvp(pb, U0, V, 1, [])
        rel = abs(np.sum(outs[0] * V) - np.sum(lam * JV)) / np.sum(np.abs(lam * JV))
    else:
        rel = np.linalg.norm(outs[0] - ref) / np.linalg.norm(ref)
    print(n, bc, "FP32 %.2e" % rel, flush=True)
    assert rel <= 1e-4


def step_us(n, precision, lines):
    h = H().from_workload(W.small_event(1, n=n, with_jet=False), precision=precision, adjoint_k=1)
    h.set_option(H().OPT_ADJ_LINES, lines)
    U = torch.from_numpy(rough_state(n, 1)).to("cuda", h.dtype)
    lam = torch.zeros_like(U)
    best = 1e30
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            h.adjoint_step(U, 0, None, 1, lam, None)
        b.record()
        torch.cuda.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b) / 5)
    h.close()
    return best


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("lines", [1, 2])
def test_a_limit_on_the_lines_costs_no_time(precision, lines):
    """HYDRO_OPT_ADJ_LINES = 1 or 2, the best settings of the one-lane-per-face
    form, were taken literally by the runs of faces: 128x64x64 2.9 ms a step
    against 0.8 (FP64), 1.1 against 0.55 (FP32)."""
    n = (128, 64, 64)
    free, limited = step_us(n, precision, 0), step_us(n, precision, lines)
    print("%s: no limit %.0f us, %d lines %.0f us" % (precision, free, lines, limited), flush=True)
    assert limited <= 1.3 * free


# y and z lines in segments: two and three, even and with a shorter last one
SEGMENTED = [(3, 161, 2), (2, 200, 3), (4, 256, 3), (2, 3, 257), (3, 5, 163), (5, 328, 2)]


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", SEGMENTED)
def test_lines_in_segments(n, bc):
    for weno in ("z", "js", "linear"):
        test_runs_and_turns_of_every_weight(n, weno, bc)


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", [(3, 256, 2), (2, 3, 257), (4, 401, 2), (2, 500, 3), (3, 2, 670)])
def test_single_precision_lines_in_segments(n, bc):
    test_single_precision_turns(n, bc)
