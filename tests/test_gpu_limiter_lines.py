"""Limited faces against the oracle where the x tiles differ from the y and z
ones (16 rows of any plane, pitch 17) and from the marches that those are
compared with: extents around tiles of 31, 32 and 15 cells, ragged rows, and
batches that walk tiles of both lengths."""
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


def decades(n, seed):
    """An admissible state whose cells differ by up to six decades: many faces are limited."""
    rng = np.random.default_rng(seed)
    shape = (n[2], n[1], n[0])
    U = np.empty((5,) + shape)
    U[0] = rng.uniform(1.0, 3.0, shape)
    U[1:4] = U[0] * rng.uniform(-0.4, 0.4, (3,) + shape)
    U[4] = rng.uniform(0.1, 1.0, shape)
    return U * 10.0 ** rng.uniform(-6.0, 0.0, shape)


XSHAPES = [(1, 3, 2), (14, 17, 3), (15, 5, 7), (16, 9, 2), (31, 5, 3), (32, 7, 3), (33, 1, 20), (62, 3, 5), (63, 5, 4),
           (64, 5, 2), (65, 2, 9), (96, 3, 1)]


@pytest.mark.parametrize("bc", ["outflow", "periodic"])
@pytest.mark.parametrize("n", XSHAPES)
def test_limited_rhs_against_the_oracle(n, bc):
    """Bar: 128 roundings of max |U| sum 1/dx as for the unlimited faces, or ten
    times what the oracle's own right-hand side moves by when every value of the
    state changes by four roundings (the limiter's weight is a quotient of
    differences that may be small), whichever is more."""
    w = W.small_event(1, n=n, with_jet=False)
    rng = np.random.default_rng(sum(n))
    for precision, weno, u in (("f64", "z", 2.0 ** -53), ("f64", "z5", 2.0 ** -53), ("f64", "js", 2.0 ** -53),
                               ("f32", "z", 2.0 ** -24)):
        U = decades(n, sum(n) + 2)
        if precision == "f32":
            U = U.astype(np.float32).astype(np.float64)
        pb = O.Problem(n=w.n, dx=w.dx, t0=w.t0, dt=w.dt, bc=(bc,) * 3, weno=weno, limiter="pp")
        Lo, _, _ = O.rhs(pb, U, 1.0, [])
        Lu, _, _ = O.rhs(O.Problem(n=w.n, dx=w.dx, t0=w.t0, dt=w.dt, bc=(bc,) * 3, weno=weno), U, 1.0, [])
        moves = 0.0
        for _ in range(3):
            Lp, _, _ = O.rhs(pb, U * (1.0 + 4.0 * u * rng.choice([-1.0, 1.0], U.shape)), 1.0, [])
            moves = max(moves, np.abs(Lp - Lo).max())
        h = H().from_workload(w, precision=precision, weno=weno, bc=(bc,) * 3, limiter="pp")
        L = h.rhs(torch.from_numpy(U).to("cuda", h.dtype), 1.0).double().cpu().numpy()
        h.close()
        bar = max(128 * u * np.abs(U).max() * 30.0, 10.0 * moves)
        err, acts = np.abs(L - Lo).max(), np.abs(Lu - Lo).max()
        print(n, bc, precision, weno, "max |dL| %.2e bar %.2e, the limiter moves L by %.2e" % (err, bar, acts), flush=True)
        assert err <= bar
        assert acts > 100.0 * bar  # a face left as it was would show


@pytest.mark.parametrize("blocks", [1, 3, 5])
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("limiter", ["none", "pp"])
def test_walked_batch_of_mixed_tile_lengths_is_bitwise(precision, limiter, blocks):
    # tile lengths 31 and 32 in one batch: a few workgroups walk all the tiles
    # and use their LDS again
    ws = [W.small_event(k, n=n) for k, n in enumerate([(31, 64, 20), (32, 31, 33), (5, 40, 62)])]
    single = []
    for w in ws:
        h = H().from_workload(w, precision=precision, limiter=limiter)
        h.step(2)
        torch.cuda.synchronize()
        single.append(h.U.clone())
        h.close()
    b = H().batch_from_workloads(ws, precision=precision, limiter=limiter)
    for a in (H().BOPT_BLOCKS_X, H().BOPT_BLOCKS_Y, H().BOPT_BLOCKS_Z):
        b.set_option(a, blocks)
    b.run(2)
    torch.cuda.synchronize()
    for e, U in enumerate(single):
        assert torch.equal(b.U[e], U), e
    b.close()
