"""Launch shapes of the batch API: what the options report, what the tuner
takes from its cache, and batches of more tiles than one launch holds."""
import pytest

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


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_default_launch_shape_is_reported(precision):
    """The shape that a new batch reports is the one that it launches, one
    workgroup per tile (0)."""
    b = H().batch_from_workloads([W.small_event(1, n=(20, 18, 16)), W.small_event(2, n=(40, 9, 33))],
                                 precision=precision)
    for a in (H().BOPT_BLOCKS_X, H().BOPT_BLOCKS_Y, H().BOPT_BLOCKS_Z):
        assert b.get_option(a) == 0, (a, b.get_option(a))
    b.close()


def test_shapes_timed_with_other_kernels_are_not_taken(tmp_path):
    """A cache line written before the x faces took line tiles (its key names no
    form of the kernels, bx counts groups of whole rows) is a miss: the batch is
    timed and its line appended, which the next batch takes."""
    p = torch.cuda.get_device_properties(0)
    n = (20, 18, 16)
    key = "%s:%d:p1:w0:l0:f0:0:%s" % (p.gcnArchName, p.multi_processor_count, "x".join(map(str, n)))

    def line(key):
        h = 1469598103934665603
        for c in key.encode():
            h = ((h ^ c) * 1099511628211) % 2 ** 64
        return "%016x 512 768 1024 1\n" % h

    cache = tmp_path / "tune.txt"
    # musta_k is part of the key whatever the flux is
    b = H().batch_from_workloads([W.small_event(1, n=n)], precision="f32")
    old = key.replace(":f0:0:", ":f0:%d:" % b.cfgs[0].musta_k)
    cache.write_text(line(old))
    assert b.autotune(str(cache)) is False
    lines = cache.read_text().splitlines()
    assert len(lines) == 2 and lines[1].split()[0] != lines[0].split()[0]
    picks = [b.get_option(a) for a in (0, 1, 2)]
    b.close()
    b = H().batch_from_workloads([W.small_event(1, n=n)], precision="f32")
    assert b.autotune(str(cache)) is True
    assert [b.get_option(a) for a in (0, 1, 2)] == picks
    b.close()


@pytest.mark.parametrize("graph", [1, 0])
def test_more_tiles_than_one_launch_holds(graph):
    """129 events of 1 x 1 x 65535 cells: 129 x 65535 x tiles, above the 2^32 / 512
    workgroups of one launch; the first and last events step bit for bit as alone."""
    n, k = (1, 1, 65535), 129
    assert n[2] * k > 2 ** 32 // 512
    w = W.Workload(name="thin", n=n, dx=(0.1,) * 3, t0=1.0, dt=0.02, steps=1,
                   prim0=W.ellipsoid_prim(n, (0.1,) * 3, (1.0, 1.0, 500.0), 30.0), jets=[])
    h = H().from_workload(w, precision="f32")
    h.step(1)
    torch.cuda.synchronize()
    one = h.U.clone()
    h.close()
    prim = torch.from_numpy(w.prim0).cuda()
    b = H().Batch([H().make_config(n, dt=w.dt, precision="f32")] * k, [prim] * k)
    b.set_option(H().BOPT_GRAPH, graph)
    b.run(1)
    torch.cuda.synchronize()
    assert torch.equal(b.U[0], one) and torch.equal(b.U[k - 1], one)
    b.close()
