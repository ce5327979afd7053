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
