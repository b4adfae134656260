"""Host-side checks of the two-stream step wrapper (no GPU needed): the
package exports it, and a bad schedule name is rejected before any stream or
device is touched."""
import pytest

import paper_1905_07931_amd as L1


def test_step_api_is_exported():
    assert "l1_step" in L1.__all__ and "side_stream" in L1.__all__
    assert callable(L1.l1_step) and callable(L1.side_stream)


@pytest.mark.parametrize("bad", ["parallel", "", "Serial", None])
def test_unknown_schedule_rejected_before_any_device_work(bad):
    with pytest.raises(ValueError):
        L1.l1_step(None, None, None, 0.01, 1e-4, Y=None, dX=None, dW=None, csc=None, out=None,
                   schedule=bad)


def test_schedule_asks_which_path_a_product_takes():
    # both schedules timed: the fork pays for tiled products and for packed ones of 2 million
    # weights on; row kernels (short products, batches that are no multiple of 4) run serially
    from paper_1905_07931_amd.step import two_stream_pays

    def pays(N, K, B, density):
        return two_stream_pays(L1.CSR(N, K, None, None, None, int(density * N * K)), B)

    for case in [(4096, 9216, 1024, .09), (4096, 4096, 512, .05), (4096, 4096, 512, .5), (2000, 2000, 512, .3),
                 (2049, 3001, 333, .1), (500, 8000, 1024, .05)]:
        assert pays(*case), case
    for case in [(300, 784, 64, .1), (1024, 1024, 1024, .4), (2000, 700, 1000, .25), (2049, 3001, 333, .05),
                 (4096, 4096, 333, .05), (2048, 4096, 333, .05), (4096, 4096, 512, .02)]:
        assert not pays(*case), case
