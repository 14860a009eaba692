"""Slots of templates whose stages are joined hold what those touch and no more (host
only): the input, the output, the blocks' partial results and arrival words."""
import pytest

from paper_2606_05495_amd import _abi as A


def _slot(pipeline, w, h, flags=0):
    cfg = A.set_config()
    cfg.abi_version = A.SET_ABI_VERSION
    cfg.num_workers, cfg.slots_per_worker = 2, 3
    t = A.set_job_template()
    t.pipeline, t.width, t.height, t.flags = pipeline, w, h, flags
    slot, total = A.set_template_footprint(cfg, t)
    assert total == 6 * slot
    return slot


@pytest.mark.parametrize("w,h", [(1, 1), (17, 65), (256, 256), (640, 639), (2048, 2048)])
def test_box_histogram(w, h):
    """The input, a kilobyte for the output and for every 4096 pixels, and rounding."""
    assert _slot(A.SET_PIPE_BOX_HIST_U8, w, h) <= w * h + 1024 * (-(-w * h // 4096)) + 1024 + 6 * 256
    # the template that returns its images still has three bytes a pixel for them
    assert _slot(A.SET_PIPE_BOX_HIST_U8, w, h, A.SET_TF_DEBUG) >= 4 * w * h


@pytest.mark.parametrize("w,h", [(1, 1), (17, 65), (256, 256), (1020, 1024), (1037, 771), (2099, 2101)])
def test_one_kernel_image(w, h):
    """The input, ten bytes a tile of 16 x 64 pixels (partials and arrivals), and rounding."""
    tiles = -(-w // 64) * -(-h // 16)
    assert _slot(A.SET_PIPE_GAUSS_SOBEL_F32, w, h) <= 4 * w * h + 10 * tiles + 8 * 256
    assert _slot(A.SET_PIPE_GAUSS_SOBEL_F32, w, h, A.SET_TF_DEBUG) >= 9 * w * h
