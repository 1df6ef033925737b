"""The expert GEMMs at the edges of their launches, in every weight format, against the float64
oracle: reductions with a partial last step (and shorter than one step), under one- and
two-tile gate/up launches and narrow and wide down launches."""
import pytest

import test_gpu_ffn
import test_gpu_fp8
import test_gpu_mxfp4

pytestmark = pytest.mark.gpu
RUN = {"bf16": test_gpu_ffn._run, "fp8": test_gpu_fp8._run, "mxfp4": test_gpu_mxfp4._run}
FORMATS = pytest.mark.parametrize("fmt", list(RUN))


def _case(fmt, T, N, k, d, f, M, label):
    RUN[fmt](dict(N=N, k=k, d=d, f=f, T=T, logits="domains", Q=3), 5, 1, M,
             label=f"{label} {fmt} T{T} N{N} d{d} f{f} M{M}")


# the steps are 64, 128 or 256 elements: every count of 32-element groups in a partial step,
# alone (d or f below one step) and after whole ones
@FORMATS
@pytest.mark.parametrize("d,f", [(32, 32), (64, 96), (96, 224), (160, 192), (224, 288),
                                 (288, 320), (352, 480), (544, 160), (480, 416)])
def test_partial_steps(fmt, d, f):
    for T, N, k, M in [(5, 6, 2, 3), (41, 5, 2, 3)]:      # 1-8 rows an expert; up to 41
        _case(fmt, T, N, k, d, f, M, "partial step")


# grids of at least 768 blocks: two column tiles per gate/up wave, wide down waves
@FORMATS
def test_partial_steps_wide_launches(fmt):
    _case(fmt, 40, 120, 16, 288, 928, 110, "two tiles")
    _case(fmt, 40, 120, 16, 1760, 160, 110, "wide down")
