"""The linear calls on lengths that keep the runtime plan (no compiled stages).

Rows and columns beyond 1024 points or below 32, Z lengths beyond 128; some are no
multiple of eight, whose twiddles are folded into an eighth turn one by one.  The
check and its bounds are those of the ragged shapes."""

import pytest

from tests.test_gpu_ragged import test_linear_calls as check

pytestmark = pytest.mark.gpu

SHAPES = [(2, 36, 1250), (3, 1250, 36), (2, 32, 1350), (2, 1350, 30), (1, 1280, 1250), (2, 40, 1536), (2, 1620, 32),
          (135, 30, 32), (225, 32, 30), (150, 36, 40), (250, 30, 36), (2, 24, 20), (3, 10, 24)]


@pytest.mark.parametrize("shape", SHAPES)
def test_linear_calls(gpu_lib, shape):
    check(gpu_lib, shape)
