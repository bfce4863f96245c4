"""The paths a call takes by its sizes: each side of a dispatch rule against
the FP64 oracle, at the sizes where a rule or a remainder changes."""
import numpy as np
import pytest

from paper_2505_07814_amd import synth

from test_gpu_parity import Case, _check_grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,H,W", [(1, 97, 130), (2, 353, 340)])
def test_scatter_tiles_and_more_than_64_rows(S, H, W):
    """Object gradient with 8-row tiles (few tiles) and 32-row tiles, over a
    batch of more rows than one wave tests at once; ragged object sides."""
    print(f"scatter S={S} H={H} W={W} B=67", flush=True)
    c = Case(synth.small_case(N=64, S=S, M=1, B=67, H=H, W=W, seed=41))
    _check_grads(c, c.engine())
