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


@pytest.mark.parametrize("B,M,budget", [(3, 1, None), (130, 4, None), (6, 2, 0)])
def test_gradient_by_chains_per_compute_unit(B, M, budget):
    """N = 64 with few chains, with more than two chains per compute unit, and
    with no wave kept (the gradient recomputes them)."""
    print(f"gradient N=64 S=3 B={B} M={M} budget={budget}", flush=True)
    c = Case(synth.small_case(N=64, S=3, M=M, B=B, H=110, W=121, seed=43))
    _check_grads(c, c.engine(wave_budget=budget))
