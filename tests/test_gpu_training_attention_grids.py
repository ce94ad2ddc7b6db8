"""Training attention on grids large enough for 32 query rows per wavefront (small
or badly filled grids run 16 rows per wavefront), at row counts around the edges of
the 128-row workgroup and the 32-row wavefront that reach it, and around the border
of M_D's two halves: two heads' inputs repeated over the grid, the first two outputs
against the masked reference within the tolerance of the other shapes, every repeat
bit for bit the same."""
import pytest

import kf_synth as S
import oracle as O
from tests.test_gpu_training_attention import KIND, _bd, _check, _run

pytestmark = pytest.mark.gpu
np = pytest.importorskip("numpy")

# (mask, N, k, d_head, heads): rows N (1 + k) of 66 to 800 under M_S
LARGE = [(0, 33, 1, 128, 384), (0, 32, 2, 128, 384), (0, 32, 3, 128, 384), (0, 100, 1, 128, 256),
         (0, 127, 1, 64, 512), (0, 85, 2, 64, 512), (0, 128, 1, 64, 512), (0, 128, 4, 64, 256),
         (0, 127, 1, 32, 512), (0, 160, 3, 32, 256),
         (0, 129, 1, 128, 200), (0, 43, 2, 128, 200), (0, 32, 4, 128, 200), (0, 160, 4, 32, 512),
         (1, 64, 1, 128, 384), (1, 16, 4, 128, 384)]
# M_D halves of N k rows: a workgroup and a wavefront across the border (25, 50, 100, 492,
# 495, 511: blocks cut from row 0 on), each half by itself (512, 513, 535, 600, 1250)
HALVES = [(1, 25, 2, 128, 384), (1, 50, 1, 128, 400), (1, 100, 1, 128, 256), (1, 100, 1, 64, 512),
          (1, 123, 4, 64, 128), (1, 123, 4, 32, 128), (1, 165, 3, 128, 64), (1, 73, 7, 128, 64),
          (1, 64, 8, 128, 64), (1, 128, 4, 64, 128), (1, 171, 3, 128, 64), (1, 107, 5, 128, 64),
          (1, 200, 3, 128, 64), (1, 250, 5, 64, 64), (1, 250, 5, 32, 64)]


@pytest.mark.parametrize("mask,N,k,dh,heads", LARGE + HALVES)
def test_large_grid(mask, N, k, dh, heads):
    Bd = _bd()
    rows, keys = Bd.training_attention_shapes(mask, N, k)
    print(f"large grid {KIND[mask]} N={N} k={k} dh={dh} heads={heads}", flush=True)
    q, k_, v = S.attention_batch(11 + N, 1, 2, rows, keys, dh, 1.0)
    rep = (heads // 8, 4, 1, 1)
    got = _run(Bd, mask, *(np.tile(x, rep) for x in (q, k_, v)), N, k, dh ** -0.5)
    ref = O.masked_attention(q, k_, v, O.training_mask(KIND[mask], N, k), dh ** -0.5)
    _check(got[:1, :2], ref, f"{KIND[mask]} N={N} k={k} dh={dh}")
    assert np.array_equal(got, np.tile(got[:1, :2], rep))
