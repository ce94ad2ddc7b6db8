"""Training attention on grids large enough for 32 query rows per wavefront (256
heads; small grids of d_head 32 and 64 run 16 rows per wavefront), at row counts
around the edges of the 128-row workgroup and the 32-row wavefront: two heads'
inputs repeated over the grid, the first two outputs against the masked reference
within the tolerance of the other shapes, every repeat bit for bit the same."""
import pytest

import kf_synth as S
import oracle as O
from tests.test_gpu_training_attention import KIND, _bd, _check, _run

pytestmark = pytest.mark.gpu
np = pytest.importorskip("numpy")


@pytest.mark.parametrize("mask,N,k,dh", [(0, 43, 2, 64), (0, 32, 3, 64), (0, 127, 1, 64), (0, 129, 2, 64),
                                         (1, 21, 3, 64), (1, 65, 1, 64), (1, 16, 5, 64),
                                         (0, 129, 1, 32), (1, 130, 2, 32)])
def test_large_grid(mask, N, k, dh):
    Bd = _bd()
    rows, keys = Bd.training_attention_shapes(mask, N, k)
    print(f"large grid {KIND[mask]} N={N} k={k} dh={dh}", flush=True)
    q, k_, v = S.attention_batch(11 + N, 1, 2, rows, keys, dh, 1.0)
    got = _run(Bd, mask, *(np.tile(x, (32, 4, 1, 1)) for x in (q, k_, v)), N, k, dh ** -0.5)
    ref = O.masked_attention(q, k_, v, O.training_mask(KIND[mask], N, k), dh ** -0.5)
    _check(got[:1, :2], ref, f"{KIND[mask]} N={N} k={k} dh={dh}")
    assert np.array_equal(got, np.tile(got[:1, :2], (32, 4, 1, 1)))
