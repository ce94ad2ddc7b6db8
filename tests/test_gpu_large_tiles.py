"""GPU parity of the large GEMM tiles, reached through prefills of many rows: 256 x
256 tiles on whole rounds with the rest of the rows in smaller ones, 160 x 128 and
128 x 128 tiles of four wavefronts (residual and folded-norm GEMMs, heads of more
than 128 rows), at row counts on and off the tile edges and at the shortest K of
the pipelined loop (two slabs); logits within 2e-2 of the oracle."""
import numpy as np
import pytest

import kf_synth as S
import oracle as O
from tests.parity_util import TOL, compare_head

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,H,f,B,N,k", [
    (1024, 16, 8192, 64, 60, 4),  # MLP-up: 4096 rows, exactly two rounds of 256 x 256 tiles
    (1024, 16, 8192, 65, 62, 3),  # 4225 rows: two rounds and 129 rows
    (512, 8, 256, 128, 60, 4),    # 8192 rows: residual GEMMs in 128 x 128 tiles
    (512, 8, 256, 129, 62, 3),    # 8385 rows: residual GEMMs in 160 x 128 tiles, the last ragged
    (128, 2, 256, 65, 61, 3),     # heads of 195 rows at the shortest K, two slabs
    (1024, 16, 256, 25, 58, 5),   # 1575 rows, K = 1024: QKV in 128 x 128 tiles, the last ragged
])
def test_large_tiles(d, H, f, B, N, k):
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = S.ModelConfig(2, d, H, f, 384, 72, S.DTYPE_BF16)
    blob = S.pack_blob(cfg, S.make_weights(cfg, seed=6, random_affine=True))
    kf = Bd.KForcing(Bd.make_config(2, d, H, f, 384, 72, cfg.dtype, B, k, N, Bd.KF_FLAG_DEBUG_LOGITS))
    kf.load_weights(blob)
    model = O.Model(blob)
    prompt = S.prompts_uniform(3, B, N, cfg.vocab)
    u = S.noise_block(8, B, N, k)
    print(f"large tiles d={d} f={f} rows={B * (N + k)}", flush=True)
    toks = kf.prefill(prompt, k, u).cpu().numpy()
    logits = kf.debug_logits(B * k).cpu().numpy().reshape(B, k, -1)
    for b in sorted({0, 1, 3, B // 2, B - 2, B - 1}):
        ol, _ = model.seq().step(list(prompt[b]), u[b].astype(np.float64), commit=True)
        compare_head(logits[b], ol, toks[b], TOL[1], where=f"seq {b}")
    assert kf.device_errors() == 0
