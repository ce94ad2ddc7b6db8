"""GPU parity of the GEMM epilogues that stage their tile as 16-bit rows (QKV
with the KV append, MLP-up), at the places where a tile is not whole: a QKV tile
of 96 columns that starts in the keys and ends in the values (d_model 1024 at
384 rows), value rows whose runs are not aligned to the cache's blocks of 4
slots, ragged rows, and rotary positions; logits within 2e-2 of the oracle."""
import numpy as np
import pytest

import kf_synth as S
import oracle as O
from tests.parity_util import TOL, compare_head

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rope", [False, True], ids=["positions", "rope"])
@pytest.mark.parametrize("d,H,B", [(1024, 16, 48), (1024, 16, 55), (128, 4, 5), (320, 5, 33)])
def test_half_epilogues(d, H, B, rope):
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = S.ModelConfig(2, d, H, 256, 384, 64, S.DTYPE_BF16, rms_rope=rope)
    blob = S.pack_blob(cfg, S.make_weights(cfg, seed=6, random_affine=True))
    kf = Bd.KForcing(Bd.make_config(2, d, H, 256, 384, 64, cfg.dtype, B, 5, 5,
                                    Bd.KF_FLAG_DEBUG_LOGITS | (Bd.KF_FLAG_RMS_ROPE if rope else 0)))
    kf.load_weights(blob)
    model = O.Model(blob)
    prompt = S.prompts_uniform(3, B, 5, cfg.vocab)
    rows = sorted({0, 1, B // 2, B - 1})
    seqs = {b: model.seq() for b in rows}
    pending = {b: list(prompt[b]) for b in rows}
    p = 5
    for step, k in enumerate([3, 5, 2, 1, 4]):  # rows 8, 8, 7, 3, 5; contexts 0, 5, 8, 13, 15
        print(f"half epilogues d={d} B={B} rope={rope} step {step}", flush=True)
        u = S.noise_block(8, B, p, k)
        out = kf.prefill(prompt, k, u) if step == 0 else kf.decode_block(u)
        torch.cuda.synchronize()
        logits = kf.debug_logits(B * k).cpu().numpy().reshape(B, k, -1)
        toks = out.cpu().numpy()
        for b in rows:
            ol, _ = seqs[b].step(pending[b], u[b].astype(np.float64), commit=True)
            compare_head(logits[b], ol, toks[b], TOL[1], where=f"step {step} seq {b}")
            pending[b] = list(toks[b])
        p += k
    assert kf.device_errors() == 0
