"""GPU parity of the bf16 decode attention at d_head 32 with contexts of more
than one key tile per wavefront (past 128 keys without a key split): prefill
and decode blocks against the oracle, logits within 2e-2 of the row maximum."""
import numpy as np
import pytest

import kf_synth as S
import oracle as O
from tests.parity_util import TOL, compare_head

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("B", [1, 3, 64])  # key splits of several tiles; fewer splits; no split
def test_dh32_many_key_tiles(B):
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = S.ModelConfig(2, 128, 4, 256, 512, 640, S.DTYPE_BF16)
    blob = S.pack_blob(cfg, S.make_weights(cfg, seed=4, random_affine=True))
    N, k = 301, 3
    kf = Bd.KForcing(Bd.make_config(cfg.n_layer, cfg.d_model, cfg.n_head, cfg.d_mlp, cfg.vocab,
                                    cfg.n_ctx, cfg.dtype, B, k, N, Bd.KF_FLAG_DEBUG_LOGITS))
    kf.load_weights(blob)
    model = O.Model(blob)
    prompt = S.prompts_uniform(7, B, N, cfg.vocab)
    rows = sorted({0, B // 2, B - 1})
    seqs = {b: model.seq() for b in rows}
    pending = {b: list(prompt[b]) for b in rows}
    for step in range(3):
        print(f"dh 32 B={B} step {step}", flush=True)
        u = S.noise_block(9, B, N + step * k, k)
        out = kf.prefill(prompt, k, u) if step == 0 else kf.decode_block(u)
        torch.cuda.synchronize()
        logits = kf.debug_logits(B * k).cpu().numpy().reshape(B, k, -1)
        toks = out.cpu().numpy()
        for b in rows:
            ol, _ = seqs[b].step(pending[b], u[b].astype(np.float64), commit=True)
            compare_head(logits[b], ol, toks[b], TOL[1], where=f"step {step} seq {b}")
            pending[b] = list(toks[b])
