"""GPU parity of the prefill's block attention: steps of many rows per sequence
over the paged KV cache, at row counts on both sides of the kernel's edges (32
rows per wavefront, 64 keys per tile, 128 keys per page), every d_head, in
lock-step and through a served sequence's page table.

The state buffer is filled with NaN bit patterns first: slots of a page that no
row of the step wrote must not reach any output.  Tolerance: the models' own
(logits within 2e-2 of the oracle's row maximum, bf16)."""
import numpy as np
import pytest

import kf_synth as S
import oracle as O
from tests.parity_util import TOL, compare_head

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (at d_head 64 grids of 64 to 255 blocks of 16 rows stay with the decode kernel,
# so 2 heads cover the small row counts and 8 heads the large ones)
MODELS = {"32": S.ModelConfig(2, 128, 4, 256, 512, 384, S.DTYPE_BF16),
          "64": S.ModelConfig(2, 128, 2, 256, 512, 384, S.DTYPE_BF16),
          "64x8": S.ModelConfig(2, 512, 8, 256, 512, 384, S.DTYPE_BF16),
          "128": S.ModelConfig(2, 256, 2, 256, 512, 384, S.DTYPE_BF16)}
# (prompt, k): rows prompt + k of 32, 33, 63, 65, 127, 128, 131, 257, 384 (the whole context)
SHAPES = [(30, 2), (29, 4), (60, 3), (64, 1), (124, 3), (124, 4), (127, 4), (255, 2), (380, 4)]


def _ctx(cfg, blob, B, N, k, served):
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kf = Bd.KForcing(Bd.make_config(cfg.n_layer, cfg.d_model, cfg.n_head, cfg.d_mlp, cfg.vocab,
                                    cfg.n_ctx, cfg.dtype, B, k, N, Bd.KF_FLAG_DEBUG_LOGITS |
                                    (Bd.KF_FLAG_SERVING if served else 0)))
    kf.state.fill_(0xFF)
    torch.cuda.synchronize()
    kf.load_weights(blob)
    return kf


@pytest.mark.parametrize("served", [False, True], ids=["lockstep", "served"])
@pytest.mark.parametrize("dh", list(MODELS))
def test_prefill_rows(dh, served):
    cfg = MODELS[dh]
    blob = S.pack_blob(cfg, S.make_weights(cfg, seed=4, random_affine=True))
    model = O.Model(blob)
    B = 3
    kf = _ctx(cfg, blob, B, 380, 4, served)
    slots = [2, 0, 1]
    for N, k in SHAPES:
        print(f"prefill attention dh={dh} served={served} rows={N + k}", flush=True)
        prompt = S.prompts_uniform(N, B, N, cfg.vocab)
        u = S.noise_block(N, B, N, k)
        out = kf.serve_admit(slots, prompt, k, u) if served else kf.prefill(prompt, k, u)
        torch.cuda.synchronize()
        logits = kf.debug_logits(B * k).cpu().numpy().reshape(B, k, -1)
        toks = out.cpu().numpy()
        for b in range(B):
            ol, _ = model.seq().step(list(prompt[b]), u[b].astype(np.float64), commit=True)
            compare_head(logits[b], ol, toks[b], TOL[1], where=f"rows {N + k} seq {b}")
        if served:
            kf.serve_release(slots)
    assert kf.device_errors() == 0
