"""GPU parity of the fp32 block attention (MFMA, 32-key tiles dealt to four
wavefronts up to 128 keys of context, to eight beyond) at key counts on both sides
of a 32-key tile, of a round of the wavefronts and of a 128-slot page, with 1, 15
and more than 16 query rows, every d_head, on a state buffer of NaN patterns (slots
past the end must not reach any output); logits within 1e-4 of the oracle."""
import numpy as np
import pytest

import kf_synth as S
import oracle as O
from tests.parity_util import TOL, compare_head

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_ctx,N", [(128, 1), (128, 27), (128, 97), (384, 122), (384, 249), (384, 300)])
@pytest.mark.parametrize("d,H", [(128, 4), (128, 2), (256, 2)], ids=["dh32", "dh64", "dh128"])
def test_fp32_attention(d, H, n_ctx, N):
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = S.ModelConfig(2, d, H, 256, 384, n_ctx, S.DTYPE_FP32)
    blob = S.pack_blob(cfg, S.make_weights(cfg, seed=5, random_affine=True))
    B = 3
    kf = Bd.KForcing(Bd.make_config(2, d, H, 256, 384, n_ctx, cfg.dtype, B, 8, N, Bd.KF_FLAG_DEBUG_LOGITS))
    kf.state.fill_(0xFF)
    torch.cuda.synchronize()
    kf.load_weights(blob)
    model = O.Model(blob)
    prompt = S.prompts_uniform(3, B, N, cfg.vocab)
    seqs, pending, p = [model.seq() for _ in range(B)], [list(x) for x in prompt], N
    for step, k in enumerate([4, 8, 7, 1, 3]):  # rows N + 4, 12, 15, 8, 4
        print(f"fp32 attention d={d} H={H} n_ctx={n_ctx} N={N} step {step}", flush=True)
        u = S.noise_block(8, B, p, k)
        out = kf.prefill(prompt, k, u) if step == 0 else kf.decode_block(u)
        torch.cuda.synchronize()
        logits = kf.debug_logits(B * k).cpu().numpy().reshape(B, k, -1)
        toks = out.cpu().numpy()
        for b in range(B):
            ol, _ = seqs[b].step(pending[b], u[b].astype(np.float64), commit=True)
            compare_head(logits[b], ol, toks[b], TOL[0], where=f"step {step} seq {b}")
            pending[b] = list(toks[b])
        p += k
    assert kf.device_errors() == 0
