"""The AR step's inverse-CDF selection from the head's tile partials, at
vocabularies on both sides of its edges: 128 columns per tile, 64 lanes with 8
tiles each in registers (65536 columns), a run of tiles per lane; u at both
ends of [0, 1).  The rule is the AR tests': the GPU's token equals the oracle's
inverse CDF (fp64) on the GPU's own fp32 logits, except where u lies within
1e-5 of a CDF boundary."""
import numpy as np
import pytest

import kf_synth as S
import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", [S.DTYPE_FP32, S.DTYPE_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("V", [2, 127, 128, 129, 8192, 8321, 65536, 65537, 70001])
def test_icdf_select(V, dtype):
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = S.ModelConfig(1, 64, 2, 64, V, 16, dtype)
    w = S.make_weights(cfg, seed=3)
    w["lnf_g"] = w["lnf_g"] * 30.0  # logits of standard deviation about 5: a few tokens hold the mass
    blob = S.pack_blob(cfg, w)
    B = 5 if V < 60000 else 40  # 32- and 64-row head tiles
    kf = Bd.KForcing(Bd.make_config(1, 64, 2, 64, V, 16, dtype, B, 1, 4, Bd.KF_FLAG_DEBUG_LOGITS))
    kf.load_weights(blob)
    prompt = S.prompts_uniform(5, B, 4, V)
    close = total = 0
    for step in range(4):
        u = S.noise_block(6, B, 4 + step, 1)[:, 0]
        u[:2] = (0.0, np.float32(1.0 - 2.0 ** -24))
        print(f"icdf V={V} dtype={dtype} step {step}", flush=True)
        out = kf.prefill_ar(prompt, u) if step == 0 else kf.decode_ar(u)
        torch.cuda.synchronize()
        logits = kf.debug_logits(B).cpu().numpy().astype(np.float64)
        toks = out.cpu().numpy()
        for b in range(B):
            total += 1
            if O.cdf_margin(logits[b], float(u[b])) < 1e-5:
                close += 1
                assert 0 <= toks[b] < V
                continue
            assert toks[b] == O.icdf(O.softmax(logits[b]), float(u[b])), (step, b)
    assert close <= total // 2 + 1
    assert kf.get_state() == (7, 1, B)
