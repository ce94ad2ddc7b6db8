"""The prefill attention's softmax denominator is a sum of fp32 probabilities, not of
the bf16 ones that the value product uses.  A model of exact weights makes the first
key's probability 1 and gives all others one value that bf16 rounds up by 0.3 % and
more; only the first key has a value.  The output is then its value over the
denominator: a sum of rounded probabilities is off by that 0.3 % in every channel,
while the outputs' own rounding to bf16 (2^-8 at most, either way) averages out over
the channels (standard error 0.02 % over 59)."""
import math

import numpy as np
import pytest

import kf_synth as S
import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _bf16(x):
    return O._bf16_np(np.atleast_1d(np.float32(x)))


def _scores(dh):
    """bf16 query and key elements (q, w) whose probability exp(-q w / sqrt(dh)) bf16 rounds up most
    (at least 0.02 % away from the tie at 0.39 %)."""
    best = (0.0, 1.0, 1.0)
    for q in np.arange(1, 2, 1 / 128):
        for w in np.arange(3, 8, 1 / 32) * math.sqrt(dh) / 8:
            w = float(_bf16(w)[0])
            p = math.exp(-q * w / math.sqrt(dh))
            up = float(_bf16(p)[0]) / p - 1
            if best[0] < up < 0.0037 and 0.4 < p < 0.6:
                best = (up, q, w)
    return best


@pytest.mark.parametrize("d,H", [(64, 1), (64, 2), (128, 1)], ids=["dh64", "dh32", "dh128"])
def test_denominator_in_fp32(d, H):
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dh, N, V = d // H, 100, d + 2
    up, q, w = _scores(dh)
    assert up > 0.003
    cfg = S.ModelConfig(2, d, H, 64, V, 256, S.DTYPE_BF16)
    t = {name: np.zeros(shape, np.float32) for name, shape in S.tensor_table(cfg)}
    for name in t:
        if name.split(".")[-1].endswith("_g"):
            t[name][:] = 1.0
    signs = np.where(np.arange(d) % 2 == 0, 1.0, -1.0)
    signs[4], signs[5] = -1.0, 1.0          # channel 5 is +1, the sum stays 0
    t["tok_emb"][0] = signs                 # the first token: normalised channel 5 is 1
    t["tok_emb"][1] = signs
    t["tok_emb"][1, 4:6] = 0.0              # every other token: 0
    t["tok_emb"][2:] = np.eye(d)            # head rows that read the residual's channels
    t["noise_b2"][[d - 1, d - 3]] = 4.0, -4.0  # the noise row: channel 5 is 0 as well
    used = [c for c in range(d) if c not in (4, 5, d - 1, d - 2, d - 3)]
    v = _bf16(40.0 + 0.37 * np.arange(d))
    for h in range(H):
        t["l0.b_qkv"][h * dh] = q
        t["l0.w_qkv"][d + h * dh, 5] = w
    t["l0.w_qkv"][[2 * d + c for c in used], 5] = v[used]
    t["l0.w_o"][:] = np.eye(d)
    kf = Bd.KForcing(Bd.make_config(2, d, H, 64, V, 256, cfg.dtype, 1, 1, N, Bd.KF_FLAG_DEBUG_LOGITS))
    kf.load_weights(S.pack_blob(cfg, t))
    prompt = np.ones((1, N), np.int32)
    prompt[0, 0] = 0
    kf.prefill(prompt, 1, np.full((1, 1), 0.5, np.float32))
    torch.cuda.synchronize()
    l = kf.debug_logits(1).cpu().numpy().astype(np.float64)[0, 2:]
    out = 4.0 * (l - l[d - 2]) / (l[d - 1] - l[d - 2])
    p = math.exp(-q * w / math.sqrt(dh))
    want = v / (1.0 + N * p)
    ratio = out[used] / want[used]
    print(f"d={d} H={H}: rounding of the probabilities {up:.4%}, outputs {ratio.mean() - 1:+.4%}, "
          f"spread {ratio.std():.4%}", flush=True)
    assert np.abs(ratio - 1).max() < 2.0 ** -8 + 1e-4
    assert abs(ratio.mean() - 1) < 1e-3
