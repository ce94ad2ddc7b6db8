"""The AR step's inverse-CDF selection from the head's tile partials, at
vocabularies on both sides of its edges: 128 columns per tile, 64 lanes with 8
tiles each in registers (65536 columns), a run of tiles per lane; u at both
ends of [0, 1).  The rule is the AR tests': the GPU's token equals the oracle's
inverse CDF (fp64) on the GPU's own fp32 logits, except where u lies within
1e-5 of a CDF boundary; there the token has mass and its interval of the CDF holds
u up to 1e-5.  At u = 0 it is the first token with mass."""
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
    exact = 0
    for step in range(4):
        u = S.noise_block(6, B, 4 + step, 1)[:, 0]
        u[:2] = (0.0, np.float32(1.0 - 2.0 ** -24))
        print(f"icdf V={V} dtype={dtype} step {step}", flush=True)
        out = kf.prefill_ar(prompt, u) if step == 0 else kf.decode_ar(u)
        torch.cuda.synchronize()
        logits = kf.debug_logits(B).cpu().numpy().astype(np.float64)
        toks = out.cpu().numpy()
        for b in range(B):
            mass = np.exp(logits[b] - logits[b].max()).astype(np.float32)
            F = np.cumsum(O.softmax(logits[b]))
            t = int(toks[b])
            assert 0 <= t < V and mass[t] > 0, (step, b, t)
            if u[b] == 0.0:
                assert t == np.nonzero(mass)[0][0], (step, b, t)
            elif O.cdf_margin(logits[b], float(u[b])) < 1e-5:
                assert (F[t - 1] if t else 0.0) <= u[b] + 1e-5 and u[b] < F[t] + 1e-5, (step, b, t)
            else:
                exact += 1
                assert t == O.icdf(O.softmax(logits[b]), float(u[b])), (step, b)
    # small vocabularies have few boundaries: of the other 12 rows hardly any lies within 1e-5 of one
    assert V > 1000 or exact >= 11
    assert kf.get_state() == (7, 1, B)


def _crafted(rng, V):
    """Logits (exact in bf16) of a few tokens with mass among tokens without any
    (exp(-200) is 0 in fp32), and uniforms at the CDF's boundaries and up to
    three fp32 steps to both sides of them."""
    logits = np.full(V, -200.0, np.float32)
    at = np.sort(rng.choice(V, rng.integers(2, 40), replace=False))
    logits[at] = rng.integers(-16, 17, at.size) / 4.0
    logits[at[rng.random(at.size) < 0.3]] = -24.0  # too little to show in a sum with the others
    logits[at[-1]] = 4.0
    F = np.cumsum(O.softmax(logits.astype(np.float64)))
    us = [0.0, np.float32(1.0 - 2.0 ** -24)]
    for m in rng.choice(at, 9):
        lo = hi = np.float32(F[m])
        us.append(lo)
        for _ in range(3):
            lo, hi = np.nextafter(lo, np.float32(0)), np.nextafter(hi, np.float32(2))
            us += [lo, hi]
    us = np.array(us, np.float32)
    return logits, F, np.where(us < 1, us, us[1])


@pytest.mark.parametrize("dtype", [S.DTYPE_FP32, S.DTYPE_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("V", [257, 8321, 70001])
def test_only_tokens_with_mass(V, dtype):
    """At and beside the boundaries of the CDF, where rounding decides, the token
    has positive probability (at u = 0 it is the first that has) and its interval of the CDF holds u up to the fp32
    error of the sums (under 40 terms and 64 tiles: 4e-6 is 64 roundings).  A
    final-norm gain of 0 makes the logits the table's products with the shift."""
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = S.ModelConfig(1, 64, 2, 64, V, 16, dtype)
    w = S.make_weights(cfg, seed=3)
    w["lnf_g"][:] = 0.0
    w["lnf_b"][:] = 0.0
    w["lnf_b"][0] = 1.0
    rng = np.random.default_rng(V)
    kf = None
    for trial in range(12):
        logits, F, us = _crafted(rng, V)
        w["tok_emb"][:, 0] = logits
        if kf is None:
            kf = Bd.KForcing(Bd.make_config(1, 64, 2, 64, V, 16, dtype, us.size, 1, 4, Bd.KF_FLAG_DEBUG_LOGITS))
        kf.load_weights(S.pack_blob(cfg, w))
        print(f"icdf mass V={V} dtype={dtype} trial {trial}", flush=True)
        toks = kf.prefill_ar(S.prompts_uniform(5, us.size, 2, V), us).cpu().numpy()
        assert np.array_equal(kf.debug_logits(us.size).cpu().numpy(), np.tile(logits, (us.size, 1)))
        assert (logits[toks] > -200).all(), (trial, toks[logits[toks] == -200])
        assert (toks[us == 0] == np.nonzero(logits > -200)[0][0]).all(), trial
        below = np.where(toks > 0, F[toks - 1], 0.0)
        assert (below <= us + 4e-6).all() and (us < F[toks] + 4e-6).all(), trial
