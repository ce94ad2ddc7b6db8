"""GPU parity of the block attention of steps of 32 rows and more through each of its
kernels (key splits, eight wavefronts, the tiled kernel of prefills): decode blocks of
k = 16 and 17 at contexts that are no multiples of a tile or a page, in lock-step and
through served sequences' page tables, and prefills of many sequences, on a state
buffer of NaN patterns (slots past the end must not reach any output); logits within
2e-2 of the oracle's row maximum.  That each shape reaches the kernel it names is
tested on the CPU (test_routes.py)."""
import numpy as np
import pytest

import kf_synth as S
import oracle as O
from tests.parity_util import TOL, compare_head

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (kernel, d_model, heads, sequences, context capacity, prompt)
DECODE = [("tiled", 512, 8, 16, 384, 70), ("tiled", 512, 16, 18, 384, 70), ("tiled", 256, 2, 3, 256, 103),
          ("tiled", 128, 4, 3, 384, 190), ("tiled", 256, 2, 43, 384, 61),
          ("split", 128, 2, 3, 384, 190), ("split", 256, 2, 3, 384, 190), ("split", 128, 4, 3, 640, 440),
          ("wide", 512, 8, 4, 384, 103)]
KS = [17, 16, 17, 16, 16, 17]  # the prefill's k, then decode blocks of 33, 33, 33, 32, 33 rows
# (d_model, heads, sequences, rows), the tiled kernel without splits in its place
PREFILL = [(512, 8, 5, 257), (512, 8, 16, 97), (512, 16, 4, 257), (512, 16, 3, 384), (256, 2, 11, 200)]


def _context(cfg, B, k, N, served):
    from paper_2606_10820_amd import binding as Bd
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    blob = S.pack_blob(cfg, S.make_weights(cfg, seed=4, random_affine=True))
    kf = Bd.KForcing(Bd.make_config(cfg.n_layer, cfg.d_model, cfg.n_head, cfg.d_mlp, cfg.vocab, cfg.n_ctx, cfg.dtype,
                                    B, k, N, Bd.KF_FLAG_DEBUG_LOGITS | (Bd.KF_FLAG_SERVING if served else 0)))
    kf.state.fill_(0xFF)
    torch.cuda.synchronize()
    kf.load_weights(blob)
    return kf, O.Model(blob)


@pytest.mark.parametrize("served", [False, True], ids=["lockstep", "served"])
@pytest.mark.parametrize("kernel,d,H,B,n_ctx,N", DECODE)
def test_decode_blocks_of_many_rows(kernel, d, H, B, n_ctx, N, served):
    cfg = S.ModelConfig(2, d, H, 256, 384, n_ctx, S.DTYPE_BF16)
    kf, model = _context(cfg, B, 17, N, served)
    prompt = S.prompts_uniform(N, B, N, cfg.vocab)
    slots = np.random.default_rng(1).permutation(B).astype(np.int32)
    rows = sorted({0, B // 2, B - 1})
    seqs = {b: model.seq() for b in rows}
    pending = {b: list(prompt[b]) for b in rows}
    p = N
    for step, k in enumerate(KS):
        print(f"{kernel} d={d} H={H} B={B} served={served} step {step} at {p}", flush=True)
        u = S.noise_block(8, B, p, k)
        if served:
            out = kf.serve_admit(slots, prompt, k, u) if step == 0 else kf.serve_step(slots, u)
        else:
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


@pytest.mark.parametrize("d,H,B,rows", PREFILL)
def test_prefills_of_many_sequences(d, H, B, rows):
    cfg = S.ModelConfig(2, d, H, 256, 384, 384, S.DTYPE_BF16)
    k, N = 3, rows - 3
    kf, model = _context(cfg, B, k, N, False)
    prompt = S.prompts_uniform(N, B, N, cfg.vocab)
    u = S.noise_block(N, B, N, k)
    print(f"prefill d={d} H={H} B={B} rows={rows}", flush=True)
    toks = kf.prefill(prompt, k, u).cpu().numpy()
    logits = kf.debug_logits(B * k).cpu().numpy().reshape(B, k, -1)
    for b in sorted({0, B // 2, B - 1}):
        ol, _ = model.seq().step(list(prompt[b]), u[b].astype(np.float64), commit=True)
        compare_head(logits[b], ol, toks[b], TOL[1], where=f"seq {b}")
    assert kf.device_errors() == 0
