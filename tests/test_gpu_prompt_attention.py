"""The prompt's attention (head_dim 128) at the edges of its 32-key steps: the
rows of a state's buffer past the last key a block sees are never read into the
result, whatever they hold; and the softmax sum of the prompt is that of a
forward (fp32 probabilities, not the rounded ones of the value product); and a
non-finite prompt row reaches no token before its group of 16.

Tolerance: TOL_STAGE, the stage tolerance every parity test uses, unless the
test states its own."""
import numpy as np
import pytest
import torch

import oracle
import oracle.stage_oracle as math
import synth
from gpu_cases import TOL_STAGE, Pair, full_mask, host, rel_err, req, run_gpu

pytestmark = pytest.mark.gpu

# one kv head of two query heads: a block of 64 query vectors is 32 tokens, so
# every block of a prompt after P0 rows sees a multiple of 32 keys plus P0 (the
# last one, P0 + n)
# (GROUPED: 1024 query vectors per block of 64 tokens; prompts of more than 1,024
# tokens, on 256 CUs, take two query tiles per wave)
NARROW = synth.StageShape("narrow128", 7, n_layers=2, hidden=256, n_q_heads=2, n_kv_heads=1, head_dim=128, ffn=512)

SINGLE = synth.StageShape("narrow128mha", 10, n_layers=2, hidden=256, n_q_heads=2, n_kv_heads=2, head_dim=128, ffn=512)
THREE = synth.StageShape("narrow128three", 12, n_layers=2, hidden=256, n_q_heads=3, n_kv_heads=1, head_dim=128, ffn=512)
GROUPED = synth.StageShape("narrow128gqa", 11, n_layers=2, hidden=256, n_q_heads=16, n_kv_heads=1, head_dim=128, ffn=2048)


@pytest.fixture(scope="module")
def narrow():
    p = Pair(NARROW, 430)
    yield p
    p.close()


def _state(p, P0, n, seed):
    """A state of P0 rows whose buffer holds NaN in every later row."""
    g, o = p.states(1, P0, P0 + n + 96, seed)
    sh = p.shape
    bad = torch.full((sh.n_layers, 1, sh.n_kv_heads, n + 96, sh.head_dim), float("nan"), dtype=torch.bfloat16)
    g.append(bad, bad)
    g.truncate(P0)
    return g, o


@pytest.mark.parametrize("P0,n,holes", [(0, 5, 0), (0, 33, 0), (32, 32, 0), (37, 40, 0.2), (3, 100, 0), (47, 77, 0.2)])
def test_rows_past_the_last_key_are_not_read(narrow, P0, n, holes):
    """Last steps of 1..15, 16..31 and 32 keys: finite and equal to the oracle."""
    g, o = _state(narrow, P0, n, 431 + n)
    past = np.ones(P0, np.uint8)
    if holes:
        past = synth.hole_mask(P0, holes, 431 + n, 0)
        past[0] = 1
    x = synth.make_hidden(NARROW, n, 431 + n, 1)
    pos = int(past.sum()) + np.arange(n)
    out = host(narrow.gpu.prefill(g, pos, x.cuda(), past if holes else None))
    assert np.isfinite(out).all()
    ref = oracle.forward(narrow.orc, o, host(x), pos[None], None, np.concatenate([past, np.ones(n, np.uint8)])[None])
    assert rel_err(out, ref) <= TOL_STAGE
    g.free()


def test_softmax_sum_is_that_of_a_forward():
    """Keys whose probability 0.5 (1 + 0.8 / 256) lies below the middle of two
    bf16 values: the value product takes them as 0.5, the sum must not, in the
    prompt as in a forward.  A sum of rounded probabilities would change the
    attention output by 0.8 / 256 = 3.1e-3 of it; the two paths otherwise differ
    by fp16 / fp32 roundings (hidden_out fp16: 2^-11 at most)."""
    sh = synth.StageShape("narrow128f16", 9, n_layers=1, hidden=256, n_q_heads=2, n_kv_heads=1, head_dim=128, ffn=512,
                          act_dtype=synth.F16)
    layers = synth.make_weights(sh, 450)
    for m in ("wk", "wv", "wd"):                             # own rows: score 0, value 0; no FFN output
        layers[0].mats[m] = synth.zero_quant_like(layers[0].mats[m])
    p = Pair(sh, 450, layers=layers)
    P, n, D = 512, 2, 128
    x = (synth.make_hidden(sh, n, 450).float() / 256).half()
    pos = P + np.arange(n)
    w = p.orc.weights(0)
    h = math.rmsnorm(host(x), w["attn_norm"], sh.rms_eps)
    q = math.apply_rope(math.gemv_rows(h, w["wq"]).reshape(n, 2, D), pos[:, None], sh.rope_theta).reshape(2 * n, D)
    key = np.linalg.pinv(q) @ np.full(2 * n, np.log(0.5 * (1 + 0.8 / 256)) * np.sqrt(D))
    k = torch.zeros((1, 1, 1, P, D))
    k[0, 0, 0, :] = torch.from_numpy(key).float()
    k[0, 0, 0, ::32] = 0                                     # the largest score, 0, in every step
    v = torch.ones_like(k)
    outs = []
    for prompt in (True, False):
        g = p.gpu.new_state(1, P + 8)
        g.append(k.bfloat16(), v.bfloat16())
        outs.append(host(p.gpu.prefill(g, pos, x.cuda())) if prompt
                    else run_gpu(p, [req(g, pos[None], full_mask(1, P + n))], x))
        g.free()
    a, b = (o - host(x) for o in outs)
    e = float(np.linalg.norm(a - b) / np.linalg.norm(b))
    print(f"prompt against forward: {e:.2e}")
    assert e <= 1e-3
    p.close()


@pytest.mark.parametrize("shape,P0,n,bad", [(SINGLE, 0, 100, 41), (SINGLE, 21, 100, 60), (NARROW, 5, 100, 62), (THREE, 0, 100, 37),
                                            (GROUPED, 3, 70, 36), (GROUPED, 0, 1100, 805)])
def test_non_finite_row_reaches_no_earlier_group(shape, P0, n, bad):
    p = Pair(shape, 460, with_oracle=False)
    x = synth.make_hidden(shape, n, 460)
    outs = []
    for poison in (False, True):
        g, _ = p.states(1, P0, P0 + n, 460, with_oracle=False)
        if poison:
            x[bad] = float("inf")
        outs.append(host(p.gpu.prefill(g, P0 + np.arange(n), x.cuda())))
        g.free()
    assert np.isnan(outs[1][bad:]).any(axis=1).all()
    assert np.array_equal(outs[0][:bad // 16 * 16], outs[1][:bad // 16 * 16])
    p.close()
