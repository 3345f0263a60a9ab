"""The prompt's attention (head_dim 128) at the edges of its 32-key steps: the
rows of a state's buffer past the last key a block sees are never read into the
result, whatever they hold.

Tolerance: TOL_STAGE, the stage tolerance every parity test uses."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_cases import TOL_STAGE, Pair, host, rel_err

pytestmark = pytest.mark.gpu

# one kv head of two query heads: a block of 64 query vectors is 32 tokens, so
# every block of a prompt after P0 rows sees a multiple of 32 keys plus P0 (the
# last one, P0 + n)
NARROW = synth.StageShape("narrow128", 7, n_layers=2, hidden=256, n_q_heads=2, n_kv_heads=1, head_dim=128, ffn=512)


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
