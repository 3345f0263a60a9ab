"""Edges of the prompt and product kernels against the oracle and each other:
prompt lengths around the 64-token block and the 8-block band (tiny stage, FFN
688: a ragged last group of k; its products are too short to be split over K),
past rows with masked holes at lengths around the attention's 32-key step and
64-query block; residual products split over K with two query tiles per wave, two
passes, and hidden sizes above 4,096 and 8,192 (narrow stages of two layers, so
that a split product's sums enter the next layer and the output); hidden states
at 2-byte aligned addresses; a row's result
in a forward must be bitwise the same whichever product form its batch selects
(16 rows or fewer, 17-32, 33-64).

Tolerance: TOL_STAGE, the stage tolerance every parity test uses (fp16 product
inputs and 16-bit cache rows; 2.8e-3 measured on these paths)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_cases import TOL_STAGE, Pair, full_mask, host, rel_err, req, run_gpu

pytestmark = pytest.mark.gpu

TINY2 = synth.with_layers(synth.TINY, 2)


@pytest.fixture(scope="module")
def tiny():
    p = Pair(TINY2, 410)
    yield p
    p.close()


@pytest.mark.parametrize("P0,n,holes", [(0, 17, 0), (0, 128, 0), (0, 129, 0), (31, 33, 0.2), (32, 63, 0.2), (33, 64, 0.2),
                                        (65, 200, 0.1), (1, 520, 0)])
def test_prompt_edges(tiny, P0, n, holes):
    g, o = tiny.states(1, P0, P0 + n + 8, 411 + n)
    past = np.ones(P0, np.uint8)
    if holes:
        past = synth.hole_mask(P0, holes, 411 + n, 0)
        past[0] = 1
    x = synth.make_hidden(TINY2, n, 411 + n, 1)
    pos = int(past.sum()) + np.arange(n)
    out = host(tiny.gpu.prefill(g, pos, x.cuda(), past if holes else None))
    ref = oracle.forward(tiny.orc, o, host(x), pos[None], None, np.concatenate([past, np.ones(n, np.uint8)])[None])
    assert rel_err(out, ref) <= TOL_STAGE
    for l in range(TINY2.n_layers):
        k, v = g.read(l, 0, P0, n)
        assert rel_err(host(k), o.K[l][0][:, P0:P0 + n]) <= TOL_STAGE
        assert rel_err(host(v), o.V[l][0][:, P0:P0 + n]) <= TOL_STAGE
    g.free()


def _splits(tiles, groups, cus):
    """The K splits that a prompt's residual product of so many workgroup tiles and groups of 128 k takes."""
    best = (1 << 30, 1)
    for S in range(1, min(8, groups // 8) + 1):
        per = -(-groups // S)
        used = -(-groups // per)
        best = min(best, (-(-tiles * used // cus) * (per + 6), used))     # the first of equal costs
    return best[1]


def _query_tiles(n, heads, kv_heads, cus):
    """Query tiles per wave of a prompt's attention."""
    rounds = [-(-(-(-n * heads // kv_heads // v) * kv_heads) // cus) for v in (64, 128)]
    return 2 if heads // kv_heads % 2 == 0 and 5 * rounds[1] <= 3 * rounds[0] else 1


# head_dim 128; (shape, P0, n, holes, query tiles per wave, o and down split over K)
WIDE = [
    (dict(hidden=256, n_q_heads=16, n_kv_heads=1, ffn=2048), 37, 1100, 0.2, 2, (True, True)),
    (dict(hidden=256, n_q_heads=2, n_kv_heads=1, ffn=512), 19, 2100, 0.2, 1, (False, False)),     # passes of 2,048 and 52 rows
    (dict(hidden=4104, n_q_heads=2, n_kv_heads=1, ffn=2048), 0, 70, 0, 1, (False, True)),
    (dict(hidden=8200, n_q_heads=2, n_kv_heads=1, ffn=2048), 5, 70, 0, 1, (False, True)),
]


@pytest.mark.parametrize("dims,P0,n,holes,tiles,split", WIDE, ids=["two-tiles-split", "two-passes", "hidden4104", "hidden8200"])
def test_prompt_forms(dims, P0, n, holes, tiles, split):
    shape = synth.StageShape("wide", 14, n_layers=2, head_dim=128, **dims)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    m = min(n, 2048)                                        # rows of the first pass
    assert _query_tiles(m, shape.n_q_heads, shape.n_kv_heads, cus) == tiles
    blocks = -(-(-(-shape.hidden // 64)) // 4) * -(-m // 64)
    for k, want in zip((shape.n_q_heads * shape.head_dim, shape.ffn), split):
        assert (_splits(blocks, -(-k // 128), cus) > 1) == want
    p = Pair(shape, 470)
    g, o = p.states(1, P0, P0 + n + 8, 470)
    past = np.ones(P0, np.uint8)
    if holes:
        past = synth.hole_mask(P0, holes, 470, 0)
        past[0] = 1
    x = synth.make_hidden(shape, n, 470, 1)
    pos = int(past.sum()) + np.arange(n)
    out = host(p.gpu.prefill(g, pos, x.cuda(), past if holes else None))
    ref = oracle.forward(p.orc, o, host(x), pos[None], None, np.concatenate([past, np.ones(n, np.uint8)])[None])
    print(f"{dims}: {rel_err(out, ref):.2e}")
    assert rel_err(out, ref) <= TOL_STAGE
    for l in range(shape.n_layers):
        k, v = g.read(l, 0, P0, n)
        assert rel_err(host(k), o.K[l][0][:, P0:P0 + n]) <= TOL_STAGE
        assert rel_err(host(v), o.V[l][0][:, P0:P0 + n]) <= TOL_STAGE
    p.close()


@pytest.mark.parametrize("hidden", [256, 4104])
def test_prompt_at_odd_addresses(hidden):
    """hidden_in and hidden_out one element (2 bytes) past a 16-byte boundary: the
    result is that of aligned ones, and the elements beside hidden_out stay."""
    shape = synth.StageShape("odd", 16, n_layers=1, head_dim=128, hidden=hidden, n_q_heads=2, n_kv_heads=1, ffn=2048)
    p = Pair(shape, 480, with_oracle=False)
    n = 70
    x = synth.make_hidden(shape, n, 480, 1).cuda()
    outs = []
    for off in (0, 1):
        g, _ = p.states(1, 0, n, 480, with_oracle=False)
        src, dst = (torch.full((n * hidden + 8,), 7.0, dtype=x.dtype, device="cuda") for _ in range(2))
        view = src[off:off + n * hidden].view(n, hidden)
        view.copy_(x)
        p.gpu.prefill(g, np.arange(n), view, hidden_out=dst[off:off + n * hidden].view(n, hidden))
        torch.cuda.synchronize()
        outs.append(dst[off:off + n * hidden].cpu())
        assert (dst[:off] == 7).all() and (dst[off + n * hidden:] == 7).all()
        g.free()
    assert torch.equal(*outs)
    p.close()


def test_row_result_does_not_depend_on_the_product_form():
    """One 8B layer: a 5-token request alone (one tile per workgroup), with 15 more
    rows (gate|up in pairs) and with 55 more (two 32-row workgroups per tile)."""
    p = Pair(synth.with_layers(synth.LLAMA8B_HALF, 1), 420)
    x = synth.make_hidden(p.shape, 60, 420)
    outs = []
    for others in ((), (15,), (55,)):
        states = [p.states(1, 40, 120, 420, stream=r, with_oracle=False)[0] for r in range(1 + len(others))]
        reqs = [req(s, (40 + np.arange(n))[None], full_mask(1, 40 + n)) for s, n in zip(states, (5,) + others)]
        outs.append(run_gpu(p, reqs, x[:5 + sum(others)])[:5].copy())
        for s in states:
            s.free()
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])
    p.close()


@pytest.mark.parametrize("n", [5, 40])
def test_padded_matrix(n):
    """The down matrix of this shape (249 chunks of 32 k) is stored with 64 groups
    of 128 k where the prepared rows hold the 63 that K = 7968 takes."""
    shape = synth.StageShape("padded", 8, n_layers=1, hidden=2048, n_q_heads=2, n_kv_heads=1, head_dim=128, ffn=7968)
    p = Pair(shape, 440)
    g, o = p.states(1, 70, 70 + n, 440)
    x = synth.make_hidden(shape, n, 440)
    pos = (70 + np.arange(n))[None]
    out = run_gpu(p, [req(g, pos, full_mask(1, 70 + n))], x)
    ref = oracle.forward(p.orc, o, host(x), pos, None, full_mask(1, 70 + n))
    assert rel_err(out, ref) <= TOL_STAGE
    p.close()
