"""GPU tests of both delta-rule chains against the float64 oracle (MI355X only).

Launches of at most 256 blocks of 16 state columns (items x value heads x d / 16) take the
direct chain, larger ones the staged one, and so do those of more than 128 blocks beside
attention over many rows or with a long tail: every head size and chunk length on both sides
of the limits, whole and ragged chunks, one chunk.
"""
import pytest
import torch

import synth
import paper_2609_18935_amd as tu
from gpu_cases import DEV, AttnCase, DeltaCase, assert_close, delta_oracle_heads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tu.lib()


def _params(s):
    return tu.delta_params(s.n_k_heads, s.n_v_heads, s.d_k, s.d_v, s.chunk, s.scale)


@pytest.mark.parametrize("d,hv", [(128, 32), (128, 34), (64, 64), (64, 66)])   # 256 blocks, and a few more
@pytest.mark.parametrize("chunk", [16, 32, 64])
@pytest.mark.parametrize("T", [33, 64, 127])
def test_chains_match_oracle(d, hv, chunk, T):
    print(f"[case] delta chain hv={hv} d={d} chunk={chunk} T={T}", flush=True)
    s = synth.DeltaShape(hv // 2, hv, d, d, chunk)
    c = DeltaCase(s, 41, 0, 0, T)
    ws = tu.delta_rule_continue(c.state, c.q, c.k, c.v, c.beta_d, c.g_d, _params(s), c.out)
    torch.cuda.synchronize()
    assert tu.workspace_faults(ws) == 0
    vh, o, S = delta_oracle_heads(c.S0, c.q_b, c.k_b, c.v_b, c.beta, c.g, s.scale, [0, hv // 4, hv // 2 - 1])
    assert_close(c.out.cpu().numpy()[:, vh], o, "out")
    assert_close(c.state.cpu().numpy()[vh], S, "state")


@pytest.mark.parametrize("chunk", [16, 64])
def test_direct_chain_over_many_chunks_and_contexts(chunk):
    """Three contexts of different lengths (one of a single chunk, in the chunked form from 21
    tokens on) in one call: each
    matches the oracle and equals its own call."""
    s = synth.DeltaShape(2, 4, 128, 128, chunk)
    tails = (700, chunk, 1025)
    print(f"[case] direct chain, chunk {chunk}, tails {tails}", flush=True)
    cases = [DeltaCase(s, 42, 0, 0, T, char=i) for i, T in enumerate(tails)]
    out = torch.full((sum(tails), 4, 128), float("nan"), device=DEV)
    states = [c.state.clone() for c in cases]
    cat = lambda name: torch.cat([getattr(c, name) for c in cases])  # noqa: E731
    layer = tu.LayerIO(tu.TU_LAYER_DELTA, cat("q"), cat("k"), cat("v"), out, state=states, beta=cat("beta_d"),
                       g=cat("g_d"))
    tu.update_layer_stack([tu.Context(2048, device=DEV) for _ in tails], [[]] * 3, list(tails), [layer],
                          tu.attn_params(2, 1, 64), _params(s))
    at = 0
    for c, st, T in zip(cases, states, tails):
        tu.delta_rule_continue(c.state, c.q, c.k, c.v, c.beta_d, c.g_d, _params(s), c.out)
        assert torch.equal(c.out, out[at:at + T]) and torch.equal(c.state, st)
        o, S = c.oracle()
        assert_close(out[at:at + T].cpu().numpy(), o, f"T={T} out")
        assert_close(st.cpu().numpy(), S, f"T={T} state")
        at += T


# Beside attention: launches of more than 128 blocks (16 heads of 128) up to 12,288 cache rows
# over the attention layers, without the rows the call removes, and 1,792 tokens; others always.
@pytest.mark.parametrize("layers,rows,removed,T,hv,direct", [
    (1, 12288, 0, 100, 32, True),
    (1, 12289, 0, 100, 32, False),
    (2, 6144, 0, 100, 32, True),
    (2, 6145, 0, 100, 32, False),
    (1, 12288, 50, 100, 32, True),
    (1, 12289, 50, 100, 32, False),
    (1, 4000, 0, 1792, 18, True),
    (1, 4000, 0, 1793, 18, False),
    (1, 12289, 0, 100, 16, True),
    (1, 12289, 0, 100, 18, False),
])
def test_chains_beside_attention_match_oracle(layers, rows, removed, T, hv, direct):
    print(f"[case] delta chain, {hv} heads, {T} tokens, beside {layers} attention layers of {rows} rows", flush=True)
    a, s = synth.AttnShape(2, 1, 64), synth.DeltaShape(hv // 2, hv, 128, 128, 32)
    old = rows - T + removed
    acs = [AttnCase(a, 43, 0, i, old, T) for i in range(layers)]
    c = DeltaCase(s, 43, 0, layers, T)
    ctx = tu.Context(old + T, device=DEV)
    ctx.pos[:old] = torch.arange(old, dtype=torch.int32, device=DEV)
    ctx.set_metadata([(0, old)], old)
    io = [tu.LayerIO(tu.TU_LAYER_ATTN, x.q, x.k, x.v, x.out, k_cache=[x.k_cache], v_cache=[x.v_cache]) for x in acs]
    io.append(tu.LayerIO(tu.TU_LAYER_DELTA, c.q, c.k, c.v, c.out, state=[c.state], beta=c.beta_d, g=c.g_d))
    tu.profile_enable(True)
    try:
        tu.update_layer_stack([ctx], [[(500, 500 + removed)] if removed else []], [T], io,
                              tu.attn_params(2, 1, 64, a.rdim, a.rope_theta), _params(s))
        kernels = tu.profile_collect()
    finally:
        tu.profile_enable(False)
    assert ("delta_chain_direct" in kernels, "delta_chain" in kernels) == (direct, not direct)
    vh, o, S = delta_oracle_heads(c.S0, c.q_b, c.k_b, c.v_b, c.beta, c.g, s.scale, [0, hv // 4, hv // 2 - 1])
    assert_close(c.out.cpu().numpy()[:, vh], o, "out")
    assert_close(c.state.cpu().numpy()[vh], S, "state")
