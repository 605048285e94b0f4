"""GPU tests of the token-by-token delta rule against the float64 oracle (MI355X only).

Tails of at most 20 tokens run the recurrence in fp32 instead of the chunked form, in
launches of any size, alone or beside longer tails; both sides of the limit are checked.
"""
import numpy as np
import pytest
import torch

import synth
import paper_2609_18935_amd as tu
from gpu_cases import DEV, DeltaCase, errors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tu.lib()


def _params(s):
    return tu.delta_params(s.n_k_heads, s.n_v_heads, s.d_k, s.d_v, s.chunk, s.scale)


# fp32 sums of at most 128 products per dot, 20 steps of a contracting recurrence: a few
# 2^-24 per term and step, far below 1e-5; 21 tokens take the chunked form (f16 operands)
@pytest.mark.parametrize("hk,hv,d,chunk,T", [
    (16, 32, 128, 64, 1), (16, 32, 128, 64, 2), (2, 4, 128, 16, 19), (1, 1, 128, 32, 20), (3, 3, 64, 16, 17),
    (2, 4, 64, 64, 20), (2, 4, 128, 64, 21), (2, 4, 128, 16, 31), (8, 136, 64, 16, 20), (8, 136, 64, 16, 21),
])
def test_step_matches_oracle(hk, hv, d, chunk, T):
    print(f"[case] delta step hk={hk} hv={hv} d={d} chunk={chunk} T={T}", flush=True)
    s = synth.DeltaShape(hk, hv, d, d, chunk)
    c = DeltaCase(s, 31, 0, 0, T)
    ws = tu.delta_rule_continue(c.state, c.q, c.k, c.v, c.beta_d, c.g_d, _params(s), c.out)
    torch.cuda.synchronize()
    assert tu.workspace_faults(ws) == 0
    o, S = c.oracle()
    bar = 1e-5 if T <= 20 else 1e-3
    for got, want, what in ((c.out, o, "out"), (c.state, S, "state")):
        ma, mr = errors(got.cpu().numpy(), want)
        print(f"[parity] {what}: max_abs={ma:.3e} mean_rel={mr:.3e}", flush=True)
        assert mr <= bar and ma <= 20 * bar * float(np.abs(want).max())


def test_step_flags_values_beyond_f16_and_reports_its_call():
    s = synth.DeltaShape(2, 4, 128, 128, 64)
    ws = torch.full((1 << 16,), 0xAB, dtype=torch.uint8, device=DEV)   # stale bytes
    for big in (False, True):
        c = DeltaCase(s, 32, 0, 0, 3)
        if big:
            c.v[2, 3, 100] = 1.0e5
        tu.delta_rule_continue(c.state, c.q, c.k, c.v, c.beta_d, c.g_d, _params(s), c.out, workspace=ws)
        assert bool(tu.workspace_faults(ws) & tu.TU_FAULT_RANGE) == big


@pytest.mark.parametrize("T", [3, 20, 21])
@pytest.mark.parametrize("name", ["q", "k", "v", "state"])
def test_nan_is_no_overflow_in_either_form(name, T):
    """A NaN reaches the outputs without a range report, token by token as in chunks; an
    infinity is reported."""
    s = synth.DeltaShape(2, 4, 128, 128, 64)
    for bad, faults in ((float("nan"), 0), (float("inf"), tu.TU_FAULT_RANGE)):
        print(f"[case] delta rule, {bad} in {name}, T={T}", flush=True)
        c = DeltaCase(s, 35, 0, 0, T)
        getattr(c, name)[(2 if name != "state" else 0, 1, 7)] = bad
        ws = tu.delta_rule_continue(c.state, c.q, c.k, c.v, c.beta_d, c.g_d, _params(s), c.out)
        assert tu.workspace_faults(ws) == faults
        assert not bool(torch.isfinite(c.out).all())


def test_step_in_a_stack_of_mixed_tails():
    """A call with tails of 0, 1 and 20 tokens, and one whose longest tail is chunked."""
    s = synth.DeltaShape(2, 4, 128, 128, 64)
    for tails in ((1, 0, 20), (5, 33)):
        print(f"[case] delta step, tails {tails} in one call", flush=True)
        cases = [DeltaCase(s, 33, 0, 0, T, char=i) for i, T in enumerate(tails)]
        ctxs = [tu.Context(64, device=DEV) for _ in tails]
        out = torch.full((sum(tails), s.n_v_heads, s.d_v), float("nan"), device=DEV)
        cat = lambda name: torch.cat([getattr(c, name) for c in cases])  # noqa: E731
        layer = tu.LayerIO(tu.TU_LAYER_DELTA, cat("q"), cat("k"), cat("v"), out, state=[c.state for c in cases],
                           beta=cat("beta_d"), g=cat("g_d"))
        tu.update_layer_stack(ctxs, [[] for _ in tails], list(tails), [layer], tu.attn_params(2, 1, 64), _params(s))
        torch.cuda.synchronize()
        at = 0
        for c, T in zip(cases, tails):
            if T:
                o, S = c.oracle()
                assert errors(out[at:at + T].cpu().numpy(), o)[1] <= 1e-3
                assert errors(c.state.cpu().numpy(), S)[1] <= 1e-3
            at += T


@pytest.mark.parametrize("d,chunk", [(128, 64), (128, 16), (64, 32)])
def test_results_do_not_depend_on_the_other_contexts(d, chunk):
    """Every context of a call gives the bits of its own call: tails on both sides of the
    token-by-token limit and of a chunk, in a call of few blocks (direct chain) and in one
    of many (staged chain, other slice widths)."""
    for hv, copies in ((4, 1), (32, 2)):
        s = synth.DeltaShape(hv // 2, hv, d, d, chunk)
        tails = (1, 20, 21, 31, 64, 300) * copies
        print(f"[case] delta rule, {len(tails)} contexts of {hv} heads, d={d} chunk={chunk}", flush=True)
        cases = [DeltaCase(s, 34, 0, 0, T, char=i) for i, T in enumerate(tails)]
        states = [c.state.clone() for c in cases]
        out = torch.full((sum(tails), hv, d), float("nan"), device=DEV)
        cat = lambda name: torch.cat([getattr(c, name) for c in cases])  # noqa: E731
        layer = tu.LayerIO(tu.TU_LAYER_DELTA, cat("q"), cat("k"), cat("v"), out, state=states, beta=cat("beta_d"),
                           g=cat("g_d"))
        tu.update_layer_stack([tu.Context(512, device=DEV) for _ in tails], [[] for _ in tails], list(tails), [layer],
                              tu.attn_params(2, 1, 64), _params(s))
        at = 0
        for c, st, T in zip(cases, states, tails):
            tu.delta_rule_continue(c.state, c.q, c.k, c.v, c.beta_d, c.g_d, _params(s), c.out)
            assert torch.equal(c.out, out[at:at + T]) and torch.equal(c.state, st), f"T={T}"
            at += T
