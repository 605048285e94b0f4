"""GPU tests of the attention launch's dispatch branches against the float64 oracle (MI355X only)."""
import pytest
import torch

import synth
import paper_2609_18935_amd as tu
from gpu_cases import DEV, AttnCase, assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tu.lib()


def _run(shape, L, T, splits, seed=21):
    case = AttnCase(shape, seed, 0, 0, L, T)
    ctx = tu.Context(case.capacity, device=DEV)
    ctx.pos[:L] = torch.arange(L, dtype=torch.int32, device=DEV)
    ctx.set_metadata([(0, L)] if L else [], L)
    p = tu.attn_params(shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rdim, shape.rope_theta,
                       shape.softmax_scale, kv_splits=splits)
    ws = tu.tail_prefill_attention(ctx, case.k_cache, case.v_cache, p, case.q, case.k, case.v, case.out,
                                   q_hat=case.q_hat)
    torch.cuda.synchronize()
    assert tu.workspace_faults(ws) == 0
    return case


# More than 256 workgroups whose query tiles see 1 .. all key tiles: the longest-first
# order. Group counts (KV heads x splits) that do and do not divide the 8 dies, a last
# query tile with few rows, and a context in front of the tail.
@pytest.mark.parametrize("Hq,Hkv,D,L,T,splits", [
    (64, 4, 64, 0, 1100, 1),
    (48, 3, 64, 300, 1501, 1),
    (32, 2, 128, 129, 900, 3),
    (16, 1, 256, 0, 1025, 5),
])
def test_longest_first_order(Hq, Hkv, D, L, T, splits):
    print(f"[case] longest first Hq={Hq} Hkv={Hkv} D={D} L={L} T={T} splits={splits}", flush=True)
    case = _run(synth.AttnShape(Hq, Hkv, D), L, T, splits)
    ref = case.oracle([], L)
    assert_close(case.out.cpu().numpy(), ref["out"], "longest-first attention")
