"""GPU tests of the attention launch's dispatch branches against the float64 oracle (MI355X only)."""
import numpy as np
import pytest
import torch

import synth
import paper_2609_18935_amd as tu
from gpu_cases import DEV, AttnCase, DeltaCase, assert_close, sample_rows

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


# The long kernel at its smallest: query tiles with few rows or with rows in some waves only,
# whole and in splits (chosen and forced), past the short kernel's limits of rows (256) and
# of units.
@pytest.mark.parametrize("Hq,Hkv,D,L,T,splits", [
    (16, 2, 256, 300, 33, 0),       # 264 rows: a second tile of 8
    (16, 2, 256, 300, 33, 1),
    (16, 2, 256, 300, 33, 5),
    (16, 2, 256, 0, 36, 0),
    (32, 4, 128, 777, 61, 3),       # 488 rows
    (32, 8, 128, 11000, 17, 0),     # 68 rows over 345 units a row tile
    (16, 4, 64, 8200, 64, 0),       # 256 rows
    (16, 4, 64, 8200, 63, 64),
    (16, 8, 64, 65530, 17, 0),      # 34 rows
])
def test_long_kernel_with_few_rows(Hq, Hkv, D, L, T, splits):
    print(f"[case] long kernel Hq={Hq} Hkv={Hkv} D={D} L={L} T={T} splits={splits}", flush=True)
    p = tu.attn_params(Hq, Hkv, D, kv_splits=1)
    tiles = tu.lib().tail_prefill_attention_workspace_size(p, T, L) - 2 * T * Hq * D
    assert tiles > 2 * Hkv * (L + T) * D, "no V^T tiles: the short kernel"
    case = _run(synth.AttnShape(Hq, Hkv, D), L, T, splits)
    assert_close(case.out.cpu().numpy(), case.oracle([], L)["out"], "long kernel")


def _rel2(got, want):
    return float(np.linalg.norm(got.cpu().numpy().astype(np.float64) - want) / np.linalg.norm(want))


# Launches split only for their uneven query tiles write fp32 partials: no further from
# float64 than the same launch whole (probabilities in f16 on both sides; f16 partials are 1.5
# times as far).
@pytest.mark.parametrize("Hq,Hkv,D,L,T", [(16, 2, 256, 0, 2721), (16, 4, 64, 0, 3000)])
def test_uneven_tiles_in_splits_lose_no_precision(Hq, Hkv, D, L, T):
    print(f"[case] split for uneven tiles Hq={Hq} Hkv={Hkv} D={D} L={L} T={T}", flush=True)
    shape = synth.AttnShape(Hq, Hkv, D)
    rows = sample_rows(T, 200, 5)
    case = _run(shape, L, T, 0)
    want = case.oracle([], L, rows=rows)["out"]
    split, whole = (_rel2(c.out[rows], want) for c in (case, _run(shape, L, T, 1)))
    print(f"[parity] error {split:.3e}, whole {whole:.3e}", flush=True)
    assert split <= 1.05 * whole


# Short tails over few rows in splits: the bf16 rounding of the rotated queries is the oracle's
# too, P has 16 bits and the partials are fp32, so only 2^-16 and fp32 sums remain; alone and
# beside contexts whose partials are f16.
@pytest.mark.parametrize("others", [(), (9000, 20000)])
@pytest.mark.parametrize("Hq,Hkv,D,L,T", [(16, 2, 256, 300, 1), (16, 4, 64, 600, 16)])
def test_short_tails_that_would_run_whole_lose_no_precision(Hq, Hkv, D, L, T, others):
    print(f"[case] short tail Hq={Hq} Hkv={Hkv} D={D} L={L} T={T} beside {others}", flush=True)
    shape = synth.AttnShape(Hq, Hkv, D)
    cases = [AttnCase(shape, 26, 0, 0, n, T, char=i) for i, n in enumerate((L,) + others)]
    ctxs = []
    for c in cases:
        ctx = tu.Context(c.capacity, device=DEV)
        ctx.pos[:c.L_old] = torch.arange(c.L_old, dtype=torch.int32, device=DEV)
        ctx.set_metadata([(0, c.L_old)], c.L_old)
        ctxs.append(ctx)
    out = torch.full((len(cases) * T, Hq, D), float("nan"), device=DEV)
    layer = tu.LayerIO(tu.TU_LAYER_ATTN, torch.cat([c.q for c in cases]), torch.cat([c.k for c in cases]),
                       torch.cat([c.v for c in cases]), out, k_cache=[c.k_cache for c in cases],
                       v_cache=[c.v_cache for c in cases])
    tu.update_layer_stack(ctxs, [[] for _ in cases], [T] * len(cases), [layer],
                          tu.attn_params(Hq, Hkv, D, shape.rdim, shape.rope_theta, shape.softmax_scale))
    for i, c in enumerate(cases):
        err = _rel2(out[i * T:(i + 1) * T], c.oracle([], c.L_old)["out"])
        print(f"[parity] context {i}: {err:.3e}", flush=True)
        # beside longer contexts the first of 616 rows (10 key tiles) was split in f16 all along
        assert err <= (2e-5 if i == 0 and (L == 300 or not others) else 1e-3)


# The short-tail kernel: one to eight row tiles of 32, contexts of none to a few rows per
# wave and of many, ragged last units (32 keys) and row tiles, every head size, group
# sizes that leave row tiles partly empty, forced and automatic splits.
@pytest.mark.parametrize("Hq,Hkv,D,rdim,L,T,splits", [
    (16, 2, 256, 256, 0, 1, 0),
    (16, 2, 256, 256, 31, 1, 0),
    (16, 2, 256, 256, 4097, 4, 0),
    (16, 2, 256, 256, 4000, 32, 0),
    (16, 2, 256, 256, 700, 5, 64),
    (32, 8, 128, 64, 1999, 9, 0),
    (3, 3, 128, 128, 5000, 63, 2),
    (16, 4, 64, 64, 9001, 64, 0),
    (20, 4, 64, 32, 250, 7, 1),
])
def test_short_tail(Hq, Hkv, D, rdim, L, T, splits):
    print(f"[case] short tail Hq={Hq} Hkv={Hkv} D={D} rdim={rdim} L={L} T={T} splits={splits}", flush=True)
    case = _run(synth.AttnShape(Hq, Hkv, D, rotary_dim=rdim), L, T, splits)
    ref = case.oracle([], L)
    assert_close(case.out.cpu().numpy(), ref["out"], "short-tail attention")


@pytest.mark.parametrize("vt", [False, True])
def test_short_tail_many_contexts_in_one_call(vt):
    """Seven contexts of different lengths, three tokens each or fewer, in one launch."""
    shape = synth.AttnShape(16, 2, 128)
    sizes = [(0, 1), (33, 3), (2500, 2), (64, 1), (700, 3), (1, 2), (6000, 1)]
    print(f"[case] short tails of {len(sizes)} contexts, V^T copies {vt}", flush=True)
    cases = [AttnCase(shape, 23, 0, 0, L, T, char=i) for i, (L, T) in enumerate(sizes)]
    ctxs, vts = [], []
    for c in cases:
        ctx = tu.Context(c.capacity, device=DEV)
        ctx.pos[:c.L_old] = torch.arange(c.L_old, dtype=torch.int32, device=DEV)
        ctx.set_metadata([(0, c.L_old)] if c.L_old else [], c.L_old)
        v = tu.new_vt_cache(c.capacity, shape.n_kv_heads, shape.head_dim, DEV)
        if vt and c.L_old:
            tu.refresh_vt_cache(ctx, [c.v_cache], [v])
        ctxs.append(ctx)
        vts.append(v)
    out = torch.full((sum(T for _, T in sizes), shape.n_q_heads, shape.head_dim), float("nan"), device=DEV)
    layer = tu.LayerIO(tu.TU_LAYER_ATTN, torch.cat([c.q for c in cases]), torch.cat([c.k for c in cases]),
                       torch.cat([c.v for c in cases]), out, k_cache=[c.k_cache for c in cases],
                       v_cache=[c.v_cache for c in cases], vt_cache=vts if vt else None)
    p = tu.attn_params(shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rdim, shape.rope_theta,
                       shape.softmax_scale)
    up = tu.update_layer_stack(ctxs, [[] for _ in sizes], [T for _, T in sizes], [layer], p)
    torch.cuda.synchronize()
    assert tu.workspace_faults(up.workspace) == 0
    at = 0
    for i, (c, (L, T)) in enumerate(zip(cases, sizes)):
        assert ctxs[i].vt_rows == L + T
        if vt:   # the copy, refreshed with rows the launch does not read from it, is a fresh one's
            fresh = tu.new_vt_cache(c.capacity, shape.n_kv_heads, shape.head_dim, DEV)
            again = tu.Context(c.capacity, device=DEV)
            again.set_metadata([(0, L + T)], L + T)
            tu.refresh_vt_cache(again, [c.v_cache], [fresh])
            assert torch.equal(vts[i].view(torch.int16), fresh.view(torch.int16)), f"context {i}: V^T copy"
        assert_close(out[at:at + T].cpu().numpy(), c.oracle([], L)["out"], f"context {i} (L={L}, T={T})")
        at += T


@pytest.mark.parametrize("D", [64, 128])
def test_many_short_tails_beside_a_delta_layer(D):
    """1,024 workgroups, of which a CU holds two or three, overlapping the delta layer."""
    shape, ds, n = synth.AttnShape(32, 32, D), synth.DeltaShape(2, 4, 64, 64, 16), 32
    print(f"[case] short tails of {n} contexts beside a delta layer, D={D}", flush=True)
    cases = [AttnCase(shape, 27, 0, 0, 40 + 3 * i, 1, char=i) for i in range(n)]
    deltas = [DeltaCase(ds, 27, 0, 1, 1, char=i) for i in range(n)]
    ctxs = []
    for c in cases:
        ctx = tu.Context(c.capacity, device=DEV)
        ctx.pos[:c.L_old] = torch.arange(c.L_old, dtype=torch.int32, device=DEV)
        ctx.set_metadata([(0, c.L_old)], c.L_old)
        ctxs.append(ctx)
    out, dout = torch.full((n, 32, D), float("nan"), device=DEV), torch.full((n, 4, 64), float("nan"), device=DEV)
    acat = lambda name: torch.cat([getattr(c, name) for c in cases])    # noqa: E731
    dcat = lambda name: torch.cat([getattr(c, name) for c in deltas])   # noqa: E731
    layers = [tu.LayerIO(tu.TU_LAYER_DELTA, dcat("q"), dcat("k"), dcat("v"), dout, state=[c.state for c in deltas],
                         beta=dcat("beta_d"), g=dcat("g_d")),
              tu.LayerIO(tu.TU_LAYER_ATTN, acat("q"), acat("k"), acat("v"), out, k_cache=[c.k_cache for c in cases],
                         v_cache=[c.v_cache for c in cases])]
    up = tu.update_layer_stack(ctxs, [[] for _ in cases], [1] * n, layers,
                               tu.attn_params(32, 32, D, shape.rdim, shape.rope_theta, shape.softmax_scale),
                               tu.delta_params(2, 4, 64, 64, 16, ds.scale))
    torch.cuda.synchronize()
    assert tu.workspace_faults(up.workspace) == 0
    for i in (0, 7, 31):
        assert_close(out[i:i + 1].cpu().numpy(), cases[i].oracle([], cases[i].L_old)["out"], f"context {i} attention")
        o, S = deltas[i].oracle()
        assert_close(dout[i:i + 1].cpu().numpy(), o, f"context {i} delta")
        assert_close(deltas[i].state.cpu().numpy(), S, f"context {i} state")


def test_short_tail_flags_values_beyond_f16():
    """A value of magnitude 1e5 in the last cache row, or in the tail, sets TU_FAULT_RANGE."""
    shape = synth.AttnShape(16, 2, 256)
    for where in ("cache", "tail"):
        print(f"[case] short tail, value 1e5 in the {where}", flush=True)
        c = AttnCase(shape, 24, 0, 0, 333, 2)
        (c.v_cache if where == "cache" else c.v)[332 if where == "cache" else 1, 1, 7] = 1.0e5
        ctx = tu.Context(c.capacity, device=DEV)
        ctx.pos[:333] = torch.arange(333, dtype=torch.int32, device=DEV)
        ctx.set_metadata([(0, 333)], 333)
        ws = tu.tail_prefill_attention(ctx, c.k_cache, c.v_cache, tu.attn_params(16, 2, 256), c.q, c.k, c.v, c.out)
        assert tu.workspace_faults(ws) & tu.TU_FAULT_RANGE
