"""GPU parity of the bf16 backward's forms: which one a shape takes is asked of lg_debug_bwd_plan, so that a change of a rule shows here
instead of leaving a form untested."""
import numpy as np
import pytest
import torch

import lg_synth
import paper_2410_01485_amd as lg
from gpu_util import DEV, TOL_OUT, TOL_REL, assert_close, assert_same_sums, dq_delta_allowance, f32np
from oracle import lg_oracle as O
from test_gpu_bwd import run_fwd_bwd
from test_gpu_varlen import check_pack

pytestmark = pytest.mark.gpu


def batch_beyond_the_shared_launch(Hq, Hkv, N, D, pattern):
    B = 1
    while lg.lg_debug_bwd_plan(B, Hq, Hkv, N, D, *pattern)["shared"]:
        B += 1
    return B


def check_heads(x, got, b, Hq, Hkv, pattern, what):
    """dq, dk, dv of a sequence's last kv head and its query heads against the oracle, element by element."""
    G = Hq // Hkv
    q, k, v, g = (f32np(t[b:b + 1, -G:]) if t.shape[1] == Hq and G > 1 else f32np(t[b:b + 1, -1:]) for t in x)
    w = O.bwd(q, k, v, g, *pattern)
    al = dq_delta_allowance(q, k, g, w["out"], *pattern)
    for name, t, n in zip(("dq", "dk", "dv"), got, (G, 1, 1)):
        assert_close(f32np(t[b:b + 1, -n:]), w[name], TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16], "%s %s of sequence %d" % (what, name, b),
                     allow=al if name == "dq" else None)


def check_apart_and_shared(Hq, Hkv, N, D, pattern):
    """A batch whose dq and dk/dv have launches of their own: its first and last sequence against the oracle, and against themselves
    alone, where they share one: the same bits of dq, and of dk and dv without groups of query heads and strided columns (else sums in
    another order).  Returns the batch's plan."""
    B = batch_beyond_the_shared_launch(Hq, Hkv, N, D, pattern)
    assert B > 1
    gen = torch.Generator(device=DEV).manual_seed(91)
    x = [torch.randn(B, h, N, D, generator=gen, device=DEV, dtype=torch.bfloat16) for h in (Hq, Hkv, Hkv, Hq)]
    got = run_fwd_bwd(*x, *pattern)
    fixed = Hq == Hkv and pattern[3] == 0
    if fixed:
        for y, z in zip(got, run_fwd_bwd(*x, *pattern)):
            assert torch.equal(y, z)
    for b in (0, B - 1):
        check_heads(x, got, b, Hq, Hkv, pattern, "apart")
        one = run_fwd_bwd(*(t[b:b + 1].contiguous() for t in x), *pattern)
        for name, y, z in zip(("dq", "dk", "dv"), got, one):
            if name == "dq" or fixed:
                assert torch.equal(y[b:b + 1], z), (name, b)
            else:
                assert_same_sums(y[b:b + 1], z, "%s of sequence %d" % (name, b))
    return lg.lg_debug_bwd_plan(B, Hq, Hkv, N, D, *pattern)


@pytest.mark.parametrize("Hq,Hkv,N,sink,window,block,stride", [
    # a sink, ragged ends; groups of query heads; blocks; strided columns; no sink, a window longer than most rows, a last tile of
    # one row; many column groups, long column parts
    (2, 2, 3001, 64, 1024, 1, 0), (4, 2, 2500, 3, 900, 1, 0), (2, 1, 3333, 64, 1024, 64, 0), (2, 2, 4100, 64, 1024, 64, 8),
    (1, 1, 2049, 0, 2048, 1, 0), (4, 2, 9000, 64, 1024, 64, 5), (3, 3, 1300, 5, 800, 1, 0), (1, 1, 1025, 0, 1025, 1, 0)])
def test_dkdv_in_64_key_form(Hq, Hkv, N, sink, window, block, stride):
    plan = check_apart_and_shared(Hq, Hkv, N, 128, (sink, window, block, stride))
    assert plan["dkdv_wide"] == -(-N // 256) and plan["dkdv"] == 0


@pytest.mark.parametrize("Hq,Hkv,N,D,sink,window,block,stride", [
    # lone sink groups of grouped heads (cut beside dq in the shared launch) and of ungrouped ones, several column groups, none
    (8, 2, 1030, 128, 64, 300, 1, 0), (8, 4, 1030, 64, 16, 100, 1, 0), (2, 1, 700, 128, 16, 100, 1, 0), (4, 1, 900, 64, 4, 130, 1, 0),
    (8, 8, 1030, 128, 64, 300, 1, 0), (8, 8, 1030, 64, 16, 100, 1, 0), (4, 2, 1150, 128, 64, 192, 64, 4), (4, 2, 700, 128, 0, 250, 1, 0)])
def test_dkdv_in_32_key_form(Hq, Hkv, N, D, sink, window, block, stride):
    plan = check_apart_and_shared(Hq, Hkv, N, D, (sink, window, block, stride))
    assert plan["dkdv"] == -(-N // (256 if D == 128 else 128)) and plan["dkdv_wide"] == 0


@pytest.mark.parametrize("H,N,D,window", [(3, 4100, 128, 4100), (2, 2300, 64, 2300), (5, 1290, 128, 600), (1, 700, 64, 700)])
def test_growing_rows_of_few_heads(H, N, D, window):
    """dk/dv's key tiles with the heads innermost beside dq, and in runs of a head apart."""
    check_apart_and_shared(H, H, N, D, (0, window, 1, 0))


@pytest.mark.parametrize("lens,Hq,Hkv,window,oracle_rows", [
    ([5000, 700, 9000], 14, 14, 4096, 1000),  # the longest takes dq with 64 rows per wave as well
    ([300, 1500, 6000, 1, 0, 257, 5000, 769], 24, 12, 1024, 400)])
def test_packs_of_both_forms_of_dkdv(lens, Hq, Hkv, window, oracle_rows):
    """Sequences of both forms of dk/dv side by side in launches of their own: against the fixed-length calls (alone the shorter ones'
    dq and dk/dv share a launch) and the oracle."""
    plan = lg.lg_debug_bwd_plan(1, Hq, Hkv, 0, 128, 64, window, cu_seqlens=np.concatenate([[0], np.cumsum(lens)]))
    assert not plan["shared"] and plan["dkdv_wide"] > 0 and plan["dkdv"] > 0
    check_pack(lens, Hq, Hkv, 128, 64, window, 1, 0, torch.bfloat16, 415, oracle_rows=oracle_rows)


@pytest.mark.parametrize("D", [64, 128])
def test_a_lone_group_beside_several_in_a_pack(D):
    """Ungrouped heads, every 16th block: the first sequence is too short for a strided column and has a lone sink group, whose sums
    whoever comes last adds; the second has several groups, summed by atomics in the same buffer; the third again a few."""
    lens = [900, 3000, 1500]
    plan = lg.lg_debug_bwd_plan(1, 4, 4, 0, D, 64, 64, 64, 16, cu_seqlens=np.concatenate([[0], np.cumsum(lens)]))
    assert plan["shared"] and plan["lone"] == 1 and plan["heads_cut"] * plan["rows_cut"] == 1
    check_pack(lens, 4, 4, D, 64, 64, 64, 16, torch.bfloat16, 416)


@pytest.mark.parametrize("H,D,cut", [(2, 128, True), (8, 128, False), (2, 64, False)])
def test_a_lone_strided_column(H, D, cut):
    """No sink, and one block in 20 whose rows reach beyond its window: a lone group of ungrouped heads, beside cut window parts (the
    pass over the parts adds its sums) and beside whole ones (whoever comes last does)."""
    N, pattern = 3000, (0, 512, 64, 20)
    plan = lg.lg_debug_bwd_plan(1, H, H, N, D, *pattern)
    assert plan["shared"] and plan["lone"] > 0 and (plan["heads_cut"] * plan["rows_cut"] > 1) == cut
    x = [t.to(DEV) for t in lg_synth.prefill_inputs(1, H, H, N, D, 92, torch.bfloat16, with_dout=True)]
    check_heads(x, run_fwd_bwd(*x, *pattern), 0, H, H, pattern, "lone column")


@pytest.mark.parametrize("D,N", [(128, 12000), (64, 3000)])
def test_heads_split_over_calls(D, N):
    """Ungrouped heads, sink and window: in calls of 17 heads and of 16 and 1 of them dk and dv have the same bits but in the sink's
    keys, whose sums are cut otherwise there, and the same bits there as well in calls of 8 and 8 of 16 heads."""
    pattern = (16, 128, 1, 0)
    x = [t.to(DEV) for t in lg_synth.prefill_inputs(1, 17, 17, N, D, 93, torch.bfloat16, with_dout=True)]
    part = lambda a, b: run_fwd_bwd(*(t[:, a:b].contiguous() for t in x), *pattern)
    whole, most, half, rest = part(0, 17), part(0, 16), part(0, 8), part(8, 16)
    assert lg.lg_debug_bwd_plan(1, 17, 17, N, D, *pattern)["lone"] != lg.lg_debug_bwd_plan(1, 16, 16, N, D, *pattern)["lone"]
    for y, z, a, b in zip(whole, most, half, rest):
        assert torch.equal(z, torch.cat([a, b], dim=1))
        assert torch.equal(y[:, :16, 16:], z[:, :, 16:])
        assert_same_sums(y[:, :16, :16], z[:, :, :16], "sink keys")


@pytest.mark.parametrize("Hq,Hkv,N,D,sink,window,block,stride,dtype", [
    (4, 4, 1500, 128, 64, 300, 1, 0, torch.bfloat16), (3, 3, 900, 64, 0, 900, 1, 0, torch.bfloat16), (8, 2, 1300, 128, 16, 500, 1, 0, torch.bfloat16),
    (2, 2, 2500, 64, 64, 64, 64, 4, torch.bfloat16), (2, 2, 700, 64, 16, 100, 1, 0, torch.float32), (2, 1, 500, 128, 0, 500, 1, 0, torch.float32)])
def test_dk_dv_over_k_v(Hq, Hkv, N, D, sink, window, block, stride, dtype):
    """Gradients written over the keys and values, either way round, of shapes whose dq, which reads all keys, shares a launch with
    dk/dv otherwise."""
    pattern = (sink, window, block, stride)
    code = lg.LG_BF16 if dtype == torch.bfloat16 else lg.LG_F32
    assert lg.lg_debug_bwd_plan(1, Hq, Hkv, N, D, *pattern, dtype=code)["shared"]
    x = [t.to(DEV) for t in lg_synth.prefill_inputs(1, Hq, Hkv, N, D, 94, dtype, with_dout=True)]
    want = run_fwd_bwd(*x, *pattern)
    for crossed in (False, True):
        q, k, v, g = (t.clone() for t in x)
        out, lse, dq = torch.empty_like(q), torch.empty(1, Hq, N, device=DEV), torch.empty_like(q)
        lg.lg_sparse_attn_fwd(q, k, v, out, lse, *pattern)
        ws = torch.empty(lg.bwd_workspace_bytes(1, Hq, Hkv, N, D, *pattern, code), dtype=torch.uint8, device=DEV)
        dk, dv = (v, k) if crossed else (k, v)
        lg.lg_sparse_attn_bwd(q, k, v, out, lse, g, dq, dk, dv, ws, *pattern)
        assert torch.equal(dq, want[0])
        for y, z in ((dk, want[1]), (dv, want[2])):
            if Hq == Hkv and stride == 0:
                assert torch.equal(y, z), crossed
            else:
                assert_same_sums(y, z, "over the inputs")
