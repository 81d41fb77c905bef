"""GPU parity: lg_sparse_attn_fwd (through the C ABI) against the fp64 oracle, element by element."""
import numpy as np
import pytest
import torch

import lg_synth
import paper_2410_01485_amd as lg
from gpu_util import DEV, TOL_LSE, TOL_OUT, TOL_REL, assert_close, check_fwd, f32np, growing_inputs, run_fwd
from oracle import lg_oracle as O

pytestmark = pytest.mark.gpu


def test_config1_fp32_sink_window():
    # B1 H1 N1024 D64 fp32, sink 16, window 128: max abs error <= 1e-4
    check_fwd(1, 1, 1, 1024, 64, 16, 128, dtype=torch.float32, seed=20241002)


# float32: 32 or 64 query rows per workgroup, by the number of workgroups (up to 128, and 257 .. 384 with a reach of 256)
F32_ROWS = [(1, 1, 1, 31, 0, 31, 1, 0), (1, 2, 1, 33, 4, 9, 1, 0), (1, 1, 1, 95, 16, 20, 1, 0), (1, 3, 1, 700, 16, 96, 16, 3),
            (2, 32, 32, 128, 0, 128, 1, 0), (2, 32, 16, 129, 4, 40, 1, 0), (2, 26, 13, 300, 0, 300, 1, 0), (2, 32, 8, 384, 16, 256, 1, 0),
            (2, 32, 8, 384, 16, 255, 1, 0), (2, 32, 8, 385, 16, 300, 1, 0)]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,N,sink,window,block,stride", F32_ROWS)
def test_float32_rows_per_workgroup(B, Hq, Hkv, N, sink, window, block, stride, D):
    check_fwd(B, Hq, Hkv, N, D, sink, window, block, stride, dtype=torch.float32, seed=12)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,N,sink,window,block,stride", [
    (2, 1, 1, 0, 1, 1, 0), (2, 2, 64, 0, 64, 1, 0), (2, 1, 129, 4, 60, 1, 0), (4, 2, 700, 64, 200, 1, 0), (2, 2, 640, 0, 640, 1, 0),
    (2, 1, 1000, 64, 128, 64, 4), (2, 2, 1090, 16, 100, 1, 0)])
def test_few_work_items_give_the_same_bits(Hq, Hkv, N, sink, window, block, stride, D):
    """Up to 256 work items of 128 rows take an instance of their own: the same bits as in a batch of more, to which the oracle
    is close."""
    check_fwd(1, Hq, Hkv, N, D, sink, window, block, stride, seed=15)
    q, k, v = (x.to(DEV) for x in lg_synth.prefill_inputs(1, Hq, Hkv, N, D, 15, torch.bfloat16))
    out, lse = torch.empty_like(q), torch.empty(1, Hq, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(q, k, v, out, lse, sink, window, block, stride)
    many = 256 // (Hq * ((N + 127) // 128)) + 1
    qm, km, vm = (x.repeat(many, 1, 1, 1) for x in (q, k, v))
    om, lm = torch.empty_like(qm), torch.empty(many, Hq, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(qm, km, vm, om, lm, sink, window, block, stride)
    assert torch.equal(om, out.expand_as(om)) and torch.equal(lm, lse.expand_as(lm))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,sink,window,block,stride", [
    (4500, 0, 4500, 1, 0), (4700, 320, 4200, 1, 0), (4230, 64, 4096, 64, 0), (9000, 0, 128, 64, 2), (8300, 64, 192, 64, 40), (450, 0, 450, 1, 0)])
def test_walks_of_few_work_items(N, sink, window, block, stride, D):
    """The instance for few work items lists its key tiles 64 at a time: rows of 3, 4 and more than 64 tiles, lists that begin in
    the middle of a rotated run, groups of 64 tiles of which most are dead: the bits of the instance that walks without a list."""
    q, k, v = (x.to(DEV) for x in lg_synth.prefill_inputs(1, 1, 1, N, D, 16, torch.bfloat16))
    out, lse = torch.empty_like(q), torch.empty(1, 1, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(q, k, v, out, lse, sink, window, block, stride)
    many = 256 // ((N + 127) // 128) + 1
    qm, km, vm = (x.repeat(many, 1, 1, 1) for x in (q, k, v))
    om, lm = torch.empty_like(qm), torch.empty(many, 1, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(qm, km, vm, om, lm, sink, window, block, stride)
    assert torch.equal(om, out.expand_as(om)) and torch.equal(lm, lse.expand_as(lm))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,N,sink,window,block,stride", [
    (4, 2, 700, 64, 200, 1, 0), (2, 1, 1000, 64, 128, 64, 4), (1, 1, 4700, 320, 4200, 1, 0), (1, 1, 4230, 64, 4096, 64, 0),
    (1, 1, 8300, 64, 192, 64, 40), (1, 1, 450, 0, 450, 1, 0), (2, 1, 129, 4, 60, 1, 0)])
def test_384_work_items_and_more_give_the_same_bits(Hq, Hkv, N, sink, window, block, stride, D):
    """The instance for few work items takes up to 384: one sequence, the most copies of it within that and one more, as a batch
    and packed (up to 128 sequences)."""
    q, k, v = (x.to(DEV) for x in lg_synth.prefill_inputs(1, Hq, Hkv, N, D, 17, torch.bfloat16))
    out, lse = torch.empty_like(q), torch.empty(1, Hq, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(q, k, v, out, lse, sink, window, block, stride)
    most = 384 // (Hq * ((N + 127) // 128))
    for many in (most, most + 1):
        qm, km, vm = (x.repeat(many, 1, 1, 1) for x in (q, k, v))
        om, lm = torch.empty_like(qm), torch.empty(many, Hq, N, dtype=torch.float32, device=DEV)
        lg.lg_sparse_attn_fwd(qm, km, vm, om, lm, sink, window, block, stride)
        assert torch.equal(om, out.expand_as(om)) and torch.equal(lm, lse.expand_as(lm))
        qp, kp, vp = (x[0].repeat(1, many, 1) for x in (q, k, v))
        op, lp = torch.empty_like(qp), torch.empty(Hq, many * N, dtype=torch.float32, device=DEV)
        lg.lg_sparse_attn_fwd_varlen(qp, kp, vp, op, lp, [N * x for x in range(many + 1)], sink, window, block, stride)
        assert torch.equal(op, out[0].repeat(1, many, 1)) and torch.equal(lp, lse[0].repeat(1, many))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,N,sink,window,block,stride", [
    # rows of a few tiles (walked), of 9 and 10 (walked, listed), of more than 64 and more than 128 (lists follow one another)
    (2, 1, 1, 0, 1, 1, 0), (2, 2, 64, 0, 64, 1, 0), (2, 1, 129, 4, 60, 1, 0), (4, 2, 700, 64, 200, 1, 0), (2, 2, 576, 0, 576, 1, 0),
    (2, 2, 577, 0, 577, 1, 0), (2, 2, 640, 0, 640, 1, 0), (2, 2, 1090, 16, 100, 1, 0), (1, 1, 4500, 0, 4500, 1, 0), (1, 1, 4700, 320, 4200, 1, 0),
    (1, 1, 4230, 64, 4096, 64, 0), (1, 1, 9000, 0, 9000, 1, 0),
    # strided columns: near (listed) and far apart (walked), most of a group of 64 tiles live, few of them, one
    (2, 1, 1000, 64, 128, 64, 4), (1, 1, 9000, 0, 128, 64, 2), (1, 1, 9000, 64, 64, 64, 16), (1, 1, 9000, 64, 64, 64, 17),
    (1, 1, 8300, 64, 192, 64, 40), (1, 1, 3000, 16, 64, 16, 64), (1, 1, 3000, 0, 64, 1, 7)])
def test_few_work_items_and_more_than_384(Hq, Hkv, N, sink, window, block, stride, D):
    """Both instances for up to 384 work items, as a batch and packed: the bits of a batch of more than 384, which takes the instance
    without a list, and whose rows are close to the oracle."""
    items = Hq * ((N + 127) // 128)
    many = 384 // items + 1
    assert items <= 384 < many * items
    q, k, v = (x.to(DEV) for x in lg_synth.prefill_inputs(1, Hq, Hkv, N, D, 18, torch.bfloat16))
    qm, km, vm = (x.repeat(many, 1, 1, 1) for x in (q, k, v))
    om, lm = torch.empty_like(qm), torch.empty(many, Hq, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(qm, km, vm, om, lm, sink, window, block, stride)
    for packed in (False, True):
        out, lse = torch.full_like(q, float("nan")), torch.full((1, Hq, N), float("nan"), dtype=torch.float32, device=DEV)
        if packed:
            lg.lg_sparse_attn_fwd_varlen(q[0], k[0], v[0], out[0], lse[0], [0, N], sink, window, block, stride)
        else:
            lg.lg_sparse_attn_fwd(q, k, v, out, lse, sink, window, block, stride)
        assert torch.equal(om, out.expand_as(om)) and torch.equal(lm, lse.expand_as(lm)), packed
    rows = (max(0, N - 300), N)
    wo, wl = O.fwd(f32np(q), f32np(k), f32np(v), sink, window, block, stride, rows=rows)
    assert_close(f32np(om[many - 1:, :, rows[0]:]), wo[:, :, rows[0]:], TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16], "out")
    assert_close(f32np(lm[many - 1:, :, rows[0]:]), wl[:, :, rows[0]:], TOL_LSE[torch.bfloat16], None, "lse")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_sink_window_ragged_gqa(D, dtype):
    check_fwd(2, 4, 2, 700, D, 64, 200, dtype=dtype, seed=2)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,sink,window,block,stride", [
    (1, 0, 1, 1, 0), (33, 4, 8, 1, 0), (257, 0, 50, 1, 0), (500, 600, 3, 1, 0), (640, 5, 1000, 1, 0),
    (1024, 64, 192, 64, 8), (1000, 48, 96, 48, 3), (900, 0, 16, 16, 1), (777, 3, 10, 1, 7),
])
def test_patterns_and_edges(dtype, N, sink, window, block, stride):
    check_fwd(1, 2, 1, N, 128, sink, window, block, stride, dtype=dtype, seed=3)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_peaked_scores_and_custom_scale(dtype):
    check_fwd(1, 2, 2, 600, 128, 16, 100, dtype=dtype, seed=4, q_mul=8.0)
    check_fwd(1, 2, 2, 300, 64, 16, 100, dtype=dtype, seed=5, scale=0.3)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_zero_queries_closed_form(dtype):
    # Q = 0: lse_i = ln(number of live keys), out_i = mean of the live value rows
    N, D, sink, window = 600, 128, 7, 90
    _, k, v = lg_synth.prefill_inputs(1, 1, 1, N, D, 6, dtype)
    q = torch.zeros(1, 1, N, D, dtype=dtype)
    out, lse = run_fwd(q, k, v, sink, window)
    cnt = np.array([min(i + 1, window) + min(sink, max(0, i - window + 1)) for i in range(N)], dtype=np.float64)
    assert_close(f32np(lse)[0, 0], np.log(cnt), 1e-5, None, "lse closed form")
    m = O.mask(N, sink, window).astype(np.float64)
    mean_v = (m @ f32np(v)[0, 0].astype(np.float64)) / cnt[:, None]
    assert_close(f32np(out)[0, 0], mean_v, TOL_OUT[dtype], TOL_REL[dtype], "uniform average")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_dead_keys_do_not_matter(dtype):
    # keys that are dead for every probed row may hold any finite garbage: results are bit-identical
    N, D, sink, window = 1500, 128, 64, 256
    q, k, v = lg_synth.prefill_inputs(1, 2, 2, N, D, 7, dtype)
    out, lse = run_fwd(q, k, v, sink, window)
    rows = np.arange(1280, 1500)
    m = O.mask(N, sink, window)
    dead = torch.as_tensor(np.where(~m[rows].any(axis=0))[0])
    assert len(dead) > 500
    k2, v2 = k.clone(), v.clone()
    k2[:, :, dead] = 3.0e4
    v2[:, :, dead] = -7.0e4
    out2, lse2 = run_fwd(q, k2, v2, sink, window)
    assert torch.equal(out[:, :, rows], out2[:, :, rows]) and torch.equal(lse[:, :, rows], lse2[:, :, rows])


def test_lse_optional_and_deterministic():
    q, k, v = lg_synth.prefill_inputs(1, 2, 1, 500, 128, 8, torch.bfloat16)
    a, la = run_fwd(q, k, v, 8, 64)
    b, _ = run_fwd(q, k, v, 8, 64, want_lse=False)
    c, lc = run_fwd(q, k, v, 8, 64)
    assert torch.equal(a, b) and torch.equal(a, c) and torch.equal(la, lc)


def sampled_full_size(Hq, Hkv, N, sink, window, block, stride, seed, heads, row_starts, nrows=48):
    """Full-size launch (the benchmark's configuration); the oracle recomputes sampled rows."""
    D = 128
    q, k, v = lg_synth.prefill_inputs(1, Hq, Hkv, N, D, seed, torch.bfloat16, device=DEV)
    out = torch.empty_like(q)
    lse = torch.empty(1, Hq, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(q, k, v, out, lse, sink, window, block, stride)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()
    G = Hq // Hkv
    for hq in heads:
        qh = f32np(q[:, hq:hq + 1])
        kh = f32np(k[:, hq // G:hq // G + 1])
        vh = f32np(v[:, hq // G:hq // G + 1])
        for r0 in row_starts:
            r0 = min(r0, N - nrows)
            wo, wl = O.fwd(qh, kh, vh, sink, window, block, stride, rows=(r0, r0 + nrows))
            tag = "full-size N%d head %d rows %d.." % (N, hq, r0)
            assert_close(f32np(out[0, hq, r0:r0 + nrows]), wo[0, 0, r0:r0 + nrows], TOL_OUT[torch.bfloat16],
                         TOL_REL[torch.bfloat16], tag + " out")
            assert_close(f32np(lse[0, hq, r0:r0 + nrows]), wl[0, 0, r0:r0 + nrows], TOL_LSE[torch.bfloat16],
                         None, tag + " lse")


def test_config2_full_size_sampled():
    # Llama-2-7B shape, block-strided: 32 heads, N=32768, 64-token blocks, own+2 preceding, sink block, every 8th
    sampled_full_size(32, 32, 32768, 64, 192, 64, 8, 20241003, heads=[0, 13, 31],
                      row_starts=[0, 200, 4090, 16384 + 100, 32768])


def test_config4_full_size_sampled():
    # Llama-2-70B shape, GQA 64/8, N=131072, sink 64 + window 4096
    sampled_full_size(64, 8, 131072, 64, 4096, 1, 0, 20241005, heads=[0, 7, 8, 37, 63],
                      row_starts=[0, 4000, 4150, 65536 + 77, 131072])


def test_work_is_enqueued_on_the_callers_stream():
    # the binding hands torch's current stream to the library: a side stream must give the same bytes
    q, k, v = lg_synth.prefill_inputs(1, 4, 2, 3000, 128, 61, torch.bfloat16)
    a, la = run_fwd(q, k, v, 64, 512)
    side = torch.cuda.Stream()
    qd, kd, vd = (x.to(DEV) for x in (q, k, v))
    out = torch.empty_like(qd)
    lse = torch.empty(1, 4, 3000, dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        lg.lg_sparse_attn_fwd(qd, kd, vd, out, lse, 64, 512)
    side.synchronize()
    assert torch.equal(out, a) and torch.equal(lse, la)


def test_binding_rejects_mixed_dtypes_and_host_tensors():
    # the library reads every buffer of a call with ONE dtype code: the binding refuses anything else
    q, k, v = lg_synth.prefill_inputs(1, 2, 2, 128, 64, 3, torch.bfloat16)
    qd, kd, vd = (x.to(DEV) for x in (q, k, v))
    out = torch.empty_like(qd)
    lse = torch.empty(1, 2, 128, dtype=torch.float32, device=DEV)
    with pytest.raises(TypeError):
        lg.lg_sparse_attn_fwd(qd, kd.float(), vd, out, lse, 4, 16)
    with pytest.raises(TypeError):
        lg.lg_sparse_attn_fwd(qd, kd, vd, out.float(), lse, 4, 16)
    with pytest.raises(TypeError):
        lg.lg_sparse_attn_fwd(qd, kd, vd, out, lse.double(), 4, 16)
    with pytest.raises(ValueError):
        lg.lg_sparse_attn_fwd(qd, k, vd, out, lse, 4, 16)          # a host tensor
    lg.lg_sparse_attn_fwd(qd, kd, vd, out, lse, 4, 16)
    dq, dk, dv = torch.empty_like(qd), torch.empty_like(kd), torch.empty_like(vd)
    ws = torch.empty(lg.bwd_workspace_bytes(1, 2, 2, 128, 64, 4, 16, 1, 0, lg.LG_BF16), dtype=torch.uint8)
    with pytest.raises(TypeError):
        lg.lg_sparse_attn_bwd(qd, kd, vd, out, lse, qd, dq, dk, dv, ws, 4, 16)  # workspace in host memory
    with pytest.raises(TypeError):
        lg.lg_sparse_attn_bwd(qd, kd, vd, out, lse, qd, dq, dk.float(), dv, ws.to(DEV), 4, 16)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_without_a_finite_score(dtype):
    """Keys 0 .. 39 score -inf (a K entry of -inf against a positive query entry).  Rows that see no other key have no
    finite score: log-sum-exp -inf, output NaN (0 / 0); the others, some with a whole half of a key tile at -inf, are
    those of the keys that are left."""
    q, k, v = lg_synth.prefill_inputs(1, 2, 1, 300, 64, 31, dtype)
    q[..., 0] = q[..., 0].abs() + 0.1
    k[:, :, :40] = 0
    k[:, :, :40, 0] = float("-inf")
    out, lse = run_fwd(q, k, v, 4, 64)
    assert torch.isnan(out[:, :, :40]).all() and torch.isneginf(lse[:, :, :40]).all()
    wo, wl = O.fwd(f32np(q), f32np(k), f32np(v), 4, 64, rows=(40, 300))
    assert_close(f32np(out[:, :, 40:]), wo[:, :, 40:], TOL_OUT[dtype], TOL_REL[dtype], "out")
    assert_close(f32np(lse[:, :, 40:]), wl[:, :, 40:], TOL_LSE[dtype], None, "lse")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,N,sink,window,block,stride", [(1, 500, 0, 500, 1, 0), (1, 257, 64, 100, 1, 0), (1, 700, 64, 128, 64, 3),
                                                          (140, 300, 0, 300, 1, 0)])
def test_scores_far_above_the_first_ones(B, N, sink, window, block, stride, D):
    """bf16: keys 130 and 131 outscore the ones before them by more than any exponent holds, keys 200 and 201 these: rows that
    see them would overflow relative to the scores they met first, their neighbours would not.  Packed, the same bits."""
    q, k, v = lg_synth.prefill_inputs(1, 2, 1, N, D, 32, torch.bfloat16)
    q[:] = q.abs() + 0.5
    for j, x in ((130, 24.0), (200, 64.0)):
        k[:, :, j:j + 2] = x
    v[:, :, 131] = 3 * v[:, :, 130]
    wo, wl = O.fwd(f32np(q), f32np(k), f32np(v), sink, window, block, stride)
    qb, kb, vb = (x.expand(B, -1, -1, -1).contiguous() for x in (q, k, v))
    out, lse = run_fwd(qb, kb, vb, sink, window, block, stride)
    assert torch.equal(out, out[:1].expand_as(out)) and torch.equal(lse, lse[:1].expand_as(lse))
    assert_close(f32np(out[:1]), wo, TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16], "out")
    assert_close(f32np(lse[:1]), wl, TOL_LSE[torch.bfloat16], None, "lse")
    qp, kp, vp = (x[0].to(DEV).repeat(1, 2, 1) for x in (q, k, v))
    op, lp = torch.empty_like(qp), torch.empty(2, 2 * N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd_varlen(qp, kp, vp, op, lp, [0, N, 2 * N], sink, window, block, stride)
    assert torch.equal(op, out[0].repeat(1, 2, 1)) and torch.equal(lp, lse[0].repeat(1, 2))


def check_lse_of_growing_scores(q, k, lse, sink, window, block, stride):
    """lse [B, Hq, N] against 64 bits.  P is rounded to bf16, by 2^-8 of the value at most, and the row sum is of the rounded
    ones: 2^-8 for any row.  Where the largest score is more than 2^8 above all others' the reference has moved to it and its
    P is 1, so that only the others' share is rounded.  Beside these a score of float32 products, 16 roundings of it."""
    B, Hq, N, D = q.shape
    live = torch.as_tensor(O.mask(N, sink, window, block, stride)).to(DEV).bool()
    strict = 0
    for b in range(B):
        for h in range(Hq):
            s = q[b, h].to(DEV).double() @ k[b, h * k.shape[1] // Hq].to(DEV).double().T / D ** 0.5
            s = s.masked_fill(~live, -float("inf"))
            want = torch.logsumexp(s, -1)
            top = s.topk(min(2, N), dim=-1).values
            moved = top[:, 0] - top[:, -1] > 6  # (2^8 is 5.55)
            share = torch.where(moved, 1 - torch.exp(top[:, 0] - want), 1.0)
            err = (lse[b, h].double() - want).abs()
            bound = 2.0 ** -8 * share + 16 * 2.0 ** -24 * want.abs().clamp(min=1)
            assert (err <= bound).all(), (b, h, int((err / bound).argmax()), float((err / bound).max()), float(err.max()))
            strict += int(moved.sum())
    return strict


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("grow", [3.0, 5.5, 8.0, 40.0, 80.0, 87.0, 88.5, 300.0])
@pytest.mark.parametrize("B,Hq,Hkv,N,sink,window,block,stride", [
    (1, 4, 2, 500, 0, 500, 1, 0), (1, 2, 2, 400, 64, 128, 64, 3),        # up to 256 work items
    (5, 32, 4, 257, 16, 200, 1, 0), (2, 32, 16, 700, 64, 128, 64, 3)])  # more
def test_scores_that_grow(B, Hq, Hkv, N, sink, window, block, stride, grow, D):
    """bf16: rows whose scores outgrow the first ones, by less and by more than the 2^8 that moves the reference.  A key that
    carries a row has the probability 1, not a rounded one, and the log-sum-exp is as exact as that."""
    q, k, v = growing_inputs(B, Hq, Hkv, N, D, grow, 51)
    out, lse = run_fwd(q, k, v, sink, window, block, stride)
    strict = check_lse_of_growing_scores(q, k, lse, sink, window, block, stride)
    assert grow < 8 or strict > B * Hq * N // 4
    for b, h in ((0, 0), (B - 1, Hq - 1)):
        hk = h * Hkv // Hq
        wo, _ = O.fwd(*(f32np(x) for x in (q[b:b + 1, h:h + 1], k[b:b + 1, hk:hk + 1], v[b:b + 1, hk:hk + 1])), sink, window, block, stride)
        assert_close(f32np(out[b:b + 1, h:h + 1]), wo, TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16], "out %d %d" % (b, h))


@pytest.mark.parametrize("D", [64, 128])
def test_scores_that_grow_packed(D):
    """More than 256 work items of sequences that differ: the bits of each by itself."""
    Hq, Hkv, lens = 32, 4, [300, 37, 129, 400, 64, 255, 513]
    seqs = [growing_inputs(1, Hq, Hkv, n, D, 12.0 * (x + 1), 52 + x) for x, n in enumerate(lens)]
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    q, k, v = (torch.cat([s[x][0] for s in seqs], dim=1).contiguous().to(DEV) for x in range(3))
    out, lse = torch.empty_like(q), torch.empty(Hq, cu[-1], device=DEV)
    lg.lg_sparse_attn_fwd_varlen(q, k, v, out, lse, cu, 16, 200, 1, 0)
    for x, s in enumerate(seqs):
        o, l = run_fwd(*s, 16, 200)
        assert torch.equal(out[:, cu[x]:cu[x + 1]], o[0]) and torch.equal(lse[:, cu[x]:cu[x + 1]], l[0]), x
        check_lse_of_growing_scores(s[0], s[1], l, 16, 200, 1, 0)


@pytest.mark.parametrize("D", [64, 128])
def test_large_values_under_scores_that_grow(D):
    """Values of 2^100: their sum weighted relative to the first scores would overflow, relative to the largest it does not."""
    q, k, v = growing_inputs(1, 4, 2, 500, D, 60.0, 53)
    wo, _ = O.fwd(f32np(q), f32np(k), f32np(v), 0, 500)
    out, lse = run_fwd(q, k, v * 2.0 ** 100, 0, 500)
    assert_close(f32np(out).astype(np.float64) * 2.0 ** -100, wo, TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16], "out")
    check_lse_of_growing_scores(q, k, lse, 0, 500, 1, 0)


@pytest.mark.parametrize("D,scale", [(64, 0.0), (128, 0.0), (64, 40.0)])
def test_float32_scores_of_any_finite_size(D, scale):
    """One key in both halves of a tile outscores the others by far, at 2^100: it takes all the weight of the rows that
    see it, and the log-sum-exp is the scaled score."""
    q, k, v = lg_synth.prefill_inputs(1, 2, 1, 200, D, 33, torch.float32)
    q[:] = 2.0 ** 50 / D
    for j in (70, 100):
        k[:, :, j] = 2.0 ** 50 * (1 if j == 70 else 2)
    out, lse = run_fwd(q, k, v, 0, 200, scale=scale)
    sc = 2.0 ** 100 * (scale if scale > 0 else D ** -0.5)
    for r0, r1, j in ((70, 100, 70), (100, 200, 100)):
        assert torch.equal(out[:, :, r0:r1].cpu(), v[:, :, j:j + 1].expand(1, 2, r1 - r0, D)), j
        assert (np.abs(f32np(lse[:, :, r0:r1]).astype(np.float64) / (sc if j == 70 else 2 * sc) - 1) < 1e-6).all()
