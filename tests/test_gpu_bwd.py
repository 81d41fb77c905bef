"""GPU parity: lg_sparse_attn_bwd (through the C ABI) against the fp64 oracle, element by element.

The GPU backward consumes the GPU forward's own out / lse (as a training step does); the oracle
computes its forward in fp64 itself."""
import numpy as np
import pytest
import torch

import lg_synth
import paper_2410_01485_amd as lg
from gpu_util import DEV, TOL_LSE, TOL_OUT, TOL_REL, assert_close, check_fwd, dq_delta_allowance, f32np, growing_inputs
from oracle import lg_oracle as O

pytestmark = pytest.mark.gpu


def run_fwd_bwd(q, k, v, g, sink, window, block=1, stride=0, scale=0.0):
    qd, kd, vd, gd = (x.to(DEV) for x in (q, k, v, g))
    B, Hq, N, D = q.shape
    Hkv = k.shape[1]
    code = lg.LG_BF16 if q.dtype == torch.bfloat16 else lg.LG_F32
    out = torch.empty_like(qd)
    lse = torch.empty(B, Hq, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(qd, kd, vd, out, lse, sink, window, block, stride, scale)
    need = lg.bwd_workspace_bytes(B, Hq, Hkv, N, D, sink, window, block, stride, code)
    assert need >= B * Hq * N * 4
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    dq = torch.full_like(qd, float("nan"))
    dk = torch.full_like(kd, float("nan"))
    dv = torch.full_like(vd, float("nan"))
    lg.lg_sparse_attn_bwd(qd, kd, vd, out, lse, gd, dq, dk, dv, ws, sink, window, block, stride, scale)
    torch.cuda.synchronize()
    return dq, dk, dv


def check_bwd(B, Hq, Hkv, N, D, sink, window, block=1, stride=0, dtype=torch.bfloat16, seed=1, q_mul=1.0,
              scale=0.0, by_tensor_max=False):
    q, k, v, g = lg_synth.prefill_inputs(B, Hq, Hkv, N, D, seed, dtype, with_dout=True, q_mul=q_mul)
    dq, dk, dv = run_fwd_bwd(q, k, v, g, sink, window, block, stride, scale)
    w = O.bwd(f32np(q), f32np(k), f32np(v), f32np(g), sink, window, block, stride, scale if scale > 0 else None)
    tag = "bwd B%d Hq%d Hkv%d N%d D%d s%d w%d b%d st%d %s" % (B, Hq, Hkv, N, D, sink, window, block, stride, dtype)
    allow = None
    if dtype == torch.bfloat16:  # Delta comes from the bf16-rounded forward output (see dq_delta_allowance)
        allow = dq_delta_allowance(f32np(q), f32np(k), f32np(g), w["out"], sink, window, block, stride,
                                   scale if scale > 0 else None)
    for name, got in (("dq", dq), ("dk", dk), ("dv", dv)):
        assert_close(f32np(got), w[name], TOL_OUT[dtype], TOL_REL[dtype], tag + " " + name, by_tensor_max,
                     allow=allow if name == "dq" else None)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_sink_window_ragged_gqa(D, dtype):
    check_bwd(2, 4, 2, 700, D, 64, 200, dtype=dtype, seed=2)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,sink,window,block,stride", [
    (1, 0, 1, 1, 0), (33, 4, 8, 1, 0), (257, 0, 50, 1, 0), (500, 600, 3, 1, 0), (640, 5, 1000, 1, 0),
    (1024, 64, 192, 64, 8), (1000, 48, 96, 48, 3), (900, 0, 16, 16, 1), (777, 3, 10, 1, 7),
])
def test_patterns_and_edges(dtype, N, sink, window, block, stride):
    check_bwd(1, 2, 1, N, 128, sink, window, block, stride, dtype=dtype, seed=3)


@pytest.mark.parametrize("Hq,N,D,window", [(16, 500, 128, 500), (16, 500, 64, 200), (32, 250, 64, 250), (16, 300, 128, 300)])
def test_heads_that_take_their_tiles_in_the_other_order(Hq, N, D, window):
    """32 kv heads, which the forward and dq take four by four, 2 to 4 tiles each.  (dk/dv takes so few key tiles head by
    head: test_heads_four_by_four.)"""
    check_fwd(2, Hq, 16, N, D, 0, window, seed=6)
    check_bwd(2, Hq, 16, N, D, 0, window, seed=6)


@pytest.mark.parametrize("B,Hq,N,D,window", [
    (33, 32, 500, 128, 500), (34, 32, 500, 128, 200), (17, 32, 500, 64, 500), (18, 32, 385, 64, 100), (33, 32, 600, 128, 600), (17, 64, 300, 128, 80),
    (52, 32, 500, 128, 300), (33, 32, 500, 64, 500)])
def test_heads_four_by_four(B, Hq, N, D, window):
    """More than 2048 (key tile, kv head) pairs of 32 or 64 heads each.  dk/dv takes heads four by four, every other four the
    other way round where the heads are a multiple of 64; in the last two cases, with more items than four rounds, two heads
    in four the other way round (33 x 32 heads of three tiles: head by head).  Without a sink and groups the same bits as
    each sequence by itself, which takes other orders and is close to the oracle."""
    gen = torch.Generator(device=DEV).manual_seed(61)
    q, k, v, g = (torch.randn(B, Hq, N, D, generator=gen, device=DEV, dtype=torch.bfloat16) for _ in range(4))
    assert Hq * B % 32 == 0 and Hq * B * -(-N // (256 if D == 128 else 128)) > 2048
    got = run_fwd_bwd(q, k, v, g, 0, window)
    for b in range(B):
        one = [x[b:b + 1].contiguous() for x in (q, k, v, g)]
        for name, x, y in zip(("dq", "dk", "dv"), got, run_fwd_bwd(*one, 0, window)):
            assert torch.equal(x[b:b + 1], y), (name, b)
    h = [f32np(x[1:2, 5:7]) for x in (q, k, v, g)]
    w = O.bwd(*h, 0, window)
    al = dq_delta_allowance(h[0], h[1], h[3], w["out"], 0, window, 1, 0)
    for name, x in zip(("dq", "dk", "dv"), got):
        assert_close(f32np(x[1:2, 5:7]), w[name], TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16], name,
                     allow=al if name == "dq" else None)


@pytest.mark.parametrize("Hq,N,sink,window,block,stride", [
    (32, 3200, 0, 2600, 1, 0), (32, 3140, 64, 2624, 64, 0), (32, 3100, 64, 2304, 64, 8),
    (44, 2049, 0, 2048, 1, 0), (32, 9000, 64, 1024, 64, 5)])  # a last query tile of one row; 29 strided columns
def test_dq_in_64_row_form(Hq, N, sink, window, block, stride):
    """32 or more key tiles per query tile, 384 or more tiles of 256 rows and a ragged length: dq with 64 rows per wave.
    Sampled rows and keys of single heads: the first rows, the sink keys, where the window starts to slide, the last rows."""
    Hkv, D = Hq // 4, 128
    assert Hq * -(-N // 256) >= 384
    q, k, v, g = lg_synth.prefill_inputs(1, Hq, Hkv, N, D, 9, torch.bfloat16, with_dout=True, device=DEV)
    dq, dk, dv = run_fwd_bwd(q, k, v, g, sink, window, block, stride)
    tol, rel = TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16]
    mid = min(2590, N - 101)
    for h, r0, r1 in ((0, 0, 40), (13, mid, mid + 50), (Hq - 1, N - 50, N)):
        a = [f32np(x) for x in (q[:, h:h + 1], k[:, h // 4:h // 4 + 1], v[:, h // 4:h // 4 + 1], g[:, h:h + 1])]
        w = O.bwd(*a, sink, window, block, stride, rows=(r0, r1), keys=(0, 1))
        al = dq_delta_allowance(a[0], a[1], a[3], w["out"], sink, window, block, stride, rows=(r0, r1))
        assert_close(f32np(dq[0, h, r0:r1]), w["dq"][0, 0, r0:r1], tol, rel, "dq head %d" % h, allow=al[0, 0, r0:r1])
    for hk, k0, k1 in ((0, 0, 30), (5, 700, 730), (Hkv - 1, N - 30, N)):  # (a kv head's gradients: four query heads)
        a = [f32np(x) for x in (q[:, 4 * hk:4 * hk + 4], k[:, hk:hk + 1], v[:, hk:hk + 1], g[:, 4 * hk:4 * hk + 4])]
        w = O.bwd(*a, sink, window, block, stride, rows=(0, 1), keys=(k0, k1))
        assert_close(f32np(dk[0, hk, k0:k1]), w["dk"][0, 0, k0:k1], tol, rel, "dk head %d" % hk)
        assert_close(f32np(dv[0, hk, k0:k1]), w["dv"][0, 0, k0:k1], tol, rel, "dv head %d" % hk)


@pytest.mark.parametrize("B,Hq,N,window", [(3, 32, 3100, 2600), (2, 48, 2100, 2100)])
def test_work_queues_over_a_batch(B, Hq, N, window):
    """dq with 64 rows per wave and dk/dv with 64 keys per wave, whose work items of all sequences one queue hands out: the
    bits of each sequence by itself."""
    D = 128
    gen = torch.Generator(device=DEV).manual_seed(16)
    q, k, v, g = (torch.randn(B, Hq, N, D, generator=gen, device=DEV, dtype=torch.bfloat16) for _ in range(4))
    assert Hq * -(-N // 256) >= 384 and (window + 256) // 64 >= 32
    got = run_fwd_bwd(q, k, v, g, 0, window)
    for b in range(B):
        one = [x[b:b + 1].contiguous() for x in (q, k, v, g)]
        for name, x, y in zip(("dq", "dk", "dv"), got, run_fwd_bwd(*one, 0, window)):
            assert torch.equal(x[b:b + 1], y), (name, b)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,N,sink,window,block,stride", [
    (2, 1, 31, 0, 31, 1, 0), (2, 2, 33, 16, 5, 1, 0), (3, 1, 65, 0, 40, 1, 0), (1, 1, 97, 17, 8, 1, 0),
    (2, 1, 700, 0, 700, 1, 0), (4, 2, 900, 16, 64, 1, 0), (2, 1, 900, 33, 64, 1, 0), (2, 1, 530, 16, 48, 16, 3)])
def test_float32_key_tiles(Hq, Hkv, N, sink, window, block, stride, D):
    """32 keys per workgroup: lengths around the tile and the step, window and column parts (a sink of one group of 16
    keys, of two, of two tiles), cut where few tiles leave the chip idle."""
    check_bwd(1, Hq, Hkv, N, D, sink, window, block, stride, dtype=torch.float32, seed=8)


@pytest.mark.parametrize("B,Hq,Hkv,N,D,sink,window", [
    (1, 2, 1, 33, 64, 4, 9), (1, 1, 1, 700, 128, 16, 90), (2, 32, 32, 128, 128, 0, 128), (2, 32, 16, 129, 64, 4, 40),
    (2, 26, 13, 300, 64, 0, 300), (2, 32, 8, 384, 64, 16, 256), (2, 32, 8, 384, 128, 16, 255)])
def test_float32_dq_rows_per_workgroup(B, Hq, Hkv, N, D, sink, window):
    """32 or 64 query rows per workgroup, by the number of workgroups (up to 128, and 257 .. 384 with a reach of 256)."""
    check_bwd(B, Hq, Hkv, N, D, sink, window, dtype=torch.float32, seed=13)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,N,sink,window,block,stride", [
    (2, 1, 700, 16, 90, 1, 0), (4, 4, 385, 0, 385, 1, 0), (8, 2, 200, 16, 48, 16, 3), (1, 1, 97, 17, 30, 1, 0)])
def test_float32_rows_do_not_depend_on_the_batch(Hq, Hkv, N, sink, window, block, stride, D):
    """Alone a sequence has up to 128 workgroups of 64 rows and takes 32 rows each, in a batch of more it takes 64: out, lse and
    dq have the same bits."""
    many = 128 // (Hq * -(-N // 64)) + 1
    gen = torch.Generator(device=DEV).manual_seed(14)
    q, k, v, g = (torch.randn(many, h, N, D, generator=gen, device=DEV) for h in (Hq, Hkv, Hkv, Hq))

    def run(*x):
        B = x[0].shape[0]
        out, lse, dq, dk, dv = torch.empty_like(x[0]), torch.empty(B, Hq, N, device=DEV), *(torch.empty_like(y) for y in x[:3])
        lg.lg_sparse_attn_fwd(*x[:3], out, lse, sink, window, block, stride)
        ws = torch.empty(lg.bwd_workspace_bytes(B, Hq, Hkv, N, D, sink, window, block, stride, lg.LG_F32), dtype=torch.uint8, device=DEV)
        lg.lg_sparse_attn_bwd(*x[:3], out, lse, x[3], dq, dk, dv, ws, sink, window, block, stride)
        return out, lse, dq

    got = run(q, k, v, g)
    for b in (0, many - 1):
        for name, x, y in zip(("out", "lse", "dq"), got, run(*(t[b:b + 1].contiguous() for t in (q, k, v, g)))):
            assert torch.equal(x[b:b + 1], y), (name, b)


@pytest.mark.parametrize("B,Hq,Hkv,N,D,sink,window,block,stride", [
    (17, 8, 4, 1030, 64, 4, 90, 1, 0), (9, 12, 12, 650, 64, 0, 650, 1, 0), (5, 4, 2, 700, 128, 16, 48, 16, 3)])
def test_float32_backward_in_one_launch_and_in_two(B, Hq, Hkv, N, D, sink, window, block, stride):
    """Up to 4096 (head dim 128: 512) workgroups dq and dk/dv share a launch, in either order: a batch on one side of the limit and
    one of its sequences on the other give the same bits of dq, and dk and dv differ by float32 rounding at most (their parts are cut
    by the batch: 2^-22 of the sum of magnitudes, taken as the tensor's largest value times 16)."""
    gen = torch.Generator(device=DEV).manual_seed(15)
    q, k, v, g = (torch.randn(B, h, N, D, generator=gen, device=DEV) for h in (Hq, Hkv, Hkv, Hq))

    def run(*x):
        n = x[0].shape[0]
        out, lse, dq, dk, dv = torch.empty_like(x[0]), torch.empty(n, Hq, N, device=DEV), *(torch.full_like(y, float("nan")) for y in x[:3])
        lg.lg_sparse_attn_fwd(*x[:3], out, lse, sink, window, block, stride)
        need = lg.bwd_workspace_bytes(n, Hq, Hkv, N, D, sink, window, block, stride, lg.LG_F32)
        ws = torch.full((need,), 255, dtype=torch.uint8, device=DEV)
        lg.lg_sparse_attn_bwd(*x[:3], out, lse, x[3], dq, dk, dv, ws, sink, window, block, stride)
        return dq, dk, dv

    got = run(q, k, v, g)
    for b in (0, B - 1):
        one = run(*(t[b:b + 1].contiguous() for t in (q, k, v, g)))
        assert torch.equal(got[0][b:b + 1], one[0])
        for x, y in zip(got[1:], one[1:]):
            assert float((x[b:b + 1] - y).abs().max()) <= 2.0 ** -18 * float(y.abs().max())


@pytest.mark.parametrize("B,Hq,Hkv,N,D,sink,window,block,stride", [
    (60, 8, 8, 1030, 64, 4, 90, 1, 0), (22, 8, 8, 1030, 128, 0, 300, 1, 0), (22, 8, 2, 1030, 128, 64, 300, 1, 0), (60, 8, 4, 1150, 64, 64, 192, 64, 4),
    (60, 8, 4, 1030, 64, 16, 100, 1, 0), (22, 8, 8, 1030, 128, 16, 100, 1, 0),
    (50, 16, 16, 129, 128, 0, 129, 1, 0)])
def test_bf16_backward_in_one_launch_and_in_two(B, Hq, Hkv, N, D, sink, window, block, stride):
    """Up to 8192 (head dim 128: 1536) workgroups dq and dk/dv share a launch: a batch beyond that and one of its sequences alone and
    packed give the same bits of dq, without groups of query heads and columns of dk and dv as well; otherwise these are sums in
    another order, and a bf16 rounding apart at most (2^-7 of a value; 2^-16 of the tensor's largest where terms cancel)."""
    gen = torch.Generator(device=DEV).manual_seed(16)
    q, k, v, g = (torch.randn(B, h, N, D, generator=gen, device=DEV, dtype=torch.bfloat16) for h in (Hq, Hkv, Hkv, Hq))
    pat = (sink, window, block, stride)

    def run(*x):
        n = x[0].shape[0]
        out, lse, dq, dk, dv = torch.empty_like(x[0]), torch.empty(n, Hq, N, device=DEV), *(torch.full_like(y, float("nan")) for y in x[:3])
        lg.lg_sparse_attn_fwd(*x[:3], out, lse, *pat)
        ws = torch.full((lg.bwd_workspace_bytes(n, Hq, Hkv, N, D, *pat, lg.LG_BF16),), 255, dtype=torch.uint8, device=DEV)
        lg.lg_sparse_attn_bwd(*x[:3], out, lse, x[3], dq, dk, dv, ws, *pat)
        return dq, dk, dv

    def run_packed(*x):  # the sequence and its first 70 rows
        x = [torch.cat([y[0], y[0, :, :70]], dim=1).contiguous() for y in x]
        cu = [0, N, N + 70]
        out, lse, dq, dk, dv = torch.empty_like(x[0]), torch.empty(Hq, N + 70, device=DEV), *(torch.full_like(y, float("nan")) for y in x[:3])
        lg.lg_sparse_attn_fwd_varlen(*x[:3], out, lse, cu, *pat)
        ws = torch.full((lg.bwd_varlen_workspace_bytes(cu, Hq, Hkv, D, *pat, lg.LG_BF16),), 255, dtype=torch.uint8, device=DEV)
        lg.lg_sparse_attn_bwd_varlen(*x[:3], out, lse, x[3], dq, dk, dv, ws, cu, *pat)
        return tuple(y[None, :, :N] for y in (dq, dk, dv))

    got = run(q, k, v, g)
    for b in (0, B - 1):
        for f in (run, run_packed):
            one = f(*(t[b:b + 1].contiguous() for t in (q, k, v, g)))
            assert torch.equal(got[0][b:b + 1], one[0]), (b, f)
            for x, y in zip(got[1:], one[1:]):
                x, y = x[b:b + 1].float(), y.float()
                if Hq == Hkv and stride == 0:
                    assert torch.equal(x, y), (b, f)
                else:
                    assert bool(((x - y).abs() <= 2.0 ** -7 * y.abs() + 2.0 ** -16 * y.abs().max()).all()), (b, f)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_peaked_scores_and_custom_scale(dtype):
    check_bwd(1, 2, 2, 600, 128, 16, 100, dtype=dtype, seed=4, q_mul=4.0, by_tensor_max=True)
    check_bwd(1, 4, 1, 300, 64, 16, 100, dtype=dtype, seed=5, scale=0.3, by_tensor_max=True)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("grow", [7.0, 8.0, 9.3, 11.0, 40.0, 80.0])
@pytest.mark.parametrize("N,sink,window", [(700, 0, 700), (900, 64, 200)])
def test_dv_of_scores_that_grow(N, sink, window, grow, D):
    """All queries of a head alike, two keys that outscore all before them, one after the other: their dv is the sum of the dO
    of the rows that they carry, and all of those rows have the same log-sum-exp, whose error would be dv's.  The other keys'
    share of a row is below x = 2 N exp(-grow): as much as their rounding, 2^-8 of it, is the log-sum-exp off, and P, 1 - x or
    more, is rounded by x or by 2^-9; dv's D roundings to bf16, of 2^-8 at most, have a standard deviation of 2^-9 / sqrt(D)
    in the mean."""
    Hq = Hkv = 4
    q, k, v, g = growing_inputs(1, Hq, Hkv, N, D, grow, 54, dout=True)
    q[:] = q[:, :, :1]
    dv = run_fwd_bwd(q, k, v, g, sink, window)[2]
    w = O.bwd(f32np(q), f32np(k), f32np(v), f32np(g), sink, window)
    assert_close(f32np(dv), w["dv"], TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16], "dv", True)
    x = 2 * N * np.exp(-grow)
    for h in range(Hkv):
        for j in (N // 5 + 7 * h, N // 2 + 5 * h):
            want = w["dv"][0, h, j]
            off = float((f32np(dv[0, h, j]).astype(np.float64) * want).sum() / (want * want).sum()) - 1
            assert abs(off) <= 6 * 2.0 ** -9 / D ** 0.5 + 2.0 ** -8 * min(1.0, x) + min(x, 2.0 ** -9), (h, j, off)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_masked_keys_get_exactly_zero_gradient(dtype):
    # upstream gradient only on a few rows: keys dead for all of them get dk = dv = 0 exactly,
    # and every other query row gets dq = 0 exactly
    N, D, sink, window = 1500, 128, 64, 256
    q, k, v, g = lg_synth.prefill_inputs(1, 2, 2, N, D, 7, dtype, with_dout=True)
    rows = np.arange(1300, 1400)
    g2 = torch.zeros_like(g)
    g2[:, :, rows] = g[:, :, rows]
    dq, dk, dv = run_fwd_bwd(q, k, v, g2, sink, window)
    m = O.mask(N, sink, window)
    dead = np.where(~m[rows].any(axis=0))[0]
    assert len(dead) > 1000
    assert (f32np(dk)[:, :, dead] == 0).all() and (f32np(dv)[:, :, dead] == 0).all()
    other = np.setdiff1d(np.arange(N), rows)
    assert (f32np(dq)[:, :, other] == 0).all()
    assert np.abs(f32np(dq)[:, :, rows]).sum() > 0


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,sink,window,block,stride", [(3000, 64, 512, 1, 0), (3000, 64, 192, 64, 8),
                                                        (2600, 0, 1100, 1, 0)])
def test_never_loaded_key_tiles_may_hold_nan_and_inf(dtype, N, sink, window, block, stride):
    """Key tiles that are dead for a whole 256-row query tile are never loaded by the forward and dq kernels
    (Section 3.2: a masked block is skipped by not loading it): NaN in K and Inf in V there leave out, lse and
    dq of those rows bit-identical.  (Rows outside the probed tile do see those keys and turn non-finite,
    and so do dk / dv of the poisoned keys themselves.)"""
    D = 128
    q, k, v, g = lg_synth.prefill_inputs(1, 2, 1, N, D, 71, dtype, with_dout=True)
    rows = np.arange(2048, 2304)                      # one 256-row query tile (a multiple of every kernel's tile)
    m = O.mask(N, sink, window, block, stride)
    tile_dead = ~m[rows].reshape(len(rows), -1)[:, :(N // 64) * 64].reshape(len(rows), N // 64, 64).any(axis=(0, 2))
    dead = np.where(np.repeat(tile_dead, 64))[0]      # every key of a 64-key tile no probed row sees
    assert len(dead) > 1000 and (dead < 2048).sum() > 500 and (dead >= 2304).sum() > 200
    k2, v2 = k.clone(), v.clone()
    k2[:, :, torch.as_tensor(dead)] = float("nan")
    v2[:, :, torch.as_tensor(dead)] = float("inf")
    g2 = torch.zeros_like(g)
    g2[:, :, rows] = g[:, :, rows]                    # upstream gradient on the probed rows only

    def run(kk, vv):
        qd, kd, vd, gd = (x.to(DEV) for x in (q, kk, vv, g2))
        out = torch.empty_like(qd)
        lse = torch.empty(1, 2, N, dtype=torch.float32, device=DEV)
        lg.lg_sparse_attn_fwd(qd, kd, vd, out, lse, sink, window, block, stride)
        code = lg.LG_BF16 if dtype == torch.bfloat16 else lg.LG_F32
        ws = torch.empty(lg.bwd_workspace_bytes(1, 2, 1, N, D, sink, window, block, stride, code), dtype=torch.uint8,
                         device=DEV)
        dq, dk, dv = torch.empty_like(qd), torch.empty_like(kd), torch.empty_like(vd)
        lg.lg_sparse_attn_bwd(qd, kd, vd, out, lse, gd, dq, dk, dv, ws, sink, window, block, stride)
        torch.cuda.synchronize()
        return out[:, :, rows].cpu(), lse[:, :, rows].cpu(), dq[:, :, rows].cpu()

    clean, poisoned = run(k, v), run(k2, v2)
    for name, a, b in zip(("out", "lse", "dq"), clean, poisoned):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b), name
    w = O.bwd(f32np(q), f32np(k), f32np(v), f32np(g2), sink, window, block, stride, rows=(2048, 2304), keys=(0, 1))
    assert_close(f32np(poisoned[0]), w["out"][:, :, rows], TOL_OUT[dtype], TOL_REL[dtype], "poisoned out")
    al = dq_delta_allowance(f32np(q), f32np(k), f32np(g2), w["out"], sink, window, block, stride, rows=(2048, 2304))
    assert_close(f32np(poisoned[2]), w["dq"][:, :, rows], TOL_OUT[dtype], TOL_REL[dtype], "poisoned dq",
                 allow=al[:, :, rows] if dtype == torch.bfloat16 else None)


@pytest.mark.parametrize("B,Hq,Hkv,N,D,sink,window,block,stride", [
    # several column groups (sink + strided blocks), column parts longer than one chunk of 4096
    # rows, GQA, ragged ends; a virtual tile with fewer than 4 groups; token-granular strided columns
    (1, 4, 2, 9000, 128, 64, 128, 64, 4),
    (2, 2, 2, 5003, 64, 16, 48, 16, 3),
    (1, 2, 1, 4700, 128, 0, 64, 64, 16),
    (1, 2, 2, 4500, 128, 2, 6, 1, 9),
])
def test_strided_columns_long_context(B, Hq, Hkv, N, D, sink, window, block, stride):
    check_bwd(B, Hq, Hkv, N, D, sink, window, block, stride, dtype=torch.bfloat16, seed=41)


@pytest.mark.parametrize("B,Hq,Hkv,N,D,sink,window,block,stride", [
    # windows of 16 or more tiles at D = 128 select dk/dv with 64 keys per wave (dq stays with 32 rows per wave, with too few
    # tiles of rows for the other form: test_dq_in_64_row_form):
    # token-granular with a ragged end (sink tile handled by the main instance); GQA with batch
    # (column instance + partial sums folded into the main instance); block-granular; block-strided
    # (both instances in the 64-keys form); no sink and a window longer than most rows
    (1, 2, 2, 3001, 128, 64, 1024, 1, 0),
    (2, 4, 2, 2500, 128, 3, 900, 1, 0),
    (1, 2, 1, 3333, 128, 64, 1024, 64, 0),
    (1, 2, 2, 4100, 128, 64, 1024, 64, 8),
    (1, 1, 1, 2049, 128, 0, 2048, 1, 0),
    # column instance of the 64-keys-per-wave kernel: 29 column groups (a last virtual tile of one), column
    # parts longer than one chunk, GQA, ragged end
    (1, 4, 2, 9000, 128, 64, 1024, 64, 5),
])
def test_long_windows_wide_kernels(B, Hq, Hkv, N, D, sink, window, block, stride):
    check_bwd(B, Hq, Hkv, N, D, sink, window, block, stride, dtype=torch.bfloat16, seed=77)


@pytest.mark.parametrize("B,Hq,Hkv,N,D,sink,window,block,stride", [
    # float32 dk/dv parts: a sink in one 16-key group (one wave per row block), in two and in five groups; window parts
    # split over workgroups; column parts of strided blocks; a window whose last rows end one tile before the sequence
    (1, 4, 2, 1500, 64, 16, 128, 1, 0),
    (2, 2, 1, 1100, 128, 40, 64, 1, 0),
    (1, 2, 2, 1000, 64, 70, 100, 1, 0),
    (1, 1, 1, 1030, 128, 0, 1030, 1, 0),
    (1, 2, 1, 900, 64, 48, 96, 48, 3),
    (1, 2, 2, 192, 64, 8, 65, 1, 0),
    # 288 key tiles of rows that grow, cut in two
    (1, 9, 9, 1000, 64, 0, 1000, 1, 0),
    (1, 10, 10, 1000, 128, 0, 1000, 1, 0),
])
def test_float32_parts(B, Hq, Hkv, N, D, sink, window, block, stride):
    check_bwd(B, Hq, Hkv, N, D, sink, window, block, stride, dtype=torch.float32, seed=83)


@pytest.mark.parametrize("B,Hq,Hkv,N,D,sink,window,block,stride", [
    # few key tiles: window parts cut by query heads and rows (a cut without rows at the end of the sequence, a group of
    # three heads, one key tile); lone column groups in one chunk, several, none (a short column part), half a group live
    (1, 8, 2, 2064, 128, 16, 673, 1, 0),
    (1, 8, 1, 1300, 64, 40, 130, 1, 0),
    (1, 6, 2, 1500, 128, 64, 64, 64, 4),
    (1, 4, 1, 260, 128, 4, 100, 1, 0),
    (2, 2, 2, 3001, 64, 64, 128, 1, 0),
    (1, 2, 2, 9000, 128, 5, 700, 1, 0),
    (1, 1, 1, 900, 128, 16, 256, 1, 0),
    (1, 2, 2, 2500, 64, 64, 64, 64, 3),
])
def test_window_parts_and_lone_columns(B, Hq, Hkv, N, D, sink, window, block, stride):
    check_bwd(B, Hq, Hkv, N, D, sink, window, block, stride, seed=84)


@pytest.mark.parametrize("Hq,Hkv,N,sink,window,block,stride", [
    (2, 1, 65, 0, 65, 1, 0),            # one key tile, two steps
    (8, 1, 300, 16, 128, 1, 0), (16, 4, 473, 0, 473, 1, 0), (4, 2, 1131, 64, 128, 64, 8), (3, 3, 1200, 64, 256, 64, 4),
    (64, 32, 2048, 64, 192, 64, 0),     # 768 work items of dq and dk/dv before the cut, and more
    (64, 32, 2049, 64, 192, 64, 0)])
def test_window_parts_beside_dq(Hq, Hkv, N, sink, window, block, stride):
    """bf16, head dim 128: up to 768 work items the window parts are cut in view of dq's, which share the launch."""
    check_bwd(1, Hq, Hkv, N, 128, sink, window, block, stride, seed=33)


@pytest.mark.parametrize("B,Hq,Hkv,N,D,sink,window", [(4, 32, 16, 2177, 64, 16, 128), (3, 32, 16, 2753, 128, 5, 128)])
def test_lone_groups_before_the_shared_launch(B, Hq, Hkv, N, D, sink, window):
    """bf16, groups of query heads, too many key tiles for a cut: the sink's column parts come before the launch of dq and dk/dv (head
    dim 64), and beyond 100 MB of out and dO (head dim 128) dq and dk/dv have one each."""
    check_bwd(B, Hq, Hkv, N, D, sink, window, seed=34)


def test_bwd_deterministic_long_window():
    q, k, v, g = lg_synth.prefill_inputs(1, 2, 2, 2000, 128, 10, torch.bfloat16, with_dout=True)
    a = run_fwd_bwd(q, k, v, g, 64, 1024)
    b = run_fwd_bwd(q, k, v, g, 64, 1024)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def test_bwd_deterministic():
    # sink + window without GQA has no atomics anywhere: bit-identical from run to run (the partial dk/dv
    # sums of column keys in strided or GQA calls are added with float atomics, in no fixed order)
    q, k, v, g = lg_synth.prefill_inputs(1, 4, 4, 900, 128, 9, torch.bfloat16, with_dout=True)
    a = run_fwd_bwd(q, k, v, g, 64, 300)
    b = run_fwd_bwd(q, k, v, g, 64, 300)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def test_config3_shape_reduced_n_all_heads():
    # config 3's heads, head dim, sink and window at a sequence the oracle finishes: N = 6144
    check_bwd(1, 32, 32, 6144, 128, 64, 4096, dtype=torch.bfloat16, seed=20241004)


def test_config3_full_size_sampled():
    """Training-step configuration as the benchmark launches it: B1, 32 heads, N=131072, D=128, sink 64,
    window 4096.  The oracle recomputes sampled query rows (dq) and sampled keys (dk, dv) of two heads."""
    B, H, N, D, sink, window = 1, 32, 131072, 128, 64, 4096
    q, k, v, g = lg_synth.prefill_inputs(B, H, H, N, D, 20241004, torch.bfloat16, with_dout=True, device=DEV)
    out = torch.empty_like(q)
    lse = torch.empty(B, H, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(q, k, v, out, lse, sink, window)
    ws = torch.empty(lg.bwd_workspace_bytes(B, H, H, N, D, sink, window, 1, 0, lg.LG_BF16),
                     dtype=torch.uint8, device=DEV)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    lg.lg_sparse_attn_bwd(q, k, v, out, lse, g, dq, dk, dv, ws, sink, window)
    torch.cuda.synchronize()
    for t in (dq, dk, dv):
        assert torch.isfinite(t.float()).all()
    tol, rel = TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16]
    for h, rows, keys in ((0, (0, 40), (0, 40)),                      # first rows; sink keys (seen by every row)
                          (0, (4080, 4120), (4140, 4180)),            # where the window starts to slide
                          (21, (70001, 70041), (99990, 100030)),      # steady state
                          (31, (N - 40, N), (N - 40, N))):            # ragged end of the sequence
        print("head", h, "rows", rows, "keys", keys, flush=True)
        a = [f32np(x[:, h:h + 1]) for x in (q, k, v, g)]
        w = O.bwd(*a, sink, window, rows=rows, keys=keys)
        al = dq_delta_allowance(a[0], a[1], a[3], w["out"], sink, window, rows=rows)
        assert_close(f32np(dq[0, h, rows[0]:rows[1]]), w["dq"][0, 0, rows[0]:rows[1]], tol, rel, "cfg3 dq h%d" % h,
                     allow=al[0, 0, rows[0]:rows[1]])
        assert_close(f32np(dk[0, h, keys[0]:keys[1]]), w["dk"][0, 0, keys[0]:keys[1]], tol, rel, "cfg3 dk h%d" % h)
        assert_close(f32np(dv[0, h, keys[0]:keys[1]]), w["dv"][0, 0, keys[0]:keys[1]], tol, rel, "cfg3 dv h%d" % h)
        assert_close(f32np(out[0, h, rows[0]:rows[1]]), w["out"][0, 0, rows[0]:rows[1]], tol, rel, "cfg3 out h%d" % h)
        assert_close(f32np(lse[0, h, rows[0]:rows[1]]), w["lse"][0, 0, rows[0]:rows[1]], TOL_LSE[torch.bfloat16], None,
                     "cfg3 lse h%d" % h)


def test_paper_block_settings_full_size_sampled():
    """Section 4.1 settings combined at the training length: 64-token blocks, 1 sink block, 32 local blocks
    and every 64th block as a strided column; B1, 32 heads, N=131072, D=128.  The oracle recomputes sampled
    query rows (dq) and sampled keys (dk, dv): sink keys, keys of a strided column (seen by every later row,
    accumulated over many workgroups), window-only keys, and the ragged end."""
    B, H, N, D, sink, window, block, stride = 1, 32, 131072, 128, 64, 2048, 64, 64
    q, k, v, g = lg_synth.prefill_inputs(B, H, H, N, D, 20241009, torch.bfloat16, with_dout=True, device=DEV)
    out = torch.empty_like(q)
    lse = torch.empty(B, H, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(q, k, v, out, lse, sink, window, block, stride)
    ws = torch.empty(lg.bwd_workspace_bytes(B, H, H, N, D, sink, window, block, stride, lg.LG_BF16),
                     dtype=torch.uint8, device=DEV)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    lg.lg_sparse_attn_bwd(q, k, v, out, lse, g, dq, dk, dv, ws, sink, window, block, stride)
    torch.cuda.synchronize()
    for t in (dq, dk, dv):
        assert torch.isfinite(t.float()).all()
    tol, rel = TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16]
    col = 63 * 64  # first strided column block
    for h, rows, keys in ((0, (0, 40), (20, 60)),                       # sink keys
                          (7, (70001, 70041), (col + 10, col + 50)),    # a strided column
                          (11, (120000, 120040), (1087 * 64 + 10, 1087 * 64 + 50)),   # a strided column past 64-key group 1024
                          (19, (100000, 100040), (90010, 90050)),       # window-only keys
                          (31, (N - 40, N), (N - 40, N))):              # the end of the sequence
        print("head", h, "rows", rows, "keys", keys, flush=True)
        a = [f32np(x[:, h:h + 1]) for x in (q, k, v, g)]
        w = O.bwd(*a, sink, window, block, stride, rows=rows, keys=keys)
        al = dq_delta_allowance(a[0], a[1], a[3], w["out"], sink, window, block, stride, rows=rows)
        assert_close(f32np(dq[0, h, rows[0]:rows[1]]), w["dq"][0, 0, rows[0]:rows[1]], tol, rel, "paper dq h%d" % h,
                     allow=al[0, 0, rows[0]:rows[1]])
        assert_close(f32np(dk[0, h, keys[0]:keys[1]]), w["dk"][0, 0, keys[0]:keys[1]], tol, rel, "paper dk h%d" % h)
        assert_close(f32np(dv[0, h, keys[0]:keys[1]]), w["dv"][0, 0, keys[0]:keys[1]], tol, rel, "paper dv h%d" % h)
        assert_close(f32np(out[0, h, rows[0]:rows[1]]), w["out"][0, 0, rows[0]:rows[1]], tol, rel, "paper out h%d" % h)
        assert_close(f32np(lse[0, h, rows[0]:rows[1]]), w["lse"][0, 0, rows[0]:rows[1]], TOL_LSE[torch.bfloat16], None,
                     "paper lse h%d" % h)


def test_one_million_tokens_sampled():
    """Index arithmetic at 2^20 tokens (8x the benchmark length), one head pair with GQA: forward and backward
    against the oracle on sampled rows and on sampled keys outside the sink (the sink keys would need the
    whole forward on the CPU)."""
    B, Hq, Hkv, N, D, sink, window = 1, 2, 1, 1 << 20, 128, 64, 4096
    q, k, v, g = lg_synth.prefill_inputs(B, Hq, Hkv, N, D, 20241010, torch.bfloat16, with_dout=True, device=DEV)
    out = torch.empty_like(q)
    lse = torch.empty(B, Hq, N, dtype=torch.float32, device=DEV)
    lg.lg_sparse_attn_fwd(q, k, v, out, lse, sink, window)
    ws = torch.empty(lg.bwd_workspace_bytes(B, Hq, Hkv, N, D, sink, window, 1, 0, lg.LG_BF16), dtype=torch.uint8,
                     device=DEV)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    lg.lg_sparse_attn_bwd(q, k, v, out, lse, g, dq, dk, dv, ws, sink, window)
    torch.cuda.synchronize()
    for t in (out, dq, dk, dv):
        assert torch.isfinite(t.float()).all()
    tol, rel = TOL_OUT[torch.bfloat16], TOL_REL[torch.bfloat16]
    a = [f32np(x) for x in (q, k, v, g)]
    for rows, keys in (((600001, 600041), (777770, 777810)), ((N - 40, N), (N - 40, N))):
        print("rows", rows, "keys", keys, flush=True)
        w = O.bwd(*a, sink, window, rows=rows, keys=keys)
        r, c = slice(*rows), slice(*keys)
        assert_close(f32np(out[0, :, r]), w["out"][0, :, r], tol, rel, "1M out")
        assert_close(f32np(lse[0, :, r]), w["lse"][0, :, r], TOL_LSE[torch.bfloat16], None, "1M lse")
        al = dq_delta_allowance(a[0], a[1], a[3], w["out"], sink, window, rows=rows)
        assert_close(f32np(dq[0, :, r]), w["dq"][0, :, r], tol, rel, "1M dq", allow=al[0, :, r])
        assert_close(f32np(dk[0, :, c]), w["dk"][0, :, c], tol, rel, "1M dk")
        assert_close(f32np(dv[0, :, c]), w["dv"][0, :, c], tol, rel, "1M dv")
