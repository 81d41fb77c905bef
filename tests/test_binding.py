"""The two ways from torch tensors to the C ABI: the extension module (csrc/lg_bind.cpp) and, where it is not built for the
interpreter, binding_ctypes.py.  Both make the same checks, raise the same errors and give the same results."""
import os
import sysconfig

import pytest
import torch

import paper_2410_01485_amd as lg
from paper_2410_01485_amd import binding, build, binding_ctypes

HERE = os.path.dirname(os.path.abspath(build.__file__))


def test_module_carries_the_interpreters_tag():
    assert build.BIND_NAME.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert os.path.exists(os.path.join(HERE, build.BIND_NAME))
    assert not os.path.exists(os.path.join(HERE, "_lg_bind.so"))


def test_the_library_is_there_when_only_the_module_fails(tmp_path, monkeypatch):
    """A machine without Python's or torch's headers gets a working package, and is told."""
    (tmp_path / "one.hip").write_text("extern \"C\" int one() { return 1; }\n")
    (tmp_path / "bind.cpp").write_text("#include <no_such_header.h>\n")
    monkeypatch.setattr(build, "sources", lambda: [str(tmp_path / "one.hip")])
    monkeypatch.setattr(build, "BIND_SRC", str(tmp_path / "bind.cpp"))
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    with pytest.raises(RuntimeError, match="through ctypes"):
        build.build(verbose=False, out=str(tmp_path / "libone.so"))
    assert os.path.exists(tmp_path / "libone.so")


def test_without_the_module_calls_go_through_ctypes(monkeypatch):
    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.setattr(build, "BIND_NAME", "no_such_module.so")
    with pytest.warns(RuntimeWarning, match="ctypes"):
        assert binding._load_native() is binding_ctypes


def z(*shape, dtype=torch.bfloat16):
    return torch.zeros(*shape, dtype=dtype)


CALLS = {
    "fwd": (z(1, 2, 8, 64), z(1, 1, 8, 64), z(1, 1, 8, 64), z(1, 2, 8, 64), None, 0, 4, 1, 0, 0.0),
    "bwd": (z(1, 2, 8, 64), z(1, 1, 8, 64), z(1, 1, 8, 64), z(1, 2, 8, 64), z(1, 2, 8), z(1, 2, 8, 64), z(1, 2, 8, 64),
            z(1, 1, 8, 64), z(1, 1, 8, 64), z(16), 0, 4, 1, 0, 0.0),
    "fwd_varlen": (z(2, 8, 64), z(1, 8, 64), z(1, 8, 64), z(2, 8, 64), None, [0, 3, 8], 0, 4, 1, 0, 0.0),
    "bwd_varlen": (z(2, 8, 64), z(1, 8, 64), z(1, 8, 64), z(2, 8, 64), z(2, 8), z(2, 8, 64), z(2, 8, 64), z(1, 8, 64),
                   z(1, 8, 64), z(16), [0, 8], 0, 4, 1, 0, 0.0),
    "decode": (z(1, 2, 64), z(1, 1, 6, 64), z(1, 1, 6, 64), z(1, 2, 64), None, None, 5, 2, 4, 1, 0, 0.0),
    "decode_cache": (z(1, 2, 64), z(1, 1, 6, 64), z(1, 1, 6, 64), z(1, 2, 64), None, None, 5, 2, 4, 1, 0, 0.0),
    "decode_cache_static": (z(1, 2, 64), z(1, 1, 6, 64), z(1, 1, 6, 64), z(1, 2, 64), None, 5, 2, 4, 1, 0, 0.0),
    "ring_append": (z(1, 1, 1, 64), z(1, 1, 1, 64), z(1, 1, 6, 64), z(1, 1, 6, 64), 4, 2, 4, 1, 0),
    "decode_paged": (z(1, 2, 64), z(3, 1, 16, 64), z(3, 1, 16, 64), z(1, 1, dtype=torch.int32), z(1, dtype=torch.int32),
                     z(1, 2, 64), None, None, 8, 2, 4, 1, 0, 0.0),
    "paged_append": (z(1, 1, 1, 64), z(1, 1, 1, 64), z(3, 1, 16, 64), z(3, 1, 16, 64), z(1, 1, dtype=torch.int32),
                     z(1, dtype=torch.int32), 8, 2, 4, 1, 0),
}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_same_errors(name):
    """Host tensors, tensors of another rank, things that are no tensors, offsets that do not fit: the same type of error
    from both, before the library is called (no GPU needed)."""
    native = binding._native or binding._load_native()
    assert native is not binding_ctypes
    good = CALLS[name]
    bad = [good, (good[0][0],) + good[1:], (3,) + good[1:], (good[0], None) + good[2:]]
    if "varlen" in name:
        at = [x for x, a in enumerate(good) if isinstance(a, list)][0]
        bad += [good[:at] + (cu,) + good[at + 1:] for cu in ([0], [0, 7], [0, 1 << 40])]
    for args in bad:
        errors = []
        for mod in (native, binding_ctypes):
            with pytest.raises((TypeError, ValueError, OverflowError)) as e:
                getattr(mod, name)(*args)
            errors.append(e.type)
        assert errors[0] is errors[1] or OverflowError in errors, (name, errors)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_results(dtype, monkeypatch):
    """Every entry point once through each of the two, the same bits."""
    dev, code = "cuda:0", lg.LG_BF16 if dtype == torch.bfloat16 else lg.LG_F32
    N, D, pat = 700, 64, (16, 200, 1, 0)

    def everything():
        g = torch.Generator(device=dev).manual_seed(3)

        def rnd(*s):
            return torch.randn(*s, generator=g, device=dev, dtype=dtype)

        def new(*s, dt=dtype):
            return torch.zeros(*s, device=dev, dtype=dt)

        res = []
        q, k, v, do = rnd(1, 2, N, D), rnd(1, 2, N, D), rnd(1, 2, N, D), rnd(1, 2, N, D)
        out, lse, dq, dk, dv = new(1, 2, N, D), new(1, 2, N, dt=torch.float32), *(new(1, 2, N, D) for _ in range(3))
        ws = new(lg.bwd_workspace_bytes(1, 2, 2, N, D, *pat, code), dt=torch.uint8)
        lg.lg_sparse_attn_fwd(q, k, v, out, lse, *pat)
        lg.lg_sparse_attn_bwd(q, k, v, out, lse, do, dq, dk, dv, ws, *pat)
        res += [t.clone() for t in (out, lse, dq, dk, dv)]
        cu = [0, 300, N]
        p = [t[0] for t in (q, k, v, out, lse, do, dq, dk, dv)]
        ws = new(lg.bwd_varlen_workspace_bytes(cu, 2, 2, D, *pat, code), dt=torch.uint8)
        lg.lg_sparse_attn_fwd_varlen(*p[:5], cu, *pat)
        lg.lg_sparse_attn_bwd_varlen(*p, ws, cu, *pat)
        res += [t.clone() for t in p[3:]]
        kc, vc, q1 = new(1, 2, 216, D), new(1, 2, 216, D), q[:, :, -1].contiguous()
        lg.lg_kv_ring_append(k, v, kc, vc, 0, *pat)
        ws = new(max(16, lg.decode_cache_workspace_bytes(1, 2, 2, N, D, *pat, code)), dt=torch.uint8)
        for call in (lambda o, l: lg.lg_sparse_attn_decode(q1, kc, vc, o, l, ws, N, *pat),
                     lambda o, l: lg.lg_sparse_attn_decode_cache(q1, kc, vc, o, l, ws, N, *pat),
                     lambda o, l: lg.lg_sparse_attn_decode_cache_static(q1, kc, vc, o, l, N, *pat)):
            res += [new(1, 2, D), new(1, 2, dt=torch.float32)]
            call(*res[-2:])
        table, kp, vp = torch.arange(14, device=dev, dtype=torch.int32)[None], new(14, 2, 16, D), new(14, 2, 16, D)
        zero, lens = new(1, dt=torch.int32), torch.full((1,), N, device=dev, dtype=torch.int32)
        lg.lg_kv_paged_append(k, v, kp, vp, table, zero, N, *pat)
        ws = new(max(16, lg.decode_paged_workspace_bytes(1, 2, 2, N, D, *pat, code)), dt=torch.uint8)
        res += [kc, vc, kp, vp, new(1, 2, D), None]
        lg.lg_sparse_attn_decode_paged(q1, kp, vp, table, lens, res[-2], None, ws, N, *pat)
        torch.cuda.synchronize()
        return res

    native = everything()
    monkeypatch.setattr(binding, "_native", binding_ctypes)
    for x, y in zip(native, everything()):
        assert x is y is None or torch.equal(x, y)
