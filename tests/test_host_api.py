"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every symbol the
header declares, validates arguments before touching the device, and its size accounting and
feature permutation are right."""
import ctypes as C
import os
import re

import numpy as np
import pytest
import torch

import paper_2412_14590_amd as mx
from paper_2412_14590_amd import binding
from oracle import ref

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    src = open(os.path.join(ROOT, "include", "mixllm.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(mixllm_[a-z0-9_]+)\s*\(", src)))


def test_library_loads_and_exports_every_declared_symbol():
    L = mx.lib()
    names = declared_functions()
    assert len(names) >= 10
    for n in names:
        assert hasattr(L, n), n
    assert mx.abi_version() >= 2


def test_query_sizes_matches_the_layout_arithmetic_and_paper_footprints():
    K, N, n8 = 4096, 4096, 410
    s = mx.query_sizes(3, K, N, n8)
    n4, n8p, n4p, ngp = N - n8, 416, 3696, 32
    assert n4p >= n4 and n8p >= n8
    assert s["w8_bytes"] == n8p * K and s["w4_bytes"] == n4p * K // 2
    assert s["scales4_bytes"] == n4p * ngp * 2 and s["zeros4_bytes"] == n4p * ngp // 2
    assert s["scales8_bytes"] == n8p * 2 and s["perm_bytes"] == 4 * N
    assert s["xq_bytes"] == 3 * K and s["xscale_bytes"] == 6 and s["y_bytes"] == 3 * N * 2
    assert s["workspace_bytes"] == 3 * K + 256      # xq, then xscale, each rounded up to 256 bytes
    # per stored weight the 4-bit part costs 0.5 + 2.5/G bytes and the group-wise 8-bit part
    # 1 + 2/G bytes (Sec. 3.5, memory traffic)
    assert (s["w4_bytes"] + s["scales4_bytes"] + s["zeros4_bytes"]) / (n4p * K) == 0.5 + 2.5 / 128
    sp = mx.query_sizes(3, K, N, n8, act_group=128, w8_group=128)
    assert (sp["w8_bytes"] + sp["scales8_bytes"]) / (n8p * K) == 1 + 2 / 128
    assert sp["xscale_bytes"] == 3 * (K // 128) * 2
    # metadata rows are padded to a multiple of 8 groups
    s2 = mx.query_sizes(0, 384, 32, 0)
    assert s2["scales4_bytes"] == 32 * 8 * 2 and s2["zeros4_bytes"] == 32 * 4


@pytest.mark.parametrize("kw,code", [
    (dict(M=1, K=4000, N=64, n8=0), -2),            # K not a multiple of the group
    (dict(M=1, K=256, N=64, n8=65), -1),            # n8 > N
    (dict(M=-1, K=256, N=64, n8=0), -1),
    (dict(M=1, K=256, N=64, n8=0, act_group=64), -2),
    (dict(M=1, K=256, N=64, n8=0, w8_group=256 * 2), -2),
    (dict(M=1, K=131072 + 128, N=64, n8=0), -2),    # beyond the K an int32 sum over all of K is safe for
])
def test_bad_descriptors_are_rejected(kw, code):
    d = binding._desc(**kw)
    s = binding._Sizes()
    assert mx.lib().mixllm_query_sizes(C.byref(d), C.byref(s)) == code


def test_null_and_misaligned_pointers_are_rejected_before_any_launch():
    L = mx.lib()
    d = binding._desc(4, 256, 64, 8)
    # null everything
    assert L.mixllm_mixed_linear(C.byref(d), None, None, None, None, None, None, None, None, None, None, 0, None) == -1
    assert L.mixllm_quantize_activations(C.byref(d), None, None, None, None) == -1
    assert L.mixllm_debug_group_partials(C.byref(d), None, None, None, None, None, None, 0, None) == -1
    assert L.mixllm_debug_channel_sums(C.byref(d), None, None, None, None, None, None, None, None, None, 0, None) == -1
    # misaligned (fake, never dereferenced: validation fails first)
    fake = 0x1000
    # the list of 8-bit channels is a device pointer: null with n8 > 0, or not 4-byte aligned
    assert L.mixllm_quantize_weights(C.byref(d), fake, None, fake, fake, fake, fake, fake, fake, None) == -1
    assert L.mixllm_quantize_weights(C.byref(d), fake, fake + 2, fake, fake, fake, fake, fake, fake, None) == -1
    # the integer sums over the groups come from the generic and the tiled kernel only: refused, nothing launched
    assert L.mixllm_debug_channel_sums(C.byref(d), fake, fake, fake, fake, fake, fake, fake, fake, fake, 2, None) == -2
    # the 128 x 128 block shape is not built for activation scales per (token, group)
    dg = binding._desc(300, 256, 64, 8, act_group=128)
    assert L.mixllm_mixed_linear_path(C.byref(dg), fake, fake, fake, fake, fake, fake, fake, fake, fake, None, 0, 10, None) == -2
    assert L.mixllm_quantize_activations(C.byref(d), fake + 2, fake, fake, None) == -1
    # bad path value
    assert L.mixllm_mixed_linear_path(C.byref(d), fake, fake, fake, fake, fake, fake, fake, fake, fake, None, 0, 11, None) == -1
    # the decode path refuses M > 16; M = 0 is a no-op that succeeds without a device
    d0 = binding._desc(0, 256, 64, 8)
    assert L.mixllm_mixed_linear(C.byref(d0), None, None, None, None, None, None, None, None, None, None, 0, None) == 0
    assert L.mixllm_status_string(-2).decode().startswith("unsupported")


def test_precision_search_calls_validate_on_the_host():
    L = mx.lib()
    d = binding._desc(0, 256, 8, 0)
    buf = (C.c_uint8 * 8192)()
    addr = (C.addressof(buf) + 15) & ~15                       # 16-byte aligned host address: never dereferenced
    vp = C.c_void_p
    # salience: null / misaligned pointers, K not a multiple of the group
    assert L.mixllm_channel_salience(C.byref(d), None, vp(addr), C.c_float(1), 0, vp(addr), None) == -1
    assert L.mixllm_channel_salience(C.byref(d), vp(addr + 2), vp(addr), C.c_float(1), 0, vp(addr), None) == -1
    bad = binding._desc(0, 200, 8, 0)
    assert L.mixllm_channel_salience(C.byref(bad), vp(addr), vp(addr), C.c_float(1), 0, vp(addr), None) == -2
    empty = binding._desc(0, 256, 0, 0)
    assert L.mixllm_channel_salience(C.byref(empty), None, None, C.c_float(1), 0, None, None) == 0
    # selection: layer list, T, workspace
    off = (C.c_int64 * 3)(0, 5, 9)
    need = L.mixllm_select_salient_workspace(2)
    assert need > 0 and L.mixllm_select_salient_workspace(0) == 0
    args = lambda o, nl, T, ws, wb: L.mixllm_select_salient(vp(addr), C.cast(o, vp), nl, C.c_int64(T), vp(addr), vp(addr),
                                                            ws, C.c_size_t(wb), None)
    assert args(off, 0, 1, vp(addr), need) == -1                 # no layers
    assert args(off, 2, 10, vp(addr), need) == -1                # T beyond the number of channels
    assert args(off, 2, -1, vp(addr), need) == -1
    assert args((C.c_int64 * 3)(0, 5, 4), 2, 1, vp(addr), need) == -1      # offsets not ascending
    assert args((C.c_int64 * 3)(1, 5, 9), 2, 1, vp(addr), need) == -1      # offsets do not start at 0
    assert args(off, 2, 3, None, need) == -1
    assert args(off, 2, 3, vp(addr), need - 1) == -3             # MIXLLM_EWORKSPACE


def test_feature_perm_matches_oracle_and_rejects_bad_lists():
    rng = np.random.default_rng(0)
    for N, n8 in ((8, 3), (100, 0), (100, 100), (4096, 410)):
        sal = rng.choice(N, n8, replace=False).astype(np.int32)
        got = mx.build_feature_perm(N, sal)
        assert np.array_equal(got, ref.feature_perm(N, sal))
        assert np.array_equal(np.sort(got), np.arange(N))
        assert np.all(np.diff(got[:n8]) > 0) and np.all(np.diff(got[n8:]) > 0)
    with pytest.raises(mx.MixllmError):
        mx.build_feature_perm(4, [1, 1])
    with pytest.raises(mx.MixllmError):
        mx.build_feature_perm(4, [7])


def test_product_path_does_not_import_the_oracle():
    # the library binding and the input generator must stand alone
    for f in ("binding.py", "synth.py", "__init__.py", "build.py"):
        src = open(os.path.join(ROOT, "paper_2412_14590_amd", f)).read()
        assert "oracle" not in src.replace("oracle-side", ""), f


def test_build_scan_flags_a_register_used_between_its_hand_issued_load_and_the_wait():
    from paper_2412_14590_amd import build
    ok = """
	;;#ASMSTART
	global_load_dwordx2 v[104:105], v119, s[98:99]
	;;#ASMEND
	v_add_u32_e32 v1, v2, v3
	;;#ASMSTART
	s_waitcnt vmcnt(6)
	;;#ASMEND
	v_lshrrev_b32_e32 v128, 16, v104
"""
    build.check_hand_issued_loads(ok, "ok")
    bad = ok.replace("v_add_u32_e32 v1, v2, v3", "v_lshrrev_b32_e32 v128, 16, v104")
    with pytest.raises(RuntimeError):
        build.check_hand_issued_loads(bad, "bad")
    # a branch ends the judged region (the two arms of a conditional load are not one sequence),
    # and a direct-to-LDS load has no destination register
    branchy = ok.replace("v_add_u32_e32 v1, v2, v3", "s_branch .LBB1_2\n.LBB1_1:\n\tv_mov_b32_e32 v104, 0")
    build.check_hand_issued_loads(branchy, "branchy")
    lds = ok.replace("global_load_dwordx2 v[104:105], v119, s[98:99]", "global_load_lds_dwordx4 v104, s[98:99]")
    build.check_hand_issued_loads(lds.replace("v_add_u32_e32 v1, v2, v3", "v_mov_b32_e32 v104, 0"), "lds")


def layer_arguments(K=256, N=40, n8=4):
    """A packed layer without data as the native calls take it: with no tokens nothing of it is read, and no GPU is needed."""
    return (K, N, n8, K, *[torch.empty(0, dtype=torch.uint8) for _ in range(6)])


def test_native_linear_takes_matrices_only():
    call = lambda xq: binding._calls().mixed_linear(xq, torch.empty((xq.shape[0], 1), dtype=torch.float16), *layer_arguments(),
                                                    mx.PATH_AUTO, None, None, 0)
    y = call(torch.empty((0, 256), dtype=torch.int8))
    assert y.shape == (0, 40) and y.dtype == torch.float16
    for shape in ((0, 256, 1), (0, 256, 3), (0, 256, 0)):
        with pytest.raises(AssertionError):
            call(torch.empty(shape, dtype=torch.int8))


def test_native_quantizer_allocates_only_where_no_buffers_are_given():
    x, q, s = (torch.empty((0, 256), dtype=t) for t in (torch.float16, torch.int8, torch.float16))
    call = lambda out: binding._calls().quantize_activations(x, None, out, 0)
    got = call(None)
    assert got[0].dtype == torch.int8 and got[0].shape == (0, 256) and got[1].dtype == torch.float16 and got[1].shape == (0, 1)
    got = call([q, s])
    assert got[0] is q and got[1] is s
    assert call((None, s)) == (None, s) and call((q, None)) == (q, None)      # no tokens: nothing is written, nothing was allocated
    for bad in ((q,), (q, s, s)):
        with pytest.raises(ValueError):
            call(bad)


def test_native_calls_take_whole_numbers_of_any_type():
    # descriptors were always filled through int(): numpy integers, and floats that are whole
    x, xs = torch.empty((0, 256), dtype=torch.float16), torch.empty((0, 1), dtype=torch.float16)
    K, N, n8, w8_group, *buffers = layer_arguments()
    for t in (int, float, np.int64, np.float32):
        y = binding._calls().linear_fp16(x, t(K), t(N), t(n8), t(w8_group), *buffers, t(128), None, None, 0)
        assert y.shape == (0, N)
        y = binding._calls().mixed_linear(x.to(torch.int8), xs, t(K), t(N), t(n8), t(w8_group), *buffers, mx.PATH_AUTO, None, None, 0)
        assert y.shape == (0, N)
        binding._calls().quantize_activations(x, t(128), (x.to(torch.int8), xs), 0)
    with pytest.raises(TypeError):
        binding._calls().linear_fp16(x, *layer_arguments(), [128], None, None, 0)
    with pytest.raises(TypeError):                     # ... nor a size to allocate by
        binding._calls().quantize_activations(x, 128.0, None, 0)
    with pytest.raises(TypeError):                     # the kernel selection is no descriptor field: an integer as before
        binding._calls().mixed_linear(x.to(torch.int8), xs, *layer_arguments(), 0.0, None, None, 0)


class Tagged(torch.Tensor):
    """A tensor subclass: its methods' results are of its type."""


def test_native_calls_allocate_results_through_the_activations_own_new_empty():
    # ... where new_empty is overridden (a subclass, a mode); plain tensors take the short way
    from torch.overrides import TorchFunctionMode
    xs = torch.empty((0, 1), dtype=torch.float16)

    def results(x):
        c = binding._calls()
        yield c.linear_fp16(x, *layer_arguments(), 256, None, None, 0)
        yield c.mixed_linear(x.to(torch.int8), xs, *layer_arguments(), mx.PATH_AUTO, None, None, 0)
        yield from c.quantize_activations(x, None, None, 0)

    x = torch.empty((0, 256), dtype=torch.float16)
    want = [((0, 40), torch.float16), ((0, 40), torch.float16), ((0, 256), torch.int8), ((0, 1), torch.float16)]
    for kind in (torch.Tensor, Tagged):
        got = list(results(x.as_subclass(kind)))
        assert [type(t) for t in got] == [kind] * 4 and [(tuple(t.shape), t.dtype) for t in got] == want
    assert type(next(results(torch.nn.Parameter(x)))) is torch.Tensor

    class Seen(TorchFunctionMode):
        count = 0

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.count += func is torch.Tensor.new_empty
            return func(*args, **(kwargs or {}))

    with Seen() as mode:
        assert len(list(results(x))) == 4
    assert mode.count >= 4


def test_native_calls_refuse_buffers_that_do_not_hold_what_is_read_or_written():
    # device buffers: their sizes and types are looked at before their address, so host tensors will do
    c, h, i8 = binding._calls(), torch.float16, torch.int8
    K, N, M = 256, 40, 3
    new = lambda *size, dtype=h: torch.empty(size, dtype=dtype)

    def refused(match, f):
        with pytest.raises(AssertionError, match=match):
            f()

    fp16 = lambda out: c.linear_fp16(new(M, K), *layer_arguments(), K, out, None, 0)
    linear = lambda xq, xs, out: c.mixed_linear(xq, xs, *layer_arguments(), mx.PATH_AUTO, out, None, 0)
    quant = lambda q, s, g=None: c.quantize_activations(new(M, K), g, (q, s), 0)
    for out in (new(M, N - 1), new(M * N - 1), new(M, N, dtype=torch.float32), new(M, N, dtype=torch.bfloat16), new(2 * M, N, dtype=torch.int8)):
        refused("^y", lambda: fp16(out))
        refused("^y", lambda: linear(new(M, K, dtype=i8), new(M, 1), out))
    for xq in (new(M, K), new(M, K, dtype=torch.float8_e4m3fn), new(M, K, dtype=torch.int32)):
        refused("^xq", lambda: linear(xq, new(M, 1), new(M, N)))
    refused("^xs", lambda: linear(new(M, K, dtype=i8), new(M, 1, dtype=torch.float32), new(M, N)))
    refused("^xs", lambda: linear(new(M, K, dtype=i8), new(M, 1, 2), new(M, N)))
    wide = 128 * 130                                   # 129 columns of scales divide to groups of 128 and are one column short
    refused("^xs", lambda: c.mixed_linear(new(M, wide, dtype=i8), new(M, 129), *layer_arguments(K=wide), mx.PATH_AUTO, new(M, N), None, 0))
    for q, s, g in ((new(M, K - 1, dtype=i8), new(M, 1), None), (new(M, K), new(M, 1), None), (new(M, K, dtype=i8), new(M - 1, 1), None),
                    (new(M, K, dtype=i8), new(M, 1), 128), (new(M, K, dtype=i8), new(M, 1, dtype=torch.float32), None)):
        refused("^x[qs]", lambda: quant(q, s, g))
    # room to spare, another shape and the raw bits as integers were always taken: these get as far as the address
    for out in (new(M, N), new(M * N + 7), new(M, N, dtype=torch.int16)):
        refused("device", lambda: fp16(out))
        refused("device", lambda: linear(new(M, K, dtype=torch.uint8), new(M, 1, dtype=torch.int16), out))
    refused("device", lambda: quant(new(M, K, dtype=torch.uint8), new(4 * M), None))


def test_static_entry_and_debug_hooks_refuse_activations_of_another_width():
    L = binding.PackedLayer(*layer_arguments())
    for K in (128, 384):
        x, xs = torch.empty((3, K), dtype=torch.float16), torch.empty((3, 1), dtype=torch.float16)
        for call in (lambda: mx.linear_fp16_static(x, L, torch.empty((3, 40), dtype=torch.float16)),
                     lambda: mx.debug_group_partials(x.to(torch.int8), L), lambda: mx.debug_channel_sums(x.to(torch.int8), xs, L)):
            with pytest.raises(AssertionError) as e:
                call()
            assert "device" not in str(e.value)        # refused for its width, before any address is taken


def test_a_variant_build_brings_the_native_calls_where_there_are_none(tmp_path, monkeypatch):
    # a library with other launch constants is loaded by the same package, which needs _calls.so beside it
    from paper_2412_14590_amd import build
    calls, made = tmp_path / "_calls.so", []
    monkeypatch.setenv("MIXLLM_EXTRA_FLAGS", "-DX=1")
    for name, value in (("SOURCES", []), ("NO_SPILL", {}), ("LIB", str(tmp_path / "lib.so")), ("CALLS", str(calls)),
                        ("_hipcc", lambda: "true"), ("build_calls", lambda: (made.append(1), calls.write_text("")))):
        monkeypatch.setattr(build, name, value)
    build.build()
    build.build()
    assert made == [1]
