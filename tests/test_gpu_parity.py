"""GPU parity: every entry point of the C-ABI library against the CPU oracle on the same
seeded inputs.  Integer results (codes, zero points, permutations, per-group partial sums and
their sums over the groups) must be bit-exact; fp16 outputs must agree within TOL
(row-L2-normalised, the workload's gate) and, element by element, within half an fp16 unit in the
last place plus the fp32 accumulation bound (util.elementwise_bound)."""
import numpy as np
import pytest
import torch

import paper_2412_14590_amd as mx
from oracle import ref
from paper_2412_14590_amd import synth

from util import (G, TOL, check_against_oracle, dev, full_size_layer, make_case, pack_from_oracle, row_rel_err,
                  stratified_rows, weight_scales_in_channel_order)

pytestmark = pytest.mark.gpu

PATHS = {"generic": mx.PATH_GENERIC, "decode": mx.PATH_DECODE, "prefill": mx.PATH_PREFILL,
         "decode_stream": mx.PATH_DECODE_STREAM, "decode_resident": mx.PATH_DECODE_RESIDENT,
         "decode_split": mx.PATH_DECODE_SPLIT, "mid": mx.PATH_MID,
         "prefill32": mx.PATH_PREFILL_32, "prefill64": mx.PATH_PREFILL_64, "prefill128": mx.PATH_PREFILL_128}
TILED = ["prefill", "prefill32", "prefill64", "prefill128"]   # the tiled kernel: block shape by grid size, or forced
DECODE_VARIANTS = ["decode_stream", "decode_resident", "decode_split"]


def say(*a):
    print(*a, flush=True)


def split_variant_covers(M, K):
    """The evenly split decode variant stages the int8 activation matrix in LDS: whole up to 128 Ki values,
    beyond that (built for 5..16 tokens) in windows over K."""
    return M <= 16 and (M * K <= 131072 or M >= 5)


def skip_unless_covered(path, M, K):
    if path == "decode_split" and not split_variant_covers(M, K):
        with pytest.raises(mx.MixllmError) as e:
            mx.mixed_linear(torch.zeros((M, K), dtype=torch.int8, device="cuda"),
                            torch.ones((M, 1), dtype=torch.float16, device="cuda"),
                            pack_from_oracle(make_case(0, K, 16, 0, seed=1)[2]), mx.PATH_DECODE_SPLIT)
        assert e.value.status == -2     # MIXLLM_EUNSUPPORTED, not a silent fallback
        pytest.skip("shape outside the split variant")


# ------------------------------------------------------------- activation quantizer --

@pytest.mark.parametrize("M,K", [(1, 4096), (16, 4096), (37, 512), (5, 128), (130, 14336)])
@pytest.mark.parametrize("grouped", [False, True])
def test_activation_quantizer_bit_exact(M, K, grouped):
    say("act", M, K, grouped)
    x = synth.make_x(M, K, seed=21)
    x[0, :7] = np.float16([0.0, -0.0, 6e-8, 65504, -65504, 1e-4, 0.5])
    if M > 2:
        x[2] = 0                                  # a degenerate (all zero) token
    ag = 128 if grouped else None
    xq_ref, xs_ref = ref.quantize_act(x, ag)
    xq, xs = mx.quantize_activations(dev(x), ag)
    assert np.array_equal(xs.cpu().numpy().view(np.uint16), xs_ref.view(np.uint16))
    assert np.array_equal(xq.cpu().numpy(), xq_ref)


def test_quantizer_division_shortcut_is_exact_for_every_fp16_pair():
    # the kernels round v / s through a reciprocal and one correction step; on the GPU, against the
    # IEEE division, for all 63488 finite fp16 values times all 31743 positive finite fp16 scales
    bad = torch.zeros(1, dtype=torch.int64, device="cuda")
    rc = mx.lib().mixllm_debug_check_fast_division(bad.data_ptr(), None)
    torch.cuda.synchronize()
    assert rc == 0 and int(bad.item()) == 0


def test_activation_quantizer_empty_batch():
    x = torch.empty((0, 256), dtype=torch.float16, device="cuda")
    xq, xs = mx.quantize_activations(x)
    assert xq.shape == (0, 256)


# ------------------------------------------------------ weight quantizer, pack, unpack --

@pytest.mark.parametrize("K,N,n8", [(256, 100, 7), (384, 33, 0), (128, 16, 16), (4096, 530, 53), (1024, 48, 17)])
@pytest.mark.parametrize("w8_group", [None, 128])
def test_weight_quantizer_codes_bit_exact(K, N, n8, w8_group):
    say("wq", K, N, n8, w8_group)
    W, sal, L, *_ = make_case(0, K, N, n8, seed=22, w8_group=w8_group)
    W = W.copy()
    W[N // 2, :128] = 0                                       # a degenerate group
    L = ref.quantize_weights(W, sal, G, w8_group)
    P = mx.quantize_weights(dev(W), sal, w8_group)
    u = mx.unpack_weights(P)
    assert np.array_equal(u["perm"].cpu().numpy(), L.perm)
    if L.n8:
        assert np.array_equal(u["s8"].cpu().numpy().view(np.uint16), L.s8.view(np.uint16))
        assert np.array_equal(u["q8"].cpu().numpy(), L.q8)
    if L.n4:
        assert np.array_equal(u["s4"].cpu().numpy().view(np.uint16), L.s4.view(np.uint16))
        assert np.array_equal(u["z4"].cpu().numpy(), L.z4)
        assert np.array_equal(u["q4"].cpu().numpy(), L.q4)


@pytest.mark.parametrize("K,N,n8", [(256, 100, 7), (384, 33, 33), (640, 35, 0)])
@pytest.mark.parametrize("w8_group", [None, 128])
def test_pack_unpack_round_trip_and_padding_is_zero(K, N, n8, w8_group):
    _, _, L, *_ = make_case(0, K, N, n8, seed=23, w8_group=w8_group)
    P = pack_from_oracle(L)
    u = mx.unpack_weights(P)
    for k in ("q8", "q4", "z4", "perm"):
        assert np.array_equal(u[k].cpu().numpy(), getattr(L, k)), k
    for k in ("s8", "s4"):
        assert np.array_equal(u[k].cpu().numpy().view(np.uint16), getattr(L, k).view(np.uint16)), k
    # packing the same codes and quantizing on the GPU give byte-identical buffers
    # (so padding rows / groups are deterministic zeros)
    W = make_case(0, K, N, n8, seed=23, w8_group=w8_group)[0]
    Q = mx.quantize_weights(dev(W), L.perm[:n8], w8_group)
    for k in ("w8", "w4", "s8", "s4", "z4", "perm"):
        assert torch.equal(getattr(P, k), getattr(Q, k)), k


def test_quantizers_on_random_shapes_and_value_ranges():
    """40 seeded random cases for the two quantizers: ragged N, K of 1..40 groups, any 8-bit share, both
    granularities, value scales from 1e-4 to 1e3 (fp16 subnormal scales up to near overflow): codes,
    zero points, scales and the channel order bit-exact against the oracle."""
    rng = np.random.default_rng(20242)
    for it in range(40):
        K = 128 * int(rng.choice([1, 2, 3, 5, 8, 16, 28, 40]))
        N = int(rng.choice([1, 3, 16, 17, 47, 100, 257, 1000]))
        n8 = int(rng.choice([0, N, N // 10, int(rng.integers(0, N + 1))]))
        M = int(rng.choice([1, 2, 7, 16, 33, 130]))
        wg = 128 if rng.integers(0, 2) else None
        ag = 128 if rng.integers(0, 2) else None
        scale = float(10.0 ** rng.uniform(-4, 3))
        W, sal, _, x, _, _ = make_case(M, K, N, n8, seed=7000 + it, w8_group=wg, act_group=ag)
        W = (W.astype(np.float32) * (scale / 0.02)).clip(-60000, 60000).astype(np.float16)
        x = (x.astype(np.float32) * scale).clip(-60000, 60000).astype(np.float16)
        L = ref.quantize_weights(W, sal, G, wg)
        u = mx.unpack_weights(mx.quantize_weights(dev(W), sal, wg))
        tag = (K, N, n8, wg, scale)
        assert np.array_equal(u["perm"].cpu().numpy(), L.perm), tag
        if L.n8:
            assert np.array_equal(u["s8"].cpu().numpy().view(np.uint16), L.s8.view(np.uint16)), tag
            assert np.array_equal(u["q8"].cpu().numpy(), L.q8), tag
        if L.n4:
            assert np.array_equal(u["s4"].cpu().numpy().view(np.uint16), L.s4.view(np.uint16)), tag
            assert np.array_equal(u["z4"].cpu().numpy(), L.z4), tag
            assert np.array_equal(u["q4"].cpu().numpy(), L.q4), tag
        xq_ref, xs_ref = ref.quantize_act(x, ag)
        xq, xs = mx.quantize_activations(dev(x), ag)
        assert np.array_equal(xs.cpu().numpy().view(np.uint16), xs_ref.view(np.uint16)), (M, K, ag, scale)
        assert np.array_equal(xq.cpu().numpy(), xq_ref), (M, K, ag, scale)


@pytest.mark.parametrize("N,n8", [(1, 0), (1, 1), (16, 5), (1000, 0), (1000, 1000), (1025, 100), (4096, 410), (57344, 5734),
                                  (3000, 2999)])
def test_feature_perm_is_built_on_the_device_from_a_device_list(N, n8):
    # mixllm_quantize_weights takes the list of 8-bit channels as a device pointer, in any order
    rng = np.random.default_rng(N + n8)
    sal = rng.permutation(N)[:n8].astype(np.int32)
    W = synth.make_w(N, 128, seed=5, n_outlier_rows=1)
    PL = mx.quantize_weights(dev(W), dev(sal))
    assert np.array_equal(PL.perm.cpu().numpy(), ref.feature_perm(N, sal))


@pytest.mark.parametrize("K,N,n8", [(128, 4097, 4096), (128, 131072, 1000), (128, 131073, 131), (1152, 15, 1), (2048, 65, 33)])
@pytest.mark.parametrize("w8_group", [None, 128])
def test_conversion_at_the_edges_of_tiles_and_units(K, N, n8, w8_group):
    # row orders on both sides of the bitmap's limit and of a block's share; rows and groups that do not
    # fill a tile of 16 or a unit of 8 groups; the 4-bit codes exported to an address that is not aligned
    rng = np.random.default_rng(N)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float16)
    sal = rng.permutation(N)[:n8].astype(np.int32)
    L = ref.quantize_weights(W, sal, G, w8_group)
    P = mx.quantize_weights(dev(W), dev(sal), w8_group)
    u = mx.unpack_weights(P)
    for k in ("q8", "q4", "z4", "perm"):
        assert np.array_equal(u[k].cpu().numpy(), getattr(L, k)), k
    for k in ("s8", "s4"):
        assert np.array_equal(u[k].cpu().numpy().view(np.uint16), getattr(L, k).view(np.uint16)), k
    import ctypes as C
    q4 = torch.full(((N - n8) * K + 32,), 99, dtype=torch.uint8, device="cuda")
    d = P.desc()
    rc = mx.lib().mixllm_unpack_weights(C.byref(d), *[t.data_ptr() for t in (P.w8, P.w4, P.s8, P.s4, P.z4, P.perm, u["q8"], u["s8"])],
                                        q4.data_ptr() + 3, *[u[k].data_ptr() for k in ("s4", "z4", "perm")], None)
    assert rc == 0
    torch.cuda.synchronize()
    assert torch.equal(q4[3:-29].view(N - n8, K), u["q4"]) and bool((q4[:3] == 99).all()) and bool((q4[-29:] == 99).all())


@pytest.mark.parametrize("K,N,n8", [
    (256, 9600, 50), (2048, 9600, 33), (1152, 9599, 33),         # whole tiles on wide layers of short rows, and one channel short of that
    (384, 4200, 4081), (512, 4200, 4080),                        # 256 tiles of 8-bit rows and one fewer (units of 8 and of 2 groups)
    (2176, 4800, 17), (2176, 4799, 17), (1152, 2400, 31), (1152, 2399, 16), (640, 1200, 15), (640, 1199, 15),   # 8, 4, 4, 2, 2, 1 rows a block
    (512, 1100, 1090), (128, 400, 390), (16, 16, 16),            # rows by the number of blocks (K is times 128 in the last)
    (33024, 20, 3), (32896, 20, 20),                             # more chunks of a row than are requested together
])
@pytest.mark.parametrize("w8_group", [None, 128])
def test_weight_quantizer_in_every_block_shape(K, N, n8, w8_group):
    # both forms of the 8-bit part, every height of its blocks and both units of the 4-bit part, with rows,
    # groups and chunks that do not fill them; the packed buffers (padding included) are those of packing the oracle's codes
    K = 128 * K if K < 128 else K
    rng = np.random.default_rng(K + N)
    W = (rng.standard_normal((N, K), dtype=np.float32) * 0.02).astype(np.float16)
    W[rng.integers(0, N), K - 1] = 3.0                           # a maximum in the last value of a row
    sal = rng.permutation(N)[:n8].astype(np.int32)
    want = pack_from_oracle(ref.quantize_weights(W, sal, G, w8_group))
    got = mx.quantize_weights(dev(W), dev(sal), w8_group)
    for k in ("w8", "w4", "s8", "s4", "z4", "perm"):
        assert torch.equal(getattr(want, k), getattr(got, k)), k


def test_conversion_of_few_long_rows_takes_as_long_as_that_of_many_short_ones():
    # the same number of weights and the same 8-bit share, 1024 rows of 28672 and 7168 of 4096, from a graph (a block per
    # tile of 8-bit rows walked its 16 long rows in sequence: 56 us against 21; in blocks of fewer rows 22 against 20)
    def us(N, K):
        W = torch.randn((N, K), device="cuda", dtype=torch.float16) * 0.02
        sal = torch.arange(0, N, 10, dtype=torch.int32, device="cuda")
        mx.quantize_weights(W, sal)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(10):
                mx.quantize_weights(W, sal)
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 100)
        return sorted(times)[4]
    narrow, wide = us(1024, 28672), us(7168, 4096)
    say(f"weight conversion, 29.4 M weights: 1024 rows {narrow:.1f} us, 7168 rows {wide:.1f} us")
    assert narrow < 1.6 * wide


@pytest.mark.parametrize("K", [4096, 4224, 8192, 8320, 16384, 16512, 32768, 32896, 131072])
@pytest.mark.parametrize("act_group", [None, 128])
@pytest.mark.parametrize("M", [1, 3])
def test_activation_quantizer_on_both_sides_of_every_block_width(M, K, act_group):
    # rows of up to 4096, 8192, 16384 and 32768 values are held in registers by 256, 512, 1024 and 1024 threads,
    # longer ones read twice; the largest value of each row in its first, a middle and its last place
    x = synth.make_x(M, K, seed=K + M)
    for m, col in zip(range(M), (K - 1, 0, K // 2 - 1)):
        x[m, col] = -1.5 * np.abs(x[m]).max()
    xq_ref, xs_ref = ref.quantize_act(x, act_group)
    xq, xs = mx.quantize_activations(dev(x), act_group)
    assert np.array_equal(xs.cpu().numpy().view(np.uint16), xs_ref.view(np.uint16))
    assert np.array_equal(xq.cpu().numpy(), xq_ref)


@pytest.mark.parametrize("K", [512, 4096, 8192, 14336, 28672, 33024])
@pytest.mark.parametrize("act_group", [None, 128])
def test_a_nan_does_not_enter_the_scale_of_its_row(K, act_group):
    # (unsupported input, but one bad value leaves its row's scale and the other codes alone, and every way through
    # the library agrees: the stand-alone quantizer in all its block widths and the quantizers inside the decode kernels)
    rng = np.random.default_rng(K)
    x = synth.make_x(4, K, seed=K)
    cols = np.array([3, K // 2 + 1, K - 1])
    clean = x.copy()
    clean[1:3, cols] = 0.0
    x[1, cols] = np.nan
    x.view(np.uint16)[2, cols] = [0xfe01, 0x7c01, 0xffff]        # negative, signalling, all bits
    x[3, rng.integers(0, K)] = clean[3].max() * 2
    clean[3] = x[3]
    xq_ref, xs_ref = ref.quantize_act(clean, act_group)
    xq_ref[1:3, cols] = -127                                     # what clamping a NaN to [-127, 127] gives
    xq, xs = mx.quantize_activations(dev(x), act_group)
    assert np.array_equal(xs.cpu().numpy().view(np.uint16), xs_ref.view(np.uint16))
    assert np.array_equal(xq.cpu().numpy(), xq_ref)
    W = synth.make_w(40, K, seed=1, n_outlier_rows=1)
    PL = mx.quantize_weights(dev(W), np.arange(4, dtype=np.int32))
    for rows in ([1], [2, 3], [0, 1, 2, 3]):
        y = mx.linear_fp16(dev(x[rows]), PL, act_group)
        two = mx.mixed_linear(dev(xq_ref[rows]), dev(xs_ref[rows]), PL)
        assert torch.isfinite(y).all() and row_rel_err(y.cpu().numpy(), two.cpu().numpy()) <= TOL


def test_a_bad_device_list_of_8bit_channels_never_writes_out_of_bounds():
    # indices out of range are ignored, duplicates count once; the order is then unspecified, but
    # every entry stays a channel number and the buffers around feature_perm are untouched
    N, K = 200, 128
    W = dev(synth.make_w(N, K, seed=6, n_outlier_rows=1))
    sal = dev(np.array([5, 5, -1, 7, 4000, 199, 7, 2 ** 30], np.int32))
    guard = torch.full((N + 64,), -77, dtype=torch.int32, device="cuda")
    L = mx.binding._alloc_layer(K, N, 8, None, W.device)
    L.perm = guard[32:32 + N]
    d = L.desc()
    import ctypes as C
    rc = mx.lib().mixllm_quantize_weights(C.byref(d), W.data_ptr(), sal.data_ptr(), L.w8.data_ptr(), L.w4.data_ptr(),
                                          L.s8.data_ptr(), L.s4.data_ptr(), L.z4.data_ptr(), L.perm.data_ptr(), None)
    torch.cuda.synchronize()
    assert rc == 0
    g = guard.cpu().numpy()
    assert (g[:32] == -77).all() and (g[32 + N:] == -77).all()
    assert ((g[32:32 + N] >= 0) & (g[32:32 + N] < N)).all()
    assert list(g[32:36]) == [5, 7, 199, 0]      # the three valid distinct channels first; the other slots of the first part stay cleared


# ------------------------------------------------------------ integer partial sums --

def check_partials(M, K, N, n8, path, seed=24):
    _, _, L, _, xq, _ = make_case(M, K, N, n8, seed)
    P_ref = ref.group_partials(xq, L)
    P = mx.debug_group_partials(dev(xq), pack_from_oracle(L), PATHS[path])
    torch.cuda.synchronize()
    assert np.array_equal(P.cpu().numpy(), P_ref)


@pytest.mark.parametrize("M,K,N,n8", [(3, 256, 7, 2), (16, 1024, 100, 9), (1, 4096, 300, 30), (9, 640, 50, 0),
                                     (5, 384, 40, 40), (2, 2048, 2070, 207), (4, 14336, 100, 12), (4, 28672, 48, 5),
                                     # more than 128 Ki activation values: the split variant walks K in windows
                                     # (14336: 16 + 12 chunk columns; 9088: 16 + 2, the last group alone in its chunk)
                                     (16, 14336, 100, 12), (9, 28672, 48, 5), (15, 9088, 70, 7),
                                     # the last window is one chunk column of which a quarter lies inside K
                                     (16, 28800, 40, 4)])
@pytest.mark.parametrize("path", ["generic", "decode"] + DECODE_VARIANTS)
def test_group_partials_bit_exact_small_m(M, K, N, n8, path):
    say("partials", path, M, K, N, n8)
    skip_unless_covered(path, M, K)
    check_partials(M, K, N, n8, path)


@pytest.mark.parametrize("M,K,N,n8", [(3, 256, 7, 2), (130, 512, 300, 30), (200, 1024, 530, 0), (33, 384, 70, 70),
                                     (257, 256, 290, 29),
                                     # grids that take the 64 x 128 and the 128 x 128 blocks (the smaller cases
                                     # above run on 32 x 128 blocks), K not a multiple of 4 groups
                                     (256, 384, 8192, 819), (384, 640, 8192, 0)])
@pytest.mark.parametrize("path", ["generic"] + TILED)
def test_group_partials_bit_exact_tiled(M, K, N, n8, path):
    # every block shape of the tiled kernel (the shape only decides which tokens share a block)
    say("partials", path, M, K, N, n8)
    check_partials(M, K, N, n8, path)


@pytest.mark.parametrize("variant", ["baseline", "paper", "w8_grouped"])
@pytest.mark.parametrize("M,K,N,n8", [(3, 256, 7, 2), (130, 512, 300, 30), (200, 1024, 530, 0), (33, 384, 70, 70),
                                     (257, 256, 290, 29), (256, 384, 8192, 819), (384, 640, 8192, 0), (300, 4096, 272, 272)])
def test_channel_sums_from_the_linears_own_kernels(M, K, N, n8, variant):
    # Sum over the groups of the int32 partials, out of the kernels the linear launches for the shape and
    # scale granularity: for 8-bit tiles with one scale per channel this is the single accumulator
    # that runs over all of K.  Bit-exact against the oracle's partials, through every block shape.
    ag, wg = {"baseline": (None, None), "paper": (128, 128), "w8_grouped": (None, 128)}[variant]
    _, _, L, _, xq, xs = make_case(M, K, N, n8, seed=33, w8_group=wg, act_group=ag)
    S_ref = ref.group_partials(xq, L).sum(axis=2, dtype=np.int64)
    assert np.abs(S_ref).max() < 2 ** 31
    PL = pack_from_oracle(L)
    for name in ["generic"] + TILED:
        try:
            S = mx.debug_channel_sums(dev(xq), dev(xs), PL, PATHS[name])
        except mx.MixllmError as e:
            # 128 x 128 blocks are not built for group-wise activation scales, nor (the sums only) for group-wise 8-bit scales
            assert e.status == -2 and name == "prefill128" and variant != "baseline", (name, variant)
            continue
        assert np.array_equal(S.cpu().numpy().astype(np.int64), S_ref), (name, variant, M, K, N, n8)


def test_group_partials_worst_case_magnitudes():
    # all activations +-127, weights at the code extremes: the largest partial sums the
    # integer pipeline can see
    K, N, n8, M = 512, 64, 16, 20
    rng = np.random.default_rng(3)
    xq = np.where(rng.random((M, K)) < 0.5, -127, 127).astype(np.int8)
    xq[0], xq[1] = 127, -127
    perm = ref.feature_perm(N, np.arange(0, 32, 2))
    q8 = np.where(rng.random((n8, K)) < 0.5, -127, 127).astype(np.int8)
    q8[0], q8[1] = 127, -127
    q4 = np.where(rng.random((N - n8, K)) < 0.5, 0, 15).astype(np.uint8)
    z4 = rng.integers(0, 16, (N - n8, K // G)).astype(np.uint8)
    q4[0], z4[0] = 15, 0
    q4[1], z4[1] = 0, 15
    s8 = np.ones((n8, 1), np.float16)
    s4 = np.ones((N - n8, K // G), np.float16)
    L = ref.QuantizedLayer(N, K, G, K, perm, q8, s8, q4, s4, z4)
    P_ref = ref.group_partials(xq, L)
    assert P_ref.max() == 128 * 127 * 127 and P_ref.min() == -128 * 127 * 127
    PL = pack_from_oracle(L)
    for path in ("generic", "prefill"):
        assert np.array_equal(mx.debug_group_partials(dev(xq), PL, PATHS[path]).cpu().numpy(), P_ref), path
    assert np.array_equal(mx.debug_group_partials(dev(xq[:16]), PL, mx.PATH_DECODE).cpu().numpy(), P_ref[:16])


# ------------------------------------------------------------------- the linear --

def check_linear(M, K, N, n8, path, variant="baseline", seed=25):
    act_group, w8_group = (None, None) if variant == "baseline" else (128, 128)
    _, _, L, _, xq, xs = make_case(M, K, N, n8, seed, w8_group, act_group)
    y = mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), PATHS[path])
    torch.cuda.synchronize()
    _, err = check_against_oracle(y.cpu().numpy(), xq, xs, L, (path, variant, M, K, N, n8))
    say(f"  linear {path} {variant} M={M} K={K} N={N} n8={n8}: row rel err {err:.2e}, every element within its bound")


@pytest.mark.parametrize("variant", ["baseline", "paper"])
@pytest.mark.parametrize("path", ["generic", "decode"] + DECODE_VARIANTS)
@pytest.mark.parametrize("M,K,N,n8", [(1, 4096, 4096, 410), (16, 1024, 100, 9), (4, 640, 50, 0), (7, 384, 40, 40),
                                     (8, 14336, 272, 27), (3, 128, 33, 3), (2, 2048, 2070, 207), (1, 14336, 1000, 90),
                                     (4, 28672, 48, 5), (3, 32768, 40, 4),
                                     # the split variant with the activations staged window by window
                                     (16, 14336, 272, 27), (10, 14336, 1000, 0), (16, 9088, 70, 70), (6, 28672, 48, 5),
                                     (16, 28800, 40, 4), (5, 28672, 8200, 820)])
def test_linear_small_m(M, K, N, n8, path, variant):
    skip_unless_covered(path, M, K)
    check_linear(M, K, N, n8, path, variant)


@pytest.mark.parametrize("variant", ["baseline", "paper"])
@pytest.mark.parametrize("path", ["generic"] + TILED)
@pytest.mark.parametrize("M,K,N,n8", [(17, 256, 7, 2), (130, 512, 300, 30), (200, 1024, 530, 0), (33, 384, 70, 70),
                                     (512, 4096, 1024, 102), (256, 384, 8192, 819), (384, 640, 8192, 0)])
def test_linear_tiled(M, K, N, n8, path, variant):
    if path == "prefill128" and variant == "paper":
        _, _, L, _, xq, xs = make_case(M, K, N, n8, 25, 128, 128)
        with pytest.raises(mx.MixllmError) as e:     # not built: refused, no other shape taken silently
            mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), PATHS[path])
        assert e.value.status == -2
        return
    check_linear(M, K, N, n8, path, variant)


def kparts_of(M, K, N, n8, act_group=None, w8_group=None, path=None):
    """K parts the tiled kernel uses for this shape when the caller brings the scratch (host-side plan)."""
    import ctypes as C
    from paper_2412_14590_amd import binding
    out = (C.c_int32 * 16)()
    d = binding._desc(M, K, N, n8, act_group, w8_group)
    assert mx.lib().mixllm_debug_work_split(C.byref(d), mx.PATH_PREFILL if path is None else path, C.cast(out, C.c_void_p)) == 0
    return out[8]


@pytest.mark.parametrize("variant", ["baseline", "paper", "w8_grouped"])
@pytest.mark.parametrize("M,K,N,n8", [(33, 8192, 300, 30), (100, 14336, 530, 53), (17, 16384, 96, 96), (64, 8576, 272, 0),
                                     (256, 28672, 140, 14), (130, 8192, 1030, 103)])
def test_tiled_path_with_k_split_over_blocks(M, K, N, n8, variant):
    # Long K, few output tiles: with the scratch mixllm_query_sizes asks for, the tiled kernel cuts K
    # into parts for several blocks and a second kernel adds the parts' fp32 sums (fixed order).
    # Against the oracle (row norm and per element), in every block shape, bit-identical between
    # runs, and through the fp16 entry point; without the scratch the same call runs unsplit.
    ag, wg = {"baseline": (None, None), "paper": (128, 128), "w8_grouped": (None, 128)}[variant]
    _, _, L, x, xq, xs = make_case(M, K, N, n8, seed=35, w8_group=wg, act_group=ag)
    PL = pack_from_oracle(L)
    need = mx.query_sizes(M, K, N, n8, ag, wg)
    assert kparts_of(M, K, N, n8, ag, wg) > 1 and need["linear_workspace_bytes"] > 0
    ws = torch.empty(need["linear_workspace_bytes"], dtype=torch.uint8, device="cuda")
    y = mx.mixed_linear(dev(xq), dev(xs), PL, mx.PATH_PREFILL, workspace=ws)
    check_against_oracle(y.cpu().numpy(), xq, xs, L, ("k split", variant, M, K, N, n8))
    ws.fill_(0xA5)                                         # the kernel may not depend on what the scratch held
    assert torch.equal(y, mx.mixed_linear(dev(xq), dev(xs), PL, mx.PATH_PREFILL, workspace=ws))
    for name in ("prefill32", "prefill64", "prefill128"):
        if name == "prefill128" and variant == "paper":
            continue
        big = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
        y2 = mx.mixed_linear(dev(xq), dev(xs), PL, PATHS[name], workspace=big)
        check_against_oracle(y2.cpu().numpy(), xq, xs, L, ("k split", name, variant, M, K, N, n8))
    y3 = mx.mixed_linear(dev(xq), dev(xs), PL, mx.PATH_PREFILL)        # no scratch: unsplit, same bound
    check_against_oracle(y3.cpu().numpy(), xq, xs, L, ("no scratch", variant, M, K, N, n8))
    small = torch.empty(need["linear_workspace_bytes"] // 3 // 16 * 16, dtype=torch.uint8, device="cuda")   # room for fewer parts
    y4 = mx.mixed_linear(dev(xq), dev(xs), PL, mx.PATH_PREFILL, workspace=small)
    check_against_oracle(y4.cpu().numpy(), xq, xs, L, ("short scratch", variant, M, K, N, n8))
    yf = mx.linear_fp16(dev(x), PL, act_group=ag)           # the fp16 entry point brings the same scratch
    assert torch.equal(yf, y) or M <= 64                    # (up to 64 tokens it may take another kernel)
    check_against_oracle(yf.cpu().numpy(), xq, xs, L, ("fp16 entry", variant, M, K, N, n8))


@pytest.mark.parametrize("variant", ["baseline", "paper", "w8_grouped"])
@pytest.mark.parametrize("M,K,N,n8", [
    (17, 1664, 16, 3), (32, 1664, 33, 33), (33, 1920, 70, 0), (65, 4224, 64, 6),      # 4 quads (one of 1 and of 3 groups), 9: uneven shares
    (17, 14336, 300, 30), (300, 4096, 257, 26), (64, 8192, 1000, 100),                # the longest K it takes; many token tiles
    (40, 1920, 4095, 409), (32, 2048, 8160, 31), (32, 2048, 8192, 31), (48, 2048, 8448, 0), (48, 2048, 8449, 0)])   # around one and two blocks a CU
def test_tiles_cut_along_k_over_the_waves_of_a_block(M, K, N, n8, variant):
    # Small grids (the library's choice, no path of its own): four waves of a block take a quarter of K each and add
    # their sums up in LDS.  Against the oracle by row norm and per element, bit-identical between runs and between the
    # entry points, nothing written outside y.
    ag, wg = {"baseline": (None, None), "paper": (128, 128), "w8_grouped": (None, 128)}[variant]
    _, _, L, x, xq, xs = make_case(M, K, N, n8, seed=37, w8_group=wg, act_group=ag)
    PL = pack_from_oracle(L)
    buf = torch.full((M * N + 64,), -3.0, dtype=torch.float16, device="cuda")
    y = mx.mixed_linear(dev(xq), dev(xs), PL, out=buf[: M * N].view(M, N))
    check_against_oracle(y.cpu().numpy(), xq, xs, L, ("slices", variant, M, K, N, n8))
    assert bool((buf[M * N:] == -3.0).all())
    assert torch.equal(y, mx.mixed_linear(dev(xq), dev(xs), PL))
    assert torch.equal(y, mx.linear_fp16(dev(x), PL, act_group=ag))


def library_choice(M, K, N, n8, act_group=None, w8_group=None):
    """The kernel MIXLLM_PATH_AUTO takes: (without scratch, with the scratch the library asks for)."""
    import ctypes as C
    from paper_2412_14590_amd import binding
    out = (C.c_int32 * 16)()
    d = binding._desc(M, K, N, n8, act_group, w8_group)
    assert mx.lib().mixllm_debug_work_split(C.byref(d), mx.PATH_AUTO, C.cast(out, C.c_void_p)) == 0
    return out[0], out[1]


SLICES = 100   # MIXLLM_PLAN_SLICES


@pytest.mark.parametrize("act_group", [None, 128])
@pytest.mark.parametrize("w8_group", [None, 128])
@pytest.mark.parametrize("M,K,N,n8", [(17, 1664, 16, 3), (33, 1920, 75, 33), (64, 4224, 64, 0), (40, 4096, 530, 530),
                                     (130, 2048, 1000, 100), (64, 8192, 257, 26),
                                     (17, 1664, 7936, 31), (32, 1664, 15488, 1549), (48, 2048, 8000, 800), (48, 4096, 8192, 819)])   # full grids of one and two blocks a CU
def test_tiles_cut_along_k_add_up_the_integer_sums(M, K, N, n8, w8_group, act_group):
    # The kernel has no debug variant that hands out its integers: scales of 1 and 2, different from group to group and
    # small codes make the outputs the integers themselves (every sum exact in fp32, converted to fp16 once).  Slices of
    # uneven length, a last slice with groups past the end of K, both parts, ragged tiles of tokens and channels.
    assert library_choice(M, K, N, n8, act_group, w8_group)[0] == SLICES
    rng = np.random.default_rng(M + K)
    ng, n4 = K // 128, N - n8
    L = make_case(0, K, N, n8, seed=45, w8_group=w8_group)[2]
    if n8:
        L.q8[:], L.s8[:] = rng.integers(-8, 9, L.q8.shape), rng.integers(1, 3, L.s8.shape)
    if n4:
        L.q4[:], L.z4[:], L.s4[:] = rng.integers(0, 16, L.q4.shape), rng.integers(0, 16, L.z4.shape), rng.integers(1, 3, L.s4.shape)
    xq = (rng.integers(-1, 2, (M, K)) * (rng.random((M, K)) < 0.25)).astype(np.int8)
    xs = rng.integers(1, 3, (M, 1 if act_group is None else ng)).astype(np.float16)
    y64 = (ref.group_partials(xq, L).astype(np.float64) * (weight_scales_in_channel_order(L)[None] * xs.astype(np.float64)[:, None, :])).sum(axis=2)
    assert np.abs(y64).max() < 65504 and (np.abs(y64) <= 2048).mean() > 0.99      # integers fp16 holds, nearly all
    y = mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L)).cpu().numpy()
    assert np.array_equal(y, y64.astype(np.float16))


@pytest.mark.parametrize("variant", ["baseline", "paper"])
@pytest.mark.parametrize("M,K,N,n8", [(40, 28672, 300, 30), (130, 16512, 530, 53), (17, 131072, 40, 20)])
def test_tiles_cut_along_k_on_long_k_without_scratch(M, K, N, n8, variant):
    ag, wg = {"baseline": (None, None), "paper": (128, 128)}[variant]
    assert library_choice(M, K, N, n8, ag, wg) == (SLICES, mx.PATH_PREFILL)
    _, _, L, x, xq, xs = make_case(M, K, N, n8, seed=46, w8_group=wg, act_group=ag)
    y = mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L))
    check_against_oracle(y.cpu().numpy(), xq, xs, L, ("slices, long K", variant, M, K, N, n8))


@pytest.mark.parametrize("M,K,N,n8", [(17, 256, 7, 2), (33, 384, 70, 70), (64, 1024, 530, 0), (50, 640, 50, 5),
                                     (64, 512, 300, 30), (20, 4096, 1000, 100), (64, 14336, 272, 27), (1, 512, 96, 9),
                                     (48, 2048, 2070, 207)])
def test_mid_path_partials_and_linear(M, K, N, n8):
    # the path for a few dozen tokens: integer partials bit-exact, outputs within tolerance, in every
    # scale granularity it covers (activation scales per token and group: up to 32 tokens)
    say("mid", M, K, N, n8)
    check_partials(M, K, N, n8, "mid")
    check_linear(M, K, N, n8, "mid")
    for ag, wg in ((None, 128), (128, None), (128, 128)):
        _, _, L, _, xq, xs = make_case(M, K, N, n8, 29, wg, ag)
        if ag == 128 and M > 32:
            with pytest.raises(mx.MixllmError) as e:
                mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), mx.PATH_MID)
            assert e.value.status == -2
            continue
        y = mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), mx.PATH_MID)
        check_against_oracle(y.cpu().numpy(), xq, xs, L, ("mid", ag, wg, M, K, N, n8))


def test_mid_path_rejects_what_it_does_not_cover():
    _, _, L, _, xq, xs = make_case(65, 256, 40, 4, seed=3)
    with pytest.raises(mx.MixllmError) as e:
        mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), mx.PATH_MID)       # more than 64 tokens
    assert e.value.status == -2
    _, _, L, _, xq, xs = make_case(40, 256, 40, 4, seed=3, w8_group=128, act_group=128)
    with pytest.raises(mx.MixllmError) as e:
        mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), mx.PATH_MID)       # activation scales per group, more than 32 tokens
    assert e.value.status == -2


def test_auto_dispatch_and_end_to_end_from_fp16():
    # x fp16 -> quantizer -> linear, everything on the GPU, weights quantized on the GPU
    for M in (1, 16, 17, 300):
        W, sal, L, x, xq, xs = make_case(M, 1024, 272, 27, seed=26)
        PL = mx.quantize_weights(dev(W), sal)
        y = mx.linear(dev(x), PL)
        y_ref = ref.mixed_linear(xq, xs, L)
        assert row_rel_err(y.cpu().numpy(), y_ref) <= TOL
    with pytest.raises(mx.MixllmError):
        mx.mixed_linear(dev(xq), dev(xs), PL, mx.PATH_DECODE)     # M = 300 > 16


@pytest.mark.parametrize("variant", ["baseline", "paper"])
@pytest.mark.parametrize("M,K,N,n8", [(1, 4096, 4096, 410), (1, 1024, 100, 9), (4, 640, 50, 0), (7, 384, 40, 40),
                                     (16, 4096, 1024, 102), (3, 128, 33, 3), (2, 2048, 2070, 207), (4, 4096, 600, 60),
                                     (3, 14336, 96, 10), (40, 512, 64, 6), (1, 14336, 272, 27), (1, 8192, 4100, 400),
                                     (1, 16384, 48, 5), (8, 2048, 300, 30), (2, 8192, 64, 6), (5, 1024, 100, 10),
                                     (8, 512, 40, 4), (16, 1024, 530, 53), (3, 4096, 1000, 100)])
def test_fused_quantizer_and_linear_from_fp16(M, K, N, n8, variant):
    # one call from fp16 activations: for M = 1 the decode kernel quantizes its own activations
    # where a variant can (K <= 4096: resident variant; K <= 16384 with per-token scales: split
    # variant), and so does the split variant for a few tokens of a short row (K a multiple of 512,
    # M K <= 16384, per-token scales); the result must equal the oracle (quantizer + linear) and
    # agree with the two-call GPU path on the same inputs
    w8g, ag = (None, None) if variant == "baseline" else (128, 128)
    W, sal, L, x, xq, xs = make_case(M, K, N, n8, seed=31, w8_group=w8g, act_group=ag)
    PL = pack_from_oracle(L)
    y = mx.linear_fp16(dev(x), PL, act_group=ag)
    torch.cuda.synchronize()
    y_ref = ref.mixed_linear(xq, xs, L)
    err = row_rel_err(y.cpu().numpy(), y_ref)
    say(f"  fused fp16 {variant} M={M} K={K} N={N} n8={n8}: row rel err {err:.2e}")
    assert err <= TOL
    y2 = mx.linear(dev(x), PL, act_group=ag)
    if M == 1:
        # decode kernel with and without the built-in quantizer (when the unfused call picks the
        # same variant the outputs are bit-identical; otherwise within tolerance)
        assert row_rel_err(y.cpu().numpy(), y2.cpu().numpy().astype(np.float64)) <= 1e-3
    else:
        assert torch.equal(y, y2)


@pytest.mark.parametrize("path", ["prefill32", "prefill64", "prefill128"])
@pytest.mark.parametrize("rows", [-1, 0, 1])
@pytest.mark.parametrize("K,groups", [(640, False), (640, True), (8192, False)])
def test_tiled_stores_at_the_last_token_tile(path, rows, K, groups):
    # a last tile that is one row short, full, and one row over, of every block shape; K = 8192 with scratch,
    # so that the parts of a K split go through the same stores; nothing is written past the last row or part
    tile = int(path[len("prefill"):])
    M, N, n8 = tile + rows, 150, 21
    act_group = 128 if groups and path != "prefill128" else None
    _, _, L, x, xq, xs = make_case(M, K, N, n8, seed=tile + rows, w8_group=128 if groups else None, act_group=act_group)
    PL = pack_from_oracle(L)
    # scratch for exactly two parts of K (sums of every token and padded row), with guard bytes right behind it
    need = 2 * M * (-(-n8 // 16) + -(-(N - n8) // 16)) * 16 * 4 if K >= 8192 else 0
    ws = torch.full((need + 256,), 77, dtype=torch.uint8, device="cuda")
    buf = torch.full((M * N + 64,), -3.0, dtype=torch.float16, device="cuda")
    y = mx.mixed_linear(dev(xq), dev(xs), PL, PATHS[path], out=buf[: M * N].view(M, N), workspace=ws[:need] if need else None)
    check_against_oracle(y.cpu().numpy(), xq, xs, L, f"{path} M={M} K={K}")
    assert bool((buf[M * N:] == -3.0).all())
    assert bool((ws[need:] == 77).all())
    assert bool((ws[:need].view(torch.int32) != 0x4d4d4d4d).all())   # K was split, and both parts stored every sum


def test_calls_go_to_the_current_stream():
    from paper_2412_14590_amd import binding
    for s in (torch.cuda.default_stream(), torch.cuda.Stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            assert binding._stream() == torch.cuda.current_stream().cuda_stream == s.cuda_stream


def test_calls_from_python_check_their_arguments_and_return_the_callers_tensors():
    _, _, L, x, xq, xs = make_case(5, 512, 64, 6, seed=41)
    PL, x, xq, xs = pack_from_oracle(L), dev(x), dev(xq), dev(xs)
    wide = torch.zeros((5, 1024), dtype=torch.float16, device="cuda")
    for bad in (x.float(), x[0], wide, wide[:, ::2], x.cpu()):      # type, dimensions, columns, strides, device
        with pytest.raises(AssertionError):
            mx.linear_fp16(bad, PL)
    for bad in (x.float(), x[0], wide[:, ::2], x.cpu()):
        with pytest.raises(AssertionError):
            mx.quantize_activations(bad)
    for bad in ((xq[:, :256], xs), (xq[:3], xs), (xq, xs.cpu()), (wide.to(torch.int8)[:, ::2], xs)):
        with pytest.raises(AssertionError):
            mx.mixed_linear(*bad, PL)
    for act_group in (64, 3):                                       # a group size the library does not have
        with pytest.raises(mx.MixllmError) as e:
            mx.linear_fp16(x, PL, act_group)
        assert e.value.status == -2
        with pytest.raises(mx.MixllmError):
            mx.quantize_activations(x, act_group)
    with pytest.raises(TypeError):
        mx.linear_fp16([1.0], PL)
    y, q, s = torch.empty((5, 64), dtype=torch.float16, device="cuda"), torch.empty_like(xq), torch.empty_like(xs)
    assert mx.linear_fp16(x, PL, out=y) is y
    qs = mx.quantize_activations(x, out=(q, s))
    assert qs[0] is q and qs[1] is s and torch.equal(q, xq) and torch.equal(s, xs)
    y2 = torch.empty_like(y)
    assert mx.mixed_linear(q, s, PL, out=y2) is y2 and torch.equal(y, y2)
    empty = mx.linear_fp16(x[:0], PL)
    assert empty.shape == (0, 64) and empty.dtype == torch.float16


def test_quantizer_refuses_a_missing_buffer():
    x = torch.ones((3, 256), dtype=torch.float16, device="cuda")
    xq, xs = mx.quantize_activations(x)
    for out in ((None, xs), (xq, None), (None, None)):
        with pytest.raises(mx.MixllmError) as e:
            mx.quantize_activations(x, out=out)
        assert e.value.status == -1


def test_fused_entry_point_rejects_a_short_workspace():
    W, sal, L, x, xq, xs = make_case(40, 512, 64, 6, seed=32)
    PL = pack_from_oracle(L)
    with pytest.raises(mx.MixllmError):
        mx.linear_fp16(dev(x), PL, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))


def test_empty_batch_is_a_no_op():
    _, _, L, *_ = make_case(0, 256, 40, 4, seed=27)
    PL = pack_from_oracle(L)
    xq = torch.empty((0, 256), dtype=torch.int8, device="cuda")
    xs = torch.empty((0, 1), dtype=torch.float16, device="cuda")
    assert mx.mixed_linear(xq, xs, PL).shape == (0, 40)


def test_output_permutation_and_determinism():
    # permuting output features only permutes y (Sec. 3.1.1), and reruns are bit-identical
    M, K, N = 8, 512, 96
    W = synth.make_w(N, K, seed=28, n_outlier_rows=4)
    sal = np.array([3, 17, 40, 41, 95], np.int32)
    x = dev(synth.make_x(M, K, seed=28))
    y1 = mx.linear(x, mx.quantize_weights(dev(W), sal))
    y1b = mx.linear(x, mx.quantize_weights(dev(W), sal))
    assert torch.equal(y1, y1b)
    sigma = np.random.default_rng(4).permutation(N)
    inv = np.argsort(sigma)
    y2 = mx.linear(x, mx.quantize_weights(dev(W[sigma]), np.sort(inv[sal]).astype(np.int32)))
    assert torch.equal(y2, y1[:, torch.from_numpy(sigma).cuda()])


# ------------------------------------------------ full-size layers of the workloads --

@pytest.mark.parametrize("M", [1, 16, 40, 130])
def test_outputs_beyond_the_fp16_range_become_infinities(M):
    # the conversion of an output that does not fit fp16 is the IEEE one (to +-inf), in the oracle and
    # in every kernel; finite outputs next to them still agree
    K, N, n8 = 512, 48, 5
    W = np.zeros((N, K), dtype=np.float16)
    W[:, :] = np.float16(0.01)
    W[3, :] = np.float16(30.0)       # a 4-bit row and (below) an 8-bit row with huge outputs
    W[7, :] = np.float16(-25.0)
    sal = np.array([7, 11, 20, 33, 40], dtype=np.int32)
    x = np.full((M, K), 20.0, dtype=np.float16)
    L = ref.quantize_weights(W, sal, G, None)
    xq, xs = ref.quantize_act(x, None)
    y_ref = ref.mixed_linear(xq, xs, L)
    assert np.isinf(y_ref[:, 3]).all() and np.isinf(y_ref[:, 7]).all() and np.isfinite(y_ref[:, 0]).all()
    for path in (mx.PATH_AUTO, mx.PATH_PREFILL, mx.PATH_GENERIC):
        y = mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), path).cpu().numpy()
        assert np.array_equal(np.isinf(y), np.isinf(y_ref))
        assert np.array_equal(np.sign(y[np.isinf(y)]), np.sign(y_ref[np.isinf(y_ref)]))
        fin = np.isfinite(y_ref)
        assert np.allclose(y[fin].astype(np.float64), y_ref[fin].astype(np.float64), rtol=2e-3)


@pytest.mark.parametrize("subnormal", ["token", "channel"])
@pytest.mark.parametrize("M,K,path", [(40, 2048, "auto"), (33, 640, "prefill32"), (70, 2048, "prefill64")])
def test_subnormal_scales_per_group_are_not_flushed(M, K, path, subnormal):
    # ... by the matrix pipe, which multiplies them: scales of a few 2^-24 on one side, large ones on the other
    N, n8 = 70, 20
    _, _, L, _, xq, xs = make_case(M, K, N, n8, seed=44, w8_group=128, act_group=128)
    rng = np.random.default_rng(44)
    for a, side in ((xs, "token"), (L.s4, "channel"), (L.s8, "channel")):
        a[:] = rng.integers(1, 1024, a.shape) * 2.0 ** -24 if side == subnormal else rng.uniform(1.0, 8.0, a.shape)
    y = mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), mx.PATH_AUTO if path == "auto" else PATHS[path])
    check_against_oracle(y.cpu().numpy(), xq, xs, L, ("subnormal", subnormal, M, K, path))


@pytest.mark.parametrize("w8_group", [None, 128])
@pytest.mark.parametrize("M,K,path", [(40, 2048, "auto"), (40, 1664, "auto"), (33, 640, "prefill32"), (33, 2048, "prefill32"), (70, 640, "prefill64"), (70, 2048, "prefill64"),
                                      (150, 1152, "auto")])
def test_infinite_and_nan_scales_per_group_reach_the_outputs_they_belong_to(M, K, path, w8_group):
    # scales per (token, group) are multiplied by the matrix pipe from bf16 halves: an infinite scale of a token or of a
    # channel gives the infinities, and the NaNs, of the sum of P s_w s_a, on its row or column only - the last
    # group of a K that ends inside a group of four included
    N, n8, ng = 70, 20, K // 128
    _, _, L, x, xq, xs = make_case(M, K, N, n8, seed=43, w8_group=w8_group, act_group=128)
    inf, nan = np.float16(np.inf), np.float16(np.nan)
    xs[0, 0], xs[1, ng - 1], xs[2, 2], xs[3, 1], xs[4, :2], xs[5, 0], xs[M - 1, ng // 2] = inf, inf, nan, -inf, inf, 0, inf
    L.s4[7, 1], L.s4[8, ng - 1], L.s8[3, 0], L.s8[4, -1], L.s4[9, 0], L.s4[30, 0] = inf, -inf, inf, nan, nan, 0
    with np.errstate(all="ignore"):
        sw = weight_scales_in_channel_order(L)
        y64 = (ref.group_partials(xq, L).astype(np.float64) * (sw[None] * xs.astype(np.float64)[:, None, :])).sum(axis=2)
        want = y64.astype(np.float16)
    assert np.isinf(want).any() and np.isnan(want).any() and np.isfinite(want[6:]).mean() > 0.8
    y = mx.mixed_linear(dev(xq), dev(xs), pack_from_oracle(L), mx.PATH_AUTO if path == "auto" else PATHS[path]).cpu().numpy()
    assert np.array_equal(np.isnan(y), np.isnan(want)) and np.array_equal(np.isinf(y), np.isinf(want))
    assert np.array_equal(y[np.isinf(want)], want[np.isinf(want)])
    fin = np.isfinite(want)
    rms = np.sqrt(np.mean(want[fin].astype(np.float64) ** 2))
    assert np.abs(y[fin].astype(np.float64) - y64[fin]).max() <= 1e-3 * max(rms, np.abs(y64[fin]).max())


def test_random_shapes_through_every_path_that_covers_them():
    """60 seeded random shapes (tokens 1..299, K of 1..40 groups, ragged N, any 8-bit share, both scale
    granularities): AUTO, the tiled kernel, every decode variant, the kernel for a few dozen tokens and
    the fp16 entry point, partials bit-exact and outputs within tolerance wherever a path takes the shape."""
    rng = np.random.default_rng(20241)
    for it in range(60):
        kind = rng.integers(0, 4)
        M = int(rng.integers(1, 17)) if kind == 0 else int(rng.integers(17, 65)) if kind == 1 else \
            int(rng.integers(65, 300)) if kind == 2 else int(rng.choice([1, 2, 3, 4, 8, 16, 32, 64, 128, 129, 256]))
        K = 128 * int(rng.choice([1, 2, 3, 4, 5, 7, 8, 12, 16, 28, 32, 40]))
        N = int(rng.choice([1, 5, 16, 17, 33, 100, 130, 500, 1030, 2070]))
        while M * K * N > 1.5e8:
            N = max(1, N // 2)
        n8 = int(rng.choice([0, N, N // 10, int(rng.integers(0, N + 1))]))
        ag, wg = (128, 128) if rng.integers(0, 3) == 0 else (None, None)
        _, _, L, x, xq, xs = make_case(M, K, N, n8, seed=5000 + it, w8_group=wg, act_group=ag)
        PL = pack_from_oracle(L)
        y_ref = ref.mixed_linear(xq, xs, L)
        P_ref = ref.group_partials(xq, L)
        paths = ["generic", "prefill"] + (DECODE_VARIANTS if M <= 16 else []) + (["mid"] if M <= 64 else [])
        taken = 0
        for name in [None] + paths:
            path = mx.PATH_AUTO if name is None else PATHS[name]
            try:
                y = mx.mixed_linear(dev(xq), dev(xs), PL, path)
                P = mx.debug_group_partials(dev(xq), PL, path)
            except mx.MixllmError as e:
                assert e.status == -2 and name in ("decode_split", "mid"), (name, M, K, N, n8)   # EUNSUPPORTED
                continue
            torch.cuda.synchronize()
            taken += 1
            assert np.array_equal(P.cpu().numpy(), P_ref), (name, M, K, N, n8, ag)
            assert row_rel_err(y.cpu().numpy(), y_ref) <= TOL, (name, M, K, N, n8, ag)
        assert taken >= 3
        yf = mx.linear_fp16(dev(x), PL, act_group=ag)
        torch.cuda.synchronize()
        assert row_rel_err(yf.cpu().numpy(), y_ref) <= TOL, ("fp16 entry", M, K, N, n8, ag)
    say("  60 random shapes: all paths agree with the oracle")


def tiled_shape_of(M, lay):
    """The forced-shape path equal to the block shape the tiled kernel picks for this layer at M tokens."""
    import ctypes as C
    from paper_2412_14590_amd import binding
    out = (C.c_int32 * 16)()
    d = binding._desc(M, lay.K, lay.N, lay.n8)
    assert mx.lib().mixllm_debug_work_split(C.byref(d), mx.PATH_PREFILL, C.cast(out, C.c_void_p)) == 0
    return {32: mx.PATH_PREFILL_32, 64: mx.PATH_PREFILL_64, 128: mx.PATH_PREFILL_128}[out[0]]


def check_cell(lay, L, PL, M, seed, act_group=None):
    """One (layer, M) cell of a workload at full size, through the call the benchmark times
    (mixllm_mixed_linear_fp16, library's choice of kernel).
    Up to 64 tokens: every row against the oracle (row norm and per element), codes, scales and the
    per-group partials bit-exact - of the kernel the library takes for them, which is the linear's own except where
    that is the tiles cut along K: their sums have a test of their own.
    More tokens (the oracle is O(MNK)): a stratified sample of rows against the oracle the same way
    (one row per 32-token tile, first and last row of every 128-token block), and ALL rows against
    the one-thread-per-output kernel on the GPU, which the sample pins to the oracle: the int32 sums
    over the groups out of the timed kernels bit-exact, the fp16 outputs within two roundings."""
    tag = (lay.name, lay.K, lay.N, lay.n8, M, act_group)
    x = synth.make_x(M, lay.K, seed=seed + M)
    xd = dev(x)
    y = mx.linear_fp16(xd, PL, act_group=act_group)
    rows = np.arange(M) if M <= 64 else stratified_rows(M, seed + M)
    xq_ref, xs_ref = ref.quantize_act(x[rows], act_group)
    P_ref, err = check_against_oracle(y.cpu().numpy()[rows], xq_ref, xs_ref, L, tag)
    xq, xs = mx.quantize_activations(xd, act_group)
    assert np.array_equal(xq.cpu().numpy()[rows], xq_ref), tag
    assert np.array_equal(xs.cpu().numpy()[rows].view(np.uint16), xs_ref.view(np.uint16)), tag
    if M <= 64:
        P = mx.debug_group_partials(xq, PL)
        assert np.array_equal(P.cpu().numpy(), P_ref), tag
        say(f"  {lay.name} K={lay.K} N={lay.N} n8={lay.n8} M={M}: all rows, row rel err {err:.2e}, elements within bound, partials exact")
        return
    S = mx.debug_channel_sums(xq, xs, PL, mx.PATH_PREFILL)
    Sg = mx.debug_channel_sums(xq, xs, PL, mx.PATH_GENERIC)
    assert torch.equal(S, Sg), tag
    assert np.array_equal(Sg.cpu().numpy()[rows].astype(np.int64), P_ref.sum(axis=2, dtype=np.int64)), tag
    del S, Sg
    yg = mx.mixed_linear(xq, xs, PL, mx.PATH_GENERIC).float()
    lws = mx.query_sizes(M, lay.K, lay.N, lay.n8, act_group, PL.w8_group)["linear_workspace_bytes"]
    yt = mx.mixed_linear(xq, xs, PL, workspace=torch.empty(max(lws, 16), dtype=torch.uint8, device="cuda")).float()
    assert torch.equal(yt.half(), y), tag        # the fp16 entry point is quantizer + this launch (K split the same way)
    rms = yg.pow(2).mean(dim=1, keepdim=True).sqrt()
    # both kernels round the same fp32-accurate value to fp16: one unit in the last place apart at
    # most, plus their accumulation errors (a few 1e-5 of the row's typical magnitude)
    assert bool(((yt - yg).abs() <= yg.abs() * 2.0 ** -10 + 2e-4 * rms + 1e-7).all()), tag
    say(f"  {lay.name} K={lay.K} N={lay.N} n8={lay.n8} M={M}: {len(rows)} sampled rows row rel err {err:.2e}, elements within "
        f"bound; all rows: integer sums exact, outputs agree with the generic kernel")


def check_block_partials(lay, L, PL, M, rows, seed):
    """Per-group int32 partials out of the tiled kernel in the block shape it uses for this layer at
    M tokens (hand-issued loads and all), on a contiguous run of token rows, against the oracle."""
    x = synth.make_x(M, lay.K, seed=seed + M)[rows]
    xq_ref, _ = ref.quantize_act(x)
    P = mx.debug_group_partials(dev(xq_ref), PL, tiled_shape_of(M, lay))
    assert np.array_equal(P.cpu().numpy(), ref.group_partials(xq_ref, L)), (lay.name, M)
    say(f"  {lay.name} K={lay.K} N={lay.N}: partials of {len(rows)} rows exact in the block shape used at M={M}")


@pytest.mark.parametrize("name", ["qkv", "o", "gate_up", "down"])
def test_llama3_8b_decode_layers_full_size(name):
    # workload 2: every layer of the block at M in {1, 4, 8, 16}, every row
    lay, L, PL = full_size_layer("8b", name)
    say("8B decode", name, lay.K, lay.N, lay.n8)
    u = mx.unpack_weights(PL)
    assert np.array_equal(u["q4"].cpu().numpy(), L.q4) and np.array_equal(u["q8"].cpu().numpy(), L.q8)
    assert np.array_equal(u["z4"].cpu().numpy(), L.z4)
    assert np.array_equal(u["s4"].cpu().numpy().view(np.uint16), L.s4.view(np.uint16))
    assert np.array_equal(u["s8"].cpu().numpy().view(np.uint16), L.s8.view(np.uint16))
    for M in (1, 4, 8, 16):
        check_cell(lay, L, PL, M, seed=100)


@pytest.mark.parametrize("name", ["qkv", "o", "gate_up", "down"])
def test_llama3_8b_prefill_layers_full_size(name):
    # workload 3: every layer at M in {512, 2048, 8192}, in the configuration the benchmark times
    lay, L, PL = full_size_layer("8b", name)
    say("8B prefill", name, lay.K, lay.N, lay.n8)
    for M in (512, 2048, 8192):
        check_cell(lay, L, PL, M, seed=200)
    # per-group partials out of the 128 x 128 block shape (the one timed at M = 2048): a whole block
    # of 128 tokens, and a ragged one
    check_block_partials(lay, L, PL, 2048, np.arange(128, 256), seed=200)
    check_block_partials(lay, L, PL, 2048, np.arange(2000, 2048), seed=200)


@pytest.mark.parametrize("name", ["qkv", "o", "gate_up", "down"])
def test_llama31_70b_layers(name):
    # workload 4: the Llama-3.1-70B-shaped layers (N(0, 0.015) weights, N/64 outlier rows), M sweep
    lay, L, PL = full_size_layer("70b", name, seed=2)
    say("70B", name, lay.K, lay.N, lay.n8)
    for M in (1, 16, 64, 256, 2048):
        check_cell(lay, L, PL, M, seed=300)
    check_block_partials(lay, L, PL, 2048, np.arange(1024, 1024 + (128 if name in ("qkv", "o") else 40)), seed=300)


def test_paper_granularity_full_size_layers():
    # the paper's scale granularity (activation scales per token and group, 8-bit weight scales per
    # group; Sec. 3.1.2, Sec. 4.1) on two full-size layers, decode and tiled path
    for name in ("o", "down"):
        lay, L, PL = full_size_layer("8b", name, w8_group=128)
        for M in (1, 16, 512, 2048):
            check_cell(lay, L, PL, M, seed=700, act_group=128)


def _check_layer(lay, Ms, seed):
    """A layer drawn for one test (8-bit share sweeps): oracle and GPU quantization, then the cells."""
    L = ref.quantize_weights(lay.W, lay.salient_idx)
    PL = mx.quantize_weights(dev(lay.W), lay.salient_idx)
    for M in Ms:
        check_cell(lay, L, PL, M, seed)


@pytest.mark.parametrize("N", [4096, 14336])
@pytest.mark.parametrize("share", [0.0, 0.20, 0.50, 0.71, 1.0])
def test_single_linear_8bit_share_sweep(N, share):
    # the grid of the paper's single-linear study (Sec. 5.2: K = 4096, N in {4096, 14336}, 8-bit shares
    # up to 100 %; 71 % is the largest per-layer share its appendix reports), 10 % being covered by
    # the Llama-shaped layer tests: decode (every row) and tiled path (sampled rows, partials)
    K = 4096
    lay = synth.make_layer(f"sweep{N}", K, N, frac8=share, seed=77)
    say(f"share sweep: N={N} share={share} n8={lay.n8}")
    _check_layer(lay, (1, 16, 1024), seed=600 + int(100 * share))


def test_uneven_8bit_share_across_a_32_layer_stack():
    # per-layer 8-bit shares drawn so that the stack averages 10 % (0 % .. 40 % per layer), plus the
    # all-4-bit and all-8-bit degenerate layers, at M = 1 and M = 256: the scatter has to put every
    # channel back in place whatever the split, and no part may be assumed non-empty
    fr = synth.uneven_fractions(32, seed=0)
    by_name = {}
    for (layer, name), f in fr.items():
        by_name.setdefault(name, []).append((f, layer))
    total = sum(synth.LLAMA3_8B[n][1] * f for (l, n), f in fr.items()) / sum(synth.LLAMA3_8B[n][1] for (l, n) in fr)
    assert abs(total - 0.10) < 5e-3 and max(fr.values()) <= 0.40 + 1e-9
    picks = []
    for name, lst in by_name.items():
        lst.sort()
        picks += [(name, lst[0][0], lst[0][1]), (name, lst[-1][0], lst[-1][1])]    # smallest and largest share
    picks += [("o", 0.0, 98), ("o", 1.0, 99)]
    for name, f, layer in picks:
        if name == "gate_up" and 0.0 < f < 0.3:
            continue   # the large layer once (its largest share) is enough for the running time
        K, N = synth.LLAMA3_8B[name]
        lay = synth.make_layer(name, K, N, frac8=f, seed=1000 + layer)
        say(f"uneven: layer {layer} {name} share {f:.3f} n8={lay.n8}")
        assert lay.n8 == synth.n8_for(N, f)
        _check_layer(lay, (1, 256), seed=500 + layer)


# ------------------------------------------------- global precision search (Sec. 3.2) --

def make_grad(N, K, seed, scale):
    """A stand-in for the loss gradient w.r.t. a layer's weights (the paper's comes from a model and
    calibration data): N(0, scale) with the same outlier input channels as the activations."""
    return (synth.make_x(N, K, seed=seed, tag="grad").astype(np.float32) * scale).astype(np.float16)


@pytest.mark.parametrize("N,K,scale", [(37, 512, 0.05), (100, 128, 3.0), (4096, 4096, 0.02), (1000, 14336, 0.5),
                                       (16, 640, 1.0)])
def test_channel_salience_matches_the_oracle(N, K, scale):
    say("salience", N, K, scale)
    W = synth.make_w(N, K, seed=41, n_outlier_rows=min(N, 8))
    g1, g2 = make_grad(N, K, 42, scale), make_grad(N, K, 43, 2 * scale)
    ref_one, s1 = ref.channel_salience(W, g1)
    got = mx.channel_salience(dev(W), dev(g1)).cpu().numpy().astype(np.float64)
    # fp32 sums against the fp64 definition: the error of S1 is bounded by the rounding of a K-term
    # fp32 sum of |g| |quantize(W) - W|; S = |S1 + S1^2/2| amplifies it by |1 + S1|
    q, s, z = ref.quantize_w4(W)
    deq = (q.astype(np.float64).reshape(N, K // G, G) - z.astype(np.float64)[:, :, None]) * s.astype(np.float64)[:, :, None]
    mag = (np.abs(g1.astype(np.float64)) * np.abs(deq.reshape(N, K) - W.astype(np.float64))).sum(axis=1)
    tol = 2e-6 * mag * (1 + np.abs(s1)) + 1e-30
    assert np.all(np.abs(got - ref_one) <= tol), float(np.max(np.abs(got - ref_one) / tol))
    # the mean over two samples, built call by call
    ref_two, _ = ref.channel_salience(W, [g1, g2])
    acc = mx.channel_salience(dev(W), dev(g1), weight=0.5)
    mx.channel_salience(dev(W), dev(g2), out=acc, weight=0.5, accumulate=True)
    assert np.allclose(acc.cpu().numpy(), ref_two, rtol=2e-4, atol=1e-12)


def test_channel_salience_uses_the_weight_quantizers_codes():
    # weights on the 4-bit grid: zero salience whatever the gradient; and the closed form where the
    # first- and second-order terms cancel (S1 = -2)
    W = np.tile(np.arange(16, dtype=np.float16) * np.float16(0.5), (3, 16))
    assert torch.all(mx.channel_salience(dev(W), dev(make_grad(3, 256, 5, 1.0))) == 0)
    W = np.zeros((2, 128), np.float16)
    W[:, 1], W[:, 2] = 15.0, 7.25
    Gd = np.zeros((2, 128), np.float16)
    Gd[0, 2], Gd[1, 2] = 8.0, -8.0
    assert mx.channel_salience(dev(W), dev(Gd)).cpu().tolist() == [0.0, 4.0]


@pytest.mark.parametrize("case", ["ties", "random", "llama_stack"])
def test_global_selection_matches_the_oracle_exactly(case):
    rng = np.random.default_rng(17)
    if case == "ties":
        layers = [rng.integers(0, 5, n).astype(np.float32) * 0.125 for n in (7, 1, 300, 4096, 12, 1025)]
    elif case == "random":
        layers = [np.abs(rng.standard_normal(n)).astype(np.float32) * 10.0 ** rng.integers(-6, 3) for n in (6144, 4096, 28672, 4096)]
    else:   # 32 blocks of Llama-3-8B-shaped layers, lognormal saliences whose scale differs per layer
        layers = [np.exp(rng.standard_normal(n) + rng.standard_normal()).astype(np.float32)
                  for _ in range(32) for n in (6144, 4096, 28672, 4096)]
    total = sum(l.size for l in layers)
    dl = [dev(l) for l in layers]
    for T in sorted({0, 1, total // 10, total // 2 + 1, total - 1, total}):
        want = ref.select_salient(layers, T)
        got = mx.select_salient(dl, T)
        assert len(got) == len(want)
        for a, b in zip(got, want):
            assert np.array_equal(a.cpu().numpy(), b), (case, T)
    say(f"selection {case}: {len(layers)} layers, {total} channels")


@pytest.mark.parametrize("case", ["empty_layers", "many_layers", "one_value", "several_chunks_per_tile", "one_channel"])
def test_global_selection_at_tile_and_layer_edges(case):
    rng = np.random.default_rng(23)
    few = lambda n: rng.integers(0, 4, n).astype(np.float32)   # many channels share the threshold's value
    layers = {
        "empty_layers": [few(0), few(1023), few(0), few(0), few(1025), few(64), few(0)],
        "many_layers": [few(int(n)) for n in rng.integers(0, 9, 1500)],          # more layers than offsets kept in LDS
        "one_value": [np.full(n, 0.25, np.float32) for n in (1024, 2048, 5)],
        "several_chunks_per_tile": [few(1 << 20), few(1025), few(3)],            # more than 1024 chunks of 1024 keys
        "one_channel": [few(1)],
    }[case]
    total = sum(l.size for l in layers)
    dl = [dev(l) for l in layers]
    for T in sorted({0, 1, total // 3, total // 2 + 1, total}):
        for a, b in zip(mx.select_salient(dl, T), ref.select_salient(layers, T), strict=True):
            assert np.array_equal(a.cpu().numpy(), b), (case, T)


def test_precision_search_end_to_end_feeds_the_linear():
    # Alg. 1 on three synthetic layers, then the chosen channels go into the weight quantizer and the
    # linear is checked against the oracle run with the same choice
    shapes = [(512, 96), (1024, 272), (512, 530)]
    Ws = [synth.make_w(N, K, seed=50 + i, n_outlier_rows=6) for i, (K, N) in enumerate(shapes)]
    Gs = [make_grad(N, K, 60 + i, 0.3) for i, (K, N) in enumerate(shapes)]
    sal = [mx.channel_salience(dev(W), dev(Gd)) for W, Gd in zip(Ws, Gs)]
    T = round(0.10 * sum(N for _, N in shapes))
    chosen = mx.select_salient(sal, T)
    want = ref.select_salient([s.cpu().numpy() for s in sal], T)     # same fp32 saliences: same decision
    assert sum(len(c) for c in chosen) == T
    for (K, N), W, idx, idx_ref in zip(shapes, Ws, chosen, want):
        # the layer's slice of the selection goes into the weight quantizer where it lies, on the
        # device: nothing between the search and the linear crosses to the host
        PL = mx.quantize_weights(dev(W), idx)
        y = mx.linear(dev(synth.make_x(5, K, seed=70)), PL)
        assert np.array_equal(idx.cpu().numpy(), idx_ref)
        L = ref.quantize_weights(W, idx_ref)
        assert np.array_equal(PL.perm.cpu().numpy(), L.perm)
        xq, xs = ref.quantize_act(synth.make_x(5, K, seed=70))
        check_against_oracle(y.cpu().numpy(), xq, xs, L, ("search", K, N))
    say("precision search: 8-bit channels per layer", [len(c) for c in chosen])
