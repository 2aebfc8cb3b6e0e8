"""GPU parity of the device-tuned path (hinm_prepare + hinm_spmm_prepared) against the CPU oracle,
and of the prepared buffer against the canonical arrays it re-orders."""
import numpy as np
import pytest

import hinm_synth as synth
from oracle import hinm_oracle as orc

pytestmark = pytest.mark.gpu

OUT_F32, RELU = 2, 1
VARIANTS = [0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 13, 14, 16, 17, 15]   # 13, 14, 16, 17 = 32-column waves; 15 = LDS-resident panel kernel (small K only)


def _ulp_bf16(y):
    e = np.floor(np.log2(np.maximum(np.abs(y), 2.0 ** -14)))
    return np.exp2(e - 7)


def _unswizzle(buf: np.ndarray, M, K, V, Kv):
    """Decode the prepared buffer (layout documented in csrc/prepared_layout.h) back into the
    canonical arrays plus the gather table and output rows."""
    T, RB = M // V, V // 32
    Kp = (Kv + 63) // 64 * 64
    S = Kp // 64
    al = lambda x: (x + 255) // 256 * 256
    a_bytes = T * S * RB * 2304
    g_off = al(a_bytes)
    o_off = g_off + al(T * Kp * 4)
    z_off = o_off + al(M * 4)
    blocks = buf[:a_bytes].reshape(T, S, RB, 2304)
    vals_u16 = blocks[..., :2048].copy().view(np.uint16).reshape(T, S, RB, 2, 64, 8)
    idx_u32 = blocks[..., 2048:].copy().view(np.uint32).reshape(T, S, RB, 64)
    G = Kp // 4
    vals = np.zeros((M, G * 2), dtype=np.uint16)
    nib = np.zeros((M, G), dtype=np.uint8)
    for lane in range(64):
        i, qa = lane % 32, lane // 32
        for sub in range(2):
            for k in range(4):
                # group 16 s + 8 sub + 4 qa + k of row 32 rb + i
                for s in range(S):
                    g = 16 * s + 8 * sub + 4 * qa + k
                    rows = (np.arange(T)[:, None] * V + 32 * np.arange(RB)[None, :] + i).reshape(-1)
                    vals[rows, 2 * g] = vals_u16[:, s, :, sub, lane, 2 * k].reshape(-1)
                    vals[rows, 2 * g + 1] = vals_u16[:, s, :, sub, lane, 2 * k + 1].reshape(-1)
                    nib[rows, g] = ((idx_u32[:, s, :, lane] >> (16 * sub + 4 * k)) & 0xF).reshape(-1)
    gather = buf[g_off:g_off + T * Kp * 4].copy().view(np.int32).reshape(T, Kp)
    out_rows = buf[o_off:o_off + M * 4].copy().view(np.int32)
    zeros = buf[z_off:z_off + 1024]
    panel = buf[z_off + 1024:z_off + 1024 + T * Kp * 4].copy().view(np.uint32).reshape(T, Kp)
    K8 = (K + 7) // 8 * 8
    g = gather.astype(np.int64)
    want_panel = np.where(g >= 0, (g << 7) | ((g & 2) << 5), K8 << 7).astype(np.uint32)
    assert np.array_equal(panel, want_panel), "LDS-address form of the gather table"
    return vals, nib, gather, out_rows, zeros


@pytest.mark.parametrize("M,K,V,Kv,dtype", [(128, 256, 32, 128, "f16"), (256, 320, 128, 200, "bf16"),
                                            (192, 256, 96, 64, "f16")])
def test_prepared_buffer_is_a_reordering(M, K, V, Kv, dtype):
    from tests import gpu_util as gu
    case = synth.small_case(M, K, V, Kv, 8, dtype, 80)
    vals, nm, vec = orc.pack(case.weights(), dtype, V, Kv)
    p = gu.upload_packed(M, K, V, Kv, dtype, vals, nm, vec)
    pin, pout = case.pi_in(), case.pi_out()
    pr = gu.gpu_prepare(p, pin, pout)
    v2, nib, gather, out_rows, zeros = _unswizzle(pr.buf.cpu().numpy(), M, K, V, Kv)
    G = Kv // 4
    assert np.array_equal(v2[:, :2 * G], vals)
    assert np.all(v2[:, 2 * G:] == 0)
    want_nib = np.stack([nm & 0xF, nm >> 4], axis=-1).reshape(M, G)
    assert np.array_equal(nib[:, :G], want_nib)
    assert np.all(nib[:, G:] == 0x4)
    assert np.array_equal(gather[:, :Kv], pin[vec])
    assert np.all(gather[:, Kv:] == -1)
    assert np.array_equal(out_rows, pout)
    assert np.all(zeros == 0)
    pr = gu.gpu_prepare(p, None, None)
    _, _, gather, out_rows, _ = _unswizzle(pr.buf.cpu().numpy(), M, K, V, Kv)
    assert np.array_equal(gather[:, :Kv], vec) and np.array_equal(out_rows, np.arange(M))


def _check(case, N, variants, relu=False, identity=False):
    from tests import gpu_util as gu
    vals, nm, vec = orc.pack(case.weights(), case.dtype, case.V, case.Kv)
    Wh = orc.unpack_fast(vals, nm, vec, case.M, case.K, case.V)
    Xb = case.activations(N)
    pin = None if identity else case.pi_in()
    pout = None if identity else case.pi_out()
    Y_acc = orc.product(Wh, Xb, case.dtype, pin, pout, relu=relu).astype(np.float64)
    p = gu.upload_packed(case.M, case.K, case.V, case.Kv, case.dtype, vals, nm, vec)
    pr = gu.gpu_prepare(p, pin, pout)
    f = RELU if relu else 0
    import paper_2407_20496_amd as hinm
    for v in variants:
        try:
            got32 = gu.gpu_spmm_prepared(pr, Xb, f | OUT_F32, variant=v).astype(np.float64)
        except hinm.HinmError as err:
            # the panel kernel refuses shapes whose panel does not fit in LDS; nothing else may refuse
            assert v == 15 and err.status == 5 and (((case.K + 7) // 8 * 8 + 8) * 128 + 8 * 32 * 144 > 160 * 1024 or N <= 32)
            continue
        gu.check_close(got32, Y_acc, what=f"{case.name} variant {v} fp32")
        got = gu.gpu_spmm_prepared(pr, Xb, f, variant=v)
        assert np.array_equal(got, orc.round_to_storage(got32.astype(np.float32), case.dtype)), f"variant {v}"
        if case.dtype == "f16":
            gu.check_close(orc.decode(got, "f16"), Y_acc, what=f"{case.name} variant {v} fp16")
        else:
            want = orc.decode(orc.round_to_storage(Y_acc.astype(np.float32), "bf16"), "bf16")
            gotd = orc.decode(got, "bf16")
            assert np.all(np.abs(gotd - want) <= np.maximum(1e-2, _ulp_bf16(want)))
            gu.check_close(gotd, want, max_abs=np.inf, what=f"{case.name} variant {v} bf16")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,K,V,Kv,N", [
    (128, 256, 32, 128, 37),
    (128, 320, 64, 160, 300),     # ragged column tail inside the second 256-column block
    (384, 512, 128, 256, 520),    # ragged tail past one 512-column block
    (192, 256, 96, 64, 40),
    (128, 512, 64, 200, 72),      # Kv % 64 != 0: padded kept columns
    (256, 1024, 128, 704, 256),   # 11 steps: odd number of 64-column steps
])
def test_prepared_small_all_variants(M, K, V, Kv, N, dtype):
    _check(synth.small_case(M, K, V, Kv, N, dtype, 81), N, VARIANTS)


@pytest.mark.parametrize("M,K,V,Kv,N,dtype", [
    (2752, 1152, 32, 576, 2048, "f16"),      # 86 tiles x 4 wide blocks: one launch of 256-column blocks is estimated ahead
    (11008, 1152, 128, 576, 2048, "bf16"),   # 64 tiles in wide blocks, 22 in narrow ones
    (5504, 1280, 64, 640, 1500, "f16"),      # 86 tiles x 3 wide blocks (ragged last block): 85 + 1
])
def test_prepared_remainder_tiles_in_a_second_launch(M, K, V, Kv, N, dtype):
    """Layers whose wide blocks make whole rounds plus a small remainder are launched in two parts (the staged tile kernel,
    pinned here, in one)."""
    import paper_2407_20496_amd as hinm
    ld = (N + 7) // 8 * 8
    text, launches = hinm.hinm_spmm_prepared_plan(M, K, V, Kv, dtype, N, ld, ld)
    assert launches == (1 if V == 32 else 2) and text.count("spmm_rings_kernel<") == launches, text
    _check(synth.small_case(M, K, V, Kv, N, dtype, 83), N, [0, 3, 16])


def test_prepared_relu_identity():
    case = synth.small_case(128, 256, 64, 128, 72, "f16", 82)
    _check(case, 72, [0, 2, 3], relu=True)
    _check(case, 72, [0, 2, 3], identity=True)


def test_prepared_c2_full():
    c = synth.c2()
    _check(c, c.N, [0, 1, 3, 8, 15])


def test_prepared_panel_kernel_edges():
    # K not a multiple of 8, ragged N, padded kept columns, one tile per wave and fewer tiles than waves
    _check(synth.small_case(64, 100, 32, 40, 70, "f16", 85), 70, [15])
    _check(synth.small_case(96, 1000, 32, 504, 130, "bf16", 86), 130, [15], relu=True)
    _check(synth.small_case(64, 512, 64, 256, 64, "f16", 87), 64, [15], identity=True)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,K,V,Kv,N", [
    (128, 256, 32, 128, 1),
    (256, 1024, 128, 704, 16),    # several workgroups per tile, odd number of steps
    (128, 2048, 64, 1032, 3),     # padded kept columns (Kv % 64 != 0)
    (192, 512, 96, 256, 17),
    (256, 4096, 128, 2048, 32),
    (128, 512, 128, 64, 8),       # a single step: no split
    (64, 4224, 32, 2200, 1),      # one column, more than 32 steps: the input vector is staged in LDS; padded steps
    (64, 4220, 32, 2112, 1),      # K % 8 != 0: same shape class without staging
    (32, 12288, 32, 8192, 1),     # 128 steps over 16 waves: the 16-row kernel stages the input vector as well
])
def test_prepared_few_columns(M, K, V, Kv, N, dtype):
    # 0 = by shape, 11 = 16-row workgroups (16x16x64 form), 12 = 32-row workgroups (32x32x32 form)
    _check(synth.small_case(M, K, V, Kv, N, dtype, 83), N, [0, 11, 12])


@pytest.mark.parametrize("M,K,V,Kv,N,dtype", [
    (128, 320, 64, 160, 300, "f16"),      # many column blocks, ragged tail, padded kept columns
    (192, 256, 96, 64, 40, "bf16"),       # a single step; 96-row tiles: three 32-row blocks
    (256, 8192, 128, 4416, 16, "bf16"),   # 69 steps: sixteen waves with more than one batch
    (8192, 256, 64, 128, 13, "f16"),      # 256 row blocks of 32: both halves of a block in one workgroup
    # many workgroups: fewer waves each, several batches per wave
    (4096, 1024, 128, 512, 136, "bf16"),  # 2304 workgroups: one wave walks all 8 steps
    (2048, 2304, 128, 1152, 72, "f16"),   # 640 workgroups: two waves, 9 steps each
    (8192, 512, 64, 384, 88, "bf16"),     # 1536 workgroups of 32 rows: one wave, 6 steps in two batches
    (512, 4608, 32, 2304, 392, "f16"),    # 36 steps, two column blocks per workgroup, ragged last block of 8
    (4096, 2048, 128, 1024, 72, "bf16"),  # 64-row workgroups with two column blocks; the last pair holds 8 columns
    (4096, 2048, 128, 1024, 200, "f16"),  # 64-row workgroups with four column blocks; the last four hold 8 columns
    (2048, 2304, 32, 1152, 136, "bf16"),  # 32-row tiles, four column blocks, 18 steps
])
def test_prepared_sixteen_row_kernel_beyond_few_columns(M, K, V, Kv, N, dtype):
    _check(synth.small_case(M, K, V, Kv, N, dtype, 88), N, [11])
    _check(synth.small_case(M, K, V, Kv, N, dtype, 89), N, [11], relu=True, identity=True)


def test_prepared_few_columns_on_a_large_layer_and_garbage_in_the_padding():
    """Up to 64 columns go to the 16-row kernel when the layer is large; columns of X beyond N (inside the
    leading dimension) may hold anything."""
    import torch
    from tests import gpu_util as gu
    case = synth.small_case(4096, 2048, 128, 1024, 40, "f16", 90)
    _check(case, 40, [0, 11])
    _padding_may_hold_anything(synth.small_case(256, 1024, 64, 512, 19, "bf16", 91), 19, 24, (0, 11, 12))
    # two column blocks per workgroup: the second pair covers columns 32..47 of the row and nothing beyond
    _padding_may_hold_anything(synth.small_case(2048, 2304, 128, 1152, 40, "f16", 92), 40, 48, (0, 11))


def _padding_may_hold_anything(case, N, ld, variants):
    from tests import gpu_util as gu
    p = gu.gpu_pack(case.weights(), case.dtype, case.V, case.Kv)
    pr = gu.gpu_prepare(p, case.pi_in(), case.pi_out())
    Xb = case.activations(N)
    Xp = np.full((case.K, ld), 0x7FC0, dtype=np.uint16)     # NaN in every padding column
    Xp[:, :N] = Xb
    for variant in variants:
        want = gu.gpu_spmm_prepared(pr, Xb, variant=variant, ldx=ld, ldy=ld)
        got = gu.gpu_spmm_prepared(pr, Xb, variant=variant, ldx=ld, ldy=ld, X_dev=gu.dev_bits(Xp))
        assert np.array_equal(got, want), f"variant {variant}"


@pytest.mark.parametrize("M,K,V,Kv,dtype", [
    (256, 512, 64, 256, "f16"),       # four steps: one wave per step
    (384, 1000, 128, 504, "bf16"),    # K % 32 != 0, Kv % 64 != 0: clamped copies, padded kept columns
    (128, 4096, 128, 2048, "f16"),    # 32 steps: the largest input that fits beside eight slabs
    (192, 2048, 64, 1024, "bf16"),
    (128, 256, 64, 128, "f16"),       # two steps, 8 KB of input rows: the waves' partial tiles (16 KB) need more LDS
    (128, 640, 128, 576, "bf16"),     # nine steps over four waves, 20 KB of input rows
])
def test_prepared_sixteen_columns_input_resident_in_lds(M, K, V, Kv, dtype):
    case = synth.small_case(M, K, V, Kv, 16, dtype, 86)
    _check(case, 16, [0, 11, 19])
    _check(case, 16, [19], relu=True)
    _check(case, 16, [19], identity=True)


def test_prepared_input_resident_variant_refuses_what_it_cannot_hold():
    import paper_2407_20496_amd as hinm
    from tests import gpu_util as gu
    for (M, K, V, Kv, N) in [(128, 8192, 128, 4096, 16),    # 256 KB of input rows
                             (128, 512, 32, 256, 16),       # V % 64 != 0
                             (128, 512, 64, 256, 8)]:       # not 16 columns
        case = synth.small_case(M, K, V, Kv, N, "f16", 87)
        p = gu.gpu_pack(case.weights(), "f16", V, Kv)
        pr = gu.gpu_prepare(p, case.pi_in(), case.pi_out())
        with pytest.raises(hinm.HinmError) as err:
            gu.gpu_spmm_prepared(pr, case.activations(N), variant=19)
        assert err.value.status == 5


def test_prepared_few_columns_repeatable_and_needs_no_workspace():
    # partial tiles are added in a fixed order: repeated calls give identical bits
    import torch
    from tests import gpu_util as gu
    import paper_2407_20496_amd as hinm
    case = synth.small_case(256, 2048, 128, 1024, 16, "bf16", 84)
    vals, nm, vec = orc.pack(case.weights(), "bf16", 128, 1024)
    p = gu.upload_packed(256, 2048, 128, 1024, "bf16", vals, nm, vec)
    pr = gu.gpu_prepare(p, case.pi_in(), case.pi_out())
    assert hinm.hinm_spmm_prepared_workspace(256, 2048, 128, 1024, "bf16", 16) == 0
    Xd = gu.dev_bits(case.activations())
    outs = []
    for _ in range(3):
        Y = torch.zeros((256, 16), dtype=torch.int16, device=gu.DEV)
        hinm.hinm_spmm_prepared(256, 2048, 128, 1024, "bf16", 16, pr.buf, Xd, 16, Y, 16, 0, None, 0)
        torch.cuda.synchronize()
        outs.append(gu.host_bits(Y))
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])
    Wh = orc.unpack_fast(vals, nm, vec, 256, 2048, 128)
    want = orc.product(Wh, case.activations(), "bf16", case.pi_in(), case.pi_out()).astype(np.float64)
    got = orc.decode(outs[0], "bf16")
    assert np.all(np.abs(got - want) <= np.maximum(1e-2, _ulp_bf16(want)))


@pytest.mark.parametrize("idx", [0, 1, 3, 4, 6, 7, 9, 10])
def test_prepared_c3_decode_full(idx):
    c = synth.c3_cases()[idx]
    assert c.N in (1, 16)
    _check(c, c.N, [0])


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("N", [1, 5, 16])
@pytest.mark.parametrize("Kv", [2056, 2112, 3072])
def test_sixteen_row_kernel_with_33_to_48_steps(Kv, N, dtype):
    """Eight waves: one step beyond 32 (the last one padded), whole ones, and the longest pass."""
    import paper_2407_20496_amd as hinm
    M, K, V = 96, 3080, 32
    ld = N if N == 1 else (N + 7) // 8 * 8
    assert "NW=8," in hinm.hinm_spmm_prepared_plan(M, K, V, Kv, dtype, N, ld, ld, 0)[0]
    _check(synth.small_case(M, K, V, Kv, N, dtype, 79), N, [0])


def test_tile_kernel_parts_run_and_store_nothing():
    """The measurement launches (copy stream alone, LDS reads and MFMAs alone) finish, leave X and the prepared
    layer as they were, and the product launched afterwards on the same buffers is still right."""
    import torch
    import paper_2407_20496_amd as hinm
    from tests import gpu_util as gu
    # the staged tile kernel's parts; the whole products run on private rings
    shapes = [(4096, 1024, 128, 512, 1100, "bf16"), (2048, 2048, 64, 512, 2056, "f16")]
    for (M, K, V, Kv, N, dtype) in shapes:
        ld = (N + 7) // 8 * 8
        assert "spmm_rings_kernel" in hinm.hinm_spmm_prepared_plan(M, K, V, Kv, dtype, N, ld, ld, 0)[0]
        case = synth.small_case(M, K, V, Kv, N, dtype, 77)
        vals, nm, vec = orc.pack(case.weights(), case.dtype, V, Kv)
        p = gu.upload_packed(M, K, V, Kv, dtype, vals, nm, vec)
        pr = gu.gpu_prepare(p, case.pi_in(), case.pi_out())
        prep = pr.buf
        ld = (N + 7) // 8 * 8
        Xh = np.zeros((K, ld), dtype=np.uint16)
        Xh[:, :N] = case.activations(N)
        X = torch.from_numpy(Xh.view(np.int16)).cuda()
        before_x, before_p = X.clone(), prep.clone()
        for part in (1, 2):
            hinm.hinm_calib_tile_part(M, K, V, Kv, dtype, N, prep, X, ld, part)
        torch.cuda.synchronize()
        assert torch.equal(X, before_x) and torch.equal(prep, before_p)
    with pytest.raises(hinm.HinmError):     # a shape served by another kernel has no tile-kernel parts
        hinm.hinm_calib_tile_part(256, 512, 64, 256, "f16", 520, prep, X, 520, 1)
    _check(synth.small_case(2048, 2048, 64, 512, 2056, "f16", 77), 2056, [0])


@pytest.mark.parametrize("forms", ["prepared", "canonical", "mixed"])
def test_chain_of_one_column(forms):
    """The intermediate of a chain at one column, long enough for the second layer to stage it in LDS, against the oracle and
    against the two calls on their own."""
    import torch
    import paper_2407_20496_amd as hinm
    from tests import gpu_util as gu
    RELU, dtype, V = 1, "bf16", 64
    shapes = [(8448, 64, 64), (64, 8448, 4232)]     # M, K, Kv: 67 steps in the second layer, the last one ragged
    layers, calls, keep, h = [], [], [], None
    for l, (M, K, Kv) in enumerate(shapes):
        case = synth.small_case(M, K, V, Kv, 1, dtype, 120 + l)
        p = gu.gpu_pack(case.weights(), dtype, V, Kv)
        vals, nm, vec = orc.pack(case.weights(), dtype, V, Kv)
        pin, pout, relu = case.pi_in(), case.pi_out(), RELU if l == 0 else 0
        form = forms if forms != "mixed" else ("canonical", "prepared")[l]
        pr = gu.gpu_prepare(p, pin, pout) if form == "prepared" else None
        if l == 0:
            Xb = h = case.activations()
        run = (lambda x, flags: gu.gpu_spmm_prepared(pr, x, flags)) if pr is not None else (
            lambda x, flags: gu.gpu_spmm(p, x, pin, pout, flags))
        want = orc.product(orc.unpack_fast(vals, nm, vec, M, K, V), h, dtype, pin, pout, relu=bool(relu))
        acc = run(h, relu | 2)
        gu.check_close(acc.astype(np.float64), want.astype(np.float64), what="layer %d on its own" % l)
        h = run(h, relu)
        assert np.array_equal(h, orc.round_to_storage(acc, dtype))
        pi = (gu.dev_i32(pin), gu.dev_i32(pout))
        keep.append((p, pr, pi))
        layers.append(hinm.Layer(M, K, V, Kv, dtype, p.vals, p.nm_idx, p.vec_idx, pi[0], pi[1], relu,
                                 pr.buf if pr is not None else None))
    nbytes = hinm.hinm_chain_sizes(layers, 1)
    scratch = torch.full((nbytes,), 0x7B, dtype=torch.uint8, device=gu.DEV)
    Y = torch.full((64, 1), 0x7B7B, dtype=torch.int16, device=gu.DEV)
    hinm.hinm_chain(layers, 1, gu.dev_bits(Xb), 1, Y, 1, scratch, nbytes)
    torch.cuda.synchronize()
    assert np.array_equal(gu.host_bits(Y), h.reshape(64, 1))


def test_chain_of_ten_layers():
    """More layers than a chain keeps routes of (eight): every layer as its own call, bit for bit."""
    import torch
    import paper_2407_20496_amd as hinm
    from tests import gpu_util as gu
    dtype, N, RELU = "bf16", 72, 1       # every layer scales by about a tenth: ten of them leave the range of f16
    sizes = [96, 64, 128, 64, 192, 64, 64, 128, 96, 64, 160]      # K of layer l, M of layer l - 1
    layers, h, keep = [], None, []
    for l in range(10):
        M, K = sizes[l + 1], sizes[l]
        case = synth.small_case(M, K, 32, K // 2, N, dtype, 140 + l)
        p = gu.gpu_pack(case.weights(), dtype, 32, K // 2)
        pr = gu.gpu_prepare(p, case.pi_in(), case.pi_out())
        if l == 0:
            Xb = h = case.activations()
        flags = RELU if l % 2 == 0 else 0
        h = gu.gpu_spmm_prepared(pr, h, flags)
        keep.append(pr)
        layers.append(hinm.Layer(M, K, 32, K // 2, dtype, None, None, None, flags=flags, prepared=pr.buf))
    nbytes = hinm.hinm_chain_sizes(layers, N)
    scratch = torch.full((nbytes,), 0x7B, dtype=torch.uint8, device=gu.DEV)
    Y = torch.full((160, N), 0x7B7B, dtype=torch.int16, device=gu.DEV)
    hinm.hinm_chain(layers, N, gu.dev_bits(Xb), N, Y, N, scratch, nbytes)
    torch.cuda.synchronize()
    assert h.any() and np.array_equal(gu.host_bits(Y), h)


def _rows16_form(c, N, variant=11):
    """What the 16-row kernel is launched with: waves, steps of a batch, 16-row blocks, and how it reads X (2: gathers of one
    column, 3: that column staged in LDS)."""
    import paper_2407_20496_amd as hinm
    ld = N if N == 1 else (N + 7) // 8 * 8
    text, launches = hinm.hinm_spmm_prepared_plan(c.M, c.K, c.V, c.Kv, c.dtype, N, ld, ld, variant << 16)
    assert launches == 1 and text.startswith("spmm_rows16_prepared_kernel<"), text
    form = dict(item.split("=") for item in text[text.index("<") + 1:text.index(">")].split(","))
    return {k: int(v) for k, v in form.items()}


# steps: (waves, batch) of one column, of 2 to 16; three column blocks differ above 16 steps
WAVES_AND_BATCH = {
    1: ((4, 1), (4, 1)), 4: ((4, 1), (4, 1)), 5: ((4, 2), (8, 1)), 8: ((4, 2), (8, 1)), 9: ((8, 2), (8, 2)), 12: ((8, 2), (8, 2)),
    13: ((8, 2), (8, 2)), 16: ((8, 2), (8, 2)), 17: ((8, 3), (8, 3)), 24: ((8, 3), (8, 3)), 25: ((8, 4), (8, 4)),
    32: ((8, 4), (8, 4)), 33: ((8, 5), (8, 5)), 40: ((8, 5), (8, 5)), 41: ((8, 3), (8, 6)), 48: ((8, 3), (8, 6)),
    49: ((16, 4), (16, 4)), 64: ((8, 4), (16, 4)), 65: ((16, 3), (16, 6)), 96: ((16, 3), (16, 6)), 97: ((16, 3), (16, 4))}


@pytest.mark.parametrize("S", list(WAVES_AND_BATCH))
@pytest.mark.parametrize("N", [1, 6, 16, 40])
def test_waves_and_batches_of_the_16_row_kernel(S, N):
    """Waves and batches change at 4, 8, 12, 16, 24, 32, 40, 48, 64 and 96 steps; the last step is ragged."""
    c = synth.small_case(96, 64 * S + 8, 32, 64 * S - 24, N, "bf16" if S % 2 else "f16", 700 + S)
    form = _rows16_form(c, N)
    want = WAVES_AND_BATCH[S][N > 1] if N <= 16 or S <= 16 else (8, 4) if S <= 32 else (16, 4) if S <= 64 else (16, 6)
    assert (form["NW"], form["KB"], form["RBW"]) == (*want, 1), form
    assert form["XMODE"] == (1 if N > 1 else 3 if S > 4 * form["NW"] else 2), form
    _check(c, N, [0, 11], relu=S % 3 == 0)


@pytest.mark.parametrize("S,one,several", [(1, (4, 1), (4, 1)), (7, (4, 2), (8, 1)), (12, (8, 2), (8, 2)), (13, (4, 4), (4, 4)),
                                           (20, (8, 3), (8, 3))])
@pytest.mark.parametrize("N", [1, 9])
def test_waves_of_the_16_row_kernel_with_many_workgroups(S, one, several, N):
    """Both halves of a 32-row block in a workgroup (256 of them and more); above 12 steps the count of workgroups decides."""
    c = synth.small_case(8320, 64 * S, 64, 64 * S - 8, N, "f16", 720 + S)
    form = _rows16_form(c, N)
    assert (form["NW"], form["KB"]) == (several if N > 1 else one) and form["RBW"] == 2, form
    _check(c, N, [11])


@pytest.mark.parametrize("S,waves,batch", [(40, 8, 5), (41, 8, 6), (48, 8, 6), (49, 16, 4)])
def test_waves_of_the_16_row_kernel_with_128_workgroups(S, waves, batch):
    c = synth.small_case(2048, 64 * S, 32, 64 * S - 8, 11, "bf16", 742)
    form = _rows16_form(c, 11)
    assert (form["NW"], form["KB"], form["RBW"]) == (waves, batch, 1), form
    _check(c, 11, [11])


def test_eight_waves_on_long_layers_of_one_column():
    """More than 256 workgroups beyond 64 steps."""
    c = synth.small_case(4128, 64 * 66, 32, 64 * 66 - 8, 1, "bf16", 741)
    form = _rows16_form(c, 1)
    assert (form["NW"], form["KB"], form["RBW"], form["XMODE"]) == (8, 3, 1, 3), form
    _check(c, 1, [11])


@pytest.mark.parametrize("M,S,waves,batch", [(8192, 33, 8, 5), (8192, 40, 8, 5), (8192, 41, 8, 3), (8192, 48, 8, 3), (8192, 57, 8, 4),
                                             (8192, 64, 8, 4), (8192, 66, 16, 3), (8224, 52, 8, 4), (8224, 66, 8, 3)])
def test_both_halves_with_one_staged_column(M, S, waves, batch):
    """256 and 257 workgroups of 32 rows, the input vector in LDS."""
    c = synth.small_case(M, 64 * S, 32, 64 * S - 8, 1, "bf16" if S % 2 else "f16", 780 + S)
    form = _rows16_form(c, 1, 0)
    assert (form["NW"], form["KB"], form["RBW"], form["XMODE"]) == (waves, batch, 2, 3), form
    _check(c, 1, [0])


@pytest.mark.parametrize("M,S,rows", [(8224, 24, 2), (8224, 25, 1), (8224, 32, 1), (8224, 33, 2), (8192, 32, 2)])
def test_halves_of_one_batch_that_spread_more_evenly(M, S, rows):
    """One column, 25 to 32 steps: 514 workgroups of 16 rows rather than 257 of 32; 512 and 256 make one round each."""
    c = synth.small_case(M, 64 * S, 32, 64 * S - 8, 1, "f16", 790 + S)
    assert _rows16_form(c, 1, 0)["RBW"] == rows
    _check(c, 1, [0])


@pytest.mark.parametrize("K", [16384, 16392, 20480, 20488, 24560, 24568, 24576])
def test_vectors_of_up_to_six_pieces_a_thread(K):
    """Eight waves stage four pieces of 4096 elements, five or six; beyond 48 KB none."""
    c = synth.small_case(64, K, 32, 64 * 40 - 8, 1, "bf16", 750)
    form = _rows16_form(c, 1, 0)
    assert (form["NW"], form["XMODE"]) == (8, 3 if K <= 24568 else 2), form
    _check(c, 1, [0])


@pytest.mark.parametrize("S,K,N,waves,batch", [(49, 9216, 1, 16, 4), (56, 9216, 1, 16, 4), (56, 9224, 1, 8, 4), (57, 4096, 1, 8, 4),
                                               (64, 4096, 9, 16, 4), (128, 8192, 9, 16, 4), (129, 8256, 9, 16, 6), (193, 12352, 16, 16, 6)])
def test_waves_and_batches_of_long_layers(S, K, N, waves, batch):
    c = synth.small_case(64, K, 32, 64 * S - 8, N, "f16", 760)
    form = _rows16_form(c, N, 0)
    assert (form["NW"], form["KB"]) == (waves, batch), form
    _check(c, N, [0])
