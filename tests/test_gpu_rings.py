"""The kernel whose waves keep private rings of gathered rows (csrc/spmm_rings.hip) against the CPU oracle, in all
four forms: fewest steps, odd and even counts of them (two groups share the steps), padded kept columns, ragged columns."""
import numpy as np
import pytest

import hinm_synth as synth
from oracle import hinm_oracle as orc
from tests.test_gpu_prepared import _check

RINGS = [20, 21, 22, 23]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [32, 64, 96, 128])
@pytest.mark.parametrize("Kv,N", [
    (136, 65),       # three steps, the last one mostly padding; one column of a second wave
    (256, 129),      # four steps: no step left over for the first group
    (320, 511),      # five: the last group has none in the last stage
    (424, 264),      # seven, padded; a column block of 8 columns
])
def test_rings(V, Kv, N, dtype):
    four = [24] if V == 128 and Kv >= 320 else []       # two stages of four steps, some of them without a step
    _check(synth.small_case(3 * V, 456, V, Kv, N, dtype, 91), N, RINGS + four, relu=(Kv == 256))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [32, 64, 96, 128])
@pytest.mark.parametrize("Kv,N", [
    (1480, 700),      # 24 steps, the last one padded; 256-column blocks two side by side, the third alone
    (2048, 129),      # 32; 128-column blocks of which the second holds one column
])
def test_rings_in_their_steady_state(V, Kv, N, dtype):
    """All slots of the rings of rows, stored values and row numbers are used several times (four groups of steps: six and
    eight stages), in every form."""
    _check(synth.small_case(3 * V, 2104, V, Kv, N, dtype, 96), N, RINGS + ([24] if V == 128 else []))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_rings_read_padding_as_zero_and_relu_clears_nan(dtype):
    """The rings of all units hold NaN when a layer with padded kept columns starts; NaN leaves the ReLU as +0."""
    import torch
    import paper_2407_20496_amd as hinm
    from tests import gpu_util as gu
    NAN = 0x7E00 if dtype == "f16" else 0x7FC0
    poison = synth.small_case(256 * 128, 512, 128, 256, 512, dtype, 92)
    W = torch.zeros((poison.M, poison.K), dtype=torch.int16, device=gu.DEV)
    nan = torch.full((poison.K, 512), NAN, dtype=torch.int16, device=gu.DEV)
    vb, nb, cb, wb = hinm.hinm_pack_sizes(poison.M, poison.K, 128, 256, dtype)
    vals = torch.empty(vb // 2, dtype=torch.int16, device=gu.DEV)
    nm = torch.empty(nb, dtype=torch.uint8, device=gu.DEV)
    vec = torch.empty(cb // 4, dtype=torch.int32, device=gu.DEV)
    work = torch.empty(wb // 8, dtype=torch.float64, device=gu.DEV)
    hinm.hinm_pack(poison.M, poison.K, 128, 256, dtype, W, vals, nm, vec, work, wb)
    size = hinm.hinm_prepare_sizes(poison.M, poison.K, 128, 256, dtype)
    prep = torch.empty(size, dtype=torch.uint8, device=gu.DEV)
    hinm.hinm_prepare(poison.M, poison.K, 128, 256, dtype, vals, nm, vec, None, None, prep, size)
    Y = torch.empty((poison.M, 512), dtype=torch.int16, device=gu.DEV)

    M, K, V, Kv, N = 64 * 64, 456, 64, 200, 512
    case = synth.small_case(M, K, V, Kv, N, dtype, 93)
    c_vals, c_nm, c_vec = orc.pack(case.weights(), dtype, V, Kv)
    pr = gu.gpu_prepare(gu.upload_packed(M, K, V, Kv, dtype, c_vals, c_nm, c_vec), case.pi_in(), case.pi_out())
    Xb = case.activations(N).copy()
    Xb[:, 7] = NAN                       # a column of NaN
    clean = Xb.copy()
    clean[:, 7] = 0
    acc = orc.product(orc.unpack_fast(c_vals, c_nm, c_vec, M, K, V), clean, dtype, case.pi_in(), case.pi_out())
    want = np.maximum(orc.decode(orc.round_to_storage(acc.astype(np.float32), dtype), dtype), 0)
    for variant in RINGS:
        hinm.hinm_spmm_prepared(poison.M, poison.K, 128, 256, dtype, 512, prep, nan, 512, Y, 512, variant << 16)
        bits = gu.gpu_spmm_prepared(pr, Xb, 1, variant)
        assert not bits[:, 7].any(), variant
        # both sides are rounded: half a unit of the last place apart from the accumulators, which differ by 1e-3 at most
        gu.check_close(orc.decode(bits, dtype), want, max_abs=1e-2 if dtype == "f16" else 2.0 ** -7 * np.abs(want).max(),
                       what="variant %d" % variant)


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["prepared", "vectors"])
@pytest.mark.parametrize("N,ldx,ldy", [(129, 200, 184), (700, 1024, 712), (264, 264, 1032)])
def test_rings_with_wider_leading_dimensions(form, N, ldx, ldy):
    """Columns of X beyond the promised extent hold NaN, and those of Y beyond N stay as they are."""
    from tests import gpu_util as gu
    import paper_2407_20496_amd as hinm
    case = synth.small_case(256, 456, 128, 328, N, "f16", 97)
    Xb = case.activations(N)
    wide = np.full((case.K, ldx), 0x7E00, dtype=np.uint16)
    wide[:, :N] = Xb
    pin, pout = case.pi_in(), case.pi_out()
    if form == "prepared":
        vals, nm, vec = orc.pack(case.weights(), "f16", 128, 328)
        pr = gu.gpu_prepare(gu.upload_packed(256, 456, 128, 328, "f16", vals, nm, vec), pin, pout)
        want = orc.product(orc.unpack_fast(vals, nm, vec, 256, 456, 128), Xb, "f16", pin, pout).astype(np.float64)
        X = gu.dev_bits(wide)
        run = lambda flags, v: gu.gpu_spmm_prepared(pr, Xb, flags, v, ldx=ldx, ldy=ldy, X_dev=X)
    else:
        p = gu.gpu_pack_vectors(case.weights(), "f16", 128, 328)
        want = gu.gpu_spmm_vectors(p, Xb, pin, pout, hinm.OUT_F32 | hinm.KERNEL_REFERENCE).astype(np.float64)
        run = lambda flags, v: gu.gpu_spmm_vectors(p, wide[:, :N], pin, pout, flags | v << 16, ldx=ldx, ldy=ldy)
    for variant in (RINGS + [24] if form == "prepared" else [20, 22, 23]):
        acc = run(hinm.OUT_F32, variant)
        gu.check_close(acc.astype(np.float64), want, what="variant %d" % variant)
        assert np.array_equal(run(0, variant), orc.round_to_storage(acc, "f16")), variant


@pytest.mark.gpu
@pytest.mark.parametrize("K,ldx", [
    (4095, 1 << 19),         # the last row ends at 4 GB: byte offsets use all 32 bits
    (4096, 400000),
])
def test_rings_with_inputs_of_more_than_2_gb(K, ldx):
    """Narrow products on a few columns of a wide matrix, against the same products on those columns alone, bit for bit."""
    import torch
    from tests import gpu_util as gu
    N, Kv = 200, 2040                # the last step is padded: row numbers of -1
    case = synth.small_case(256, K, 128, Kv, N, "bf16", 98)
    Xb, pin, pout = case.activations(N), case.pi_in(), case.pi_out()
    X = torch.empty((K, ldx), dtype=torch.int16, device=gu.DEV)
    X[:, :N] = gu.dev_bits(Xb)
    pr = gu.gpu_prepare(gu.gpu_pack(case.weights(), "bf16", 128, Kv), pin, pout)
    for variant in RINGS + [24]:
        want = gu.gpu_spmm_prepared(pr, Xb, 0, variant)
        assert want.any() and np.array_equal(gu.gpu_spmm_prepared(pr, Xb, 0, variant, ldx=ldx, X_dev=X), want), variant
    p = gu.gpu_pack_vectors(case.weights(), "bf16", 128, Kv)
    import paper_2407_20496_amd as hinm
    pins = gu.dev_i32(pin), gu.dev_i32(pout)
    for variant in (20, 22, 23):
        want = gu.gpu_spmm_vectors(p, Xb, pin, pout, variant << 16)
        Y = torch.zeros((256, N), dtype=torch.int16, device=gu.DEV)
        hinm.hinm_spmm_vectors(256, K, 128, Kv, "bf16", N, p.vals_v, p.vec_idx, *pins, X, ldx, Y, N, variant << 16)
        torch.cuda.synchronize()
        assert want.any() and np.array_equal(gu.host_bits(Y), want), variant


@pytest.mark.gpu
def test_staged_tile_kernel_beyond_4_gb():
    """What rings cannot address runs on the staged kernel, here as whole rounds of wide blocks and a remainder behind them."""
    import torch
    import paper_2407_20496_amd as hinm
    from tests import gpu_util as gu
    M, K, V, Kv, N, ldx = 2752, 4096, 32, 576, 2048, (1 << 19) + 8
    text, launches = hinm.hinm_spmm_prepared_plan(M, K, V, Kv, "f16", N, ldx, N)
    assert launches == 2 and text.count("spmm_tile_prepared_kernel<") == 2, text
    case = synth.small_case(M, K, V, Kv, N, "f16", 99)
    Xb = case.activations(N)
    X = torch.empty((K, ldx), dtype=torch.int16, device=gu.DEV)
    X[:, :N] = gu.dev_bits(Xb)
    pr = gu.gpu_prepare(gu.gpu_pack(case.weights(), "f16", V, Kv), case.pi_in(), case.pi_out())
    want = gu.gpu_spmm_prepared(pr, Xb, 2, 16)          # wide blocks alone, on the columns alone
    got = gu.gpu_spmm_prepared(pr, Xb, 2, 0, ldx=ldx, X_dev=X)
    gu.check_close(got.astype(np.float64), want.astype(np.float64), what="two launches")
    assert np.array_equal(gu.gpu_spmm_prepared(pr, Xb, 0, 0, ldx=ldx, X_dev=X), orc.round_to_storage(got, "f16"))


@pytest.mark.parametrize("M,K,V,Kv,N,form", [
    (4096, 11008, 128, 5504, 2048, "NB=256,NWK=2"),     # one round of 256-column blocks
    (16384, 16384, 128, 8192, 8192, "NB=512,NWK=1"),
    (4096, 4096, 64, 2048, 1024, "NB=256,NWK=2"),
    (4096, 4096, 128, 2048, 1024, "NB=128,NWK=2"),
    (11008, 4096, 128, 2048, 100, "RB=2,NB=128,NWK=4"),  # halves of tiles, four groups of steps
    (4096, 4096, 128, 2048, 256, "SRC=0"),              # the small blocks of the other kernel are ahead
])
def test_form_by_shape(M, K, V, Kv, N, form):
    import paper_2407_20496_amd as hinm
    ld = (N + 7) // 8 * 8
    text, n = hinm.hinm_spmm_prepared_plan(M, K, V, Kv, "bf16", N, ld, ld)
    assert n == 1 and form in text, text
    assert text.startswith("spmm_mid_kernel<" if form == "SRC=0" else "spmm_rings_kernel<"), text


@pytest.mark.parametrize("M,K,Kv,N,form", [
    (9856, 2864, 720, 288, "NB=256,NWK=1"),       # 924 workgroups of 128 columns are four rounds, not two
    (2880, 5888, 2944, 256, "NB=128,NWK=2"),      # 180 of them one short round
    (12640, 13784, 1720, 96, "NB=128,NWK=2"),     # 395: two rounds, half of what the 16-row kernel takes
    (11584, 2240, 1120, 352, "NB=256,NWK=1"),     # no launch of its own for a short remainder
    (6336, 12368, 1544, 4704, "NB=512,NWK=1"),    # few of many rows
])
def test_form_of_32_row_tiles(M, K, Kv, N, form):
    """A unit's LDS holds one workgroup of 128 columns (82944 of 163840 bytes), not two."""
    import paper_2407_20496_amd as hinm
    ld = (N + 7) // 8 * 8
    text, n = hinm.hinm_spmm_prepared_plan(M, K, 32, Kv, "f16", N, ld, ld)
    assert n == 1 and "RB=1," + form in text and "private rings" in text, text
    text, _ = hinm.hinm_spmm_prepared_plan(M, K, 32, Kv, "f16", N, ld, ld, flags=23 << 16)
    assert 2 * int(text.split("lds=")[1]) > 160 * 1024


def test_rings_leave_what_they_cannot_address():
    """Byte offsets into X are 32 bits wide: beyond, and below three steps, the staged tile kernel runs."""
    import paper_2407_20496_amd as hinm
    for K, Kv, N in ((65536, 1024, 32768), (256, 128, 4096)):
        text, _ = hinm.hinm_spmm_prepared_plan(4096, K, 128, Kv, "bf16", N, N, N)
        assert "private rings" not in text, text
        with pytest.raises(hinm.HinmError) as err:
            hinm.hinm_spmm_prepared_plan(4096, K, 128, Kv, "bf16", N, N, N, flags=20 << 16)
        assert err.value.status == 5
    text, _ = hinm.hinm_spmm_prepared_plan(4096, 65528, 128, 1024, "bf16", 32760, 32760, 32760)
    assert "private rings" in text


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [32, 64, 96, 128])
@pytest.mark.parametrize("Kv,N,orders", [
    (136, 65, True), (256, 129, False), (320, 511, True), (424, 264, False),
])
def test_rings_before_2_4(V, Kv, N, orders, dtype):
    """The same edges on the dense stored values: row numbers looked up on the way, or taken as they are."""
    from tests import gpu_util as gu
    import paper_2407_20496_amd as hinm
    case = synth.small_case(3 * V, 456, V, Kv, N, dtype, 94)
    p = gu.gpu_pack_vectors(case.weights(), dtype, V, Kv)
    pin, pout = (case.pi_in(), case.pi_out()) if orders else (None, None)
    Xb = case.activations(N)
    want = gu.gpu_spmm_vectors(p, Xb, pin, pout, hinm.OUT_F32 | hinm.KERNEL_REFERENCE).astype(np.float64)
    for variant in RINGS:
        if variant == 21 and V > 64:
            with pytest.raises(hinm.HinmError):
                gu.gpu_spmm_vectors(p, Xb, pin, pout, variant << 16)
            continue
        got = gu.gpu_spmm_vectors(p, Xb, pin, pout, hinm.OUT_F32 | variant << 16)
        gu.check_close(got.astype(np.float64), want, what="variant %d" % variant)
        bits = gu.gpu_spmm_vectors(p, Xb, pin, pout, variant << 16)
        assert np.array_equal(bits, orc.round_to_storage(got, dtype)), variant


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [32, 64, 96, 128])
@pytest.mark.parametrize("Kv,N", [
    (1096, 700),      # 18 steps, the last one padded: row numbers of most stages come through the loop's own chain
    (1280, 264),      # 20 whole ones
])
def test_rings_before_2_4_in_their_steady_state(V, Kv, N, dtype):
    """Vector indexes and channel order are followed inside the loop (from the sixth stage on; two groups have nine and ten)."""
    from tests import gpu_util as gu
    import paper_2407_20496_amd as hinm
    case = synth.small_case(2 * V, 1400, V, Kv, N, dtype, 100)
    p = gu.gpu_pack_vectors(case.weights(), dtype, V, Kv)
    Xb, pin, pout = case.activations(N), case.pi_in(), case.pi_out()
    want = gu.gpu_spmm_vectors(p, Xb, pin, pout, hinm.OUT_F32 | hinm.KERNEL_REFERENCE).astype(np.float64)
    for variant in RINGS:
        if variant == 21 and V > 64:
            continue
        got = gu.gpu_spmm_vectors(p, Xb, pin, pout, hinm.OUT_F32 | variant << 16)
        gu.check_close(got.astype(np.float64), want, what="variant %d" % variant)
        bits = gu.gpu_spmm_vectors(p, Xb, pin, pout, variant << 16)
        assert np.array_equal(bits, orc.round_to_storage(got, dtype)), variant


@pytest.mark.gpu
@pytest.mark.parametrize("M,V,Kv,N", [
    (1536, 64, 1096, 1000),      # 384 blocks of 64 x 64: the rings by estimate
    (768, 128, 1000, 2500),      # padded steps, beyond the line of the kernel for a moderate number of columns
])
def test_layers_before_2_4_run_on_rings_by_shape(M, V, Kv, N):
    """No pinned form: the result is one of the forms', bit for bit."""
    from tests import gpu_util as gu
    import paper_2407_20496_amd as hinm
    assert hinm.hinm_calib_mid_plan(M, 2200, V, Kv, "f16", N, 1) == ""
    case = synth.small_case(M, 2200, V, Kv, N, "f16", 101)
    p = gu.gpu_pack_vectors(case.weights(), "f16", V, Kv)
    Xb, pin, pout = case.activations(N), case.pi_in(), case.pi_out()
    want = gu.gpu_spmm_vectors(p, Xb, pin, pout, hinm.OUT_F32 | hinm.KERNEL_REFERENCE).astype(np.float64)
    got = gu.gpu_spmm_vectors(p, Xb, pin, pout, hinm.OUT_F32)
    gu.check_close(got.astype(np.float64), want, what="by shape")
    forms = [gu.gpu_spmm_vectors(p, Xb, pin, pout, hinm.OUT_F32 | v << 16) for v in RINGS if v != 21 or V <= 64]
    assert any(np.array_equal(got, f) for f in forms)


@pytest.mark.gpu
def test_rings_before_2_4_ignore_rows_of_padding():
    """NaN in a row of X that no kept column names does not reach the result, wherever padding happens to look."""
    from tests import gpu_util as gu
    import paper_2407_20496_amd as hinm
    case = synth.small_case(64, 456, 64, 200, 130, "f16", 95)
    p = gu.gpu_pack_vectors(case.weights(), "f16", 64, 200)
    Xb = case.activations(130).copy()
    Xb[[r for r in range(456) if r not in set(p.vec_idx.cpu().numpy().ravel().tolist())]] = 0x7E00
    want = gu.gpu_spmm_vectors(p, Xb, None, None, hinm.OUT_F32 | hinm.KERNEL_REFERENCE).astype(np.float64)
    assert np.isfinite(want).all()
    for variant in RINGS:
        got = gu.gpu_spmm_vectors(p, Xb, None, None, hinm.OUT_F32 | variant << 16)
        gu.check_close(got.astype(np.float64), want, what="variant %d" % variant)


def test_four_groups_need_two_stages_and_two_halves():
    import paper_2407_20496_amd as hinm
    for V, Kv, ok in ((128, 264, True), (128, 256, False), (64, 512, False)):
        if ok:
            assert "NWK=4" in hinm.hinm_spmm_prepared_plan(512, 600, V, Kv, "f16", 200, 200, 200, flags=24 << 16)[0]
            continue
        with pytest.raises(hinm.HinmError) as err:
            hinm.hinm_spmm_prepared_plan(512, 600, V, Kv, "f16", 200, 200, 200, flags=24 << 16)
        assert err.value.status == 5
