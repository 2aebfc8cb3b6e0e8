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
def test_rings_read_padding_as_zero_and_relu_clears_nan():
    """The rings of all units hold NaN when a layer with padded kept columns starts; NaN and -0 leave the ReLU as +0."""
    import torch
    import paper_2407_20496_amd as hinm
    from tests import gpu_util as gu
    poison = synth.small_case(256 * 128, 512, 128, 256, 512, "f16", 92)
    W = torch.zeros((poison.M, poison.K), dtype=torch.int16, device=gu.DEV)
    nan = torch.full((poison.K, 512), 0x7E00, dtype=torch.int16, device=gu.DEV)
    vb, nb, cb, wb = hinm.hinm_pack_sizes(poison.M, poison.K, 128, 256, "f16")
    vals = torch.empty(vb // 2, dtype=torch.int16, device=gu.DEV)
    nm = torch.empty(nb, dtype=torch.uint8, device=gu.DEV)
    vec = torch.empty(cb // 4, dtype=torch.int32, device=gu.DEV)
    work = torch.empty(wb // 8, dtype=torch.float64, device=gu.DEV)
    hinm.hinm_pack(poison.M, poison.K, 128, 256, "f16", W, vals, nm, vec, work, wb)
    size = hinm.hinm_prepare_sizes(poison.M, poison.K, 128, 256, "f16")
    prep = torch.empty(size, dtype=torch.uint8, device=gu.DEV)
    hinm.hinm_prepare(poison.M, poison.K, 128, 256, "f16", vals, nm, vec, None, None, prep, size)
    Y = torch.empty((poison.M, 512), dtype=torch.int16, device=gu.DEV)

    M, K, V, Kv, N = 64 * 64, 456, 64, 200, 512
    case = synth.small_case(M, K, V, Kv, N, "f16", 93)
    c_vals, c_nm, c_vec = orc.pack(case.weights(), "f16", V, Kv)
    pr = gu.gpu_prepare(gu.upload_packed(M, K, V, Kv, "f16", c_vals, c_nm, c_vec), case.pi_in(), case.pi_out())
    Xb = case.activations(N).copy()
    Xb[:, 7] = 0x7E00                    # a column of NaN
    Xb[:, 9] = 0x8000                    # and one of -0
    clean = Xb.copy()
    clean[:, 7] = 0
    want = np.maximum(orc.product(orc.unpack_fast(c_vals, c_nm, c_vec, M, K, V), clean, "f16", case.pi_in(),
                                  case.pi_out()).astype(np.float64), 0)
    for variant in RINGS:
        hinm.hinm_spmm_prepared(poison.M, poison.K, 128, 256, "f16", 512, prep, nan, 512, Y, 512, variant << 16)
        bits = gu.gpu_spmm_prepared(pr, Xb, 1, variant)
        assert not bits[:, [7, 9]].any(), variant
        gu.check_close(orc.decode(bits, "f16"), want, what="variant %d" % variant)


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
