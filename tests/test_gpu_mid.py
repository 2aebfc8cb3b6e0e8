"""The kernel for a moderate number of columns (csrc/spmm_mid.hip) in every block shape its dispatch takes, from both
layer forms, against the CPU oracle: ragged columns and kept columns, waves without steps, odd numbers of steps."""
import numpy as np
import pytest

import hinm_synth as synth
from tests.test_gpu_prepared import _check as check_prepared
from tests.test_gpu_spmm import _check_full as check_canonical

pytestmark = pytest.mark.gpu

# M, K, V, Kv, N, (32-row blocks, 32-column blocks, waves) of a workgroup
PREPARED = [
    (64, 256, 32, 200, 37, (1, 1, 4)),
    (4800, 640, 96, 584, 30, (1, 1, 8)),     # ten steps on eight waves
    (4832, 2048, 32, 1992, 17, (1, 1, 8)),   # 32 steps, the last one padded
    (9600, 128, 64, 72, 20, (2, 1, 8)),      # two steps: six waves have none
    (9600, 128, 64, 72, 2, (2, 1, 8)),
    (4800, 1088, 32, 1032, 9, (1, 1, 8)),
    (640, 640, 64, 584, 965, (2, 2, 8)),
    (1280, 320, 64, 264, 965, (2, 2, 4)),
    (640, 320, 64, 264, 1765, (2, 2, 4)),     # beyond 1024 columns: fewer than 1024 rows
    (2560, 320, 64, 264, 965, (2, 2, 2)),
    (1280, 2304, 128, 2000, 965, (4, 2, 4)),
    (320, 1152, 32, 1032, 965, (1, 2, 8)),
    (640, 320, 32, 264, 965, (1, 2, 4)),
    (1152, 320, 32, 264, 965, (1, 2, 2)),
]
CANONICAL = [c for c in PREPARED if c[5] not in ((2, 1, 8), (4, 2, 4))] + [
    (1280, 1152, 64, 1048, 965, (2, 4, 4)),
    (320, 320, 160, 168, 70, (1, 1, 4)),     # tiles beyond 128 rows: packed arrays only
    (64, 64, 32, 8, 33, (1, 1, 4)),          # a single, mostly empty step
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,K,V,Kv,N,block", PREPARED)
def test_mid_prepared(M, K, V, Kv, N, block, dtype):
    import paper_2407_20496_amd as hinm
    ld = (N + 7) // 8 * 8
    plan, launches = hinm.hinm_spmm_prepared_plan(M, K, V, Kv, dtype, N, ld, ld, 0)
    assert launches == 1 and "spmm_mid_kernel<" in plan and "RB=%d,CB=%d,NW=%d>" % block in plan
    check_prepared(synth.small_case(M, K, V, Kv, N, dtype, 84), N, [0], relu=(N % 2 == 0), identity=(V == 96))


def _runs_on(block, form, M, K, V, Kv, N, dtype):
    import paper_2407_20496_amd as hinm
    plan = hinm.hinm_calib_mid_plan(M, K, V, Kv, dtype, N, form)
    return "SRC=%d,RB=%d,CB=%d,NW=%d>" % (form + 1, *block) in plan


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,K,V,Kv,N,block", CANONICAL)
def test_mid_canonical(M, K, V, Kv, N, block, dtype):
    assert _runs_on(block, 0, M, K, V, Kv, N, dtype)
    check_canonical(synth.small_case(M, K, V, Kv, N, dtype, 85), N, [0], relu=(N % 2 == 0), identity=(V == 96), ld_pad=8)


@pytest.mark.parametrize("prepared", [True, False])
def test_mid_ignores_what_lies_beside_the_kept_columns(prepared):
    """Input rows that no tile keeps, the padding columns of X and the values of the next row hold infinities and NaN:
    none may reach an output (the ragged last step multiplies zeros there)."""
    import torch
    import paper_2407_20496_amd as hinm
    from oracle import hinm_oracle as orc
    from tests import gpu_util as gu
    M, K, V, Kv, N = 64, 192, 32, 72, 37
    case = synth.small_case(M, K, V, Kv, N, "f16", 86)
    vals, nm, vec = orc.pack(case.weights(), "f16", V, Kv)
    Wh = orc.unpack_fast(vals, nm, vec, M, K, V)
    Xb = case.activations(N)
    want = orc.product(Wh, Xb, "f16", None, None).astype(np.float64)
    ld = 48
    Xp = np.full((K, ld), 0x7C00, dtype=np.uint16)
    Xp[:, :N] = Xb
    unused = np.setdiff1d(np.arange(K), vec.reshape(-1))
    Xp[unused] = 0x7E00
    vals[1::2, 0] = 0x7C00          # every other row starts with an infinity: its outputs are not looked at
    p = gu.upload_packed(M, K, V, Kv, "f16", vals, nm, vec)
    if prepared:
        got = gu.gpu_spmm_prepared(gu.gpu_prepare(p, None, None), Xb, 2, ldx=ld, ldy=ld, X_dev=gu.dev_bits(Xp))
    else:
        got = gu.gpu_spmm(p, Xb, None, None, 2, ldx=ld, ldy=ld, X_dev=gu.dev_bits(Xp))
    gu.check_close(got[0::2].astype(np.float64), want[0::2], what="rows without infinities")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,K,V,Kv,N,block", CANONICAL)
def test_mid_vectors(M, K, V, Kv, N, block, dtype):
    assert _runs_on(block, 1, M, K, V, Kv, N, dtype)
    from oracle import hinm_oracle as orc
    from tests import gpu_util as gu
    case = synth.small_case(M, K, V, Kv, N, dtype, 87)
    pv = gu.gpu_pack_vectors(case.weights(), dtype, V, Kv)
    Wv = orc.unpack_vectors(*orc.pack_vectors(case.weights(), dtype, V, Kv), M, K, V)
    pin, pout = (None, None) if V == 96 else (case.pi_in(), case.pi_out())
    Xb, relu = case.activations(N), int(N % 2 == 0)
    want = orc.product(Wv, Xb, dtype, pin, pout, acc=np.float32, relu=bool(relu)).astype(np.float64)
    got32 = gu.gpu_spmm_vectors(pv, Xb, pin, pout, flags=2 | relu)
    gu.check_close(got32.astype(np.float64), want, what="layer before its 2:4 step")
    assert np.array_equal(gu.gpu_spmm_vectors(pv, Xb, pin, pout, flags=relu), orc.round_to_storage(got32, dtype))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,K,Kv,N,ld_pad", [
    (48, 272, 264, 220, 0),     # ragged last step and ragged last block of columns
    (48, 272, 264, 5, 0),       # rows of eight elements: the second half of a block lies past their end
    (48, 272, 264, 9, 8),
    (32, 40, 8, 17, 0),         # nothing but a ragged step
    (32, 320, 312, 1, 0),
    (32, 2120, 2112, 9, 0),     # eight waves with batches of six: 33 whole steps, 48 and a ragged one
    (32, 3120, 3112, 16, 0),
    (32, 3080, 3072, 1, 0),
])
def test_sixteen_row_tiles_with_ragged_ends(M, K, Kv, N, ld_pad, dtype):
    check_canonical(synth.small_case(M, K, 16, Kv, N, dtype, 88), N, [0], ld_pad=ld_pad)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,K,V,Kv,ldx", [
    (48, 40, 16, 8, 1),             # one piece per row
    (60, 600, 20, 520, 8),          # rows past the tile in the last workgroup; a strided column
    (2048, 96, 64, 72, 1),          # two rows per wave
    (8192, 64, 128, 64, 1),         # four
    (8, 17000, 8, 16904, 1),        # three chunks, the last ragged
    (8, 8192, 8, 8192, 1),          # exactly one chunk
])
def test_vectors_single_column(M, K, V, Kv, ldx, dtype):
    from oracle import hinm_oracle as orc
    from tests import gpu_util as gu
    case = synth.small_case(M, K, V, Kv, 1, dtype, 89)
    pv = gu.gpu_pack_vectors(case.weights(), dtype, V, Kv)
    Wv = orc.unpack_vectors(*orc.pack_vectors(case.weights(), dtype, V, Kv), M, K, V)
    Xb = case.activations(1)
    for pin, pout, relu in ((case.pi_in(), case.pi_out(), 1), (None, None, 0)):
        want = orc.product(Wv, Xb, dtype, pin, pout, acc=np.float32, relu=bool(relu)).astype(np.float64)
        got32 = gu.gpu_spmm_vectors(pv, Xb, pin, pout, flags=2 | relu, ldx=ldx, ldy=ldx)
        gu.check_close(got32.astype(np.float64), want, what="single column")
        got = gu.gpu_spmm_vectors(pv, Xb, pin, pout, flags=relu, ldx=ldx, ldy=ldx)
        assert np.array_equal(got, orc.round_to_storage(got32, dtype))
