"""hinm_pack and hinm_prepare where their launches change: how many columns a score thread owns and how many rows it
requests at a time, how many keys a select thread holds and where its digits start, and how prepare loads the packed
arrays.  Bit for bit."""
import numpy as np
import pytest

import hinm_synth as synth
from oracle import hinm_oracle as orc
from tests.test_gpu_pack import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,V,Kv", [
    (33, 129, 33, 64),         # odd K: one column a thread, rows beyond one batch of 32
    (62, 130, 31, 64),         # two columns a thread, fewer rows than a batch
    (130, 1026, 65, 512),      # ... and a remainder behind two batches
    (64, 130, 16, 64),         # batches of eight: two, with a remainder, none
    (40, 129, 20, 64),
    (14, 130, 7, 64),
    (256, 8192, 1, 64),        # eight columns a thread (enough threads for it)
    (2, 16384, 1, 8192),       # sixteen keys a select thread
    (2, 16392, 1, 8192),       # keys re-read in every pass
])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_pack_launch_edges(M, K, V, Kv, dtype):
    _compare(synth.small_case(M, K, V, Kv, 1, dtype, 500).weights(), dtype, V, Kv)


@pytest.mark.parametrize("K", [64, 5000])
@pytest.mark.parametrize("values", [(1.0,), (1.0, 1.0625), (0.0, 2.0**-14), (0.0, 64.0), (1.0, 1.5, 2.0, 4.0)])
def test_select_digits(K, values):
    # few distinct scores: all equal (no digit at all), apart in low bits only, apart in the leading bits
    rng = np.random.default_rng(K)
    W = np.broadcast_to(np.array(values, dtype=np.float32)[rng.integers(0, len(values), size=(4, 1, K))], (4, 8, K))
    _compare(synth.to_bits(np.ascontiguousarray(W.reshape(32, K)), "bf16"), "bf16", 8, K // 16 * 8)


@pytest.mark.parametrize("V", [8, 20, 24])           # rows in batches of eight, with and without a remainder
@pytest.mark.parametrize("K", [640, 5000, 16392])    # four, sixteen or no keys held per select thread
@pytest.mark.parametrize("case", ["zeros cut", "zeros below", "ones cut", "near ties cut"])
def test_select_among_many_equal_scores(case, K, V):
    """A third to two thirds of the columns tie, in the middle of distinct scores: the threshold among the equal ones, above
    them, and among scores that differ from them in low bits only."""
    rng = np.random.default_rng(K + V)
    W = rng.uniform(0.5, 2.0, size=(2, V, K)).astype(np.float32)
    tied = rng.random(K) < (0.4 if case == "zeros below" else 0.6)
    W[:, :, tied] = 0.0 if case.startswith("zeros") else 1.25
    if case == "near ties cut":
        W[:, 0, tied & (rng.random(K) < 0.5)] = 1.2578125      # one bf16 step in a single row
    _compare(synth.to_bits(np.ascontiguousarray(W.reshape(2 * V, K)), "bf16"), "bf16", V, K // 16 * 8)


@pytest.mark.parametrize("Kv", [64, 72, 576, 1088])  # whole steps or not; one to nine workgroup-loads of steps
def test_prepare_does_not_depend_on_alignment(Kv):
    import torch
    import paper_2407_20496_amd as hinm
    from tests import gpu_util as gu
    M, K, V = 192, 1096, 96
    c = synth.small_case(M, K, V, Kv, 1, "f16", 501)
    p = gu.gpu_pack(c.weights(), c.dtype, V, Kv)
    want = gu.gpu_prepare(p, c.pi_in(), c.pi_out()).buf.cpu().numpy()
    nbytes = want.size
    vals = torch.empty(p.vals.numel() + 1, dtype=torch.int16, device=gu.DEV)[1:]
    nm = torch.empty(p.nm_idx.numel() + 1, dtype=torch.uint8, device=gu.DEV)[1:]
    vals.copy_(p.vals)
    nm.copy_(p.nm_idx)
    for v, m in ((vals, p.nm_idx), (p.vals, nm), (vals, nm)):
        buf = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device=gu.DEV)
        hinm.hinm_prepare(M, K, V, Kv, c.dtype, v, m, p.vec_idx, gu.dev_i32(c.pi_in()), gu.dev_i32(c.pi_out()), buf, nbytes)
        torch.cuda.synchronize()
        assert np.array_equal(buf.cpu().numpy(), want)
