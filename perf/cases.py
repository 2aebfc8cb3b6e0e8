"""The work whose speed counts: calls of this package as a program that runs or compresses HiNM layers makes them.

A case names one call path (`kind`) and its sizes:

  prepared   hinm_spmm_prepared   one layer in the device-tuned form, Y = P_out (W (P_in X)): how a layer is served
  chain      hinm_chain           consecutive prepared layers, ReLU between them, each with its own channel orders
  canonical  hinm_spmm            the product straight from the packed arrays, with no prepare step
  vectors    hinm_spmm_vectors    a layer of a gradually pruned model before its 2:4 step
  compress   hinm_pack + hinm_prepare      dense weights to the two layer forms (re-run whenever the weights change)
  search     gyro.gyro_permute    the channel-permutation search of one layer, its packing included

All paths have one direction (inference and compression): the package holds no backward pass.  Sizes are those of this
repository's own workloads (hinm_synth.py: encoder feed-forward layer, MLP layers for decoding and prefill, two-layer
chain, large layer, convolutions as matrix products) with ragged column counts beside the even ones; `draw` spreads
over the same ranges.
"""
import math

import torch

import paper_2407_20496_amd as hinm
from paper_2407_20496_amd.gyro import gyro_permute

TORCH_DTYPE = {"f16": torch.float16, "bf16": torch.bfloat16}
DEV = "cuda:0"


def _case(kind, M, K, V, Kv, dtype, N=0, relu=False, name=None):
    c = {"kind": kind, "M": M, "K": K, "V": V, "Kv": Kv, "dtype": dtype, "N": N, "relu": relu}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest call: a tiny layer with 16-row tiles from its packed arrays; launch and call overhead
        _case("canonical", 256, 256, 16, 128, "f16", N=64, name="tiny_canonical"),
        # decoding one token through an MLP block: up- and down-projection, bound by the weights
        _case("chain", 11008, 4096, 128, 2048, "bf16", N=1, relu=True, name="decode_mlp_1_token"),
        # decoding a batch of 16 sequences through a down-projection at 87.5 % total sparsity
        _case("prepared", 4096, 11008, 128, 2752, "bf16", N=16, name="decode_16_tokens"),
        # a serving batch of ragged size: between decoding and prefill
        _case("prepared", 11008, 4096, 128, 2048, "bf16", N=100, name="serve_100_tokens"),
        # a 3x3 convolution as a matrix product (32-row tiles), odd column count, from its packed arrays
        _case("canonical", 256, 2304, 32, 1152, "f16", N=1571, relu=True, name="conv_canonical_ragged"),
        # feed-forward layer of an encoder, 32 sequences of 128 tokens
        _case("prepared", 3072, 768, 64, 384, "f16", N=4096, relu=True, name="encoder_ffn"),
        # prefill of 2048 tokens through a down-projection
        _case("prepared", 4096, 11008, 128, 5504, "bf16", N=2048, name="prefill_down"),
        # two square layers with channel orders of their own, 1024 tokens
        _case("chain", 4096, 4096, 64, 2048, "f16", N=1024, relu=True, name="chain_square"),
        # the largest product: bound by arithmetic
        _case("prepared", 16384, 16384, 128, 8192, "bf16", N=8192, name="large_layer"),
        # a layer between its two pruning steps, ragged token count
        _case("vectors", 4096, 4096, 64, 2048, "f16", N=1000, name="vectors_ragged"),
        # compressing an up-projection: dense weights -> packed arrays -> device-tuned form
        _case("compress", 11008, 4096, 128, 2048, "bf16", name="compress_mlp"),
        # permutation search of the encoder's feed-forward layer
        _case("search", 3072, 768, 64, 384, "f16", name="search_encoder_ffn"),
    ]


# ---- drawn cases ----------------------------------------------------------------------------------

def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(x, m):
    return max(m, int(round(x / m)) * m)


def _columns(rng, hi):
    """Column counts over 1..hi: single tokens, small batches, ragged and even large ones."""
    if rng.random() < 0.15:
        return 1
    n = int(round(_log(rng, 2, hi)))
    return n if rng.random() < 0.6 else _multiple(n, 16) if n >= 16 else n


def draw(rng):
    kind = rng.choices(["prepared", "chain", "canonical", "vectors", "compress", "search"], [45, 15, 15, 10, 8, 7])[0]
    dtype = rng.choice(["f16", "bf16"])
    V = rng.choice([32, 64, 64, 128, 128])
    keep = rng.choice([0.125, 0.25, 0.25, 0.5, 0.5, 0.5])
    relu = rng.random() < 0.5
    if kind == "search":
        V = rng.choice([32, 64])
        M, K = _multiple(_log(rng, 512, 3072), V), _multiple(_log(rng, 256, 768), 8)
        return _case(kind, M, K, V, _multiple(K * rng.choice([0.25, 0.5]), 8), dtype)
    if kind == "compress":
        M, K = _multiple(_log(rng, 256, 11008), V), _multiple(_log(rng, 256, 11008), 8)
        while M * K > 11008 * 4096:
            M, K = _multiple(M / 2, V), _multiple(K / 2, 8)
        return _case(kind, M, K, V, _multiple(K * keep, 8), dtype)
    if kind == "canonical" and rng.random() < 0.3:
        V = 16  # small tiles: served by the packed-array path only
        M, K = _multiple(_log(rng, 128, 1024), V), _multiple(_log(rng, 128, 1024), 8)
        return _case(kind, M, K, V, _multiple(K * 0.5, 8), dtype, N=_columns(rng, 256), relu=relu)
    big = 16384 if kind == "prepared" else 11008 if kind == "chain" else 8192
    M, K = _multiple(_log(rng, 256, big), V), _multiple(_log(rng, 256, big), 8)
    if kind == "chain":  # the second layer leads back to K channels: both have to be whole tiles
        K = _multiple(K, V)
    Kv = _multiple(K * keep, 8)
    N = _columns(rng, 8192 if kind == "prepared" else 4096)
    return _case(kind, M, K, V, Kv, dtype, N=N, relu=relu)


# ---- preparation ------------------------------------------------------------------------------------

def _weights(M, K, dtype, gen):
    return (torch.randn(M, K, device=DEV, generator=gen) * 0.02).to(TORCH_DTYPE[dtype])


def _order(n, gen):
    return torch.randperm(n, device=DEV, generator=gen, dtype=torch.int32)


def _pack_buffers(M, K, V, Kv, dtype):
    vb, nb, cb, wb = hinm.hinm_pack_sizes(M, K, V, Kv, dtype)
    return {
        "vals": torch.empty((M, Kv // 2), dtype=torch.int16, device=DEV),
        "nm_idx": torch.empty((M, Kv // 8), dtype=torch.uint8, device=DEV),
        "vec_idx": torch.empty((M // V, Kv), dtype=torch.int32, device=DEV),
        "workspace": torch.empty(wb // 8, dtype=torch.float64, device=DEV),
        "workspace_bytes": wb,
    }


def _packed_layer(M, K, V, Kv, dtype, flags, prepare, gen):
    """A packed layer with random channel orders; in the device-tuned form too when `prepare` is set."""
    b = _pack_buffers(M, K, V, Kv, dtype)
    W = _weights(M, K, dtype, gen)
    hinm.hinm_pack(M, K, V, Kv, dtype, W, b["vals"], b["nm_idx"], b["vec_idx"], b["workspace"], b["workspace_bytes"])
    pi_in, pi_out = _order(K, gen), _order(M, gen)
    prepared = None
    if prepare:
        nbytes = hinm.hinm_prepare_sizes(M, K, V, Kv, dtype)
        prepared = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        hinm.hinm_prepare(M, K, V, Kv, dtype, b["vals"], b["nm_idx"], b["vec_idx"], pi_in, pi_out, prepared, nbytes)
    return hinm.Layer(M, K, V, Kv, dtype, b["vals"], b["nm_idx"], b["vec_idx"], pi_in, pi_out, flags, prepared)


def _ld(N):
    return N if N == 1 else (N + 7) // 8 * 8


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind, M, K, V, Kv, dtype, N = (case[k] for k in ("kind", "M", "K", "V", "Kv", "dtype", "N"))
    flags = hinm.EPI_RELU if case["relu"] else 0
    s = {"kind": kind, "M": M, "K": K, "V": V, "Kv": Kv, "dtype": dtype, "N": N, "flags": flags}
    if kind == "search":
        W = _weights(M, K, dtype, gen)
        # second-order saliency of every weight: w^2 times a positive curvature
        curvature = torch.empty(M, K, device=DEV).exponential_(generator=gen) + 0.1
        s.update(W=W, rho=(W.float() * W.float() * curvature).contiguous(), seed=seed)
        return s
    if kind == "compress":
        s.update(_pack_buffers(M, K, V, Kv, dtype))
        nbytes = hinm.hinm_prepare_sizes(M, K, V, Kv, dtype)
        s.update(W=_weights(M, K, dtype, gen), pi_in=_order(K, gen), pi_out=_order(M, gen), prepared_bytes=nbytes,
                 prepared=torch.empty(nbytes, dtype=torch.uint8, device=DEV))
        return s
    ld = _ld(N)
    X = torch.zeros((K, ld), dtype=TORCH_DTYPE[dtype], device=DEV)
    X[:, :N] = torch.randn(K, N, device=DEV, generator=gen).to(TORCH_DTYPE[dtype])
    rows_out = K if kind == "chain" else M
    Y = torch.empty((rows_out, ld), dtype=TORCH_DTYPE[dtype], device=DEV)
    s.update(X=X, Y=Y, ld=ld, out=Y[:, :N])
    if kind == "chain":
        keep = Kv / K
        layers = [_packed_layer(M, K, V, Kv, dtype, flags, True, gen),
                  _packed_layer(K, M, V, _multiple(M * keep, 8), dtype, 0, True, gen)]
        nbytes = hinm.hinm_chain_sizes(layers, N)
        s.update(layers=layers, scratch=torch.empty(nbytes, dtype=torch.uint8, device=DEV), scratch_bytes=nbytes)
    elif kind == "vectors":
        b = _pack_buffers(M, K, V, Kv, dtype)
        vals_v = torch.empty((M, Kv), dtype=torch.int16, device=DEV)
        hinm.hinm_pack_vectors(M, K, V, Kv, dtype, _weights(M, K, dtype, gen), None, None, vals_v, b["vec_idx"],
                               b["workspace"], b["workspace_bytes"])
        s.update(vals_v=vals_v, vec_idx=b["vec_idx"], pi_in=_order(K, gen), pi_out=_order(M, gen))
    else:
        s["layer"] = _packed_layer(M, K, V, Kv, dtype, flags, kind == "prepared", gen)
    return s


# ---- one pass ---------------------------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    M, K, V, Kv, dtype, N = s["M"], s["K"], s["V"], s["Kv"], s["dtype"], s["N"]
    if kind == "prepared":
        hinm.hinm_spmm_prepared(M, K, V, Kv, dtype, N, s["layer"].prepared, s["X"], s["ld"], s["Y"], s["ld"], s["flags"])
        return s["out"]
    if kind == "chain":
        hinm.hinm_chain(s["layers"], N, s["X"], s["ld"], s["Y"], s["ld"], s["scratch"], s["scratch_bytes"])
        return s["out"]
    if kind == "canonical":
        l = s["layer"]
        hinm.hinm_spmm(M, K, V, Kv, dtype, N, l.vals, l.nm_idx, l.vec_idx, l.pi_in, l.pi_out, s["X"], s["ld"], s["Y"],
                       s["ld"], s["flags"])
        return s["out"]
    if kind == "vectors":
        hinm.hinm_spmm_vectors(M, K, V, Kv, dtype, N, s["vals_v"], s["vec_idx"], s["pi_in"], s["pi_out"], s["X"],
                               s["ld"], s["Y"], s["ld"], s["flags"])
        return s["out"]
    if kind == "compress":
        hinm.hinm_pack(M, K, V, Kv, dtype, s["W"], s["vals"], s["nm_idx"], s["vec_idx"], s["workspace"],
                       s["workspace_bytes"])
        hinm.hinm_prepare(M, K, V, Kv, dtype, s["vals"], s["nm_idx"], s["vec_idx"], s["pi_in"], s["pi_out"],
                          s["prepared"], s["prepared_bytes"])
        # the device-tuned form is opaque (its layout is the library's own); the packed arrays say it all
        return {"vals": s["vals"], "nm_idx": s["nm_idx"], "vec_idx": s["vec_idx"]}
    return gyro_permute(s["W"], V, Kv, dtype, rho=s["rho"], seed=s["seed"])


# ---- what a pass cannot do without --------------------------------------------------------------------

def _layer_bytes(M, K, V, Kv):
    """Stored values, NM index, vector index, both channel orders."""
    return M * Kv + M * Kv // 8 + M // V * Kv * 4 + (K + M) * 4


def work(case):
    kind, M, K, V, Kv, N = (case[k] for k in ("kind", "M", "K", "V", "Kv", "N"))
    T = M // V
    if kind == "chain":
        Kv2 = _multiple(M * (Kv / K), 8)
        return {"bytes": _layer_bytes(M, K, V, Kv) + _layer_bytes(K, M, V, Kv2) + 2 * K * N * 2,
                "flops": M * Kv * N + K * Kv2 * N}
    if kind == "vectors":
        return {"bytes": M * Kv * 2 + T * Kv * 4 + (K + M) * 4 + (K + M) * N * 2, "flops": 2 * M * Kv * N}
    if kind == "compress":
        return {"bytes": M * K * 2 + 2 * _layer_bytes(M, K, V, Kv), "flops": 2 * M * K}
    if kind == "search":
        # eight iterations of each search with their default sample counts: cost matrices (Eq. 4) of both, two rounds
        # of distances of the sampled channels to the T centroids where channels are sampled by more than one
        P = Kv // 4
        icp = 8 * T * P * P * V * 3
        ocp = 8 * T * T * K * 2
        return {"bytes": M * K * 6 + _layer_bytes(M, K, V, Kv), "flops": icp + ocp}
    return {"bytes": _layer_bytes(M, K, V, Kv) + (K + M) * N * 2, "flops": M * Kv * N}


def tolerance(case):
    """16-bit results: sums in another order round the other way now and then, one unit in the last place apart; a chain
    rounds its intermediate too.  Against the same products with sums in binary64 the listed sizes showed, in f16 and
    bf16, at most 4e-5 and 1.1e-4 (2-norm) and one unit in the last place, 1e-3 and 7.8e-3: four times that."""
    if case["kind"] == "compress":
        return "exact"
    if case["kind"] == "search":
        return {"rel": 1e-9, "max": 1e-8, "differ": 0.0}  # objectives in binary64; orders and packed arrays are whole numbers
    return {"rel": 1.6e-4, "max": 4e-3} if case["dtype"] == "f16" else {"rel": 4.6e-4, "max": 3.1e-2}
