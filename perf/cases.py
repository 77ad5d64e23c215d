"""What a user of the library has it do, as timed cases.

`listed()` names them; `draw(rng)` gives more of the same ranges.  `prepare` makes what the
caller's program holds before the call (token rows, packed weights, the output buffers it
reuses), `run` is one pass through the public entry points.  Kinds:

  layer       moe_layer_chunked: one MoE layer forward
  stages      moe_route, moe_dispatch, moe_expert_ffn, moe_combine called one by one, as a
              caller that runs its own exchange between them does
  stack       inference stack: layers in sequence, each feeding the next its 16-bit output
  train       moe_layer_forward_keep, then moe_layer_backward: one training step of a layer
  offload     moe_expert_ffn_offloaded: expert weights in page-locked host memory
  popularity  the inference scheduler on one batch: per layer the estimate, its sums to the
              host, both scheduling phases there
  tables      the offline profiling stage: sample-path counts and their top-k tables
"""
import math

import numpy as np
import torch

import paper_2210_17223_amd as moe

DEV = "cuda:0"


# ---------------------------------------------------------------------------- the cases
def _layer(name, T, d, E, h, k, C, kind="layer", dtype="bf16", act="gelu", renorm=False, biases=False,
           skew="none", chunks=1, layers=1, resident=0):
    return dict(name=name, kind=kind, T=T, d=d, E=E, h=h, k=k, C=C, dtype=dtype, act=act, renorm=renorm,
                biases=biases, skew=skew, chunks=chunks, layers=layers, resident=resident)


def _paths(name, kind, T, L=12, E=16, k=1, l=3, N=16, max_pack=4):
    return dict(name=name, kind=kind, T=T, L=L, E=E, k=k, l=l, N=N, max_pack=max_pack)


def listed():
    return [
        # correctness-sized fp32 layer (configuration 1): launches and host time
        _layer("tiny_fp32", 512, 128, 4, 256, 1, 128, dtype="f32"),
        # a decode step of 16 sequences through a GPT-2-small-shaped layer, nothing dropped
        _layer("decode_gpt2s", 16, 768, 16, 3072, 2, 16),
        # prefill / training-batch forward of the same layer (configuration 2)
        _layer("gpt2s_moe", 4096, 768, 16, 3072, 2, 640),
        # odd sizes, every option, the four entry points called one by one
        _layer("ragged_stages", 3001, 1000, 13, 2600, 3, 867, kind="stages", act="gelu_tanh", renorm=True,
               biases=True),
        # popularity follows Zipf(1.2): full, overflowing and nearly empty experts (configuration 3)
        _layer("skewed", 16384, 1024, 32, 4096, 2, 1280, skew="zipf"),
        # the large chunked layer (configuration 4)
        _layer("large_chunked", 32768, 2048, 64, 8192, 2, 1024, chunks=4),
        # serving: four large layers, 256 tokens a step, correlated expert choices (configuration 5)
        _layer("infer_stack", 256, 4096, 8, 14336, 2, 256, kind="stack", skew="markov", layers=4),
        # training steps at the ordinary and at the large size
        _layer("gpt2s_train", 4096, 768, 16, 3072, 2, 640, kind="train"),
        _layer("large_train", 32768, 2048, 64, 8192, 2, 1024, kind="train"),
        # serving with the experts in host memory, two slots on the device
        _layer("offload_serve", 256, 1024, 16, 4096, 2, 256, kind="offload", resident=2),
        # the scheduler's shape of the inference runs: 12 layers, 16 experts, paths of length 3
        _paths("popularity_batch", "popularity", 8192),
        _paths("path_tables", "tables", 1 << 20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(v, m):
    return max(m, (int(v) + m // 2) // m * m)


def _slots(rng, T, E, k):
    cf = rng.choice([0.0, 1.0, 1.25, 1.5])          # 0: nothing is dropped
    return T if cf == 0.0 else min(T, max(1, math.ceil(cf * k * T / E)))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer_f32", "stages", "stack", "train", "train", "offload",
                       "popularity", "tables"])
    if kind == "layer_f32":
        T, d = _log_int(rng, 64, 4096), _mult(_log_int(rng, 64, 1024), 4)
        E, k = rng.randint(2, 16), rng.randint(1, 2)
        c = _layer("", T, d, E, _mult(d * rng.uniform(1.5, 4.0), 4), k, _slots(rng, T, E, k), dtype="f32",
                   act=rng.choice(["gelu", "relu"]))
    elif kind in ("layer", "stages", "train"):
        lo, hi = (128, 16384) if kind == "train" else (8, 32768)
        T = _log_int(rng, lo, hi)
        step = rng.choice([8, 64])
        d = _mult(_log_int(rng, 256, 2048), step)
        E, k = rng.choice([4, 8, 13, 16, 32, 64]), rng.randint(1, 3)
        h = _mult(d * rng.uniform(2.0, 4.0), step)
        c = _layer("", T, d, E, h, k, _slots(rng, T, E, k), kind=kind,
                   act="gelu" if rng.random() < 0.7 else rng.choice(["gelu_tanh", "relu"]),
                   skew=rng.choice(["none", "none", "zipf"]))
        if kind == "layer":
            c["chunks"] = rng.choice([1, 2, 4, 8])
        if kind == "stages":
            c["renorm"], c["biases"] = rng.random() < 0.5, rng.random() < 0.5
    elif kind == "stack":
        T, d = _log_int(rng, 8, 512), _mult(_log_int(rng, 1024, 4096), 128)
        c = _layer("", T, d, rng.choice([4, 8]), _mult(3.5 * d, 128), 2, T, kind="stack", skew="markov",
                   layers=rng.randint(2, 4))
    elif kind == "offload":
        T, d = _log_int(rng, 32, 2048), _mult(_log_int(rng, 256, 2048), 64)
        c = _layer("", T, d, rng.choice([4, 8, 16]), _mult(d * rng.uniform(2.0, 4.0), 64), 2, T, kind="offload",
                   resident=rng.randint(2, 4))
    elif kind == "popularity":
        E = rng.choice([8, 16, 32])
        c = _paths("", "popularity", _log_int(rng, 256, 32768), rng.randint(6, 12), E, rng.randint(1, 2),
                   rng.randint(2, 3), E, 4)
    else:
        E = rng.choice([8, 16, 32])
        c = _paths("", "tables", _log_int(rng, 1 << 16, 1 << 21), rng.randint(6, 12), E, rng.randint(1, 2),
                   rng.randint(2, 3), E, 4)
    del c["name"]
    return c


# ---------------------------------------------------------------------------- inputs
class _State:
    pass


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype, std=1.0):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=g)


def _zipf(E, alpha):
    p = np.arange(1, E + 1, dtype=np.float64) ** -alpha
    return p / p.sum()


def _zipf_gate_bias(seed, E, d):
    """Per-expert logit offset under which expert popularity follows Zipf(1.2)."""
    p = _zipf(E, 1.2)[np.random.default_rng(seed).permutation(E)]
    scale = 0.02 * math.sqrt(d) * math.sqrt(6.0) / math.pi
    return torch.tensor(scale * np.log(p), dtype=torch.float32, device=DEV)


def _choices(g, T, E, k, logp):
    """[T, k] distinct experts drawn from exp(logp), first choice first."""
    u = torch.rand((T, E), generator=g, device=DEV).clamp_min_(1e-20)
    return torch.topk(logp - torch.log(-torch.log(u)), k, dim=1).indices


def _markov_choices(g, L, T, E, k, order):
    """[L, T, k]: a token keeps its previous layer's experts with probability 0.7, otherwise
    draws them from Zipf(1.0) over the seeded order of the experts."""
    logp = torch.tensor(np.log(_zipf(E, 1.0)), dtype=torch.float32, device=DEV)[order]
    out = [_choices(g, T, E, k, logp)]
    for _ in range(1, L):
        keep = torch.rand((T, 1), generator=g, device=DEV) < 0.7
        out.append(torch.where(keep, out[-1], _choices(g, T, E, k, logp)))
    return torch.stack(out)


def _prepare_layer(c, seed, g, keep_canonical=False):
    """One layer's weights, gate and the buffers its outputs go to."""
    s = moe.Shape.make(c["T"], c["d"], c["E"], c["h"], c["k"], c["C"], dtype=c["dtype"], act=c["act"],
                       renorm_topk=c["renorm"])
    dt = s.torch_dtype
    L = _State()
    L.s, L.chunks = s, c["chunks"]
    L.b = moe.alloc_buffers(s, c["chunks"], DEV, y_act=c["kind"] == "stack")
    for key in ("src_of", "xe", "ye"):
        L.b[key].zero_()                        # rows past the last kept one stay as they are
    Wg = _normal(g, (c["d"], c["E"]), dt, 0.02)
    W1 = _normal(g, (c["E"], c["d"], c["h"]), dt, 0.02)
    W2 = _normal(g, (c["E"], c["h"], c["d"]), dt, 0.02)
    moe.moe_pack_gate(s, Wg, L.b["Wgp"])
    moe.moe_pack_weights(s, W1, W2, L.b["W1p"], L.b["W2p"])
    L.W1, L.W2 = (W1, W2) if keep_canonical else (None, None)
    L.b1 = _normal(g, (c["E"], c["h"]), torch.float32, 0.05) if c["biases"] else None
    L.b2 = _normal(g, (c["E"], c["d"]), torch.float32, 0.05) if c["biases"] else None
    L.gate_bias, L.stride = None, 0
    if c["skew"] == "zipf":
        L.gate_bias = _zipf_gate_bias(seed, c["E"], c["d"])
    return L


def _prepare_paths(c, seed, g):
    s = moe.PathShape(c["L"], c["E"], c["k"], c["l"])
    P, tables = moe.moe_path_count(s), c["L"] - c["l"]
    st = _State()
    st.s, st.P, st.tables = s, P, tables
    st.counts = torch.zeros(tables * P * c["E"], dtype=torch.int32, device=DEV)
    st.top_e = torch.zeros(tables * P * c["k"], dtype=torch.int32, device=DEV)
    st.top_q = torch.zeros(tables * P * c["k"], dtype=torch.int64, device=DEV)
    order = torch.randperm(c["E"], generator=g, device=DEV)
    T = c["T"] if c["kind"] == "tables" else 1 << 17
    st.sel = _markov_choices(g, c["L"], T, c["E"], c["k"], order).to(torch.int32).contiguous()
    if c["kind"] == "popularity":
        moe.moe_path_profile(s, st.sel, T, st.counts)
        moe.moe_path_finalize(s, st.counts, st.top_e, st.top_q)
        st.sel = _markov_choices(g, c["L"], c["T"], c["E"], c["k"], order).to(torch.int32).contiguous()
        st.S = torch.zeros((tables, c["E"]), dtype=torch.int64, device=DEV)
        # what the gates of the estimated layers report for this batch
        st.gate_counts = torch.stack([torch.bincount(st.sel[a + c["l"]].reshape(-1).long(), minlength=c["E"])
                                      for a in range(tables)]).to(torch.int32)
    return st


def prepare(case, seed):
    c = dict(case)
    g = _gen(seed)
    if c["kind"] in ("popularity", "tables"):
        st = _prepare_paths(c, seed, g)
        st.case, st.kind = c, c["kind"]
        return st
    st = _State()
    st.case, st.kind = c, c["kind"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    st.x = _normal(g, (c["T"], c["d"]), dt)
    st.layers = [_prepare_layer(c, seed + 7919 * i, g, c["kind"] == "train") for i in range(c["layers"])]
    L = st.layers[0]
    if c["skew"] == "markov":
        order = torch.randperm(c["E"], generator=g, device=DEV)
        forced = _markov_choices(g, c["layers"], c["T"], c["E"], c["k"], order)
        for i, layer in enumerate(st.layers):
            layer.gate_bias = torch.zeros((c["T"], c["E"]), device=DEV).scatter_(1, forced[i], 64.0)
            layer.stride = c["E"]
    if c["kind"] == "train":
        rows, f32 = moe.moe_max_rows(L.s), torch.float32
        st.pre = torch.zeros(rows * c["h"], dtype=torch.float16, device=DEV)
        st.hid = torch.zeros(rows * c["h"], dtype=torch.float16, device=DEV)
        st.dy = _normal(g, (c["T"], c["d"]), f32)
        st.dx = torch.empty((c["T"], c["d"]), dtype=f32, device=DEV)
        st.dWg = torch.empty((c["d"], c["E"]), dtype=f32, device=DEV)
        st.dW1 = torch.empty((c["E"], c["d"], c["h"]), dtype=f32, device=DEV)
        st.dW2 = torch.empty((c["E"], c["h"], c["d"]), dtype=f32, device=DEV)
        st.dgate = torch.empty(c["T"] * c["k"], dtype=f32, device=DEV)
        st.ws = torch.empty(moe.moe_backward_workspace_bytes(L.s), dtype=torch.uint8, device=DEV)
    if c["kind"] == "offload":
        # the routed rows are there; the packed weights move to the host and leave the device
        b = L.b
        moe.moe_route(L.s, st.x, b["Wgp"], L.gate_bias, L.stride, b["expert_idx"], b["gate"])
        moe.moe_dispatch(L.s, st.x, b["expert_idx"], b["counts"], b["offsets"], b["slot_of"], b["src_of"],
                         b["xe"], b["workspace"])
        host = {}
        for key in ("W1p", "W2p"):
            host[key] = torch.empty(b[key].shape, dtype=b[key].dtype, pin_memory=True)
            host[key].copy_(b[key])
            del b[key]
        st.W1h, st.W2h = host["W1p"], host["W2p"]
        st.staging = torch.empty(moe.moe_offload_staging_bytes(L.s, c["resident"]), dtype=torch.uint8, device=DEV)
        st.ws = torch.empty(moe.moe_offload_workspace_bytes(L.s), dtype=torch.uint8, device=DEV)
    return st


# ---------------------------------------------------------------------------- one pass
_OUT = ("expert_idx", "gate", "counts", "offsets", "slot_of", "src_of", "xe", "ye", "y")


def _outputs(b):
    return {key: b[key] for key in _OUT}


def run(st):
    if st.kind in ("layer", "stack"):
        x, out = st.x, []
        for L in st.layers:
            b = L.b
            moe.moe_layer_chunked(L.s, L.chunks, x, b["Wgp"], L.gate_bias, L.stride, b["W1p"], L.b1, b["W2p"],
                                  L.b2, b["expert_idx"], b["gate"], b["counts"], b["offsets"], b["slot_of"],
                                  b["src_of"], b["xe"], b["ye"], b["y"], b["y_act"], b["workspace"])
            x = b["y_act"]
            out.append(_outputs(b))
        return out
    if st.kind == "stages":
        L = st.layers[0]
        s, b = L.s, L.b
        moe.moe_route(s, st.x, b["Wgp"], L.gate_bias, L.stride, b["expert_idx"], b["gate"])
        moe.moe_dispatch(s, st.x, b["expert_idx"], b["counts"], b["offsets"], b["slot_of"], b["src_of"],
                         b["xe"], b["workspace"])
        moe.moe_expert_ffn(s, b["xe"], b["offsets"], b["W1p"], L.b1, b["W2p"], L.b2, b["ye"], b["workspace"])
        moe.moe_combine(s, b["ye"], b["slot_of"], b["gate"], b["y"])
        return _outputs(b)
    if st.kind == "train":
        L = st.layers[0]
        s, b = L.s, L.b
        moe.moe_layer_forward_keep(s, st.x, b["Wgp"], L.gate_bias, L.stride, b["W1p"], None, b["W2p"], None,
                                   b["expert_idx"], b["gate"], b["counts"], b["offsets"], b["slot_of"],
                                   b["src_of"], b["xe"], b["ye"], st.pre, st.hid, b["y"], b["workspace"])
        moe.moe_layer_backward(s, st.x, b["Wgp"], L.gate_bias, L.stride, L.W1, L.W2, b["W1p"],
                               b["expert_idx"], b["gate"], b["offsets"], b["slot_of"], b["src_of"], b["xe"],
                               b["ye"], st.pre, st.hid, st.dy, st.dx, st.dWg, st.dW1, st.dW2, st.dgate, st.ws)
        return dict(_outputs(b), dx=st.dx, dWg=st.dWg, dW1=st.dW1, dW2=st.dW2, dgate=st.dgate)
    if st.kind == "offload":
        L = st.layers[0]
        b = L.b
        moe.moe_expert_ffn_offloaded(L.s, b["xe"], b["offsets"], st.W1h, st.W2h, L.b1, L.b2, b["ye"],
                                     st.staging, st.case["resident"], st.ws)
        return b["ye"]
    c, s, P, k = st.case, st.s, st.P, st.case["k"]
    if st.kind == "popularity":
        out = []
        for a in range(st.tables):
            rows = slice(a * P * k, (a + 1) * P * k)
            moe.moe_popularity_estimate(s, st.sel[a:a + c["l"]], c["T"], st.top_e[rows], st.top_q[rows], st.S[a])
            S = st.S[a].cpu().numpy().view(np.uint64)
            counts = st.gate_counts[a].cpu().numpy()
            out.append(moe.moe_schedule_layer(c["N"], c["E"], k, c["T"], S, counts, c["max_pack"]))
        return {"S": st.S, "schedules": out}
    st.counts.zero_()
    moe.moe_path_profile(s, st.sel, c["T"], st.counts)
    moe.moe_path_finalize(s, st.counts, st.top_e, st.top_q)
    return [st.counts, st.top_e, st.top_q]


# ---------------------------------------------------------------------------- yardsticks
def _kept_rows(c):
    """Expected kept assignments."""
    T, E, k, C = c["T"], c["E"], c["k"], c["C"]
    if c["skew"] == "zipf":
        return sum(min(C, T, T * k * p) for p in _zipf(E, 1.2))
    return min(T * k, E * C)


def work(case):
    c = dict(case)
    T, E, k = c["T"], c["E"], c["k"]
    if c["kind"] in ("popularity", "tables"):
        tables, P = c["L"] - c["l"], E ** c["l"]
        if c["kind"] == "popularity":
            return {"bytes": tables * (T * (c["l"] * k * 4 + k * 12) + E * 8), "flops": 0}
        return {"bytes": c["L"] * T * k * 4 + tables * P * (E * 4 + k * 12), "flops": 0}
    d, h, e = c["d"], c["h"], 2 if c["dtype"] == "bf16" else 4
    A = _kept_rows(c)
    used = E * (1.0 - (1.0 - 1.0 / E) ** (T * k))       # experts that get at least one row
    weights = 2 * used * d * h * e
    if c["kind"] == "offload":
        return {"bytes": 2 * E * d * h * e + 2 * A * d * e, "flops": 4 * A * d * h}
    byt = T * d * e + d * E * 4 + weights + T * k * 12 + A * 4 + 2 * A * d * e + T * d * 4
    ops = 2 * T * d * E + 4 * A * d * h
    if c["kind"] == "stages":                           # between the calls xe and ye are inputs again
        byt += 2 * A * d * e + 2 * T * k * 4
    if c["kind"] == "train":
        byt += weights + 2 * A * h * 2 + 2 * T * d * 4 + 2 * E * d * h * 4 + d * E * 4 + T * k * 4
        ops = 3 * ops
    return {"bytes": c["layers"] * byt, "flops": c["layers"] * ops}


def tolerance(case):
    if case["kind"] in ("popularity", "tables"):
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}               # 32-bit sums of up to 4096 terms
    if case["kind"] == "train":
        return {"rel": 1e-2, "max": 0.2}                # two chained bf16 operand roundings
    if case["kind"] == "stack":
        # roundings add up from layer to layer; a token whose two gate logits are all but equal
        # may list its experts the other way round
        return {"rel": 2e-2, "max": 0.3, "differ": 0.01}
    return {"rel": 5e-3, "max": 0.05}                   # 16-bit hidden activations and expert outputs
