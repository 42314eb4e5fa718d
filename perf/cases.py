"""The routed MoE FFN's performance cases: what a program that serves or
evaluates a Mixture-of-Experts layer has this library do.

A layer's weights stay in HBM and every call brings a batch of tokens: one
token to a few dozen while decoding, thousands while a prompt is read.  Most
callers make one call per layer (``moe.forward``; ``moe.forward_noalloc``
where nothing may be allocated); expert-parallel callers run the steps
themselves with their own exchange in between (``moe.route``,
``moe.permute``, ``moe.ffn_group``, ``moe.combine``), and a dense or shared
FFN goes through ``moe.ffn_dense``.  The layer shapes are the package's named
workloads: Mixtral-8x7B and DBRX tensor-parallel shards, the DeepSeekV2
expert-parallel share with and without its shared experts (the latter under a
Zipf router bias), and the Mixtral expert-parallel share.
"""
import math

import torch

from paper_2410_12247_amd import moe, synth

#: tokens of the largest batch of each layer shape
MAX_TOKENS = {"mixtral": 16384, "dbrx": 8192, "dsv2": 16384, "zipf": 16384, "mixtral_ep": 8192}

#: share of a token's k slots that land on the local experts under the Zipf
#: bias, over the share uniform routing gives them
ZIPF_LOCAL = 1.68


def listed():
    return [
        # one sequence being decoded: launches, latency and the weights of k experts
        {"name": "decode_mixtral_1", "call": "forward", "layer": "mixtral", "tokens": 1},
        # a small ragged batch inside a serving loop that may not allocate
        {"name": "decode_mixtral_13_noalloc", "call": "noalloc", "layer": "mixtral",
         "tokens": 13},
        # a full decode batch: every expert's weights are streamed once
        {"name": "decode_dbrx_64", "call": "forward", "layer": "dbrx", "tokens": 64},
        # the same with 160 router outputs, few rows per expert, shared experts
        {"name": "decode_dsv2_61", "call": "forward", "layer": "dsv2", "tokens": 61},
        # a short prompt, skewed expert loads, an odd token count
        {"name": "prompt_zipf_1027", "call": "forward", "layer": "zipf", "tokens": 1027},
        # long prompts through each of the three layer shapes
        {"name": "prefill_mixtral_16384", "call": "forward", "layer": "mixtral",
         "tokens": 16384},
        {"name": "prefill_dbrx_8192", "call": "forward", "layer": "dbrx", "tokens": 8192},
        {"name": "prefill_dsv2_16384", "call": "forward", "layer": "dsv2", "tokens": 16384},
        # full-width experts in two pipeline stages, bits that do not depend on
        # how the work is cut
        {"name": "pipeline_mixtral_ep_4099", "call": "forward", "layer": "mixtral_ep",
         "tokens": 4099, "pipeline_n": 2, "exact_order": True},
        # the steps one by one, as an expert-parallel caller runs them
        {"name": "steps_dbrx_2050", "call": "steps", "layer": "dbrx", "tokens": 2050},
        # the router alone, over the largest batch of the load sweep
        {"name": "route_zipf_65536", "call": "route", "layer": "zipf", "tokens": 65536},
        # one dense SwiGLU FFN (a shared expert) over a ragged row count
        {"name": "dense_dsv2_shared_3001", "call": "dense", "hidden": 5120, "inter": 3072,
         "tokens": 3001},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    call = rng.choice(["forward", "forward", "forward", "forward", "noalloc", "steps", "route",
                       "dense"])
    if call == "dense":
        return {"call": call, "hidden": 64 * rng.randint(32, 96), "inter": 64 * rng.randint(16, 64),
                "tokens": _log_int(rng, 1, 8192)}
    layer = rng.choice(["mixtral", "dbrx", "dsv2", "zipf"])
    if call == "route":
        return {"call": call, "layer": layer, "tokens": _log_int(rng, 1, 65536)}
    if call == "noalloc":
        return {"call": call, "layer": layer, "tokens": _log_int(rng, 1, 256)}
    if call == "steps":
        return {"call": call, "layer": rng.choice(["mixtral", "dbrx", "zipf"]),
                "tokens": _log_int(rng, 1, 4096)}
    if rng.random() < 0.2:
        layer = "mixtral_ep"
    c = {"call": call, "layer": layer, "tokens": _log_int(rng, 1, MAX_TOKENS[layer])}
    if rng.random() < 0.2:
        c["exact_order"] = True
        if rng.random() < 0.5:
            c["pipeline_n"] = 2
    return c


def _shape(case):
    return synth.SHAPES[case["layer"]].with_tokens(case["tokens"])


def _opts(case):
    return moe.opts(pipeline_n=case.get("pipeline_n", 1),
                    exact_order=case.get("exact_order", False))


class _Inputs:
    """Gaussian tensors of the case: x ~ N(0, 1), weights ~ N(0, 0.02)."""

    def __init__(self, case, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        if case["call"] == "dense":
            H, I = case["hidden"], case["inter"]
            self.x = self._bf16((case["tokens"], H), 1.0)
            self.w_gate, self.w_up = self._bf16((I, H)), self._bf16((I, H))
            self.w_down = self._bf16((H, I))
            return
        s = _shape(case)
        self.x = self._bf16((s.T, s.H), 1.0)
        self.w_router = self._normal((s.E, s.H), 0.02)
        self.bias = (torch.from_numpy(synth.zipf_bias(s.E, s.EL, s.H)).cuda()
                     if s.zipf_bias else None)
        if case["call"] == "route":
            return
        self.w_gate = self._bf16((s.EL, s.I, s.H))
        self.w_up = self._bf16((s.EL, s.I, s.H))
        self.w_down = self._bf16((s.EL, s.H, s.I))
        self.sg = self.su = self.sd = None
        if s.n_shared and case["call"] != "steps":
            self.sg = self._bf16((s.shared_inter, s.H))
            self.su = self._bf16((s.shared_inter, s.H))
            self.sd = self._bf16((s.H, s.shared_inter))

    def _normal(self, shape, sigma):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(
            0.0, sigma, generator=self.gen)

    def _bf16(self, shape, sigma=0.02):
        return self._normal(shape, sigma).to(torch.bfloat16)


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    st = {"case": case, "in": _Inputs(case, seed)}
    call, T = case["call"], case["tokens"]
    if call == "dense":
        st["act"] = _empty((T, case["inter"]), torch.bfloat16)
        st["y"] = _empty((T, case["hidden"]), torch.float32)
        return st
    s = _shape(case)
    d = moe.dims(s.T, s.H, s.I, s.E, s.k, s.e0, s.EL, s.renorm,
                 s.shared_inter if call in ("forward", "noalloc") else 0)
    st["d"], st["o"] = d, _opts(case)
    if call == "forward":
        st["buf"] = moe.MoEBuffers(d, st["o"])
        return st
    st["topk_ids"] = _empty((T, s.k), torch.int32)
    st["topk_w"] = _empty((T, s.k), torch.float32)
    if call == "route":
        return st
    st["y"] = _empty((T, s.H), torch.float32)
    st["counts"] = _empty((s.EL,), torch.int32)
    if call == "steps":
        rows = T * min(s.k, s.EL)
        st["offsets"] = _empty((s.EL + 1,), torch.int32)
        st["sorted_slot"] = torch.zeros((rows,), dtype=torch.int32, device="cuda")
        st["slot_row"] = _empty((T * s.k,), torch.int32)
        st["x_perm"] = _empty((rows, s.H), torch.bfloat16)
        st["act"] = _empty((rows, s.I), torch.bfloat16)
        st["y_perm"] = _empty((rows, s.H), torch.float32)
        st["ws"] = _empty((max(moe.workspace_bytes(d), 1),), torch.uint8)
    return st


def run(st):
    call, i = st["case"]["call"], st["in"]
    if call == "dense":
        moe.ffn_dense(st["case"]["tokens"], st["case"]["hidden"], st["case"]["inter"], i.x,
                      i.w_gate, i.w_up, i.w_down, st["act"], st["y"])
        return {"y": st["y"]}
    if call == "forward":
        b = st["buf"]
        b.run(i.x, i.w_router, i.bias, i.w_gate, i.w_up, i.w_down, i.sg, i.su, i.sd)
        return {"y": b.y, "topk_w": b.topk_w, "topk_ids": b.topk_ids, "counts": b.counts}
    if call == "noalloc":
        moe.forward_noalloc(st["d"], st["o"], i.x, i.w_router, i.bias, i.w_gate, i.w_up,
                            i.w_down, i.sg, i.su, i.sd, st["y"], st["topk_ids"], st["topk_w"],
                            st["counts"])
        return {k: st[k] for k in ("y", "topk_w", "topk_ids", "counts")}
    d = st["d"]
    moe.route(d, i.x, i.w_router, i.bias, st["topk_ids"], st["topk_w"])
    if call == "route":
        return {"topk_w": st["topk_w"], "topk_ids": st["topk_ids"]}
    moe.permute(d, st["topk_ids"], i.x, st["counts"], st["offsets"], st["sorted_slot"],
                st["slot_row"], st["x_perm"], st["ws"])
    moe.ffn_group(d, 0, d.local_count, st["offsets"], st["x_perm"], i.w_gate, i.w_up, i.w_down,
                  st["act"], st["y_perm"])
    moe.combine(d, 0, d.local_count, st["y_perm"], st["topk_ids"], st["slot_row"],
                st["topk_w"], st["y"], 0)
    return {k: st[k] for k in ("y", "topk_w", "topk_ids", "counts", "offsets", "sorted_slot",
                               "slot_row")}


def work(case):
    """Inputs read once (of the expert weights, those of experts expected to
    have rows), outputs written once; the router's, experts' and shared FFN's
    multiply-adds."""
    T = case["tokens"]
    if case["call"] == "dense":
        H, I = case["hidden"], case["inter"]
        return {"bytes": T * H * 2 + 3 * H * I * 2 + T * H * 4, "flops": 6 * T * H * I}
    s = _shape(case)
    b = T * s.H * 2 + s.E * s.H * 4 + T * s.k * 8
    f = 2 * T * s.E * s.H
    if case["call"] != "route":
        rows = T * s.k * s.EL / s.E * (ZIPF_LOCAL if s.zipf_bias else 1.0)
        active = s.EL * (1.0 - (1.0 - s.k / s.E) ** T)
        b += active * 3 * s.H * s.I * 2 + T * s.H * 4
        f += 6 * rows * s.H * s.I
        if s.n_shared and case["call"] != "steps":
            b += 3 * s.H * s.shared_inter * 2
            f += 6 * T * s.H * s.shared_inter
    return {"bytes": int(b), "flops": int(f)}


def tolerance(case):
    # Routing is exact: whole numbers must agree.  The router's weights are
    # fp32 (1e-6 to 4e-6 from the 64-bit softmax).  The FFN rounds its SwiGLU
    # activation to bf16, which puts y about 1.7e-3 from the 64-bit result.
    if case["call"] == "route":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
    return {"rel": 6e-3, "max": 0.06, "differ": 0.0}


def _ffn64(x, g, u, d):
    a = x @ g.double().t()
    a = a * torch.sigmoid(a)
    return (a * (x @ u.double().t())) @ d.double().t()


def exact(case, seed):
    i = _Inputs(case, seed)
    x = i.x.double()
    if case["call"] == "dense":
        return {"y": _ffn64(x, i.w_gate, i.w_up, i.w_down)}
    s = _shape(case)
    z = torch.cat([xs @ i.w_router.double().t() for xs in x.split(8192)])
    if i.bias is not None:
        z = z + i.bias.double()
    top, ids = torch.topk(z, s.k, dim=1)
    w = torch.softmax(top, 1) if s.renorm else torch.exp(top - torch.logsumexp(z, 1, keepdim=True))
    if case["call"] == "route":
        return {"topk_w": w, "topk_ids": None}
    y = torch.zeros_like(x) if i.sg is None else _ffn64(x, i.sg, i.su, i.sd)
    for e in range(s.EL):
        tok, slot = (ids == s.e0 + e).nonzero(as_tuple=True)
        if tok.numel():
            r = _ffn64(x[tok], i.w_gate[e], i.w_up[e], i.w_down[e])
            y.index_add_(0, tok, r * w[tok, slot].unsqueeze(1))
    out = {"y": y, "topk_w": w, "topk_ids": None, "counts": None}
    if case["call"] == "steps":
        out.update(offsets=None, sorted_slot=None, slot_row=None)
    return out
