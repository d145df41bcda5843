"""The calls whose speed matters, over the range a program makes them in.

Every case goes through the binding's entry points as a serving or training program calls them: decode steps of one
to 256 tokens, chunked and whole-prompt prefill layers, routed stacks, the attention sub-block, and the two backward
calls of training.  Shapes are those of the repository's workloads (Llama-3.1-8B, Llama-2-7B, Llama-2-13B, the tiny
fp32 stack, the rank-896 operating point) and, when drawn, other sizes of the same ranges.

Inputs are seeded Gaussians as in the package's synthetic workloads, made on the GPU.  Gates are those of a trained
router: the per-token logit bias puts every token clearly on one side of the decision, in runs of neighbouring
positions, so that no branch hangs on the last bit of a logit.  A stack's residual projections (W_d, W_2) are scaled
by 1/sqrt(2 L), as models of that depth are initialised, so that the hidden states keep their scale over depth.
"""
import math

import torch

from paper_2609_08189_amd import hero as H

DEV = "cuda:0"
MODELS = {  # d, d_ff of the backbones the workloads name, and the tiny fp32 one
    "8b": (4096, 14336), "7b": (4096, 11008), "13b": (5120, 13824), "tiny": (256, 688),
}
D_S, D_H, D_A, D_E, D_P, D_HEAD = 64, 48, 16, 256, 64, 256
EPS_NORM, EPS, T_HIST = 1e-5, 1e-6, 0.9
ETA = math.log(49.0)
RUN = 64  # neighbouring positions that take the same branch in a prefill


def _c(name, kind, model, T, **kw):
    c = dict(name=name, kind=kind, model=model, T=T, dtype="bf16", L=32, j=17, d_r=64, d_m=128, mode="budget",
             skip=0.27, memory="f32", tiled=False, graph=False, batch=1, n_heads=32, n_kv=8)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the fp32 stack of four narrow layers (launches and latency)
        _c("tiny_f32_stack_64", "stack", "tiny", 64, dtype="f32", L=4, d_r=16, d_m=32),
        # one sequence decoding, layer by layer on the library's own scratch
        _c("decode_8b_layer_1", "layer_noalloc", "8b", 1, tiled=True, mode="threshold", skip=0.0),
        # a small decode batch with the memory in depth-history form and the plain weights
        _c("decode_8b_hist_layer_48", "layer", "8b", 48, memory="history", j=24),
        # a full decode batch through all 32 layers, captured once and replayed
        _c("decode_7b_stack_256", "stack", "7b", 256, tiled=True, graph=True),
        # a chunk of a prompt
        _c("chunk_8b_layer_640", "layer", "8b", 640, mode="threshold", skip=0.39, j=9),
        # whole prompts through one layer: the 8B shape at the looser skip rate
        _c("prefill_8b_layer_4096", "layer", "8b", 4096, skip=0.2687),
        # a ragged prompt at the 13B shape, threshold rule, second routed layer
        _c("prefill_13b_layer_2777", "layer", "13b", 2777, L=40, j=2, mode="threshold", skip=0.29),
        # the operating point with adapters of rank 896 and a memory of width 64, kept in bf16
        _c("prefill_rank896_layer_4096", "layer", "8b", 4096, d_r=896, d_m=64, skip=0.25, memory="bf16"),
        # the headline: 16 prompts of 2048 through the 32-layer stack
        _c("prefill_8b_stack_32768", "stack", "8b", 32768, skip=0.3882),
        # dense attention of one decoder block over two prompts
        _c("attention_8b_2x2048", "attention", "8b", 4096, batch=2),
        # training: the routed block's backward and the router's backward of one layer
        _c("block_backward_8b_4096", "block_backward", "8b", 4096, skip=0.2687),
        _c("router_backward_8b_4096", "router_backward", "8b", 4096),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    what = rng.choice(("tiny", "decode", "decode", "decode_stack", "chunk", "prefill", "prefill", "stack", "attention",
                       "block_backward", "router_backward"))
    model = rng.choice(("8b", "7b", "13b"))
    kw = dict(L=40 if model == "13b" else 32, skip=round(rng.uniform(0.0, 0.6), 3),
              mode=rng.choice(("budget", "threshold")))
    kw["j"] = rng.randint(1, kw["L"])
    if what == "tiny":
        c = _c("", "stack", "tiny", _log_int(rng, 1, 512), **dict(kw, dtype="f32", L=rng.randint(2, 6), d_r=16, d_m=32))
    elif what == "decode":
        memory = rng.choice(("f32", "f32", "bf16", "history"))
        kind = "layer" if memory == "history" else rng.choice(("layer", "layer_noalloc"))
        c = _c("", kind, model, _log_int(rng, 1, 256), memory=memory, tiled=rng.random() < 0.7, **kw)
    elif what == "decode_stack":
        c = _c("", "stack", model, _log_int(rng, 1, 256), tiled=True, graph=rng.random() < 0.7, **dict(kw, L=rng.randint(2, 16)))
    elif what == "chunk":
        c = _c("", "layer", model, _log_int(rng, 257, 1500), **kw)
    elif what == "prefill":
        d_r, d_m = rng.choice(((64, 128), (64, 128), (32, 64), (128, 256), (896, 64)))
        c = _c("", "layer", model, _log_int(rng, 1500, 12000), d_r=d_r, d_m=d_m,
               memory=rng.choice(("f32", "f32", "bf16", "history")), **kw)
    elif what == "stack":
        c = _c("", "stack", model, _log_int(rng, 2000, 20000), **dict(kw, L=rng.randint(2, 8)))
    elif what == "attention":
        n_heads, n_kv = {"8b": (32, 8), "7b": (32, 32), "13b": (40, 40)}[model]
        batch = rng.randint(1, 6)
        c = _c("", "attention", model, batch * _log_int(rng, 16, 8192 // batch), batch=batch, n_heads=n_heads, n_kv=n_kv)
    elif what == "block_backward":
        c = _c("", "block_backward", model, _log_int(rng, 100, 6000), d_r=rng.choice((64, 64, 896)), **kw)
    else:
        # from the third routed layer: before it the memory read does not depend on the query
        c = _c("", "router_backward", model, _log_int(rng, 16, 6000), d_m=rng.choice((64, 128, 128)),
               **dict(kw, j=rng.randint(3, kw["L"])))
    del c["name"]
    return c


# ---- inputs -----------------------------------------------------------------------------------------------------


def _n_skip(case):
    return int(math.floor(case["skip"] * case["T"] + 0.5))


class _Draw:
    """Seeded draws, one stream a tensor, in the order they are asked for."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(1000003 * (seed + 1))
        self.dtype = torch.bfloat16 if dtype == "bf16" else torch.float32

    def f32(self, *shape, std=1.0):
        x = torch.randn(*shape, device=DEV, generator=self.g)
        return x.mul_(std) if std != 1.0 else x

    def store(self, *shape, std=1.0, mean=0.0):
        """N(mean, std) in the storage dtype; large matrices are drawn in it."""
        if mean == 0.0:
            x = torch.randn(*shape, device=DEV, generator=self.g, dtype=self.dtype)
            return x.mul_(std) if std != 1.0 else x
        return (self.f32(*shape, std=std) + mean).to(self.dtype)

    def uniform(self, *shape, lo=0.0, hi=1.0):
        return torch.rand(*shape, device=DEV, generator=self.g).mul_(hi - lo).add_(lo)


def _dims(case):
    d, d_ff = MODELS[case["model"]]
    return H.hero_dims(d=d, d_ff=d_ff, d_r=case["d_r"], L_R=case["L"], d_m=case["d_m"], d_s=D_S, d_h=D_H, d_a=D_A,
                       d_e=D_E, d_p=D_P, d_head=D_HEAD, dtype=H.HERO_BF16 if case["dtype"] == "bf16" else H.HERO_F32,
                       eps_norm=EPS_NORM, eps=EPS, T_hist=T_HIST,
                       state_dtype=H.HERO_BF16 if case["memory"] == "bf16" else H.HERO_F32)


def _router(r, case):
    d, d_m = MODELS[case["model"]][0], case["d_m"]
    pitch = (D_S + d_m + 1 + 7) // 8 * 8
    shapes = dict(w_hd=(D_E, d), w_hu=(D_H, D_E), w_p1=(D_P, 6), w_p2=(D_A, D_P), w_q=(d_m, D_S), w_k=(d_m, D_S),
                  w_v=(d_m, D_S), w_n=(d_m, D_S), w_c=(d_m, d_m), th1=(D_HEAD, pitch), th2=(D_HEAD,), ps1=(D_HEAD, d),
                  ps2=(D_HEAD,))
    w = {k: r.store(*s, std=0.02) for k, s in shapes.items()}
    w["th1"][:, D_S + d_m + 1:] = 0
    return w


def _ffn(r, case, std_out):
    d, d_ff = MODELS[case["model"]]
    return dict(norm_w=r.store(d, std=0.02, mean=1.0), w_gate=r.store(d_ff, d, std=0.02),
                w_up=r.store(d_ff, d, std=0.02), w_down=r.store(d, d_ff, std=std_out),
                w1=r.store(case["d_r"], d, std=0.02), w2=r.store(d, case["d_r"], std=std_out))


def _pairs(r, case, T):
    """phi(k) and v of the routed layers before this one."""
    n = case["j"] - 1
    return r.f32(T, n, case["d_m"], std=0.5).exp_(), r.f32(T, n, case["d_m"])


def _decays(n):
    rho = 1.0 / (1.0 + math.exp(-ETA))
    return torch.tensor([rho ** (n - 1 - i) for i in range(n)], dtype=torch.float64, device=DEV)


def _memory(a, b, dtype):
    """S and zeta after the layers whose pairs these are."""
    n, T, d_m = a.shape[1], a.shape[0], a.shape[2]
    if n == 0:
        return torch.zeros(T, d_m, d_m, device=DEV, dtype=dtype), torch.zeros(T, d_m, device=DEV, dtype=dtype)
    aw = a.to(dtype) * _decays(n).to(dtype)[None, :, None]
    return torch.bmm(aw.transpose(1, 2).contiguous(), b.to(dtype)), aw.sum(1)


def _bias(r, case):
    """A logit bias that puts floor(skip T + 1/2) tokens on the adapter's side, by runs of positions."""
    T, n_skip = case["T"], _n_skip(case)
    run = RUN if T > 256 else 1
    n_runs = (T + run - 1) // run
    order = torch.rand(n_runs, device=DEV, generator=r.g).argsort()
    rank = torch.empty_like(order)
    rank[order] = torch.arange(n_runs, device=DEV)
    place = rank.repeat_interleave(run)[:T].argsort(stable=True)   # tokens, run after run in the drawn order
    sign = torch.ones(T, device=DEV)
    sign[place[:n_skip]] = -1.0
    return sign * (2.5 + r.f32(T).abs_())


def _layer_inputs(case, seed):
    """Everything one layer call reads, as tensors (exact() computes from these too)."""
    r = _Draw(seed, case["dtype"])
    T, j, d = case["T"], case["j"], MODELS[case["model"]][0]
    x = dict(hbar=r.store(T, d), router=_router(r, case), bias=_bias(r, case), prev1=None, prev2=None)
    if j >= 2:
        x["prev1"] = (x["hbar"].float() - r.f32(T, d, std=0.5)).to(r.dtype)
    if j >= 3:
        x["prev2"] = (x["prev1"].float() - r.f32(T, d, std=0.5)).to(r.dtype)
    x["ka"], x["vb"] = _pairs(r, case, T)
    x["p"] = r.uniform(T, lo=0.2, hi=0.8) if j > 1 else torch.ones(T, device=DEV)
    x["m"] = r.uniform(T) * x["p"] if j > 1 else torch.ones(T, device=DEV)
    if case["memory"] != "history":
        x["S"], x["zeta"] = _memory(x["ka"], x["vb"], torch.float32)
        if case["memory"] == "bf16":
            x["S"] = x["S"].to(torch.bfloat16)
    x["ffn"] = _ffn(r, case, 0.02)
    return x


def _ptrs(w, names):
    return [w[n].data_ptr() for n in names]


def _ffn_struct(dims, f, tiled):
    s = H.hero_ffn_weights(*_ptrs(f, ("norm_w", "w_gate", "w_up", "w_down")))
    if tiled:
        f["gu_t"] = torch.empty(2 * f["w_gate"].numel(), dtype=f["w_gate"].dtype, device=DEV)
        f["dn_t"] = torch.empty(f["w_down"].numel(), dtype=f["w_down"].dtype, device=DEV)
        H.check(H.hero_ffn_decode_weights_make(dims, s, f["gu_t"], f["dn_t"], _stream()), "decode weights")
        s.w_gate_up_tiled, s.w_down_tiled = f["gu_t"].data_ptr(), f["dn_t"].data_ptr()
    return s


def _stream():
    return torch.cuda.current_stream().cuda_stream


class _Stats:
    """The optional per-layer outputs, a row a layer."""

    def __init__(self, case, layers):
        T, n_skip = case["T"], _n_skip(case)
        P = (T + 63) // 64 * 64
        new = lambda dt, w=P: torch.zeros(layers, w, dtype=dt, device=DEV)   # noqa: E731
        self.mask, self.ffn, self.ad, self.counts = new(torch.uint8), new(torch.int32), new(torch.int32), new(torch.int32, 4)
        self.logit, self.gate, self.lam = new(torch.float32), new(torch.float32), new(torch.float32, 4)
        self.structs = [H.hero_layer_stats(*(t[l].data_ptr() for t in (self.mask, self.ffn, self.ad, self.counts,
                                                                        self.logit, self.gate, self.lam)))
                        for l in range(layers)]
        self.out = dict(mask=self.mask[:, :T], idx_ffn=self.ffn[:, :T - n_skip], idx_ad=self.ad[:, :n_skip],
                        counts=self.counts[:, :2], logit=self.logit[:, :T], gate=self.gate[:, :T], lam=self.lam[:, :1])


def _routing(case, bias):
    budget = case["mode"] == "budget"
    return H.hero_routing(H.HERO_MODE_BUDGET if budget else H.HERO_MODE_THRESHOLD, 0.5, case["skip"],
                          bias.data_ptr(), 0)


def _prepare_layer(case, seed):
    x = _layer_inputs(case, seed)
    dims, T, j = _dims(case), case["T"], case["j"]
    s = dict(case=case, x=x, dims=dims, h=torch.empty_like(x["hbar"]), stats=_Stats(case, 1))
    if case["memory"] == "history":
        x["kv"] = torch.zeros(T, case["L"], 2, case["d_m"], device=DEV)
        x["kv"][:, :j - 1, 0], x["kv"][:, :j - 1, 1] = x["ka"], x["vb"]
        s["mem"] = H.hero_history(*_ptrs(x, ("kv", "p", "m")))
    else:
        s["mem"] = H.hero_state(*_ptrs(x, ("S", "zeta", "p", "m")))
    del x["ka"], x["vb"]
    s["ffn"] = _ffn_struct(dims, x["ffn"], case["tiled"])
    s["router"] = H.hero_router_weights(*_ptrs(x["router"], H.ROUTER_FIELDS))
    s["adapter"] = H.hero_adapter_weights(*_ptrs(x["ffn"], ("w1", "w2")))
    s["routing"] = _routing(case, x["bias"])
    if case["kind"] != "layer_noalloc":
        s["ws_bytes"] = H.hero_workspace_size(dims, T, False)
        s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=DEV)
    return s


def _run_layer(s):
    case, x = s["case"], s["x"]
    args = (s["dims"], case["j"], case["T"], x["hbar"], x["prev1"], x["prev2"], s["h"], s["mem"], s["ffn"], s["router"],
            s["adapter"])
    stats = s["stats"]
    if case["memory"] == "history":
        H.check(H.hero_routed_layer_hist(*args, [ETA] * case["j"], s["routing"], stats.structs[0], s["ws"],
                                         s["ws_bytes"], _stream()), "layer")
        return dict(stats.out, h=s["h"], kv=x["kv"], p=x["p"], m=x["m"])
    if case["kind"] == "layer_noalloc":
        H.check(H.hero_routed_layer_noalloc(*args, ETA, s["routing"], stats.structs[0], _stream()), "layer")
    else:
        H.check(H.hero_routed_layer(*args, ETA, s["routing"], stats.structs[0], s["ws"], s["ws_bytes"], _stream()),
                "layer")
    return dict(stats.out, h=s["h"], S=x["S"], zeta=x["zeta"], p=x["p"], m=x["m"])


def _stack_inputs(case, seed):
    r = _Draw(seed, case["dtype"])
    d = MODELS[case["model"]][0]
    x = dict(hbar=r.store(case["T"], d), router=_router(r, case), bias=_bias(r, case))
    std = 0.02 / math.sqrt(2.0 * case["L"])
    x["ffn"] = (_ffn(r, case, std) for _ in range(case["L"]))
    return x


def _prepare_stack(case, seed):
    x = _stack_inputs(case, seed)
    x["ffn"] = list(x["ffn"])
    dims, T, d_m = _dims(case), case["T"], case["d_m"]
    s = dict(case=case, x=x, dims=dims, h=torch.empty_like(x["hbar"]), stats=_Stats(case, case["L"]))
    st = s["state"] = dict(S=torch.zeros(T, d_m, d_m, device=DEV), zeta=torch.zeros(T, d_m, device=DEV),
                           p=torch.ones(T, device=DEV), m=torch.ones(T, device=DEV))
    s["mem"] = H.hero_state(*_ptrs(st, ("S", "zeta", "p", "m")))
    s["ffn"] = [_ffn_struct(dims, f, case["tiled"]) for f in x["ffn"]]
    s["adapter"] = [H.hero_adapter_weights(*_ptrs(f, ("w1", "w2"))) for f in x["ffn"]]
    s["router"] = H.hero_router_weights(*_ptrs(x["router"], H.ROUTER_FIELDS))
    s["routing"] = _routing(case, x["bias"])
    s["ws_bytes"] = H.hero_workspace_size(dims, T, True)
    s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=DEV)
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _call_stack(s)
        torch.cuda.current_stream().wait_stream(side)
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _call_stack(s)
    return s


def _call_stack(s):
    H.check(H.hero_routed_stack(s["dims"], s["case"]["T"], s["x"]["hbar"], s["h"], s["mem"], s["ffn"], s["router"],
                                s["adapter"], [ETA] * s["case"]["L"], s["routing"], s["stats"].structs, s["ws"],
                                s["ws_bytes"], _stream()), "stack")


def _run_stack(s):
    if s["case"]["graph"]:
        s["graph"].replay()
    else:
        _call_stack(s)
    return dict(s["stats"].out, h=s["h"], **s["state"])


def _attention_inputs(case, seed):
    r = _Draw(seed, "bf16")
    d, hd = MODELS[case["model"]][0], 128
    return dict(h=r.store(case["T"], d), norm_w=r.store(d, std=0.02, mean=1.0),
                w_qkv=r.store((case["n_heads"] + 2 * case["n_kv"]) * hd, d, std=0.02),
                w_o=r.store(d, case["n_heads"] * hd, std=0.02),
                inv_freq=[500000.0 ** (-2.0 * i / hd) for i in range(hd // 2)])


def _prepare_attention(case, seed):
    x = _attention_inputs(case, seed)
    s = dict(case=case, x=x, dims=_dims(case), adims=H.hero_attn_dims(case["n_heads"], case["n_kv"], 128),
             hbar=torch.empty_like(x["h"]), seq=case["T"] // case["batch"])
    s["w"] = H.hero_attn_weights(*_ptrs(x, ("norm_w", "w_qkv", "w_o")))
    s["ws_bytes"] = H.hero_decoder_workspace_size(s["dims"], s["adims"], 0, case["batch"], s["seq"])
    s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=DEV)
    return s


def _run_attention(s):
    H.check(H.hero_attention_block(s["dims"], s["adims"], s["case"]["batch"], s["seq"], s["x"]["h"], s["hbar"], s["w"],
                                   s["x"]["inv_freq"], s["ws"], s["ws_bytes"], _stream()), "attention")
    return s["hbar"]


def _block_inputs(case, seed):
    r = _Draw(seed, "bf16")
    T, d = case["T"], MODELS[case["model"]][0]
    x = dict(hbar=r.store(T, d), dh=r.store(T, d), gate=r.uniform(T, lo=0.02, hi=0.98))
    place = torch.rand(T, device=DEV, generator=r.g).argsort()
    n = _n_skip(case)
    x["idx_ad"], x["idx_ffn"] = place[:n].sort().values, place[n:].sort().values
    x["ffn"] = _ffn(r, case, 0.02)
    return x


def _prepare_block(case, seed):
    x = _block_inputs(case, seed)
    dims, T = _dims(case), case["T"]
    d, d_ff = MODELS[case["model"]]
    f = x["ffn"]
    s = dict(case=case, x=x, dims=dims)
    s["ffn"] = H.hero_ffn_weights(*_ptrs(f, ("norm_w", "w_gate", "w_up", "w_down")))
    f["down_t"] = torch.empty(d_ff, d, dtype=torch.bfloat16, device=DEV)
    f["gu_t"] = torch.empty(d, 2 * d_ff, dtype=torch.bfloat16, device=DEV)
    H.check(H.hero_ffn_backward_weights_make(dims, s["ffn"], f["down_t"], f["gu_t"], _stream()), "backward weights")
    s["ffn_t"] = H.hero_ffn_backward_weights(*_ptrs(f, ("down_t", "gu_t")))
    s["adapter"] = H.hero_adapter_weights(*_ptrs(f, ("w1", "w2")))
    idx = s["idx"] = {}
    for k in ("idx_ffn", "idx_ad"):
        idx[k] = torch.zeros(T, dtype=torch.int32, device=DEV)
        idx[k][:x[k].numel()] = x[k].int()
    s["counts"] = torch.tensor([T - _n_skip(case), _n_skip(case), 0, 0], dtype=torch.int32, device=DEV)
    s["routing"] = H.hero_routing(H.HERO_MODE_BUDGET if case["mode"] == "budget" else H.HERO_MODE_THRESHOLD, 0.5,
                                  case["skip"], None, 0)
    new = lambda *sh: torch.zeros(*sh, device=DEV)   # noqa: E731
    s["out"] = dict(dhbar=torch.empty_like(x["hbar"]), dgate=new(T), dlogit=new(T), dw1=new(case["d_r"], d),
                    dw2=new(d, case["d_r"]))
    s["grads"] = H.hero_block_grads(*_ptrs(s["out"], ("dhbar", "dgate", "dlogit", "dw1", "dw2")))
    s["ws_bytes"] = H.hero_backward_workspace_size(dims, T)
    s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=DEV)
    return s


def _run_block(s):
    x = s["x"]
    H.check(H.hero_routed_block_backward(s["dims"], s["case"]["T"], x["hbar"], x["dh"], x["gate"], s["idx"]["idx_ffn"],
                                         s["idx"]["idx_ad"], s["counts"], s["routing"], None, s["ffn"], s["ffn_t"],
                                         s["adapter"], s["grads"], s["ws"], s["ws_bytes"], _stream()), "block backward")
    return s["out"]


def _router_bwd_inputs(case, seed):
    r = _Draw(seed, "bf16")
    T, d, d_m = case["T"], MODELS[case["model"]][0], case["d_m"]
    x = dict(hbar=r.store(T, d), router=_router(r, case))
    x["prev1"] = (x["hbar"].float() - r.f32(T, d, std=0.5)).to(r.dtype)
    x["prev2"] = (x["prev1"].float() - r.f32(T, d, std=0.5)).to(r.dtype)
    ka, vb = _pairs(r, case, T)
    x["S"], x["zeta"] = _memory(ka, vb, torch.float32)
    x["p"] = r.uniform(T, lo=0.2, hi=0.8)
    x["m"] = r.uniform(T) * x["p"]
    x["dlogit"], x["dS"] = r.f32(T), r.f32(T, d_m, d_m, std=0.05)
    x["dzeta"], x["dp"], x["dm"] = r.f32(T, d_m, std=0.1), r.f32(T, std=0.1), r.f32(T, std=0.1)
    return x


def _prepare_router_bwd(case, seed):
    x = _router_bwd_inputs(case, seed)
    dims, T, d = _dims(case), case["T"], MODELS[case["model"]][0]
    s = dict(case=case, x=x, dims=dims)
    with torch.no_grad():   # the forward's memory read, which a training program has kept
        s["c_read"] = _router_forward(case, _wide(x))["c"].float().contiguous()
    s["state"] = H.hero_state(*_ptrs(x, ("S", "zeta", "p", "m")), s["c_read"].data_ptr())
    s["router"] = H.hero_router_weights(*_ptrs(x["router"], H.ROUTER_FIELDS))
    s["carry"] = H.hero_router_carry(*_ptrs(x, ("dS", "dzeta", "dp", "dm")))
    s["dh"] = [torch.zeros(T, d, device=DEV) for _ in range(3)]
    s["g"] = {k: torch.zeros(v.shape, device=DEV) for k, v in x["router"].items()}
    s["grads"] = H.hero_router_grads(*_ptrs(s["g"], H.ROUTER_FIELDS))
    s["deta"] = torch.zeros(4, device=DEV)
    s["ws_bytes"] = H.hero_router_backward_workspace_size(dims, T)
    s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=DEV)
    return s


def _run_router_bwd(s):
    x, case = s["x"], s["case"]
    H.check(H.hero_router_backward(s["dims"], case["j"], case["T"], x["hbar"], x["prev1"], x["prev2"], s["state"],
                                   s["router"], ETA, x["dlogit"], s["carry"], *s["dh"], s["grads"], s["deta"], s["ws"],
                                   s["ws_bytes"], _stream()), "router backward")
    return dict(s["g"], dh0=s["dh"][0], dh1=s["dh"][1], dh2=s["dh"][2], deta=s["deta"][:1],
                **{k: x[k] for k in ("dS", "dzeta", "dp", "dm")})


_PREPARE = {"layer": _prepare_layer, "layer_noalloc": _prepare_layer, "stack": _prepare_stack,
            "attention": _prepare_attention, "block_backward": _prepare_block, "router_backward": _prepare_router_bwd}
_RUN = {"layer": _run_layer, "layer_noalloc": _run_layer, "stack": _run_stack, "attention": _run_attention,
        "block_backward": _run_block, "router_backward": _run_router_bwd}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    return _RUN[state["case"]["kind"]](state)


# ---- what a pass cannot do without ------------------------------------------------------------------------------


def _layer_work(case, j):
    T, n_ad = case["T"], _n_skip(case)
    n_ffn, (d, d_ff), r, m = T - n_ad, MODELS[case["model"]], case["d_r"], case["d_m"]
    e = 2 if case["dtype"] == "bf16" else 4
    w_router = D_E * d + D_H * D_E + D_P * 6 + D_A * D_P + 4 * m * D_S + m * m + D_HEAD * (D_S + m + 2) + D_HEAD * (d + 1)
    b = e * (w_router + d + (3 * d * d_ff if n_ffn else 0) + (2 * d * r if n_ad else 0))
    b += T * e * d * (1 + min(j, 3))                       # hbar and the earlier states in, h out
    if case["memory"] == "history":
        b += T * 4 * 2 * m * j
    else:
        b += T * (2 if j > 1 else 1) * (m * m * (2 if case["memory"] == "bf16" else 4) + 4 * m)
    b += T * (4 * 4 + 4 + 1 + 4 + 8)                       # p, m both ways, bias, mask, index, logit, gate
    f = n_ffn * 6.0 * d * d_ff + n_ad * 4.0 * d * r + T * (2.0 * w_router + 6.0 * m * m)
    return b, f


def work(case):
    kind, T, (d, d_ff) = case["kind"], case["T"], MODELS[case["model"]]
    if kind in ("layer", "layer_noalloc"):
        b, f = _layer_work(case, case["j"])
    elif kind == "stack":
        each = [_layer_work(case, j) for j in range(1, case["L"] + 1)]
        b, f = sum(x[0] for x in each), sum(x[1] for x in each)
    elif kind == "attention":
        nq, nkv, seq = case["n_heads"] * 128, case["n_kv"] * 128, T // case["batch"]
        b = 2 * (2 * T * d + (2 * nq + 2 * nkv) * d)
        f = 2.0 * T * d * (2 * nq + 2 * nkv) + 4.0 * 128 * case["n_heads"] * case["batch"] * seq * (seq + 1) / 2
    elif kind == "block_backward":
        n_ad = _n_skip(case)
        b = 2 * (3 * T * d + 3 * d * d_ff + 2 * d * case["d_r"]) + 4 * 2 * d * case["d_r"] + T * 16
        f = (T - n_ad) * 10.0 * d * d_ff + n_ad * 10.0 * d * case["d_r"]
    else:
        m = case["d_m"]
        w = (D_E + D_HEAD) * d + 4 * m * D_S + m * m + D_HEAD * (D_S + m)
        b = T * (4 * 3 * m * m + 3 * 2 * d + 3 * 4 * d) + 6 * w
        f = T * (6.0 * w + 10.0 * m * m)
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """About four times the distance from exact(): 8 significant bits of the stored hidden states and of the products'
    operands, gathered over depth in a stack; 32-bit sums in the fp32 path and in the router's backward."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["kind"] == "router_backward":
        return {"rel": 2e-5}
    return {"rel": 3e-2 if case["kind"] == "stack" else 1.2e-2}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------


def _wide(x):
    """The tensors of x in float64."""
    if isinstance(x, dict):
        return {k: _wide(v) for k, v in x.items()}
    return x.double() if isinstance(x, torch.Tensor) and x.is_floating_point() else x


def _silu(x):
    return x * torch.sigmoid(x)


def _phi(x):
    return torch.where(x > 0, x + 1.0, torch.exp(x.clamp(max=0.0)))


def _rms(h):
    return h * torch.rsqrt((h * h).mean(-1, keepdim=True) + EPS_NORM)


def _cos(a, b):
    return (a * b).sum(-1) / (a.norm(dim=-1) * b.norm(dim=-1) + EPS)


def _router_forward(case, x, j=None, eta=None):
    """The router of layer j on float64 tensors: c, the new state and the logit without its bias."""
    j = case["j"] if j is None else j
    R, hbar, T, m, L = x["router"], x["hbar"], case["T"], case["d_m"], case["L"]
    z_h = _silu(_rms(hbar) @ R["w_hd"].T) @ R["w_hu"].T
    zero = torch.zeros(T, dtype=torch.float64, device=DEV)
    d_j = gam = zero
    if j >= 2:
        delta = hbar - x["prev1"]
        d_j = delta.norm(dim=-1)
        if j >= 3:
            gam = _cos(delta, x["prev1"] - x["prev2"])
    path = torch.stack([zero + j / L, zero + (L - j) / L, d_j, gam, x["p"], x["m"]], -1)
    s = torch.cat([z_h, _silu(path @ R["w_p1"].T) @ R["w_p2"].T], -1)
    q, k, v = (s @ R[n].T for n in ("w_q", "w_k", "w_v"))
    fq, fk = _phi(q), _phi(k)
    rho = 1.0 / (1.0 + math.exp(-ETA)) if eta is None else torch.sigmoid(eta)
    if j == 1:
        c, nu = torch.zeros_like(q), zero
        S, zeta = fk[:, :, None] * v[:, None, :], fk
    else:
        c = torch.bmm(fq[:, None, :], x["S"])[:, 0] / ((fq * x["zeta"]).sum(-1, keepdim=True) + EPS)
        nu = 1.0 - _cos(s @ R["w_n"].T, c @ R["w_c"].T)
        S, zeta = rho * x["S"] + fk[:, :, None] * v[:, None, :], rho * x["zeta"] + fk
    n_in = D_S + m + 1
    a = _silu(torch.cat([s, c, nu[:, None]], -1) @ R["th1"][:, :n_in].T) @ R["th2"]
    p = torch.sigmoid(a / T_HIST)
    b = _silu(hbar @ R["ps1"].T) @ R["ps2"]
    return dict(c=c, fk=fk, v=v, S=S, zeta=zeta, p=p, m=x["m"] * p, logit=a + b)


def _branches(case, hbar, gate, ffn, idx_f, idx_a):
    """hbar + g FFN(u) on the rows idx_f, hbar + (1 - g) Adapter(u) on idx_a; ffn holds stored weights."""
    u = _rms(hbar) * ffn["norm_w"].double()
    h = hbar.clone()
    if idx_f.numel():
        uf = u[idx_f]
        act = _silu(uf @ ffn["w_gate"].double().T) * (uf @ ffn["w_up"].double().T)
        h = h.index_add(0, idx_f, gate[idx_f, None] * (act @ ffn["w_down"].double().T))
    if idx_a.numel():
        hid = _silu(u[idx_a] @ ffn["w1"].double().T)
        h = h.index_add(0, idx_a, (1.0 - gate[idx_a, None]) * (hid @ ffn["w2"].double().T))
    return h


def _decide(case, logit):
    """Mask, both index lists and lambda by the call's rule."""
    T, n_skip = case["T"], _n_skip(case)
    if case["mode"] == "threshold":
        mask, lam = logit >= 0.0, torch.zeros(1, dtype=torch.float64, device=DEV)
    else:
        order = logit.sort(stable=True)
        mask = torch.ones(T, dtype=torch.bool, device=DEV)
        mask[order.indices[:n_skip]] = False
        lam = order.values[n_skip:n_skip + 1] if n_skip < T else torch.full((1,), math.inf, dtype=torch.float64, device=DEV)
    return mask, mask.nonzero()[:, 0], (~mask).nonzero()[:, 0], lam


def _exact_layer(case, x, j, ffn):
    R = _router_forward(case, x, j)
    logit = R["logit"] + x["bias"]
    gate = torch.sigmoid(logit)
    mask, idx_f, idx_a, lam = _decide(case, logit)
    h = _branches(case, x["hbar"], gate, ffn, idx_f, idx_a)
    counts = torch.tensor([idx_f.numel(), idx_a.numel()], dtype=torch.int32, device=DEV)
    stats = dict(mask=mask.to(torch.uint8), idx_ffn=idx_f.int(), idx_ad=idx_a.int(), counts=counts, logit=logit, gate=gate,
                 lam=lam)
    return R, h, stats


def exact(case, seed):
    with torch.no_grad():
        if case["kind"] in ("layer", "layer_noalloc"):
            x = _layer_inputs(case, seed)
            ffn, ka, vb = x.pop("ffn"), x.pop("ka"), x.pop("vb")
            x = _wide(x)
            if case["memory"] == "history":
                x["S"], x["zeta"] = _memory(ka, vb, torch.float64)
            R, h, stats = _exact_layer(case, x, case["j"], ffn)
            out = dict({k: v[None] for k, v in stats.items()}, h=h, p=R["p"], m=R["m"])
            if case["memory"] == "history":
                kv = torch.zeros(case["T"], case["L"], 2, case["d_m"], dtype=torch.float64, device=DEV)
                n = case["j"] - 1
                kv[:, :n, 0], kv[:, :n, 1], kv[:, n, 0], kv[:, n, 1] = ka, vb, R["fk"], R["v"]
                return dict(out, kv=kv)
            return dict(out, S=R["S"], zeta=R["zeta"])
        if case["kind"] == "stack":
            x = _stack_inputs(case, seed)
            ffn = x.pop("ffn")
            x = _wide(x)
            x.update(prev1=None, prev2=None, p=torch.ones(case["T"], dtype=torch.float64, device=DEV),
                     m=torch.ones(case["T"], dtype=torch.float64, device=DEV))
            rows = []
            for j, f in enumerate(ffn, 1):
                R, h, stats = _exact_layer(case, x, j, f)
                rows.append(stats)
                x.update(hbar=h, prev1=x["hbar"], prev2=x["prev1"], S=R["S"], zeta=R["zeta"], p=R["p"], m=R["m"])
            return dict({k: torch.stack([s[k] for s in rows]) for k in rows[0]}, h=x["hbar"], S=x["S"], zeta=x["zeta"],
                        p=x["p"], m=x["m"])
        if case["kind"] == "attention":
            return _exact_attention(case, _attention_inputs(case, seed))
    if case["kind"] == "block_backward":
        x = _block_inputs(case, seed)
        hbar, gate = x["hbar"].double().requires_grad_(), x["gate"].double().requires_grad_()
        f = dict(x["ffn"], w1=x["ffn"]["w1"].double().requires_grad_(), w2=x["ffn"]["w2"].double().requires_grad_())
        h = _branches(case, hbar, gate, f, x["idx_ffn"], x["idx_ad"])
        g = torch.autograd.grad((h * x["dh"].double()).sum(), (hbar, gate, f["w1"], f["w2"]), allow_unused=True)
        g = [torch.zeros_like(w) if v is None else v for v, w in zip(g, (hbar, gate, f["w1"], f["w2"]))]
        gd = gate.detach()
        return dict(dhbar=g[0], dgate=g[1], dlogit=g[1] * gd * (1.0 - gd), dw1=g[2], dw2=g[3])
    x = _wide(_router_bwd_inputs(case, seed))
    names = list(H.ROUTER_FIELDS)
    leaves = [x["router"][n] for n in names] + [x[n] for n in ("hbar", "prev1", "prev2", "S", "zeta", "p", "m")]
    eta = torch.tensor([ETA], dtype=torch.float64, device=DEV)
    leaves.append(eta)
    for t in leaves:
        t.requires_grad_()
    R = _router_forward(case, x, eta=eta)
    J = sum((R[a] * x[b]).sum() for a, b in (("logit", "dlogit"), ("S", "dS"), ("zeta", "dzeta"), ("p", "dp"), ("m", "dm")))
    g = torch.autograd.grad(J, leaves)
    keys = names + ["dh0", "dh1", "dh2", "dS", "dzeta", "dp", "dm", "deta"]
    return dict(zip(keys, g))


def _exact_attention(case, x):
    nh, nkv, hd, B, seq = case["n_heads"], case["n_kv"], 128, case["batch"], case["T"] // case["batch"]
    h = x["h"].double()
    qkv = (_rms(h) * x["norm_w"].double()) @ x["w_qkv"].double().T
    freq = torch.tensor(x["inv_freq"], dtype=torch.float32).double().to(DEV)   # the entry point takes float32
    ang = torch.arange(seq, dtype=torch.float64, device=DEV)[:, None] * freq
    cos, sin = ang.cos(), ang.sin()

    def turned(y):
        a, b = y[..., 0::2], y[..., 1::2]
        return torch.stack([a * cos - b * sin, a * sin + b * cos], -1).flatten(-2)

    q, k, v = (t.reshape(B, seq, -1, hd).transpose(1, 2).contiguous() for t in qkv.split([nh * hd, nkv * hd, nkv * hd], 1))
    q, k = turned(q), turned(k)
    o = torch.empty(B, seq, nh * hd, dtype=torch.float64, device=DEV)
    hidden = torch.ones(seq, seq, dtype=torch.bool, device=DEV).triu(1)
    for b in range(B):
        for n in range(nh):
            g = n // (nh // nkv)
            p = ((q[b, n] @ k[b, g].T) / math.sqrt(hd)).masked_fill(hidden, -math.inf).softmax(-1)
            o[b, :, n * hd:(n + 1) * hd] = p @ v[b, g]
    return h + o.reshape(B * seq, -1) @ x["w_o"].double().T
