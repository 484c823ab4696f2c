"""The work that a user of this library has it do, as measurable cases.

A pass starts where a serving or training step hands over to the library: the batch's token -> (adapter, kind) arrays,
the activations and the adapters lie in device memory, and the step calls the segment builder and then the LoRA update of
its linear layers.  Every case is a plain dict; `what` names the calls of its pass:

  linear    segment builder + the forward of one linear layer
  layer     segment builder + the forward of a decoder layer's seven linears as four calls (q,k,v and gate,up read one x
            each, o and down their own)
  backward  the gradients of such a layer's linears on the fine-tune rows (segment tables and saved h in hand)
  train     segment builder + dropout + forward + backward + dropout of the input gradient for one linear layer: a
            fine-tuning step of a module as an autograd function would issue it
  rows      kind offsets + split of a projection's rows by kind + concatenation (around the attention of a mixed batch)

and the rest of it the sizes: `ft` fine-tune rows as `ft_seqs` sequences, `prefill` requests of `prefill_len` rows,
`decode` rows; `zipf` rows with segment lengths drawn from a truncated Zipf law; `adapters` adapters whose ranks cycle
through `ranks`; `shuffle`: rows in arrival order instead of the batch order fine-tune | prefill | decode; `drop`: share
of the rows without an adapter; `per_request_scale`: the dynamic scale, one value per request.

Calls of a loop that repeats on fixed buffers (serving, the layer stack) are prepared once, the rest is called directly.
The library's own choice of kernel (LQ_VARIANT_AUTO) is used throughout.
"""
import math

import numpy as np
import torch

from paper_2511_00101_amd import binding as lq
from paper_2511_00101_amd import synth

FT, PREFILL, DECODE = synth.KIND_FINETUNE, synth.KIND_PREFILL, synth.KIND_DECODE
LAYER = {name: (d_in, d_out) for name, d_in, d_out in synth.LAYER_PROJECTIONS}
GROUPS = (("q", "k", "v"), ("o",), ("gate", "up"), ("down",))   # the projections of a group read one x

_BASE = dict(what="linear", d_in=4096, d_out=4096, ft=0, ft_seqs=1, prefill=0, prefill_len=64, decode=0, zipf=0, adapters=16, ranks="16",
             shuffle=False, drop=0.0, per_request_scale=False, dropout=0.0)


def _case(**kw):
    return dict(_BASE, **kw)


def listed():
    return [
        # a few requests on a small layer: nothing but launches and latency
        _case(name="tiny", d_in=256, d_out=256, ft=64, prefill=1, prefill_len=32, decode=6, adapters=4, ranks="8"),
        # interactive serving, a decode step of sixteen requests through one decoder layer
        _case(name="decode_layer_16", what="layer", decode=16, adapters=16, ranks="16"),
        # a busy server's decode step: 256 requests over 64 adapters, one layer's attention projection
        _case(name="decode_256", decode=256, adapters=64, ranks="16"),
        # a unified step: two fine-tune sequences, eight prefills and 256 decodes in one batch
        _case(name="unified", ft=4096, ft_seqs=2, prefill=8, prefill_len=64, decode=256, adapters=32, ranks="16"),
        # the same kind of step through a whole decoder layer at rank 32
        _case(name="unified_layer", what="layer", ft=4096, ft_seqs=2, prefill=16, prefill_len=64, decode=512, adapters=16, ranks="32"),
        # an MLP of a server with many users: Zipf-distributed request lengths, adapters of different ranks
        _case(name="zipf_mlp_up", d_in=4096, d_out=11008, zipf=8192, adapters=32, ranks="8,16,32,64"),
        _case(name="zipf_mlp_down", d_in=11008, d_out=4096, zipf=8192, adapters=32, ranks="8,16,32,64"),
        # long prompts: 8 x 2048 prefill rows with larger adapters
        _case(name="prefill_16k", d_in=4096, d_out=4096, prefill=8, prefill_len=2048, adapters=8, ranks="64"),
        # the backward of the unified step's decoder layer
        _case(name="backward_layer", what="backward", ft=4096, ft_seqs=2, prefill=16, prefill_len=64, decode=512, adapters=16, ranks="32"),
        # fine-tuning one module with the paper's LoRA configuration (rank 8, dropout 0.05)
        _case(name="train_dropout", what="train", ft=2048, ft_seqs=2, adapters=2, ranks="8", dropout=0.05),
        # everything odd at once: ragged widths, ranks up to the maximum, rows in arrival order, some of them without an
        # adapter, requests with scales of their own
        _case(name="train_ragged", what="train", d_in=1032, d_out=776, ft=900, ft_seqs=5, prefill=7, prefill_len=37, decode=141, adapters=5,
              ranks="16,128,5,24,33", shuffle=True, drop=0.1, per_request_scale=True),
        # the rows of a projection split by kind for the attention kernels, and put together again
        _case(name="split_concat", what="rows", ft=4096, ft_seqs=2, prefill=8, prefill_len=64, decode=256, adapters=32, ranks="16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["linear", "linear", "linear", "layer", "backward", "train", "rows"])
    adapters = _log(rng, 1, 64)
    ranks = rng.choice(["8", "16", "32", "64", "128", "16", "32", "8,16,32,64", "16,5,24,33", "8,12,31"])
    c = _case(what=what, adapters=adapters, ranks=ranks, shuffle=rng.random() < 0.3, per_request_scale=rng.random() < 0.3,
              drop=rng.choice([0.0, 0.0, 0.1]))
    if what not in ("layer", "backward"):
        widths = [1024, 4096, 11008, 14336, 8 * _log(rng, 32, 1024)]
        c["d_in"], c["d_out"] = rng.choice(widths), rng.choice(widths)
    mix = rng.choice(["mixed", "mixed", "decode", "prefill", "finetune", "zipf"])
    if what in ("backward", "train"):
        mix = rng.choice(["mixed", "finetune"])
    most = 5000 if what in ("layer", "backward") else 12000
    T = _log(rng, 16, most)
    if mix == "zipf":
        c["zipf"] = T
    if mix == "decode":
        c["decode"] = min(T, 1024)
    if mix in ("finetune", "mixed"):
        c["ft_seqs"] = rng.randint(1, min(4, max(1, T // 8)))
        c["ft"] = T if mix == "finetune" else max(1, int(T * rng.uniform(0.3, 0.8)))
    if mix in ("prefill", "mixed"):
        left = T - c["ft"]
        c["prefill"] = max(1, min(_log(rng, 1, 64), left // 2))
        c["prefill_len"] = max(1, int(left * (0.7 if mix == "mixed" else 1.0)) // c["prefill"])
        if mix == "mixed":
            c["decode"] = max(1, left - c["prefill"] * c["prefill_len"])
    if what == "train" and rng.random() < 0.5:
        c["dropout"] = 0.05
    while work(c)["bytes"] > 1.0e9:    # no more than the largest listed case
        if what in ("layer", "backward"):
            c["adapters"] = max(1, c["adapters"] // 2)
            for rows in ("ft", "prefill_len", "decode", "zipf"):
                c[rows] = (c[rows] * 3 + 3) // 4
        else:
            c["d_in"], c["d_out"] = max(256, c["d_in"] // 16 * 8), max(256, c["d_out"] // 16 * 8)
    return c


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def _ranks(c):
    cycle = [int(r) for r in c["ranks"].split(",")]
    return [cycle[i % len(cycle)] for i in range(c["adapters"])]


def _tokens(c):
    return c["ft"] + c["prefill"] * c["prefill_len"] + c["decode"] + c["zipf"]


def _ft_rows(c):
    return c["ft"] + c["zipf"] // 10


def _adapters_in_use(c):
    """Expected number of adapters that a batch of these sizes touches: (all kinds, fine-tune rows)."""
    n, ft = c["adapters"], min(c["adapters"], c["ft_seqs"] if c["ft"] else 0)
    draws = c["decode"] + (c["zipf"] // 40)           # (a Zipf segment has some forty rows on average)
    once = max(ft, min(n, c["prefill"]))              # sequences and requests take the adapters in turn
    used = once + (n - once) * (1.0 - (1.0 - 1.0 / n) ** draws)
    return used, ft + (n - ft) * (1.0 - (1.0 - 1.0 / n) ** (c["zipf"] // 400))


def work(case):
    c = dict(_BASE, **case)
    T, n_ft = int(_tokens(c) * (1.0 - c["drop"])), int(_ft_rows(c) * (1.0 - c["drop"]))
    r = sum(_ranks(c)) / c["adapters"]
    used, used_ft = _adapters_in_use(c)
    if c["what"] == "rows":
        return {"bytes": 2 * T * c["d_in"] * 4, "flops": 0}
    groups = [[LAYER[p] for p in g] for g in GROUPS] if c["what"] in ("layer", "backward") else [[(c["d_in"], c["d_out"])]]
    n_bytes = flops = 0.0
    for g in groups:
        if c["what"] != "backward":
            n_bytes += T * g[0][0] * 2     # x, once for the projections that share it
        for d_in, d_out in g:
            adapter = r * (d_in + d_out)
            if c["what"] != "backward":
                # y read and written, the adapters in use, saved h
                n_bytes += T * d_out * 4 + used * adapter * 2 + n_ft * r * 4
                flops += 2 * T * adapter
            if c["what"] in ("backward", "train"):
                # dy, x, dx read and written, adapters, their gradients read and written, saved h
                n_bytes += n_ft * (2 * d_out + 2 * d_in + 4 * d_in) + used_ft * adapter * (2 + 8) + n_ft * r * 4
                flops += 4 * n_ft * adapter
            if c["what"] == "train" and c["dropout"]:
                n_bytes += T * d_in * 4 + n_ft * d_in * 4     # masked copy of x; mask of the input gradient in place
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    if case["what"] == "rows":
        return "exact"
    # Against the same path with its sums in another order: 5e-5 and one bf16 unit in the last place (7.8e-3 of the value)
    # where a rounding of y or dx falls the other way, 5e-6 for the fp32 outputs.  (Against 64 bits, unrounded: 1.7e-3, the
    # rounding itself.)  Rates of such flips grow with the widths, and a pass may add into a y that an earlier one rounded.
    return {"rel": 1e-3, "max": 1.6e-2}


# ---- inputs -----------------------------------------------------------------------------------------------------------
def _batch(c, rng):
    """token_adapter, token_kind and the request of every row, in batch order or in arrival order."""
    n, runs = c["adapters"], []
    if c["ft"]:
        cut = np.linspace(0, c["ft"], c["ft_seqs"] + 1).astype(int)
        runs += [(i % n, FT, int(cut[i + 1] - cut[i])) for i in range(c["ft_seqs"])]
    runs += [(i % n, PREFILL, c["prefill_len"]) for i in range(c["prefill"])]
    runs += [(int(a), DECODE, 1) for a in rng.integers(0, n, size=c["decode"])]
    if c["zipf"]:
        b = synth.batch_zipf(rng, total=c["zipf"], n_adapters=n)
        start = np.flatnonzero(np.concatenate([[True], (np.diff(b.token_adapter) != 0) | (np.diff(b.token_kind) != 0)]))
        runs += [(int(b.token_adapter[s]), int(b.token_kind[s]), int(m)) for s, m in zip(start, np.diff(np.append(start, c["zipf"])))]
    lens = np.array([m for _, _, m in runs], dtype=np.int64)
    adapter = np.repeat(np.array([a for a, _, _ in runs], dtype=np.int32), lens)
    kind = np.repeat(np.array([k for _, k, _ in runs], dtype=np.uint8), lens)
    request = np.repeat(np.arange(len(runs)), lens)
    adapter[rng.random(len(adapter)) < c["drop"]] = -1
    if c["shuffle"]:
        order = rng.permutation(len(adapter))
        adapter, kind, request = adapter[order], kind[order], request[order]
    return adapter, kind, request


def prepare(case, seed):
    c = dict(_BASE, **case)
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    adapter, kind, request = _batch(c, rng)
    T, n = len(adapter), c["adapters"]
    ranks = _ranks(c)
    top = max(ranks)

    def normal(rows, cols, std=1.0):
        return (torch.randn(rows, cols, generator=gen, device="cuda") * std).to(torch.bfloat16)

    def adapters(d_in, d_out):
        return lq.AdapterTable.from_tensors([normal(r, d_in, 0.02) for r in ranks], [normal(r, d_out, 0.02) for r in ranks],
                                            [2.0] * n)

    s = {"case": c, "ta": torch.from_numpy(adapter).cuda(), "tk": torch.from_numpy(kind).cuda()}
    s["ranks"] = torch.tensor(ranks, dtype=torch.int32, device="cuda")
    s["scales"] = None
    if c["per_request_scale"] or c["dropout"]:
        per_request = rng.choice([0.5, 1.0, 2.0], size=int(request.max()) + 1) if c["per_request_scale"] else np.full(int(request.max()) + 1, 2.0)
        scale = per_request[request]
        scale[kind == FT] /= 1.0 - c["dropout"]      # the dropout's factor travels with the row's scale
        s["scales"] = torch.from_numpy(scale.astype(np.float32)).cuda()
    s["seg"] = lq.SegmentTables.empty(T, n)
    s["build_ws"] = lq.workspace(lq.lora_build_workspace_bytes(T, n))
    if c["what"] == "rows":
        s["src"], s["parts"], s["dst"] = normal(T, c["d_in"]), torch.zeros(T, c["d_in"], dtype=torch.bfloat16, device="cuda"), normal(T, c["d_in"])
        s["offsets"] = torch.zeros(4, dtype=torch.int32, device="cuda")
        lq.lora_build_segments(s["ta"], s["tk"], s["ranks"], s["seg"], s["build_ws"])
        return s
    s["build"] = lq.prepare_build_segments(s["ta"], s["tk"], s["ranks"], s["seg"], s["build_ws"])
    names = GROUPS if c["what"] in ("layer", "backward") else (("linear",),)
    h_rows = T if c["zipf"] else c["ft"]
    ws_bytes, s["groups"] = 4096, []
    for g in names:
        shapes = [LAYER.get(p, (c["d_in"], c["d_out"])) for p in g]
        d_in = shapes[0][0]
        grp = {"x": normal(T, d_in), "y": [normal(T, do) for _, do in shapes], "ad": [adapters(di, do) for di, do in shapes],
               "h": [torch.zeros(h_rows * top, device="cuda") if h_rows else None for _ in g]}   # (inference only: nothing saved)
        if c["what"] in ("backward", "train"):
            grp["dy"] = [normal(T, do) for _, do in shapes]
            grp["dx"] = [normal(T, d_in) for _ in g]
            on = sorted(set(adapter[(kind == FT) & (adapter >= 0)].tolist()))
            grp["dA"] = [{a: torch.zeros(ranks[a], di, device="cuda") for a in on} for di, _ in shapes]
            grp["dB"] = [{a: torch.zeros(ranks[a], do, device="cuda") for a in on} for _, do in shapes]
            table = lambda grads: [torch.tensor([m[a].data_ptr() if a in m else 0 for a in range(n)], dtype=torch.int64).cuda() for m in grads]
            grp["dA_ptrs"], grp["dB_ptrs"] = table(grp["dA"]), table(grp["dB"])
            ws_bytes = max([ws_bytes] + [lq.lora_workspace_bytes(T, n, top, di, do) for di, do in shapes])
            if c["what"] == "train":
                grp["xd"] = torch.zeros_like(grp["x"])
        ws_bytes = max([ws_bytes, lq.lora_forward_group_workspace_bytes(len(g), T, top)] +
                       [lq.lora_forward_workspace_bytes(T, top, di, do, lq.LQ_VARIANT_AUTO) for di, do in shapes])
        s["groups"].append(grp)
    s["ws"] = lq.workspace(ws_bytes)
    s["calls"] = []
    for g in s["groups"]:
        if len(g["y"]) > 1:
            s["calls"].append(lq.prepare_forward_group(g["x"], g["y"], g["ad"], s["seg"], g["h"], s["ws"], lq.LQ_VARIANT_AUTO,
                                                       token_scales=s["scales"]))
        else:
            s["calls"].append(lq.prepare_forward(g["x"], g["y"][0], g["ad"][0], s["seg"], g["h"][0], s["ws"], lq.LQ_VARIANT_AUTO,
                                                 token_scales=s["scales"]))
    if c["what"] == "backward":
        s["build"]()
        for call in s["calls"]:
            call()                                   # the forward that saved h
    return s


# ---- one pass ---------------------------------------------------------------------------------------------------------
def _tables(s):
    seg = s["seg"]
    return [seg.perm, seg.seg_starts, seg.seg_adapter, seg.seg_kind, seg.h_offsets, seg.n_segments]


def _backward(s, g, k, x):
    lq.lora_segmented_backward(x, g["dy"][k], g["dx"][k], g["ad"][k], g["dA_ptrs"][k], g["dB_ptrs"][k], s["seg"], g["h"][k], s["ws"],
                               lq.LQ_VARIANT_AUTO, token_scales=s["scales"])


def run(state):
    s, c = state, state["case"]
    if c["what"] == "rows":
        lq.lora_kind_offsets(s["seg"], s["offsets"])
        lq.lora_split_rows(s["src"], s["seg"], s["parts"])
        lq.lora_concat_rows(s["parts"], s["seg"], s["dst"])
        return [s["offsets"], s["parts"], s["dst"]]
    if c["what"] == "backward":
        for g in reversed(s["groups"]):
            for k in range(len(g["y"])):
                _backward(s, g, k, g["x"])
        return [[g["dx"], [list(m.values()) for m in g["dA"]], [list(m.values()) for m in g["dB"]]] for g in s["groups"]]
    s["build"]()
    if c["what"] == "train":
        g, n = s["groups"][0], c["adapters"]
        x = g["x"]
        if c["dropout"]:
            lq.lora_dropout_rows(g["x"], g["xd"], s["ta"], s["tk"], n, 1234, c["dropout"])
            x = g["xd"]
        lq.lora_segmented_forward(x, g["y"][0], g["ad"][0], s["seg"], g["h"][0], s["ws"], lq.LQ_VARIANT_AUTO, token_scales=s["scales"])
        _backward(s, g, 0, x)
        if c["dropout"]:
            lq.lora_dropout_rows(g["dx"][0], g["dx"][0], s["ta"], s["tk"], n, 1234, c["dropout"])
        return _tables(s) + [g["y"], g["h"], g["dx"], [list(m.values()) for m in g["dA"]], [list(m.values()) for m in g["dB"]]]
    for call in s["calls"]:
        call()
    return _tables(s) + [[g["y"], g["h"]] for g in s["groups"]]


# ---- the same pass in 64 bits, in plain torch ----------------------------------------------------------------------------
def _hash32(v):
    s = (v * 747796405 + 2891336453) & 0xffffffff
    w = (((s >> ((s >> 28) + 4)) ^ s) * 277803737) & 0xffffffff
    return (w >> 22) ^ w


def _kept(T, d, seed, p):
    """The dropout contract's mask: one 32-bit word per pair of columns, its halves compared with round(p 65536)."""
    key = _hash32(_hash32(torch.arange(T, device="cuda", dtype=torch.int64)) ^ seed)
    word = _hash32((key[:, None] + torch.arange(d // 2, device="cuda", dtype=torch.int64)) & 0xffffffff)
    return torch.stack([word & 0xffff, word >> 16], dim=2).reshape(T, d) >= int(round(p * 65536))


def exact(case, seed):
    c = dict(_BASE, **case)
    if c["what"] == "rows":
        return None                                       # (copies and whole numbers)
    s = prepare(case, seed)
    ranks, T = _ranks(c), len(s["ta"])
    ta, tk = s["ta"].long(), s["tk"].long()
    scale = s["scales"].double() if s["scales"] is not None else torch.full((T,), 2.0, dtype=torch.float64, device="cuda")
    live_ft = (tk == FT) & (ta >= 0)
    groups = []
    for g in s["groups"]:
        x = g["x"].double()
        keep = _kept(T, x.shape[1], 1234, c["dropout"]) | ~live_ft[:, None] if c["dropout"] else None
        if keep is not None:
            x = x * keep
        ys, hs, dxs, dAs, dBs = [], [], [], [], []
        for k, ad in enumerate(g["ad"]):
            y = g["y"][k].double() if c["what"] != "backward" else None
            h_out = torch.zeros(g["h"][k].numel(), dtype=torch.float64, device="cuda") if g["h"][k] is not None else None
            back = c["what"] in ("backward", "train")
            dx = g["dx"][k].double() if back else None
            dA, dB, at = {}, {}, 0
            for a in range(c["adapters"]):
                A, B = ad.A[a].double(), ad.B[a].double()
                for kind in ((FT,) if c["what"] == "backward" else (FT, PREFILL, DECODE)):
                    rows = torch.nonzero((ta == a) & (tk == kind)).flatten()
                    if not len(rows):
                        continue
                    h = x[rows] @ A.T
                    if y is not None:
                        y[rows] += scale[rows, None] * (h @ B)
                    if kind == FT and h_out is not None:
                        h_out[at: at + h.numel()] = h.flatten()
                        at += h.numel()
                    if kind == FT and back:
                        dy = g["dy"][k][rows].double()
                        gr = scale[rows, None] * (dy @ B.T)
                        dx[rows] += gr @ A
                        dA[a], dB[a] = gr.T @ x[rows], (scale[rows, None] * h).T @ dy
            if back and keep is not None:
                dx = dx * keep
            on = list(g["dA"][k]) if back else []
            ys.append(y), hs.append(h_out), dxs.append(dx)
            dAs.append([dA[a] for a in on]), dBs.append([dB[a] for a in on])
        groups.append([ys, hs, dxs, dAs, dBs])
    if c["what"] == "backward":
        return [g[2:] for g in groups]
    if c["what"] == "train":
        return [None] * 6 + groups[0]
    return [None] * 6 + [[g[0], g[1]] for g in groups]
