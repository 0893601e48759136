"""What the library's speed is measured on: whole expert-parallel steps through the public entry points.

A case is one step of one source rank as a program that serves or trains a mixture-of-experts model runs it:
routing table -> ep_layout -> dispatch of the token rows -> combine of the experts' outputs, which sit in a buffer
of their own (as they do behind real experts).  The kinds of step:

  decode   low-latency mode: the routing of all ranks is known, one command per row, the GPU waits for the posted
           completion counters (ep_recv_wait), nothing on the host waits
  prefill  one batch of a source rank, commands per row / per chunk / per sequenced chunk, the host waits (ep_wait)
  place    ring off: layout, placement and combine only (what a caller without a proxy runs)
  dedup    high-throughput mode with deduplication: one copy per (token, rank group), two-level reduce
  rings    high-throughput mode through the ring-buffer channels (ep_ht_dispatch)
  moved    the proxy performs the peer writes between registered heaps: one message per row out of the tokens' own
           buffer (decode sizes), or chunks out of a packed send heap (prefill sizes)

The handle (rings, proxy threads, scratch) and the workspaces a program keeps beside it (chunk rings, send heap) are
shared by all states of one case and stopped with the last of them.  Inputs, receive buffers and outputs belong to a
state.
"""
import math
import weakref

import torch

import paper_2512_19849_amd as ep
from paper_2512_19849_amd.runner import EPRunner

CMDS = {"row": ep.EP_CMD_PER_TOKEN, "chunk": ep.EP_CMD_CHUNK32, "ordered": ep.EP_CMD_CHUNK32_ORDERED,
        "none": ep.EP_CMD_NONE}


def _case(kind, T, H, E, K, R, S=1, cap=0, payload="bf16", cmds="chunk", routing="softmax", masked=0.0, group=1,
          slices=0, slots=0):
    """T tokens of a source rank, H hidden, E experts, top-K, R ranks, S sources whose routing is given; cap: the
    handle's capacity in tokens (0: T); masked: share of dropped (token, expert) pairs; group: ranks per group."""
    return dict(kind=kind, T=T, H=H, E=E, K=K, R=R, S=S, cap=cap or T, payload=payload, cmds=cmds, routing=routing,
                masked=masked, group=group, slices=slices, slots=slots)


def listed():
    return [
        # the smallest step: nothing but latency, launches and one trip through the proxy
        dict(_case("decode", 64, 1024, 16, 2, 4, cmds="row"), name="decode_tiny"),
        # a decode step of a 256-expert model over 32 ranks, routing of all 32 sources known
        dict(_case("decode", 128, 7168, 256, 8, 32, S=32, cmds="row"), name="decode_bf16"),
        # FP8 rows, 128 experts over 8 ranks, a batch that does not fill the handle's capacity
        dict(_case("decode", 57, 4096, 128, 8, 8, S=8, cap=128, payload="fp8", cmds="row"), name="decode_fp8_ragged"),
        # prefill batch of 4096 tokens with the skewed routing of real gates, chunk commands: bf16 and FP8 rows
        dict(_case("prefill", 4096, 7168, 256, 8, 16, routing="zipf"), name="prefill_bf16"),
        dict(_case("prefill", 4096, 7168, 256, 8, 16, routing="zipf", payload="fp8"), name="prefill_fp8"),
        # the largest batch: 8192 tokens, balanced routing, one command per row
        dict(_case("prefill", 8192, 4096, 128, 8, 8, routing="uniform", cmds="row"), name="prefill_large_row"),
        # a mid-sized ragged batch with sequenced chunks (the ordered high-throughput commands)
        dict(_case("prefill", 1531, 5120, 128, 6, 8, cap=2048, routing="zipf", cmds="ordered"),
             name="prefill_ordered_ragged"),
        # placement only, odd sizes, a tenth of the pairs dropped by capacity limits
        dict(_case("place", 777, 2944, 96, 6, 6, cap=1024, cmds="none", masked=0.1), name="place_ragged"),
        # high-throughput mode: deduplicated rows per destination GPU, two-level reduce
        dict(_case("dedup", 4096, 7168, 256, 8, 16, routing="zipf"), name="dedup_bf16"),
        # high-throughput mode: chunks through rings with head and tail flow control
        dict(_case("rings", 4096, 7168, 256, 8, 16, routing="zipf", slices=128, slots=2), name="rings_bf16"),
        # the proxy moves the rows: a decode step's FP8 messages, a prefill batch's bf16 chunks
        dict(_case("moved", 128, 7168, 256, 8, 32, payload="fp8", cmds="row"), name="moved_decode_fp8"),
        dict(_case("moved", 4096, 7168, 256, 8, 16, routing="zipf"), name="moved_prefill_bf16"),
    ]


def _between(rng, lo, hi, step=1):
    """Spread over the logarithm, a multiple of step."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "place", "dedup", "rings",
                       "moved", "moved"])
    E, R = rng.choice([(16, 4), (64, 8), (96, 6), (128, 8), (128, 16), (256, 16), (256, 32)])
    H = _between(rng, 1024, 8192, 128)
    K = rng.choice([2, 4, 5, 6, 8, 8, 8])
    payload = rng.choice(["bf16", "bf16", "fp8"])
    routing = rng.choice(["softmax", "zipf", "uniform"])
    masked = rng.choice([0.0, 0.0, 0.0, 0.1])
    few = 256  # tokens of a decode step, at most

    def tokens(lo, hi, heaviest=4096 * 8 * 7168):
        T = _between(rng, lo, min(hi, heaviest // (K * H)))
        return T, rng.choice([T, T, (T + 255) // 256 * 256])

    if kind == "decode":
        T, cap = tokens(1, few)
        return _case(kind, T, H, E, K, R, S=rng.choice([1, R, R]), cap=cap, payload=payload, cmds="row",
                     routing=routing, masked=masked)
    if kind == "prefill":
        T, cap = tokens(256, 8192)
        return _case(kind, T, H, E, K, R, cap=cap, payload=payload, cmds=rng.choice(["chunk", "chunk", "row", "ordered"]),
                     routing=routing, masked=masked)
    if kind == "place":
        T, cap = tokens(1, 8192)
        return _case(kind, T, H, E, K, R, cap=cap, payload=payload, cmds="none", routing=routing, masked=masked)
    if kind == "dedup":
        T, cap = tokens(256, 8192)
        return _case(kind, T, H, E, K, R, cap=cap, routing=routing, masked=masked, group=rng.choice([1, 1, 2]))
    if kind == "rings":
        T, cap = tokens(512, 4096)
        return _case(kind, T, H, E, K, min(R, 16), cap=cap, payload=payload, routing=routing, masked=masked,
                     slices=rng.choice([64, 128, 256]), slots=rng.choice([2, 4]))
    if rng.random() < 0.5:
        T, cap = tokens(1, few)
        return _case(kind, T, H, E, K, R, cap=cap, payload=payload, cmds="row", routing=routing, masked=masked)
    T, cap = tokens(256, 4096)
    return _case(kind, T, H, E, K, R, cap=cap, payload=payload, cmds=rng.choice(["chunk", "chunk", "ordered"]),
                 routing=routing, masked=masked)


def _row_bytes(H, payload):
    """Bytes of a row on its way to an expert: bf16, or E4M3 codes and one fp32 scale per 128 channels."""
    return 2 * H if payload == "bf16" else H + H // 32


def work(case):
    c = case
    T, H, K, S, NG = c["T"], c["H"], c["K"], c["S"], c["R"] // c["group"]
    rows = T * K * (1.0 - c["masked"])
    table = 12 * S * T * K + 16 * T * K          # layout in and out; (expert, row) and (weight, row) of the source
    combine = 2 * H * (rows + T)
    if c["kind"] == "dedup":
        # distinct groups a token's experts fall into, were they spread evenly
        kept = T * NG * (1.0 - (1.0 - 1.0 / NG) ** (rows / T))
        send = 2 * H * (T + kept)
        combine = 2 * H * (rows + kept) + 2 * H * (kept + T)
        table += 24 * T * K
    else:
        send = 2 * H * T + _row_bytes(H, c["payload"]) * rows
    return {"bytes": send + combine + table, "flops": 2.0 * rows * H}


def tolerance(case):
    # Layout, placed rows, FP8 codes and scales, posted counts: no arithmetic that may come out otherwise.  The
    # combined rows: an fp32 chain of at most 8 products rounded once to bf16.  Against the same sums in 64 bits
    # 3 to 5 values in 100000 round to the neighbouring bf16 (measured: 1.0e-5 to 1.7e-5 in the 2-norm); one bf16
    # step is at most 2^-7 = 0.0078 of the value, also where the two-level reduce flips one rounded partial sum.
    return {"rel": 8e-5, "max": 0.01}


class _Engine:
    """The handle of a case, and the second, group-level one of the deduplicating mode, with their workspaces."""

    def __init__(self, c):
        many = dict(max_tokens=c["cap"], spin_timeout_ms=10000)
        self.group = None
        if c["kind"] in ("place", "dedup"):
            self.runner = EPRunner(c["R"], c["E"], c["K"], c["H"], S=c["S"], num_proxy_threads=0, **many)
        else:
            self.runner = EPRunner(c["R"], c["E"], c["K"], c["H"], S=c["S"], ht_slices=c["slices"],
                                   ht_ring_slots=c["slots"], **many)
        if c["kind"] == "dedup":
            NG = c["R"] // c["group"]
            self.group = EPRunner(NG, NG, c["K"], c["H"], **many)
        self.ring = self.heap = None
        if c["kind"] == "rings":
            self.ring = torch.zeros(self.runner.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        if c["kind"] == "moved":
            # the source heap that rows or messages are packed into (bf16 rows that travel on their own leave from x)
            rows = c["cap"] if c["cmds"] == "row" else c["cap"] * c["K"]
            self.heap = torch.zeros((rows, _message_bytes(c)), dtype=torch.uint8, device="cuda")

    def __del__(self):
        for r in (getattr(self, "runner", None), getattr(self, "group", None)):
            if r is not None:
                r.close()


_engines = weakref.WeakValueDictionary()


def _engine(c):
    key = tuple(sorted((k, v) for k, v in c.items() if k != "name"))
    e = _engines.get(key)
    if e is None:
        e = _engines[key] = _Engine(c)
    return e


def _message_bytes(c):
    """An FP8 row that travels as one message is padded to 16 bytes."""
    return 2 * c["H"] if c["payload"] == "bf16" else (c["H"] + c["H"] // 32 + 15) // 16 * 16


def _route(c, gen):
    """The router's choice for all sources: int32 [S, T, K] (distinct experts, -1 where dropped) and fp32 weights."""
    shape = (c["S"], c["T"], c["E"])
    if c["routing"] == "uniform":
        idx = torch.rand(shape, generator=gen, device="cuda").topk(c["K"], dim=-1).indices
        w = torch.randn(idx.shape, generator=gen, device="cuda").softmax(-1)
    else:
        logits = torch.randn(shape, generator=gen, device="cuda")
        if c["routing"] == "zipf":  # expert popularity ~ 1/rank over a random order of the experts
            order = torch.randperm(c["E"], generator=gen, device="cuda")
            logits -= (order + 1).float().log()
        w, idx = logits.softmax(-1).topk(c["K"], dim=-1)
        w = w / w.sum(-1, keepdim=True)
    idx = idx.to(torch.int32)
    if c["masked"]:
        idx = torch.where(torch.rand(idx.shape, generator=gen, device="cuda") < c["masked"], -1, idx)
    return idx.contiguous(), w.float().contiguous()


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    T, H, K, E = c["T"], c["H"], c["K"], c["E"]

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)

    def zeros(shape, dtype=torch.bfloat16):
        return torch.zeros(shape, dtype=dtype, device="cuda")

    idx, w = _route(c, gen)
    s = {"c": c, "engine": _engine(c), "idx": idx, "w": w[0].contiguous(), "x": normal(T, H)}
    rows = c["S"] * T * K                 # buffers hold the most that routing can ask for: it is known only on the GPU
    s["y"] = normal(rows, H)              # the experts' outputs, one row per received row
    s["out"] = zeros((T, H))
    s["recv"], s["scale"], s["messages"] = zeros((rows, H)), None, None
    if c["kind"] == "dedup":
        rows_g = T * min(K, c["R"] // c["group"])
        s["recv"], s["partial"] = zeros((rows_g, H)), zeros((rows_g, H))
        s["group_idx"], s["first_k"] = torch.empty_like(idx), torch.empty_like(idx)
        s["index"], s["ones"] = zeros((rows,), torch.int32), torch.ones_like(s["w"])
    if c["payload"] == "fp8":
        s["recv"], s["scale"] = zeros((rows, H), torch.uint8), zeros((rows, H // 128), torch.float32)
        if c["kind"] == "moved":
            s["messages"] = zeros((rows, _message_bytes(c)), torch.uint8)
    s["counts"] = zeros((E,), torch.int32)
    return s


def _layout_of(lay, prefix=""):
    return {prefix + k: getattr(lay, k) for k in lay.__dataclass_fields__}


def run(s):
    c, e = s["c"], s["engine"]
    r, kind, x, idx = e.runner, c["kind"], s["x"], s["idx"]
    payload = ep.EP_BF16 if c["payload"] == "bf16" else ep.EP_FP8_E4M3
    cmds = CMDS[c["cmds"]]
    if kind == "dedup":
        return _run_dedup(s)
    lay = r.layout(idx)
    got = _layout_of(lay)
    if kind == "rings":
        r.ht_dispatch(x, idx[0], lay, e.ring, s["recv"], recv_scale=s["scale"])
    elif kind == "moved":
        target = s["recv"] if s["messages"] is None else s["messages"]  # rows land here as they travelled
        n = target.shape[0]
        if c["cmds"] == "row":
            source = x if s["messages"] is None else e.heap
            r.register_heaps(source, target)
            packed = target if s["messages"] is None else e.heap  # (bf16 rows leave from x: nothing is packed)
            r.dispatch(x, idx[0], lay, packed, payload=payload, cmd_mode=cmds | ep.EP_CMD_NO_PLACEMENT, recv_rows=n)
        else:
            r.register_heaps(e.heap, target)
            r.dispatch(x, idx[0], lay, e.heap, payload=payload, cmd_mode=cmds, recv_rows=n)
        r.wait()
        if s["messages"] is not None:
            r.fp8_unpack(s["messages"], s["recv"], s["scale"])
    else:
        r.dispatch(x, idx[0], lay, s["recv"], s["scale"], payload=payload, cmd_mode=cmds)
        if kind == "decode":
            r.recv_wait(s["counts"])
            got["counts"] = s["counts"]
    r.combine(s["y"], s["w"], lay.dst_row[0], s["out"])
    if kind in ("prefill", "rings"):
        r.wait()
    got.update(recv=s["recv"], scale=s["scale"], out=s["out"])
    return got


def _run_dedup(s):
    c, r, g = s["c"], s["engine"].runner, s["engine"].group
    idx, gi, fk, T = s["idx"], s["group_idx"], s["first_k"], c["T"]
    ep.ep_dedup(r.h, idx, T, c["group"], gi, fk)
    lay, lay_g = r.layout(idx), g.layout(gi)
    g.dispatch(s["x"], gi[0], lay_g, s["recv"], cmd_mode=ep.EP_CMD_CHUNK32)
    ep.ep_gather_index(r.h, lay.dst_row[0], lay_g.dst_row[0], fk[0], T, s["index"].shape[0], s["index"])
    ep.ep_combine_partial(r.h, s["y"], s["w"], lay.dst_row[0], fk[0], lay_g.dst_row[0], T, s["y"].shape[0],
                          s["partial"].shape[0], s["partial"])
    g.combine(s["partial"], s["ones"], lay_g.dst_row[0], s["out"])
    g.wait()
    got = dict(_layout_of(lay), **_layout_of(lay_g, "group_"))
    got.update(group_idx=gi, first_k=fk, recv=s["recv"], index=s["index"], partial=s["partial"], out=s["out"])
    return got
