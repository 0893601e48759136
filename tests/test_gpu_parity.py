"""Parity of the HIP path (through the C ABI) against the CPU oracle, element by
element on the same seeded inputs.  Integer / byte work is compared bit-exactly;
combine within 1 bf16 ulp of the oracle and within the fp64 bound."""
import numpy as np
import pytest

import ep_inputs as g

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def epmod():
    import paper_2512_19849_amd as ep
    ep.load_library(build_if_missing=False)      # the built library must be there: no fallback
    return ep


def _runner(epmod, cfg, T=None, **kw):
    from paper_2512_19849_amd.runner import EPRunner
    kw.setdefault("spin_timeout_ms", 3000)
    return EPRunner(cfg.R, cfg.E, cfg.K, cfg.H, T if T is not None else cfg.T, S=cfg.S, **kw)


def _dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return t if dtype is None else t.to(dtype)


def _check_layout(oracle, got: dict, idx, E, R):
    want = oracle.layout(idx, E, R)
    for name in ("count", "expert_total", "rank_total", "base", "expert_offset", "rank_offset", "slot", "dst_row"):
        assert np.array_equal(got[name], want[name]), name
    return want


# ------------------------------------------------------------------ layout
@pytest.mark.parametrize("one_launch", ["1", "0"])
@pytest.mark.parametrize("cid,T,mask", [(1, None, 0.0), (1, 37, 0.3), (2, None, 0.0), (2, 100, 0.1),
                                        (4, None, 0.0), (4, 4095, 0.05), (5, None, 0.0), (5, 1, 0.0),
                                        (4, 65, 0.0), (1, 0, 0.0)])
def test_layout_parity(epmod, oracle, cid, T, mask, one_launch, monkeypatch):
    monkeypatch.setenv("EP_LAYOUT_SMALL", one_launch)
    cfg = g.config(cid)
    idx, _ = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=17)
    with _runner(epmod, cfg, idx.shape[1] or 1) as r:
        for rep in range(2):                                   # second call: scratch must have reset itself
            lay = r.layout(_dev(idx))
            torch.cuda.synchronize()
            _check_layout(oracle, lay.numpy(), idx, cfg.E, cfg.R)
        assert r.stats()["device_error"] == 0


def test_layout_hand_over_between_workgroups_many_times(epmod, oracle, monkeypatch):
    """The two-kernel form, which the table would not take by itself: its tile histograms cross workgroups through
    write-through stores, a ticket and cache-bypassing loads (no L2 write-back or invalidate).  300 layouts of the full
    4096-token table, each compared on the device with the oracle's arrays, other kernels' dirty lines in the caches in
    between."""
    monkeypatch.setenv("EP_LAYOUT_SMALL", "0")
    cfg = g.config(4)
    idx, _ = g.routing_all(cfg)
    want = {k: _dev(v) for k, v in oracle.layout(idx, cfg.E, cfg.R).items()}
    noise = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
    with _runner(epmod, cfg) as r:
        d_idx = _dev(idx)
        bad = torch.zeros((), dtype=torch.int64, device="cuda")
        for it in range(300):
            if it % 3 == 0:
                noise.add_(1)                                    # leaves dirty lines in every L2
            lay = r.layout(d_idx)
            for name, v in want.items():
                bad += (getattr(lay, name) != v).sum()
        torch.cuda.synchronize()
        assert int(bad.item()) == 0
        assert r.stats()["device_error"] == 0


def test_layout_special_shapes(epmod, oracle):
    rng = np.random.default_rng(0)
    for (S, T, K, E, R) in [(1, 300, 1, 1, 1), (3, 129, 4, 8, 8), (2, 64, 6, 96, 3), (1, 1000, 8, 1024, 4),
                            (5, 77, 3, 12, 2)]:
        idx = np.stack([np.stack([rng.permutation(E)[:K] for _ in range(T)]) for _ in range(S)]).astype(np.int32)
        cfg = g.EPConfig("x", T=T, H=128, E=E, K=K, R=R, S=S)
        with _runner(epmod, cfg) as r:
            lay = r.layout(_dev(idx))
            torch.cuda.synchronize()
            _check_layout(oracle, lay.numpy(), idx, E, R)
    # all tokens to one expert; everything masked
    cfg = g.EPConfig("x", T=500, H=128, E=16, K=1, R=4)
    for idx in (np.full((1, 500, 1), 9, np.int32), np.full((1, 500, 1), -1, np.int32)):
        with _runner(epmod, cfg) as r:
            lay = r.layout(_dev(idx))
            torch.cuda.synchronize()
            _check_layout(oracle, lay.numpy(), idx, 16, 4)


@pytest.mark.parametrize("one_launch", ["1", "0"])
def test_layout_small_tables_both_forms(epmod, oracle, one_launch, monkeypatch):
    """Small tables with the one-launch form of the layout, which they take, and with it switched off: a dozen 64-token
    tiles and one more, ragged last tiles, several sources with few tiles each, 392 experts over 8
    ranks, masked and fully masked entries, one expert for everybody."""
    monkeypatch.setenv("EP_LAYOUT_SMALL", one_launch)
    rng = np.random.default_rng(12)
    for (S, T, K, E, R, maskp) in [(1, 768, 8, 256, 16, 0.0), (1, 769, 8, 256, 16, 0.0), (4, 130, 3, 24, 4, 0.2),
                                   (5, 130, 3, 24, 4, 0.2), (12, 64, 2, 16, 4, 0.0), (13, 1, 1, 4, 2, 0.0),
                                   (1, 700, 8, 384, 8, 0.5), (1, 640, 5, 392, 8, 0.0), (2, 333, 7, 64, 64, 1.0),
                                   (3, 200, 1, 1, 1, 0.1), (1, 1, 8, 8, 1, 0.0)]:
        idx = np.stack([np.stack([rng.permutation(E)[:K] for _ in range(T)]) for _ in range(S)]).astype(np.int32)
        if maskp:
            idx = g.mask_random(idx, maskp, seed=S * 100 + T)
        cfg = g.EPConfig("small", T=T, H=128, E=E, K=K, R=R, S=S)
        with _runner(epmod, cfg) as r:
            for rep in range(2):
                lay = r.layout(_dev(idx))
                torch.cuda.synchronize()
                _check_layout(oracle, lay.numpy(), idx, E, R)
            assert r.stats()["device_error"] == 0
    # an expert id out of range is reported by whichever form runs, and the entry is dropped
    cfg = g.EPConfig("small", T=100, H=128, E=8, K=2, R=2, S=1)
    idx = np.stack([rng.permutation(8)[:2] for _ in range(100)]).astype(np.int32)[None]
    idx[0, 41, 1] = 8
    with _runner(epmod, cfg) as r:
        lay = r.layout(_dev(idx))
        torch.cuda.synchronize()
        got = lay.numpy()
        assert got["slot"][0, 41, 1] == -1 and got["dst_row"][0, 41, 1] == -1
        assert r.stats()["device_error"] == epmod.EP_EBOUNDS


@pytest.mark.parametrize("S,T,K,E,R,maskp", [
    (1, 51, 5, 16, 4, 0.0), (1, 64, 4, 16, 4, 0.0), (1, 257, 1, 64, 8, 0.1),           # 255 / 256 / 257 entries
    (1, 585, 7, 24, 3, 0.0), (3, 683, 2, 40, 5, 0.2), (1, 513, 8, 256, 16, 0.0),       # 15 to 17 groups of 256
    (7, 5, 3, 8, 2, 0.3), (256, 3, 2, 4, 4, 0.0), (65, 9, 6, 12, 1, 0.1),              # many sources in one group
    (1, 8192, 8, 64, 8, 0.05), (1, 8193, 8, 64, 8, 0.0), (5, 1024, 8, 256, 32, 0.0),   # both sides of the line between
    (5, 1025, 8, 256, 32, 0.0), (1, 5120, 8, 63, 7, 0.0), (1, 5121, 8, 63, 7, 0.0),    # the two forms
    (1, 2000, 8, 1024, 256, 0.0), (1, 700, 64, 64, 2, 0.0)])
def test_layout_one_workgroup_per_expert(epmod, oracle, S, T, K, E, R, maskp):
    """The one-launch form at the edges of its groups (256 entries), of its waves' shares and of its range in entries."""
    rng = np.random.default_rng(S * 1000 + T)
    idx = np.argsort(rng.random((S, T, E)), axis=-1)[..., :K].astype(np.int32)
    idx[:, ::3, 0] = np.where((idx[:, ::3, 1:] == E - 1).any(-1), idx[:, ::3, 0], E - 1)  # a busy last expert
    if maskp:
        idx = g.mask_random(idx, maskp, seed=T)
    with _runner(epmod, g.EPConfig("edges", T=T, H=128, E=E, K=K, R=R, S=S)) as r:
        lay = r.layout(_dev(idx))
        torch.cuda.synchronize()
        _check_layout(oracle, lay.numpy(), idx, E, R)
        assert r.stats()["device_error"] == 0


# several workgroups per expert: their shares of the waves (9 waves in 9 and in 6 parts, 16 in 16, 2 and 1), lists longer
# than 64 quads with one and with several sources in 64 of them, both sides of the lines in tokens
@pytest.mark.parametrize("S,T,K,E,R", [(1, 2048, 1, 7, 7), (1, 2049, 1, 7, 7), (1, 2049, 1, 40, 8), (1, 4097, 1, 1, 1),
                                       (1, 13000, 3, 3, 1), (1, 6000, 8, 100, 10), (1, 3000, 8, 130, 10),
                                       (1, 16384, 4, 64, 8), (1, 16385, 2, 64, 8), (3, 2048, 1, 2, 1), (2, 3072, 3, 5, 5),
                                       (8, 768, 1, 1, 1), (64, 96, 2, 4, 2), (3, 2049, 1, 2, 1), (7, 1170, 5, 64, 4),
                                       (7, 1171, 5, 64, 4), (5, 4000, 2, 256, 8)])
def test_layout_busy_expert(epmod, oracle, S, T, K, E, R):
    """Nearly every token names one expert, first among its entries or last."""
    rng = np.random.default_rng(T)
    score = rng.random((S, T, E))
    score[:, :, E // 2] -= rng.random((S, T)) < 0.97
    idx = np.argsort(score, axis=-1)[..., :K].astype(np.int32)
    idx[:, T // 2:] = idx[:, T // 2:, ::-1]
    idx[:, ::5, 0] = -1
    with _runner(epmod, g.EPConfig("busy", T=T, H=128, E=E, K=K, R=R, S=S)) as r:
        lay = r.layout(_dev(idx))
        torch.cuda.synchronize()
        _check_layout(oracle, lay.numpy(), idx, E, R)
        assert r.stats()["device_error"] == 0


# less than a group of 256, full groups, full groups and a rest, a lane's largest share, several sources
@pytest.mark.parametrize("S,T,K,E,R", [(1, 41, 2, 8, 2), (1, 1024, 4, 256, 16), (1, 771, 5, 1024, 8), (1, 8192, 8, 128, 8),
                                       (4, 300, 3, 40, 5)])
def test_layout_ids_that_are_no_expert(epmod, oracle, S, T, K, E, R):
    """Ids beyond the experts, in 16 bits and not (their low halves name experts), and negative ones: dropped, reported."""
    rng = np.random.default_rng(E)
    idx = np.argsort(rng.random((S, T, E)), axis=-1)[..., :K].astype(np.int32)
    bad = np.array([E, 65535, 65536 + 3, 131072, 2**31 - 1, -2, -65536 + 1, -2**31], np.int32)
    where = rng.random(idx.shape) < 0.2
    idx = np.where(where, bad[rng.integers(0, len(bad), idx.shape)], idx).astype(np.int32)
    with _runner(epmod, g.EPConfig("bad", T=T, H=128, E=E, K=K, R=R, S=S)) as r:
        lay = r.layout(_dev(idx))
        torch.cuda.synchronize()
        _check_layout(oracle, lay.numpy(), np.where(where, -1, idx).astype(np.int32), E, R)
        assert r.stats()["device_error"] == epmod.EP_EBOUNDS


# smallest, a decode table over 32 sources, a batch (each of a size that takes one launch otherwise), more than 8 ids per
# token, and a table that takes the two kernels anyway
@pytest.mark.parametrize("S,T,K,E,R", [(1, 5, 2, 8, 2), (32, 128, 8, 256, 32), (1, 4096, 8, 256, 16), (2, 300, 12, 64, 8),
                                       (1, 9000, 8, 64, 8)])
@pytest.mark.parametrize("name", ["slot", "dst_row"])
def test_layout_over_the_routing_table(epmod, oracle, S, T, K, E, R, name):
    """An output that is the routing table's own buffer: with a handle, and from static scratch."""
    rng = np.random.default_rng(T)
    idx = g.mask_random(np.argsort(rng.random((S, T, E)), axis=-1)[..., :K].astype(np.int32), 0.05, seed=T)
    i32 = dict(dtype=torch.int32, device="cuda")
    with _runner(epmod, g.EPConfig("over", T=T, H=128, E=E, K=K, R=R, S=S)) as r:
        for static in (False, True):
            d_idx = _dev(idx)
            out = dict(count=torch.empty((S, E), **i32), expert_total=torch.empty(E, **i32), rank_total=torch.empty(R, **i32),
                       base=torch.empty((S, E), **i32), expert_offset=torch.empty(E + 1, **i32),
                       rank_offset=torch.empty(R + 1, **i32), slot=torch.empty_like(d_idx), dst_row=torch.empty_like(d_idx))
            out[name] = d_idx
            if static:
                epmod.ep_layout_static(d_idx, S, T, K, E, R, *out.values())
            else:
                epmod.ep_layout(r.h, d_idx, T, *out.values())
            torch.cuda.synchronize()
            _check_layout(oracle, {k: v.cpu().numpy() for k, v in out.items()}, idx, E, R)
        assert r.stats()["device_error"] == 0


# ---------------------------------------------------------- dispatch bf16
def _dispatch_case(epmod, oracle, cfg, T, mask, cmd_mode, rank_filter=-1, src=0, extra_rows=3, proxy_writes=False,
                   extra_flags=0, **kw):
    idx, w = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=23)
    T = idx.shape[1]
    x = g.activations(cfg, src, T=T)
    flags = epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS | extra_flags
    rows = int((idx >= 0).sum()) + extra_rows
    with _runner(epmod, cfg, T, flags=flags, heap_rows=rows, **kw) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        recv = torch.full((rows, cfg.H), -1.5, dtype=torch.bfloat16, device="cuda")     # sentinel 0xBFC0
        from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
        d_x = bits_to_bf16(x)
        target = recv
        if proxy_writes:
            # the proxy moves the rows: per token straight out of x, chunks out of a packed send heap
            if (cmd_mode & 0xFF) == epmod.EP_CMD_PER_TOKEN:
                cmd_mode |= epmod.EP_CMD_NO_PLACEMENT
                r.register_heaps(d_x, recv)
            else:
                target = torch.full((rows, cfg.H), 2.5, dtype=torch.bfloat16, device="cuda")
                r.register_heaps(target, recv)
        r.dispatch(d_x, d_idx[src], lay, target, src=src, rank_filter=rank_filter, cmd_mode=cmd_mode)
        if (cmd_mode & 0xFF) != epmod.EP_CMD_NONE:
            r.wait()
        torch.cuda.synchronize()
        layn = lay.numpy()
        want_lay = _check_layout(oracle, layn, idx, cfg.E, cfg.R)
        want, wc = oracle.dispatch_bf16(x, idx[src], want_lay["dst_row"][src], cfg.E_loc, rows, rank_filter,
                                        fill=0xBFC0)
        got = bf16_to_bits(recv)
        assert np.array_equal(got, want)
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        if proxy_writes:
            assert st["copied_bytes"] == st["write_bytes"] > 0 and 1 <= st["copy_batches"] <= st["writes"]
        else:
            assert st["copied_bytes"] == 0 and st["copy_batches"] == 0
        return dict(stats=st, cmds=epmod.ep_cmd_log(r.h), events=epmod.ep_event_log(r.h), lay=want_lay, idx=idx,
                    counters=r.counters().copy(), x=x, recv=got)


@pytest.mark.parametrize("cid,T,mask", [(1, None, 0.0), (1, 50, 0.25), (2, None, 0.0), (4, 300, 0.0),
                                        (5, 257, 0.1), (4, 1, 0.0)])
def test_dispatch_bf16_ring_off(epmod, oracle, cid, T, mask):
    cfg = g.config(cid)
    out = _dispatch_case(epmod, oracle, cfg, T, mask, epmod.EP_CMD_NONE)
    assert out["stats"]["cmds"] == 0


def test_dispatch_bf16_other_source_and_rank_filter(epmod, oracle):
    cfg = g.config(2)                                           # 32 sources, inbound share of rank 0
    _dispatch_case(epmod, oracle, cfg, 64, 0.0, epmod.EP_CMD_NONE, rank_filter=0, src=7)
    _dispatch_case(epmod, oracle, cfg, 64, 0.0, epmod.EP_CMD_PER_TOKEN, rank_filter=5, src=31)


@pytest.mark.parametrize("pipeline", ["1", "0"])
@pytest.mark.parametrize("vpl", [1, 2, 4, 7, 8, 14, 16])
def test_dispatch_bf16_every_row_split(epmod, oracle, vpl, pipeline, monkeypatch):
    """Every way of cutting a row into wavefronts, in the plain form and in the form with a command wave
    (EP_DISPATCH_PIPELINE=1), with the ring off as well."""
    monkeypatch.setenv("EP_DISPATCH_VPL", str(vpl))
    monkeypatch.setenv("EP_DISPATCH_PIPELINE", pipeline)
    _dispatch_case(epmod, oracle, g.config(4), 70, 0.05, epmod.EP_CMD_CHUNK32)
    _dispatch_case(epmod, oracle, g.config(1), 33, 0.0, epmod.EP_CMD_PER_TOKEN)
    if pipeline == "1":
        _dispatch_case(epmod, oracle, g.config(4), 70, 0.05, epmod.EP_CMD_NONE)


@pytest.mark.parametrize("pipeline", ["1", "0"])
@pytest.mark.parametrize("mode", ["per_token", "chunk32", "ordered"])
def test_ring_on_dispatch_with_and_without_a_command_wave(epmod, oracle, mode, pipeline, monkeypatch):
    """With EP_DISPATCH_PIPELINE=1 ring-on dispatches run persistent workgroups whose command wave lags one batch
    of tokens behind the data waves; the default is the plain form.  Both: payload and command multiset equal the oracle's,
    with rings of 8 slots (back-pressure reaches the command wave, then the data waves), with more batches than
    workgroups (14 000 tokens of 128-wide rows, 12 tokens per batch: up to three batches per workgroup, so both
    LDS slots are reused) and with a Drain at the end."""
    monkeypatch.setenv("EP_DISPATCH_PIPELINE", pipeline)
    cm = {"per_token": epmod.EP_CMD_PER_TOKEN, "chunk32": epmod.EP_CMD_CHUNK32,
          "ordered": epmod.EP_CMD_CHUNK32_ORDERED}[mode]
    wide = g.EPConfig("narrow_many", T=14000, H=128, E=16, K=3, R=4, seed=77)
    for cfg, T, entries, extra in ((g.config(4), 900, 4096, 0), (g.config(4), 200, 8, epmod.EP_CMD_DRAIN),
                                   (wide, None, 64, 0), (g.config(2, S=1), None, 4096, epmod.EP_CMD_DRAIN)):
        if mode == "ordered" and extra:
            extra = 0                                           # (the sequenced mode ends with its own Drain)
        out = _dispatch_case(epmod, oracle, cfg, T, 0.05, cm | extra, ring_entries=entries, spin_timeout_ms=10000)
        if mode == "ordered":
            oracle.check_order_trace(out["events"])
        else:
            _check_commands(epmod, oracle, cfg, out, mode)


@pytest.mark.parametrize("pipeline", ["1", "0"])
@pytest.mark.parametrize("waves", [4, 8, 16])
def test_per_token_commands_every_push_form(epmod, oracle, waves, pipeline, monkeypatch):
    """One command per row leaves through the first wave of a workgroup that holds one token or several, through the
    last workgroup of a group (commands sorted by channel each time), or through the command wave of a persistent
    workgroup; all must hand the proxy the same multiset of commands, with rings of 8 and of 4096 slots."""
    monkeypatch.setenv("EP_PER_TOKEN_WAVES", str(waves))
    monkeypatch.setenv("EP_DISPATCH_PIPELINE", pipeline)
    for cid, T, entries in ((4, 70, 4096), (4, 70, 8), (2, None, 64), (1, 33, 8)):
        cfg = g.config(cid)
        out = _dispatch_case(epmod, oracle, cfg, T, 0.05, epmod.EP_CMD_PER_TOKEN, ring_entries=entries)
        _check_commands(epmod, oracle, cfg, out, "per_token")


# ------------------------------------------------------ commands and proxy
def _check_commands(epmod, oracle, cfg, out, mode_name, payload="bf16", src=0, rank_filter=-1):
    want = oracle.expected_cmds(out["idx"][src], out["lay"], src, cfg.E_loc, cfg.H, payload, mode_name, rank_filter)
    got = oracle.cmd_multiset(out["cmds"])
    assert got == want
    for w in out["cmds"]:
        d = oracle.decode_cmd(w)
        assert d["gen"] == d["gen_hi"]
    res = oracle.check_fence_trace(out["events"], out["lay"]["count"])
    E_loc = cfg.E_loc
    sel = np.arange(cfg.E) // E_loc == rank_filter if rank_filter >= 0 else np.ones(cfg.E, bool)
    assert np.array_equal(out["counters"][src][sel], out["lay"]["count"][src][sel])
    st = out["stats"]
    assert st["atomics_applied"] == int(sel.sum()) == st["atomics"]
    assert st["write_rows"] == int(out["lay"]["count"][src][sel].sum())
    assert st["write_bytes"] == st["write_rows"] * oracle.row_bytes(cfg.H, payload)
    return res


# groups of workgroups that push together.  One token per workgroup: 33 and 129 tokens.  Several: 301 tokens in pairs, four
# workgroups to a group (the last group and its last workgroup not full), 300 tokens by eights, two workgroups to a group.
# The last size with groups and the first without: 12288 commands, 256 MB of rows.  Groups of one: a single token, a top-k
# that does not divide 64, more than 64 / 2 pairs per token, workgroups that hold 64 pairs by themselves.
@pytest.mark.parametrize("T,K,E,R,H", [(33, 1, 8, 8, 7168), (129, 5, 48, 16, 7168), (301, 8, 64, 8, 4096),
                                       (300, 3, 64, 8, 1024), (2048, 6, 16, 4, 7168), (2049, 6, 16, 4, 7168),
                                       (488, 8, 16, 4, 32768), (489, 8, 16, 4, 32768), (1, 4, 16, 4, 7168),
                                       (57, 3, 24, 6, 4096), (300, 7, 64, 8, 1024), (70, 33, 96, 12, 5120),
                                       (2048, 6, 16, 4, 640)])
def test_per_token_commands_of_workgroup_groups(epmod, oracle, T, K, E, R, H):
    """Dispatches of one handle in per-token and chunk modes by turns (the counters they share go back to zero), taken
    from either end of the token range."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("groups", T=T, H=H, E=E, K=K, R=R, routing="uniform", seed=K)
    idx = g.mask_random(g.routing_all(cfg)[0], 0.05, seed=K)
    x = g.activations(cfg)
    rows = int((idx >= 0).sum()) + 1
    lay = oracle.layout(idx, E, R)
    want, _ = oracle.dispatch_bf16(x, idx[0], lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
    flags = epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS | epmod.EP_FLAG_CACHE_HINTS
    with _runner(epmod, cfg, flags=flags, heap_rows=rows) as r:
        d_idx, d_x = _dev(idx), bits_to_bf16(x)
        lay_d = r.layout(d_idx)
        recv = torch.empty((rows, H), dtype=torch.bfloat16, device="cuda")
        cmds = type(oracle.cmd_multiset([]))()
        for mode in ("per_token", "chunk32", "per_token", "per_token"):
            recv.fill_(-1.5)
            r.dispatch(d_x, d_idx[0], lay_d, recv, cmd_mode=epmod.CMD_MODES[mode])
            r.wait()
            torch.cuda.synchronize()
            assert np.array_equal(bf16_to_bits(recv), want), mode
            assert np.array_equal(r.counters()[0], lay["count"][0]), mode
            cmds += oracle.expected_cmds(idx[0], lay, 0, cfg.E_loc, H, "bf16", mode)
        assert oracle.cmd_multiset(epmod.ep_cmd_log(r.h)) == cmds
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0


@pytest.mark.parametrize("T,K,E,R,H,cut", [(128, 8, 256, 32, 7168, 61), (96, 4, 16, 4, 4096, 33)])
def test_per_token_commands_between_two_parts_of_a_chunked_dispatch(epmod, oracle, T, K, E, R, H, cut):
    """Sequenced chunks of a table that is dispatched in two parts: what the first part leaves half counted is not seen
    by a per-token dispatch in between, and the second part completes it."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("parts", T=T, H=H, E=E, K=K, R=R, routing="uniform", seed=K)
    idx, x = g.routing_all(cfg)[0], g.activations(cfg)
    rows = T * K
    lay = oracle.layout(idx, E, R)
    want, _ = oracle.dispatch_bf16(x, idx[0], lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
    with _runner(epmod, cfg, flags=epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS, heap_rows=rows) as r:
        d_idx, d_x = _dev(idx), bits_to_bf16(x)
        lay_d = r.layout(d_idx)
        bufs = [torch.full((rows, H), -1.5, dtype=torch.bfloat16, device="cuda") for _ in range(2)]

        def part(lo, hi):
            epmod.ep_dispatch(r.h, d_x[lo:hi], d_idx[0, lo:hi], lay_d.dst_row[0, lo:hi], lay_d.count[0], lay_d.base[0],
                              hi - lo, 0, -1, epmod.EP_BF16, epmod.EP_CMD_CHUNK32_ORDERED, bufs[0], None, rows)

        part(0, cut)
        for _ in range(2):
            bufs[1].fill_(-1.5)
            r.dispatch(d_x, d_idx[0], lay_d, bufs[1], cmd_mode=epmod.EP_CMD_PER_TOKEN)
            r.wait()
            torch.cuda.synchronize()
            assert np.array_equal(bf16_to_bits(bufs[1]), want)
            assert np.array_equal(r.counters()[0], lay["count"][0])
        part(cut, T)
        r.wait()
        torch.cuda.synchronize()
        assert np.array_equal(bf16_to_bits(bufs[0]), want)
        assert np.array_equal(epmod.ep_tail_counters(r.h, 1, R)[0], lay["count"][0].reshape(R, -1).sum(1))
        writes = type(oracle.cmd_multiset([]))()
        for _ in range(2):
            writes += oracle.expected_cmds(idx[0], lay, 0, cfg.E_loc, H, "bf16", "per_token")
        assert oracle.cmd_multiset(epmod.ep_cmd_log(r.h)) == writes
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0


@pytest.mark.parametrize("cid,T,mask,window", [(1, None, 0.0, 0), (1, None, 0.2, 4), (2, 128, 0.0, 64),
                                               (4, 200, 0.0, 0), (5, 300, 0.1, 7)])
def test_dispatch_per_token_commands(epmod, oracle, cid, T, mask, window):
    cfg = g.config(cid, S=1)
    out = _dispatch_case(epmod, oracle, cfg, T, mask, epmod.EP_CMD_PER_TOKEN, reorder_window=window, reorder_seed=5)
    _check_commands(epmod, oracle, cfg, out, "per_token")
    # the commands alone determine the receive buffer
    rows = out["recv"].shape[0]
    send = out["x"].view(np.uint8).reshape(out["x"].shape[0], -1)
    heap, hits = oracle.replay_writes_per_token(out["cmds"], send, rows, fill_byte=0)
    nvalid = int((out["idx"] >= 0).sum())
    assert (hits[:nvalid] == 1).all() and (hits[nvalid:] == 0).all()
    assert np.array_equal(heap[:nvalid], out["recv"].view(np.uint8).reshape(rows, -1)[:nvalid])


@pytest.mark.parametrize("cid,T,mask,window", [(1, None, 0.0, 0), (4, 700, 0.0, 0), (4, 700, 0.1, 16),
                                               (5, 1000, 0.0, 64)])
def test_dispatch_chunk32_commands(epmod, oracle, cid, T, mask, window):
    cfg = g.config(cid, S=1)
    out = _dispatch_case(epmod, oracle, cfg, T, mask, epmod.EP_CMD_CHUNK32, reorder_window=window, reorder_seed=9)
    _check_commands(epmod, oracle, cfg, out, "chunk32")
    oracle.check_chunk_cover(out["cmds"], out["lay"], 0, cfg.E_loc, oracle.row_bytes(cfg.H, "bf16"))


# -------------------------------------------- writes performed by the proxy
@pytest.mark.parametrize("cid,T,mask,window,threads", [(1, None, 0.0, 0, 4), (1, 50, 0.25, 5, 1), (2, 128, 0.0, 0, 2),
                                                       (4, 300, 0.05, 16, 4), (5, 700, 0.0, 0, 3)])
def test_proxy_performs_per_token_writes(epmod, oracle, cid, T, mask, window, threads):
    cfg = g.config(cid, S=1)
    out = _dispatch_case(epmod, oracle, cfg, T, mask, epmod.EP_CMD_PER_TOKEN, proxy_writes=True,
                         reorder_window=window, reorder_seed=3, num_proxy_threads=threads)
    _check_commands(epmod, oracle, cfg, out, "per_token")


@pytest.mark.parametrize("cid,T,mask,window,mode", [(1, None, 0.0, 0, "chunk32"), (4, 700, 0.1, 16, "chunk32"),
                                                    (5, 1000, 0.0, 0, "chunk32"), (1, None, 0.2, 6, "ordered"),
                                                    (4, 500, 0.0, 0, "ordered")])
def test_proxy_performs_chunk_writes(epmod, oracle, cid, T, mask, window, mode):
    cfg = g.config(cid, S=1)
    if mode == "chunk32":
        out = _dispatch_case(epmod, oracle, cfg, T, mask, epmod.EP_CMD_CHUNK32, proxy_writes=True,
                             reorder_window=window, reorder_seed=11)
        _check_commands(epmod, oracle, cfg, out, "chunk32")
    else:
        out = _dispatch_case(epmod, oracle, cfg, T, mask, epmod.EP_CMD_CHUNK32_ORDERED, proxy_writes=True,
                             reorder_window=window, reorder_seed=11)
        oracle.check_order_trace(out["events"])
        assert out["stats"]["drains"] == 8


# a row of 16 vectors, one of exactly / just over a 256-vector piece, the largest row that counts as a row (32 KiB) and
# the smallest that counts as a chunk; many copies (batches beyond one argument block) and few
@pytest.mark.parametrize("H,T", [(128, 3000), (2048, 1500), (2176, 1500), (16384, 40), (16384, 150), (16512, 120)])
def test_proxy_copies_rows_at_the_edges_of_pieces(epmod, oracle, H, T):
    cfg = g.EPConfig(f"edges{H}", T=T, H=H, E=32, K=6, R=4, routing="uniform")
    out = _dispatch_case(epmod, oracle, cfg, T, 0.03, epmod.EP_CMD_PER_TOKEN, proxy_writes=True, num_proxy_threads=1)
    _check_commands(epmod, oracle, cfg, out, "per_token")


# batches of up to 496 rows of one length travel in one argument block: one row, a full block, a row more, pieces of 256
# vectors and one vector more
@pytest.mark.parametrize("H,T,K", [(1024, 1, 1), (2048, 62, 8), (2176, 71, 7), (4096, 31, 16), (128, 124, 4)])
def test_proxy_copies_small_batches_of_rows(epmod, oracle, H, T, K):
    cfg = g.EPConfig(f"rows{H}", T=T, H=H, E=32, K=K, R=4, routing="uniform")
    out = _dispatch_case(epmod, oracle, cfg, T, 0.0, epmod.EP_CMD_PER_TOKEN, proxy_writes=True, num_proxy_threads=1,
                         num_channels=1)
    _check_commands(epmod, oracle, cfg, out, "per_token")


@pytest.mark.parametrize("cid,T,mask,window,mode,threads", [
    (3, None, 0.0, 0, "per_token", 4), (3, 50, 0.25, 5, "per_token", 1), (3, None, 0.2, 6, "chunk32", 2),
    (5, 700, 0.0, 16, "per_token", 3), (5, 1000, 0.05, 0, "chunk32", 4), (4, 300, 0.0, 8, "chunk32_ordered", 4),
    ("h128", 90, 0.1, 3, "per_token", 2), ("h128", 90, 0.0, 0, "chunk32", 2), (5, None, 0.0, 0, "per_token", 4)])
def test_proxy_performs_fp8_writes(epmod, oracle, cid, T, mask, window, mode, threads):
    """The low-latency token as the paper sends it: FP8, ONE message per row (codes, scales, padding), moved by the
    proxy between registered heaps.  Per token the kernel quantises every token once into its own message row and
    only pushes commands; in the chunk modes it packs message rows into a send heap that mirrors the receive heap.
    After ep_fp8_unpack the codes and scales equal the oracle's quantiser bit for bit, the messages equal the
    oracle's message rows, rows nobody addressed keep their bytes, and the command stream carries message lengths."""
    from paper_2512_19849_amd.runner import bits_to_bf16
    if cid == "h128":                                          # one block per row: 132 bytes padded to 144
        cfg = g.EPConfig("h128", T=T, H=128, E=8, K=2, R=4, S=1)
        rng = np.random.default_rng(3)
        idx = np.stack([rng.permutation(8)[:2] for _ in range(T)]).astype(np.int32)[None]
    else:
        cfg = g.config(cid, S=1)
        idx, _ = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=29)
    T = idx.shape[1]
    x = g.activations(cfg, 0, T=T)
    rows = int((idx >= 0).sum()) + 2
    rb = oracle.row_bytes(cfg.H, "fp8")
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    oracle.set_threads(min(16, oracle.max_threads()))
    try:
        wq, ws, wc = oracle.dispatch_fp8(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
    finally:
        oracle.set_threads(1)
    hit = wc > 0
    log = T <= 1000
    flags = (epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS) if log else 0
    with _runner(epmod, cfg, T, flags=flags, heap_rows=rows, reorder_window=window, reorder_seed=4,
                 num_proxy_threads=threads, spin_timeout_ms=10000) as r:
        d_idx, d_x = _dev(idx), bits_to_bf16(x)
        lay = r.layout(d_idx)
        dst = torch.full((rows, rb), 0xA5, dtype=torch.uint8, device="cuda")
        if mode == "per_token":
            send = torch.zeros((T, rb), dtype=torch.uint8, device="cuda")
            cm = epmod.EP_CMD_PER_TOKEN | epmod.EP_CMD_NO_PLACEMENT
        else:
            send = torch.zeros((rows, rb), dtype=torch.uint8, device="cuda")
            cm = epmod.CMD_MODES[mode]
        r.register_heaps(send, dst)
        rq = torch.zeros((rows, cfg.H), dtype=torch.uint8, device="cuda")
        rs = torch.zeros((rows, cfg.H // 128), dtype=torch.float32, device="cuda")
        for rep in range(2):
            dst.fill_(0xA5)
            r.dispatch(d_x, d_idx[0], lay, send, None, payload=epmod.EP_FP8_E4M3, cmd_mode=cm, recv_rows=rows)
            r.wait()
            r.fp8_unpack(dst, rq, rs)
            torch.cuda.synchronize()
            got = dst.cpu().numpy()
            used = cfg.H + cfg.H // 32
            assert np.array_equal(got[hit][:, :used], oracle.fp8_message_rows(wq[hit], ws[hit])[:, :used]), rep
            assert (got[~hit] == 0xA5).all(), rep
            assert np.array_equal(rq.cpu().numpy()[hit], wq[hit]), rep
            assert np.array_equal(rs.cpu().numpy()[hit].view(np.uint32), ws[hit].view(np.uint32)), rep
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert st["copied_bytes"] == st["write_bytes"] == 2 * int(hit.sum()) * rb
        if mode != "chunk32_ordered":
            assert np.array_equal(r.counters()[0], want_lay["count"][0])
        if log and mode != "chunk32_ordered":
            want_cmds = oracle.expected_cmds(idx[0], want_lay, 0, cfg.E_loc, cfg.H, "fp8", mode)
            assert oracle.cmd_multiset(epmod.ep_cmd_log(r.h)) == want_cmds + want_cmds
            oracle.check_fence_trace(epmod.ep_event_log(r.h), want_lay["count"])
        r.register_heaps(None, None)


def test_proxy_performs_writes_of_another_source_into_one_rank(epmod, oracle):
    """Config 2's inbound share: source 31's rows for rank 5 only, moved by the proxy (per token out of that
    source's x; as chunks out of a send heap), with the other ranks' partitions untouched."""
    cfg = g.config(2)
    for mode, name in ((epmod.EP_CMD_PER_TOKEN, "per_token"), (epmod.EP_CMD_CHUNK32, "chunk32")):
        out = _dispatch_case(epmod, oracle, cfg, 64, 0.0, mode, rank_filter=5, src=31, proxy_writes=True,
                             reorder_window=3)
        _check_commands(epmod, oracle, cfg, out, name, src=31, rank_filter=5)


def test_proxy_writes_follow_new_data_and_atomics_wait_for_them(epmod, oracle):
    """Three dispatches through the same registered heaps with different activations: each receive
    buffer holds that call's rows (nothing stale is forwarded), and count atomics, which do not wait for
    the copies, get ahead of their rows and are held back by the fence."""
    cfg = g.config(4, S=1)
    T = 600
    idx, _ = g.routing_all(cfg, T)
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    rows = idx.size
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    with _runner(epmod, cfg, T, num_channels=1, num_proxy_threads=1) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        send = torch.zeros((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
        recv = torch.zeros((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
        r.register_heaps(send, recv)
        for it in range(3):
            x = g.activations(cfg, it, T=T)
            r.dispatch(bits_to_bf16(x), d_idx[0], lay, send, cmd_mode=epmod.EP_CMD_CHUNK32 | epmod.EP_CMD_ATOMICS_FIRST)
            r.wait()
            torch.cuda.synchronize()
            want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
            assert np.array_equal(bf16_to_bits(recv), want), it
        st = r.stats()
        assert st["atomics_deferred"] >= 1 and st["proxy_error"] == 0 and st["device_error"] == 0
        # unregistering returns to the mode in which the kernel places the rows itself
        r.register_heaps(None, None)
        recv2 = torch.zeros_like(recv)
        r.dispatch(bits_to_bf16(x), d_idx[0], lay, recv2, cmd_mode=epmod.EP_CMD_PER_TOKEN)
        r.wait()
        torch.cuda.synchronize()
        assert np.array_equal(bf16_to_bits(recv2), want)
        assert r.stats()["copied_bytes"] == st["copied_bytes"]


@pytest.mark.parametrize("cid,T,window,limit,pack,proxy_writes", [
    (4, 600, 32, 6, 0, False), (5, 500, 0, 2, 8, True), (1, None, 4, 1, 16, False), (4, 300, 16, 5, 4, True)])
def test_pacing_and_packing_on_a_real_dispatch(epmod, oracle, cid, T, window, limit, pack, proxy_writes):
    """Per-token dispatch with the proxy's sender-side policies on: at most `limit` messages in flight per
    destination rank and thread, one-row Writes packed best-effort; the receive buffer, the counters and
    the fence trace are what they are without the policies."""
    cfg = g.config(cid, S=1)
    out = _dispatch_case(epmod, oracle, cfg, T, 0.05, epmod.EP_CMD_PER_TOKEN, proxy_writes=proxy_writes,
                         reorder_window=window, reorder_seed=13, max_outstanding=limit, pack_rows=pack)
    _check_commands(epmod, oracle, cfg, out, "per_token")
    st = out["stats"]
    assert 1 <= st["max_in_flight"] <= limit
    res = oracle.check_pacing_trace(out["events"], limit, cfg.E_loc)
    assert res["peak"] == st["max_in_flight"] and res["sent"] == st["write_msgs"] + st["atomics"]
    if pack > 1:
        assert st["write_msgs"] <= st["writes"]
        wr = out["events"][(out["events"][:, 0] & 0xFF) == oracle.EV_WRITE]
        assert len(wr) == st["write_msgs"] and wr[:, 3].sum() == st["write_rows"] and wr[:, 3].max() <= pack
    else:
        assert st["write_msgs"] == st["writes"]


def test_registered_heaps_argument_errors(epmod):
    cfg = g.config(1)
    with _runner(epmod, cfg) as r:
        x = torch.zeros((cfg.T, cfg.H), dtype=torch.bfloat16, device="cuda")
        recv = torch.zeros((cfg.T * cfg.K, cfg.H), dtype=torch.bfloat16, device="cuda")
        sc = torch.zeros((cfg.T * cfg.K, cfg.H // 128), dtype=torch.float32, device="cuda")
        idx = _dev(g.routing_all(cfg)[0])
        lay = r.layout(idx)

        def rc_of(fn):
            with pytest.raises(epmod.EPError) as ei:
                fn()
            return ei.value.rc
        # the flag needs registered heaps
        assert rc_of(lambda: r.dispatch(x, idx[0], lay, recv, cmd_mode=epmod.EP_CMD_PER_TOKEN |
                                        epmod.EP_CMD_NO_PLACEMENT)) == epmod.EP_EINVAL
        assert rc_of(lambda: r.register_heaps(x, None)) == epmod.EP_EINVAL
        r.register_heaps(x, recv)
        # per token: needs the flag, and x must be the registered source
        assert rc_of(lambda: r.dispatch(x, idx[0], lay, recv, cmd_mode=epmod.EP_CMD_PER_TOKEN)) == epmod.EP_EINVAL
        assert rc_of(lambda: r.dispatch(x.clone(), idx[0], lay, recv, cmd_mode=epmod.EP_CMD_PER_TOKEN |
                                        epmod.EP_CMD_NO_PLACEMENT)) == epmod.EP_EINVAL
        # chunks: must be packed into the registered source heap; FP8 messages carry their scales (no scale array)
        assert rc_of(lambda: r.dispatch(x, idx[0], lay, recv, cmd_mode=epmod.EP_CMD_CHUNK32)) == epmod.EP_EINVAL
        assert rc_of(lambda: r.dispatch(x, idx[0], lay, x, recv_scale=sc, payload=epmod.EP_FP8_E4M3,
                                        cmd_mode=epmod.EP_CMD_CHUNK32)) == epmod.EP_EINVAL
        # ring-off dispatch is unaffected
        r.dispatch(x, idx[0], lay, recv, cmd_mode=epmod.EP_CMD_NONE)
        torch.cuda.synchronize()
        assert r.stats()["cmds"] == 0


def test_atomics_first_forces_the_fence_path(epmod, oracle):
    cfg = g.config(1)
    for mode, name in ((epmod.EP_CMD_PER_TOKEN, "per_token"), (epmod.EP_CMD_CHUNK32, "chunk32")):
        out = _dispatch_case(epmod, oracle, cfg, None, 0.0, mode | epmod.EP_CMD_ATOMICS_FIRST, num_channels=1,
                             num_proxy_threads=1)
        res = _check_commands(epmod, oracle, cfg, out, name)
        # one channel, atomics pushed by the first wavefront before it stores anything: atomics with a
        # nonzero count reach the receiver ahead of (some of) their rows and must wait
        assert res["waited"] == out["stats"]["atomics_deferred"] and res["waited"] >= 1


@pytest.mark.parametrize("cid,T,window,proxy_writes", [(1, None, 0, False), (4, 400, 32, False), (5, 300, 8, True)])
def test_sender_side_fence_on_a_real_dispatch(epmod, oracle, cid, T, window, proxy_writes):
    """The count Atomics are pushed before any row (one channel, one thread), so each one with a nonzero
    count reaches the proxy ahead of its rows.  With the sender-side fence the sender half holds them;
    none has to wait at the receiver, and buffer, counters and fence trace are as ever."""
    cfg = g.config(cid, S=1)
    out = _dispatch_case(epmod, oracle, cfg, T, 0.0, epmod.EP_CMD_PER_TOKEN | epmod.EP_CMD_ATOMICS_FIRST,
                         proxy_writes=proxy_writes, extra_flags=epmod.EP_FLAG_SENDER_FENCE, num_channels=1,
                         num_proxy_threads=1, reorder_window=window, reorder_seed=4)
    res = _check_commands(epmod, oracle, cfg, out, "per_token")
    st = out["stats"]
    assert res["waited"] == 0 and st["atomics_deferred"] == 0
    assert st["sender_held"] >= 1
    held = out["events"][(out["events"][:, 0] & 0xFF) == oracle.EV_SENDER_HELD]
    assert len(held) == st["sender_held"]


def test_drain_blocks_until_popped_and_small_ring_backpressure(epmod, oracle):
    cfg = g.config(1)
    out = _dispatch_case(epmod, oracle, cfg, None, 0.0, epmod.EP_CMD_PER_TOKEN | epmod.EP_CMD_DRAIN,
                         ring_entries=8, num_channels=2, num_proxy_threads=2, reorder_window=3)
    _check_commands(epmod, oracle, cfg, out, "per_token")
    assert out["stats"]["drains"] == 2
    # 128 writes + 16 atomics through 2 rings of 8 slots: laps wrapped many times without loss
    assert out["stats"]["cmds"] == 128 + 16 + 2


def test_repeated_dispatch_reuses_scratch_and_counters(epmod, oracle):
    cfg = g.config(5, S=1)
    idx, _ = g.routing_all(cfg, 600)
    x = g.activations(cfg, 0, T=600)
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    with _runner(epmod, cfg, 600) as r:
        d_idx, d_x = _dev(idx), bits_to_bf16(x)
        lay = r.layout(d_idx)
        want_lay = oracle.layout(idx, cfg.E, cfg.R)
        want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, idx.size)
        for it, mode in enumerate([epmod.EP_CMD_CHUNK32, epmod.EP_CMD_PER_TOKEN, epmod.EP_CMD_CHUNK32]):
            recv = torch.zeros((idx.size, cfg.H), dtype=torch.bfloat16, device="cuda")
            r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=mode)
            r.wait()
            torch.cuda.synchronize()
            assert np.array_equal(bf16_to_bits(recv), want)
            st = r.stats()
            assert st["atomics_applied"] == cfg.E * (it + 1) and st["write_rows"] == idx.size * (it + 1)
            assert np.array_equal(r.counters()[0], want_lay["count"][0])


# ------------------------------------------------------------------- FP8
def _fp8_case(epmod, oracle, cfg, x, idx, cmd_mode):
    T = idx.shape[1]
    rows = int((idx >= 0).sum()) + 2
    from paper_2512_19849_amd.runner import bits_to_bf16
    with _runner(epmod, cfg, T, flags=epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS, heap_rows=rows) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        rq = torch.full((rows, cfg.H), 0xA5, dtype=torch.uint8, device="cuda")
        rs = torch.full((rows, cfg.H // 128), -1.0, dtype=torch.float32, device="cuda")
        r.dispatch(bits_to_bf16(x), d_idx[0], lay, rq, rs, payload=epmod.EP_FP8_E4M3, cmd_mode=cmd_mode)
        if cmd_mode != epmod.EP_CMD_NONE:
            r.wait()
        torch.cuda.synchronize()
        want_lay = oracle.layout(idx, cfg.E, cfg.R)
        wq, ws, _ = oracle.dispatch_fp8(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
        gq, gs = rq.cpu().numpy(), rs.cpu().numpy()
        assert np.array_equal(gs.view(np.uint32), ws.view(np.uint32)), "scales differ"
        bad = np.argwhere(gq != wq)
        assert bad.size == 0, f"{len(bad)} codes differ, first at {bad[:3].tolist()}"
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0
        return dict(stats=st, cmds=epmod.ep_cmd_log(r.h), events=epmod.ep_event_log(r.h), lay=want_lay, idx=idx,
                    counters=r.counters().copy())


@pytest.mark.parametrize("cid,T,mask,mode", [(3, None, 0.0, "none"), (3, None, 0.2, "per_token"),
                                             (5, 400, 0.0, "chunk32"), (4, 150, 0.0, "none")])
def test_dispatch_fp8_parity(epmod, oracle, cid, T, mask, mode):
    cfg = g.config(cid, S=1)
    idx, _ = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=29)
    x = g.activations(cfg, 0, T=idx.shape[1])
    out = _fp8_case(epmod, oracle, cfg, x, idx, epmod.CMD_MODES[mode])
    if mode != "none":
        _check_commands(epmod, oracle, cfg, out, mode, payload="fp8")


# tokens whose first expert was dropped read their row behind their pairs, the others ahead of them, those without any not at
# all (bf16: from 24 MB of tokens on); one and four tokens per workgroup
@pytest.mark.parametrize("payload", ["bf16", "fp8"])
@pytest.mark.parametrize("mode", ["none", "chunk32"])
@pytest.mark.parametrize("T,H", [(301, 7168), (1203, 1024), (1760, 7168), (12300, 1024)])
def test_dispatch_rows_ahead_of_their_pairs(epmod, oracle, T, H, mode, payload):
    cfg = g.EPConfig("ahead", T=T, H=H, E=32, K=4, R=4, routing="zipf", seed=H)
    idx, _ = g.routing_all(cfg)
    idx[0, ::3, 0] = -1
    idx[0, 1::4, :] = -1
    idx[0, -1, :] = -1
    x = np.resize(g.activations(cfg, 0, T=499), (T, H))
    if payload == "fp8":
        _fp8_case(epmod, oracle, cfg, x, idx, epmod.CMD_MODES[mode])
        return
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    rows = int((idx >= 0).sum()) + 2
    with _runner(epmod, cfg, T) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        recv = torch.full((rows, H), -1.5, dtype=torch.bfloat16, device="cuda")
        r.dispatch(bits_to_bf16(x), d_idx[0], lay, recv, cmd_mode=epmod.CMD_MODES[mode])
        if mode != "none":
            r.wait()
        torch.cuda.synchronize()
        want, _ = oracle.dispatch_bf16(x, idx[0], oracle.layout(idx, cfg.E, cfg.R)["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
        assert np.array_equal(bf16_to_bits(recv), want)
        assert r.stats()["device_error"] == 0


# a handle with one expert per rank keeps to four slices of a row per wave up to 384 MB of rows, others up to 320 MB
@pytest.mark.parametrize("E", [16, 32])
@pytest.mark.parametrize("T", [2790, 2791, 3348, 3349])
def test_dispatch_bf16_at_the_lines_of_one_slice_per_wave(epmod, E, T):
    H, K, R = 7168, 8, 16
    gen = torch.Generator(device="cuda").manual_seed(T)
    idx = torch.rand((1, T, E), generator=gen, device="cuda").topk(K, dim=-1).indices.to(torch.int32)
    idx = torch.where(torch.rand(idx.shape, generator=gen, device="cuda") < 0.1, -1, idx).contiguous()
    x = torch.randn((T, H), generator=gen, device="cuda", dtype=torch.bfloat16)
    with _runner(epmod, g.EPConfig("line", T=T, H=H, E=E, K=K, R=R), T, num_proxy_threads=0) as r:
        lay = r.layout(idx)
        recv = torch.full((T * K, H), -1.5, dtype=torch.bfloat16, device="cuda")
        r.dispatch(x, idx[0], lay, recv)
        valid = idx[0] >= 0
        got = recv[lay.dst_row[0][valid].long()]
        assert torch.equal(got, x[valid.nonzero()[:, 0]])
        assert (recv[int(valid.sum()):] == -1.5).all()
        assert r.stats()["device_error"] == 0


# one command per row beyond 12288 of them: the heads of up to 16 channels are read ahead every half ring
@pytest.mark.parametrize("channels,entries", [(1, 2), (3, 64), (16, 1024), (17, 1024), (8, 4096)])
def test_per_token_commands_read_heads_ahead(epmod, oracle, channels, entries):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    T, K = 1700, 8
    cfg = g.EPConfig("heads", T=T, H=128, E=32, K=K, R=4, routing="zipf", seed=entries)
    idx, _ = g.routing_all(cfg)
    idx = g.mask_random(idx, 0.05, seed=channels)
    rows = int((idx >= 0).sum())
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    with _runner(epmod, cfg, T, num_channels=channels, ring_entries=entries, num_proxy_threads=min(channels, 4)) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        recv = torch.empty((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
        for it in range(3):
            x = g.activations(cfg, it, T=T)
            recv.fill_(-1.5)
            r.dispatch(bits_to_bf16(x), d_idx[0], lay, recv, cmd_mode=epmod.EP_CMD_PER_TOKEN)
            r.wait()
            torch.cuda.synchronize()
            want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
            assert np.array_equal(bf16_to_bits(recv), want), it
            assert np.array_equal(r.counters()[0], want_lay["count"][0])
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert st["write_rows"] == 3 * rows


# 128 MB of rows: a row's scales leave together from there on; 9 blocks over 2 waves, 63 over 4 waves, the last of them ragged
@pytest.mark.parametrize("T,H,K,mask,mode", [(13468, 1152, 8, 0.0, "none"), (13469, 1152, 8, 0.0, "chunk32"),
                                             (3900, 8064, 4, 0.01, "chunk32_ordered"), (15200, 1024, 8, 0.001, "none")])
def test_dispatch_fp8_scales_stored_together(epmod, oracle, T, H, K, mask, mode):
    cfg = g.EPConfig("scales", T=T, H=H, E=16, K=K, R=4, routing="uniform", seed=T)
    idx, _ = g.routing_all(cfg)
    if mask:
        idx = g.mask_random(idx, mask, seed=K)
        idx[0, 7, :] = -1
    x = np.resize(g.activations(cfg, 0, T=499), (T, H))
    _fp8_case(epmod, oracle, cfg, x, idx, epmod.CMD_MODES[mode])


# a row's scales leave together from 200 MB of rows on: both sides of the line, four groups of channels per lane with a ragged last
# wave, a row that is one wave's, and messages that the proxy moves
@pytest.mark.parametrize("T,H,K,mask,mode", [(3382, 7168, 8, 0.0, "none"), (3383, 7168, 8, 0.01, "chunk32"),
                                             (2915, 8320, 8, 0.0, "chunk32_ordered"), (23700, 1024, 8, 0.0, "none")])
def test_dispatch_fp8_scales_stored_together_from_200_mb_on(epmod, oracle, T, H, K, mask, mode):
    test_dispatch_fp8_scales_stored_together(epmod, oracle, T, H, K, mask, mode)


@pytest.mark.parametrize("mode", ["chunk32", "chunk32_ordered"])
def test_proxy_performs_fp8_writes_with_scales_stored_together(epmod, oracle, mode):
    test_proxy_performs_fp8_writes(epmod, oracle, 4, 3400, 0.0, 0, mode, 4)


def test_dispatch_fp8_of_many_rows_to_one_rank(epmod):
    """One rank's part of 200 MB of rows is what the dispatch to all ranks places there; other rows keep their bytes."""
    T, H, E, K, R = 3400, 7168, 32, 8, 4
    gen = torch.Generator(device="cuda").manual_seed(5)
    idx = torch.rand((1, T, E), generator=gen, device="cuda").topk(K, dim=-1).indices.to(torch.int32)
    x = torch.randn((T, H), generator=gen, device="cuda", dtype=torch.bfloat16)
    with _runner(epmod, g.EPConfig("part", T=T, H=H, E=E, K=K, R=R), T, num_proxy_threads=0) as r:
        lay = r.layout(idx)
        rows = T * K
        got = [(torch.full((rows, H), 0xA5, dtype=torch.uint8, device="cuda"),
                torch.full((rows, H // 128), -1.0, dtype=torch.float32, device="cuda")) for _ in range(2)]
        for (rq, rs), rank in zip(got, (-1, 2)):
            r.dispatch(x, idx[0], lay, rq, rs, payload=epmod.EP_FP8_E4M3, rank_filter=rank)
        first, end = int(lay.rank_offset[2]), int(lay.rank_offset[3])
        for whole, part, untouched in zip(*got, (0xA5, -1.0)):
            assert torch.equal(whole[first:end], part[first:end])
            assert (part[:first] == untouched).all() and (part[end:] == untouched).all()
        assert r.stats()["device_error"] == 0


def test_fp8_quantiser_all_bf16_inputs_and_corner_blocks(epmod, oracle):
    """Every finite bf16 value goes through the kernel's quantiser, grouped so
    that blocks hold similar magnitudes (dense coverage of rounding cases),
    then again in a seeded shuffle (wide dynamic range inside a block); plus
    zero / tiny / threshold blocks and exact ties."""
    bits = np.arange(65536, dtype=np.uint32).astype(np.uint16)
    fin = bits[np.isfinite(g.bf16_bits_to_f32(bits))]
    by_mag = fin[np.argsort(np.abs(g.bf16_bits_to_f32(fin)), kind="stable")]
    rng = np.random.default_rng(7)
    H = 1024
    pad = (-len(fin)) % H
    parts = [np.concatenate([by_mag, by_mag[:pad]]), np.concatenate([rng.permutation(fin), fin[:pad]])]
    # neighbouring-magnitude blocks with one larger peak: exercises many inv values per value
    for mul in (2, 3, 7, 11):
        blk = np.concatenate([by_mag, by_mag[:pad]]).reshape(-1, 128).copy()
        peak = np.abs(g.bf16_bits_to_f32(blk)).max(axis=1) * mul
        ok = np.isfinite(peak.astype(np.float32)) & (peak < 3e38)
        blk[ok, 0] = g.f32_to_bf16_bits(peak[ok].astype(np.float32))
        parts.append(blk.reshape(-1))
    corner = np.zeros((8, H), np.uint16)
    corner[0, 5] = 0x8000                                       # zero block with a -0
    corner[1, :128] = 0x0080; corner[1, 1] = 0x8080             # 2^-126 everywhere
    corner[2, 0] = g.f32_to_bf16_bits(np.array([2.0 ** -100], np.float32))[0]
    corner[2, 1] = g.f32_to_bf16_bits(np.array([-(2.0 ** -101)], np.float32))[0]
    corner[3, 0] = g.f32_to_bf16_bits(np.array([2.0 ** -101], np.float32))[0]
    corner[4, :128] = g.f32_to_bf16_bits(np.array([1.5703125] * 128, np.float32)); corner[4, 0] = \
        g.f32_to_bf16_bits(np.array([2.09375], np.float32))[0]  # y = 336: exact tie between 320 and 352
    corner[5, :128] = 0x0001                                    # smallest bf16 subnormal
    corner[6, :256] = g.f32_to_bf16_bits(rng.normal(0, 1e-30, 256).astype(np.float32))
    corner[7, :] = g.f32_to_bf16_bits(rng.normal(0, 1e30, H).astype(np.float32))
    x = np.concatenate([p.reshape(-1, H) for p in parts] + [corner])
    T = x.shape[0]
    cfg = g.EPConfig("fp8sweep", T=T, H=H, E=4, K=1, R=2)
    idx = (np.arange(T, dtype=np.int32) % 4).reshape(1, T, 1)
    _fp8_case(epmod, oracle, cfg, x, idx, epmod.EP_CMD_NONE)


# --------------------------------------------------------------- combine
def _combine_check(oracle, out_bits, y, w, dst_row, K):
    want = oracle.combine(y, w, dst_row)
    ulp = oracle.bf16_ulp_distance(out_bits, want)
    assert ulp.max() <= 1, f"max distance {ulp.max()} bf16 steps"
    ref, mag = oracle.combine_f64(y, w, dst_row)
    got = g.bf16_bits_to_f32(out_bits).astype(np.float64)
    bound = 2.0 ** -8 * np.abs(ref) + K * 2.0 ** -24 * mag * (1 + 2.0 ** -7) + 2.0 ** -133
    assert (np.abs(got - ref) <= bound).all()
    return int((ulp != 0).sum())


@pytest.mark.parametrize("cid,T,mask", [(1, None, 0.0), (1, 41, 0.3), (2, None, 0.0), (4, 200, 0.0),
                                        (5, 300, 0.1)])
def test_combine_parity(epmod, oracle, cid, T, mask):
    cfg = g.config(cid, S=1)
    idx, w = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=31)
    T = idx.shape[1]
    lay = oracle.layout(idx, cfg.E, cfg.R)
    rows = max(1, int((idx >= 0).sum()))
    y = g.activations(cfg, 0, tid=g.TID_Y, T=rows)
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    with _runner(epmod, cfg, T) as r:
        out = torch.full((T, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        r.combine(bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0]), out)
        torch.cuda.synchronize()
        ndiff = _combine_check(oracle, bf16_to_bits(out), y, w[0], lay["dst_row"][0], cfg.K)
        assert ndiff == 0          # same fused chain on both sides: expected bit-equal
        assert r.stats()["device_error"] == 0


@pytest.mark.parametrize("fresh_mb", [0, 1, 4096])
def test_combine_directly_after_dispatch_reads_the_fresh_rows_first(epmod, oracle, fresh_mb, monkeypatch):
    """On a handle made with EP_FLAG_CACHE_HINTS a combine that follows a bf16 dispatch into the same buffer walks
    the tokens backwards and reads the rows of the last tokens with cached loads (none, some, or all of them, by
    the byte budget); a second combine of the same inputs takes the plain order.  Both equal the oracle's sum,
    bit for bit."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    monkeypatch.setenv("EP_COMBINE_FRESH_MB", str(fresh_mb))
    cfg = g.config(5, S=1)
    T = 333                                                      # 333 x 8 x 8 KiB = 2.6 MiB of rows
    idx, w = g.routing_all(cfg, T)
    idx = g.mask_random(idx, 0.1, seed=77)
    lay_want = oracle.layout(idx, cfg.E, cfg.R)
    rows = int((idx >= 0).sum()) + 1
    x = g.activations(cfg, 0, T=T)
    want_recv, _ = oracle.dispatch_bf16(x, idx[0], lay_want["dst_row"][0], cfg.E_loc, rows, -1, fill=0)
    with _runner(epmod, cfg, T, flags=epmod.EP_FLAG_CACHE_HINTS) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        recv = torch.zeros((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
        # three rounds into the same buffer: the dispatch takes the tokens forwards, backwards, forwards, and
        # the combine that follows finds the fresh rows at the end, at the start, at the end of the token range
        for rnd, mode in enumerate((epmod.EP_CMD_CHUNK32, epmod.EP_CMD_PER_TOKEN, epmod.EP_CMD_NONE)):
            recv.fill_(-2.0)
            recv[rows - 1].zero_()                                   # (the spare row nobody writes)
            outs = [torch.full((T, cfg.H), 3.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
            r.dispatch(bits_to_bf16(x), d_idx[0], lay, recv, cmd_mode=mode)
            r.combine(recv, _dev(w[0]), lay.dst_row[0], outs[0])       # directly after the dispatch
            r.combine(recv, _dev(w[0]), lay.dst_row[0], outs[1])       # nothing fresh any more
            r.wait()
            torch.cuda.synchronize()
            assert np.array_equal(bf16_to_bits(recv), want_recv), rnd
            for out in outs:
                assert _combine_check(oracle, bf16_to_bits(out), want_recv, w[0], lay_want["dst_row"][0], cfg.K) == 0
        assert r.stats()["device_error"] == 0


@pytest.mark.parametrize("K,vpl", [(1, 1), (3, 2), (5, 4), (6, 1), (8, 4), (2, 2), (4, 1), (8, 7), (3, 9), (8, 10),
                                   (2, 11), (4, 12), (5, 13), (8, 14), (6, 15)])
def test_combine_generic_k_and_splits(epmod, oracle, K, vpl, monkeypatch):
    monkeypatch.setenv("EP_COMBINE_VPL", str(vpl))
    cfg = g.EPConfig("ck", T=90, H=1536, E=24, K=K, R=3, seed=99)
    idx, w = g.routing_all(cfg)
    idx = g.mask_random(idx, 0.2, seed=3)
    idx[0, 5, :] = -1                                          # a token with every k masked
    lay = oracle.layout(idx, cfg.E, cfg.R)
    rows = int((idx >= 0).sum())
    y = g.activations(cfg, 0, tid=g.TID_Y, T=rows)
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    with _runner(epmod, cfg) as r:
        out = torch.full((cfg.T, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        r.combine(bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0]), out)
        torch.cuda.synchronize()
        ob = bf16_to_bits(out)
        assert _combine_check(oracle, ob, y, w[0], lay["dst_row"][0], K) == 0
        assert (ob[5] == 0).all()


@pytest.mark.parametrize("H", [4608, 4736, 5120, 5632, 6144, 6656, 7168, 7680])
def test_combine_one_wave_per_token_for_mid_sized_rows(epmod, oracle, H, monkeypatch):
    """Rows of 9 to 15 column slices (hidden 4736: a ragged last one), at 1600 tokens.  One wave per token, which is
    asked for here, is not offered any more: like any value that is not, it leaves a wave per slice."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    monkeypatch.setenv("EP_COMBINE_VPL", str((H // 8 + 63) // 64))
    cfg = g.EPConfig("cw", T=1600, H=H, E=32, K=8, R=4, routing="zipf", seed=1234 + H)
    idx, w = g.routing_all(cfg)
    idx = g.mask_random(idx, 0.05, seed=H)
    lay = oracle.layout(idx, cfg.E, cfg.R)
    rows = int((idx >= 0).sum())
    y = g.activations(cfg, 0, tid=g.TID_Y, T=rows)
    with _runner(epmod, cfg) as r:
        out = torch.full((cfg.T, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        r.combine(bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0]), out)
        torch.cuda.synchronize()
        assert _combine_check(oracle, bf16_to_bits(out), y, w[0], lay["dst_row"][0], cfg.K) == 0
        assert r.stats()["device_error"] == 0


# top-5 and top-7 with a wave per slice: the last volume with all loads of a slice in flight, the first with one at a time
@pytest.mark.parametrize("K,T", [(5, 3906), (5, 3907), (7, 1743), (7, 1744)])
def test_combine_loads_in_flight_by_volume(epmod, oracle, K, T):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("volume", T=T, H=8192, E=16, K=K, R=4, routing="uniform", seed=T)
    idx, w = g.routing_all(cfg)
    idx[0, 5, :] = -1
    lay = oracle.layout(idx, cfg.E, cfg.R)
    y = np.resize(g.activations(cfg, 0, tid=g.TID_Y, T=T), (T * K, cfg.H))
    with _runner(epmod, cfg, num_proxy_threads=0) as r:
        out = torch.full((T, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        r.combine(bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0]), out)
        torch.cuda.synchronize()
        assert _combine_check(oracle, bf16_to_bits(out), y, w[0], lay["dst_row"][0], K) == 0
        assert r.stats()["device_error"] == 0


# one expert per rank, up to top-8: masked entries load nothing (top-1 and top-9 as on other handles)
@pytest.mark.parametrize("K", range(1, 10))
def test_combine_on_a_handle_with_one_expert_per_rank(epmod, oracle, K):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("sparse", T=90, H=1152, E=12, K=K, R=12, seed=K)
    idx, w = g.routing_all(cfg)
    idx = g.mask_random(idx, 0.4, seed=K)
    idx[0, 5, :] = -1
    lay = oracle.layout(idx, cfg.E, cfg.R)
    rows = int((idx >= 0).sum())
    y = g.activations(cfg, 0, tid=g.TID_Y, T=rows)
    with _runner(epmod, cfg, num_proxy_threads=0) as r:
        out = torch.full((cfg.T, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        r.combine(bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0]), out)
        torch.cuda.synchronize()
        ob = bf16_to_bits(out)
        assert _combine_check(oracle, ob, y, w[0], lay["dst_row"][0], K) == 0
        assert (ob[5] == 0).all()
        assert r.stats()["device_error"] == 0


# the last launch without a limit on the waves of a compute unit and the first with one (84 KB / top-k; handles with one expert
# per rank: 100 KB / expected rows), two slices per token and a ragged second one; then the partial reduce's rule (96 KB)
@pytest.mark.parametrize("K,R,E,T", [(8, 4, 16, 6399), (8, 4, 16, 6400), (4, 4, 16, 13440), (8, 16, 16, 9600), (3, 2, 6, 18000),
                                     (8, 4, 16, 7680)])
def test_combine_with_few_waves_per_compute_unit(epmod, oracle, K, R, E, T):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("few", T=T, H=640, E=E, K=K, R=R, routing="uniform", seed=T)
    idx, w = g.routing_all(cfg)
    idx = g.mask_random(idx, 0.3, seed=K)
    idx[0, -1, :] = -1
    lay = oracle.layout(idx, cfg.E, cfg.R)
    rows = int((idx >= 0).sum())
    y = np.resize(g.activations(cfg, 0, tid=g.TID_Y, T=997), (rows, cfg.H))
    with _runner(epmod, cfg, num_proxy_threads=0) as r:
        d_y, d_w, d_row = bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0])
        out = torch.full((T, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        r.combine(d_y, d_w, d_row, out)
        # every entry a group of its own: a partial sum per row, in the row's own place
        own = torch.arange(K, dtype=torch.int32, device="cuda").repeat(T, 1)
        partial = torch.full((rows, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        epmod.ep_combine_partial(r.h, d_y, d_w, d_row, own, d_row, T, rows, rows, partial)
        torch.cuda.synchronize()
        assert _combine_check(oracle, bf16_to_bits(out), y, w[0], lay["dst_row"][0], K) == 0
        weight = np.zeros((rows, 1), np.float32)
        valid = lay["dst_row"][0] >= 0
        weight[lay["dst_row"][0][valid], 0] = w[0][valid]
        assert _combine_check(oracle, bf16_to_bits(partial), y, weight, np.arange(rows, dtype=np.int32)[:, None], 1) == 0
        assert r.stats()["device_error"] == 0


# two slices per token: the last launch without a limit on the waves of a compute unit and the first with one, 96 KB / top-k;
# then the same for the partial reduce, 128 KB
@pytest.mark.parametrize("K,T", [(8, 7679), (8, 7680), (7, 8319), (7, 8320), (6, 10240), (5, 12160), (4, 15360), (1, 7680),
                                 (8, 10239), (8, 10240), (6, 13440)])
def test_combine_with_as_many_waves_as_masked_entries_need(epmod, oracle, K, T):
    test_combine_with_few_waves_per_compute_unit(epmod, oracle, K, 4, 16, T)


# four waves per workgroup, three slices per token: the last workgroup holds one to four waves; the last launch that fits onto the
# chip at once and the first that does not; top-3 and less at any size
@pytest.mark.parametrize("K,T", [(8, 1), (8, 2), (4, 3), (9, 4), (8, 2730), (8, 2731), (12, 2730), (12, 2731), (3, 2733), (2, 6001),
                                 (1, 2734)])
def test_reduces_with_four_waves_per_workgroup(epmod, oracle, K, T):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("four", T=T, H=1152, E=16, K=K, R=4, routing="uniform", seed=T)
    idx, w = g.routing_all(cfg)
    idx = g.mask_random(idx, 0.2, seed=K)
    lay = oracle.layout(idx, cfg.E, cfg.R)
    rows = max(1, int((idx >= 0).sum()))
    y = np.resize(g.activations(cfg, 0, tid=g.TID_Y, T=499), (rows, cfg.H))
    with _runner(epmod, cfg, num_proxy_threads=0) as r:
        d_y, d_w, d_row = bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0])
        out = torch.full((T, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        r.combine(d_y, d_w, d_row, out)
        own = torch.arange(K, dtype=torch.int32, device="cuda").repeat(T, 1)  # every entry a group of its own
        partial = torch.full((rows, cfg.H), 7.0, dtype=torch.bfloat16, device="cuda")
        epmod.ep_combine_partial(r.h, d_y, d_w, d_row, own, d_row, T, rows, rows, partial)
        torch.cuda.synchronize()
        assert _combine_check(oracle, bf16_to_bits(out), y, w[0], lay["dst_row"][0], K) == 0
        valid = lay["dst_row"][0] >= 0
        if valid.any():
            weight = np.zeros((rows, 1), np.float32)
            weight[lay["dst_row"][0][valid], 0] = w[0][valid]
            assert _combine_check(oracle, bf16_to_bits(partial), y, weight, np.arange(rows, dtype=np.int32)[:, None], 1) == 0
        assert r.stats()["device_error"] == 0


def test_round_trip_identity_expert(epmod, oracle):
    """dispatch -> identity expert -> combine returns the input scaled by the
    sum of its weights; with K = 1 and w = 1 it is the input, bit for bit."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    for cid, K in ((1, None), (1, 1), (4, None)):
        cfg = g.config(cid, S=1) if K is None else g.config(cid, S=1, K=K)
        T = min(cfg.T, 256)
        idx, w = g.routing_all(cfg, T)
        if K == 1:
            w = np.ones_like(w)
        x = g.activations(cfg, 0, T=T)
        with _runner(epmod, cfg, T) as r:
            d_idx = _dev(idx)
            lay = r.layout(d_idx)
            recv = torch.zeros((idx.size, cfg.H), dtype=torch.bfloat16, device="cuda")
            r.dispatch(bits_to_bf16(x), d_idx[0], lay, recv, cmd_mode=epmod.EP_CMD_PER_TOKEN)
            out = torch.zeros((T, cfg.H), dtype=torch.bfloat16, device="cuda")
            r.combine(recv, _dev(w[0]), lay.dst_row[0], out)
            r.wait()
            torch.cuda.synchronize()
            ob = bf16_to_bits(out)
            if K == 1:
                assert np.array_equal(ob, x)
            else:
                xf = g.bf16_bits_to_f32(x).astype(np.float64)
                want = xf * w[0].astype(np.float64).sum(1, keepdims=True)
                got = g.bf16_bits_to_f32(ob).astype(np.float64)
                assert (np.abs(got - want) <= 2.0 ** -8 * np.abs(want) * (1 + 2.0 ** -10) + 2.0 ** -133).all()
                assert oracle.bf16_ulp_distance(ob, x).max() <= 1


# ------------------------------------------------------------- error paths
def test_ring_off_step_replays_from_a_hip_graph(epmod, oracle):
    """layout -> dispatch (ring off) -> combine touch no host state and clear their own scratch, so the three
    launches can be captured once and replayed: every replay, with new routing and new activations in the
    same buffers and eager work in between, must give what the eager calls give (= the oracle's result)."""
    cfg = g.config(1)
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    T, rows = cfg.T, cfg.T * cfg.K
    with _runner(epmod, cfg, num_proxy_threads=0) as r:
        d_idx = torch.zeros((1, T, cfg.K), dtype=torch.int32, device="cuda")
        d_x = torch.zeros((T, cfg.H), dtype=torch.bfloat16, device="cuda")
        d_w = torch.zeros((T, cfg.K), dtype=torch.float32, device="cuda")
        recv = torch.zeros((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
        out = torch.zeros((T, cfg.H), dtype=torch.bfloat16, device="cuda")

        def step():
            lay = r.layout(d_idx)
            r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=epmod.EP_CMD_NONE)
            r.combine(recv, d_w, lay.dst_row[0], out)
            return lay

        def load(seed):
            c2 = g.EPConfig(cfg.name, T=cfg.T, H=cfg.H, E=cfg.E, K=cfg.K, R=cfg.R, S=1, seed=cfg.seed + seed)
            idx, w = g.routing_all(c2)
            x = g.activations(c2)
            d_idx.copy_(_dev(idx))
            d_w.copy_(_dev(w[0]))
            d_x.copy_(bits_to_bf16(x))
            return idx, w, x

        load(0)
        step()                                       # warm-up outside the capture (first-use initialisation)
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                lay = step()
        for seed in (1, 2, 3):
            idx, w, x = load(seed)
            recv.fill_(7.0)                          # eager work between the replays
            graph.replay()
            torch.cuda.synchronize()
            want_lay = oracle.layout(idx, cfg.E, cfg.R)
            got = lay.numpy()
            for name, v in want_lay.items():
                assert np.array_equal(got[name], v), (seed, name)
            wrecv, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
            assert np.array_equal(bf16_to_bits(recv), wrecv), seed
            wout = oracle.combine(wrecv, w[0], want_lay["dst_row"][0])
            assert int(oracle.bf16_ulp_distance(bf16_to_bits(out), wout).max()) <= 1, seed
            # and the eager path on the same inputs
            out.zero_()
            step()
            torch.cuda.synchronize()
            assert int(oracle.bf16_ulp_distance(bf16_to_bits(out), wout).max()) <= 1
        assert r.stats()["device_error"] == 0


@pytest.mark.parametrize("mode_name", ["per_token", "chunk32", "chunk32_ordered", "ring_channels"])
def test_ring_on_step_replays_from_a_hip_graph(epmod, oracle, mode_name):
    """layout -> dispatch with commands through the proxy -> GPU-side wait for the posted counters -> combine,
    captured once and replayed with new routing and activations, eager work and synchronisations in between.
    A call on a capturing stream runs nothing, so what its kernel will push goes to the handle's ledger
    (ep_captured) and is handed back with ep_expect at every launch of the graph; every replay must give what
    the eager calls give (= the oracle's result), and ep_wait must cover the replayed commands."""
    cfg = g.config(1)
    mode = {"per_token": epmod.EP_CMD_PER_TOKEN, "chunk32": epmod.EP_CMD_CHUNK32,
            "chunk32_ordered": epmod.EP_CMD_CHUNK32_ORDERED, "ring_channels": None}[mode_name]
    channels = mode is None                          # ep_ht_dispatch: rows through ring slots, ends with Drains
    ordered = channels or mode == epmod.EP_CMD_CHUNK32_ORDERED
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    T, rows = cfg.T, cfg.T * cfg.K
    kw = dict(ht_slices=3, ht_ring_slots=1) if channels else {}
    with _runner(epmod, cfg, num_proxy_threads=2, spin_timeout_ms=10000, **kw) as r:
        d_idx = torch.zeros((1, T, cfg.K), dtype=torch.int32, device="cuda")
        d_x = torch.zeros((T, cfg.H), dtype=torch.bfloat16, device="cuda")
        d_w = torch.zeros((T, cfg.K), dtype=torch.float32, device="cuda")
        recv = torch.zeros((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
        out = torch.zeros((T, cfg.H), dtype=torch.bfloat16, device="cuda")
        counts = torch.zeros((cfg.E,), dtype=torch.int32, device="cuda")
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda") if channels else None

        def step():
            lay = r.layout(d_idx)
            if channels:
                r.ht_dispatch(d_x, d_idx[0], lay, ring, recv)
            else:
                r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=mode)
            if not ordered:                          # (the ordered mode announces rows per rank, not per expert)
                r.recv_wait(counts)
            r.combine(recv, d_w, lay.dst_row[0], out)
            return lay

        def load(seed):
            c2 = g.EPConfig(cfg.name, T=cfg.T, H=cfg.H, E=cfg.E, K=cfg.K, R=cfg.R, S=1, seed=cfg.seed + seed)
            idx, w = g.routing_all(c2)
            x = g.activations(c2)
            d_idx.copy_(_dev(idx))
            d_w.copy_(_dev(w[0]))
            d_x.copy_(bits_to_bf16(x))
            return idx, w, x

        load(0)
        step()                                       # warm-up outside the capture (first-use initialisation)
        r.wait()
        torch.cuda.synchronize()
        assert r.captured() == (0, 0)                # eager calls leave the ledger alone
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                lay = step()
        cap = r.captured()
        assert cap == ((0, 8) if ordered else (cfg.E, 0))   # 8 FIFOs to drain, or one count Atomic per expert
        assert r.captured() == (0, 0)                # reading it cleared it
        r.wait()                                     # nothing was launched by the capture: returns at once
        for seed in (1, 2, 3):
            idx, w, x = load(seed)
            recv.fill_(7.0)                          # eager work between the replays
            counts.fill_(-5)
            r.expect(*cap)
            graph.replay()
            r.wait()                                 # covers the replayed commands
            torch.cuda.synchronize()
            want_lay = oracle.layout(idx, cfg.E, cfg.R)
            got = lay.numpy()
            for name, v in want_lay.items():
                assert np.array_equal(got[name], v), (seed, name)
            wrecv, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
            assert np.array_equal(bf16_to_bits(recv), wrecv), seed
            wout = oracle.combine(wrecv, w[0], want_lay["dst_row"][0])
            assert int(oracle.bf16_ulp_distance(bf16_to_bits(out), wout).max()) <= 1, seed
            if not ordered:
                assert np.array_equal(counts.cpu().numpy(), want_lay["count"][0]), seed
                assert np.array_equal(r.counters()[0], want_lay["count"][0]), seed
            # and the eager path on the same inputs
            out.zero_()
            step()
            r.wait()
            torch.cuda.synchronize()
            assert int(oracle.bf16_ulp_distance(bf16_to_bits(out), wout).max()) <= 1
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        if not ordered:
            assert st["atomics_applied"] == 7 * cfg.E   # warm-up + three replays + three eager steps


def test_profile_reports_the_kernels_own_durations(epmod, oracle):
    """ep_profile: timed launches give the same results, their durations are positive, add up per call, are not
    longer than what recorded events around the same calls see, and nothing is timed while profiling is off."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.config(4, S=1)
    T = 1024
    idx, w = g.routing_all(cfg, T)
    x = g.activations(cfg, 0, T=T)
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    wrecv, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, idx.size)
    wout = oracle.combine(wrecv, w[0], want_lay["dst_row"][0])
    with _runner(epmod, cfg, T) as r:
        d_idx, d_x, d_w = _dev(idx), bits_to_bf16(x), _dev(w[0])
        recv = torch.zeros((idx.size, cfg.H), dtype=torch.bfloat16, device="cuda")
        out = torch.zeros((T, cfg.H), dtype=torch.bfloat16, device="cuda")

        def step():
            lay = r.layout(d_idx)
            r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=epmod.EP_CMD_CHUNK32)
            r.combine(recv, d_w, lay.dst_row[0], out)
            r.wait()
            return lay

        step()
        torch.cuda.synchronize()
        assert [epmod.ep_profile_read(r.h, c)[1] for c in (0, 1, 2)] == [0, 0, 0]
        epmod.ep_profile(r.h, 8)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(3):
            lay = step()
        b.record()
        epmod.ep_profile(r.h, False)
        step()                                       # not timed
        torch.cuda.synchronize()
        assert np.array_equal(lay.numpy()["dst_row"], want_lay["dst_row"])
        assert np.array_equal(bf16_to_bits(recv), wrecv) and np.array_equal(bf16_to_bits(out), wout)
        total = 0.0
        for call in (0, 1, 2):
            ms, n = epmod.ep_profile_read(r.h, call, reset=False)
            assert n == 3 and 0.003 < ms / n < 5.0, (call, ms, n)
            assert epmod.ep_profile_read(r.h, call) == (ms, n)            # unchanged until reset
            assert epmod.ep_profile_read(r.h, call) == (0.0, 0)
            total += ms
        assert total <= a.elapsed_time(b)            # the kernels ran inside the bracket
        with pytest.raises(epmod.EPError):
            epmod.ep_profile_read(r.h, 3)
        assert r.stats()["device_error"] == 0


def test_host_side_argument_errors(epmod):
    from paper_2512_19849_amd.runner import EPRunner
    with pytest.raises(epmod.EPError):
        epmod.ep_proxy_start(3, 16, 2, 1024, 64)               # E % R != 0
    with pytest.raises(epmod.EPError):
        epmod.ep_proxy_start(4, 16, 2, 1000, 64)               # H % 128 != 0
    with EPRunner(4, 16, 2, 1024, 64, num_proxy_threads=0) as r:
        idx = torch.zeros((1, 64, 2), dtype=torch.int32, device="cuda")
        lay = r.layout(idx)
        x = torch.zeros((64, 1024), dtype=torch.bfloat16, device="cuda")
        recv = torch.zeros((128, 1024), dtype=torch.bfloat16, device="cuda")
        with pytest.raises(epmod.EPError):                     # ring on but no proxy thread
            r.dispatch(x, idx[0], lay, recv, cmd_mode=epmod.EP_CMD_PER_TOKEN)
        with pytest.raises(epmod.EPError):                     # more tokens than the handle's capacity
            epmod.ep_layout(r.h, idx, 65, lay.count, lay.expert_total, lay.rank_total, lay.base,
                            lay.expert_offset, lay.rank_offset, lay.slot, lay.dst_row)
        torch.cuda.synchronize()


def test_device_side_bounds_check_reports_instead_of_faulting(epmod, oracle):
    """A destination row beyond the receive buffer is skipped by the kernel's
    own bounds check and surfaces as EP_EBOUNDS."""
    from paper_2512_19849_amd.runner import EPRunner
    cfg = g.config(1)
    idx, _ = g.routing_all(cfg)
    with EPRunner(cfg.R, cfg.E, cfg.K, cfg.H, cfg.T, spin_timeout_ms=2000) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        x = torch.zeros((cfg.T, cfg.H), dtype=torch.bfloat16, device="cuda")
        recv = torch.zeros((100, cfg.H), dtype=torch.bfloat16, device="cuda")   # 128 rows needed
        r.dispatch(x, d_idx[0], lay, recv, cmd_mode=epmod.EP_CMD_NONE)
        torch.cuda.synchronize()
        assert r.stats()["device_error"] == epmod.EP_EBOUNDS
        with pytest.raises(epmod.EPError):
            r.wait()


# ------------------------------------------- full sizes, bench launch configuration
@pytest.mark.parametrize("cid,payload,mode,threads", [(4, "bf16", "chunk32", 4), (4, "bf16", "per_token", 4),
                                                      (5, "bf16", "chunk32", 4), (5, "fp8", "chunk32", 1),
                                                      (5, "fp8", "per_token", 4), (4, "fp8", "chunk32", 4),
                                                      (4, "bf16", "chunk32_ordered", 4), (5, "bf16", "per_token", 4),
                                                      (5, "bf16", "chunk32_ordered", 4), (4, "fp8", "per_token", 4),
                                                      (4, "fp8", "chunk32_ordered", 4), (5, "fp8", "chunk32_ordered", 4),
                                                      (4, "bf16", "per_token", 1)])
def test_full_size_round_trip(epmod, oracle, cid, payload, mode, threads):
    """The whole path at the workload's full size, element by element, with the
    launch configuration bench.py times (8 channels x 4096 slots)."""
    from paper_2512_19849_amd.runner import EPRunner, bits_to_bf16, bf16_to_bits
    cfg = g.config(cid, S=1)
    idx, w = g.routing_all(cfg)
    x = g.activations(cfg)
    rows = idx.size
    oracle.set_threads(min(16, oracle.max_threads()))
    try:
        want = oracle.layout(idx, cfg.E, cfg.R)
        with EPRunner(cfg.R, cfg.E, cfg.K, cfg.H, cfg.T, num_proxy_threads=threads, spin_timeout_ms=10000) as r:
            d_idx, d_x, d_w = _dev(idx), bits_to_bf16(x), _dev(w[0])
            lay = r.layout(d_idx)
            out = torch.zeros((cfg.T, cfg.H), dtype=torch.bfloat16, device="cuda")
            if payload == "bf16":
                recv = torch.zeros((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
                r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=epmod.CMD_MODES[mode])
                y_dev = recv
            else:
                rq = torch.zeros((rows, cfg.H), dtype=torch.uint8, device="cuda")
                rs = torch.zeros((rows, cfg.H // 128), dtype=torch.float32, device="cuda")
                r.dispatch(d_x, d_idx[0], lay, rq, rs, payload=epmod.EP_FP8_E4M3, cmd_mode=epmod.CMD_MODES[mode])
                y_bits = g.activations(cfg, 0, tid=g.TID_Y, T=rows)
                y_dev = bits_to_bf16(y_bits)
            r.combine(y_dev, d_w, lay.dst_row[0], out)
            r.wait()
            torch.cuda.synchronize()
            got = lay.numpy()
            for name, v in want.items():
                assert np.array_equal(got[name], v), name
            if payload == "bf16":
                wrecv, wc = oracle.dispatch_bf16(x, idx[0], want["dst_row"][0], cfg.E_loc, rows)
                assert np.array_equal(bf16_to_bits(recv), wrecv)
                y_bits = wrecv
            else:
                wq, ws, _ = oracle.dispatch_fp8(x, idx[0], want["dst_row"][0], cfg.E_loc, rows)
                assert np.array_equal(rq.cpu().numpy(), wq)
                assert np.array_equal(rs.cpu().numpy().view(np.uint32), ws.view(np.uint32))
            wout = oracle.combine(y_bits, w[0], want["dst_row"][0])
            assert oracle.bf16_ulp_distance(bf16_to_bits(out), wout).max() <= 1
            assert np.array_equal(bf16_to_bits(out), wout)
            st = r.stats()
            assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
            assert st["write_rows"] == rows
            nchunks = int(np.ceil(want["count"][0] / 32).sum())
            assert st["writes"] == (rows if mode == "per_token" else nchunks)
            if mode == "chunk32_ordered":                      # tail counters instead of per-expert count atomics
                assert np.array_equal(epmod.ep_tail_counters(r.h, 1, cfg.R)[0], want["rank_total"])
            else:
                assert st["atomics_applied"] == cfg.E
                assert np.array_equal(r.counters()[0], want["count"][0])
    finally:
        oracle.set_threads(1)


@pytest.mark.parametrize("cid,payload", [(4, "bf16"), (5, "bf16"), (4, "fp8"), (5, "fp8")])
def test_full_size_ring_off_dispatch(epmod, oracle, cid, payload):
    """The ring-off dispatch at the workload's full size (the shape the timing suite launches: no proxy threads
    needed, no commands), element by element."""
    from paper_2512_19849_amd.runner import EPRunner, bits_to_bf16, bf16_to_bits
    cfg = g.config(cid, S=1)
    idx, _ = g.routing_all(cfg)
    x = g.activations(cfg)
    rows = idx.size
    oracle.set_threads(min(16, oracle.max_threads()))
    try:
        want = oracle.layout(idx, cfg.E, cfg.R)
        with EPRunner(cfg.R, cfg.E, cfg.K, cfg.H, cfg.T, num_proxy_threads=4, spin_timeout_ms=10000) as r:
            d_idx, d_x = _dev(idx), bits_to_bf16(x)
            lay = r.layout(d_idx)
            if payload == "bf16":
                recv = torch.full((rows, cfg.H), -1.5, dtype=torch.bfloat16, device="cuda")
                r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=epmod.EP_CMD_NONE)
                torch.cuda.synchronize()
                wrecv, _ = oracle.dispatch_bf16(x, idx[0], want["dst_row"][0], cfg.E_loc, rows)
                assert np.array_equal(bf16_to_bits(recv), wrecv)
            else:
                rq = torch.full((rows, cfg.H), 0x55, dtype=torch.uint8, device="cuda")
                rs = torch.full((rows, cfg.H // 128), -1.0, dtype=torch.float32, device="cuda")
                r.dispatch(d_x, d_idx[0], lay, rq, rs, payload=epmod.EP_FP8_E4M3, cmd_mode=epmod.EP_CMD_NONE)
                torch.cuda.synchronize()
                wq, ws, _ = oracle.dispatch_fp8(x, idx[0], want["dst_row"][0], cfg.E_loc, rows)
                assert np.array_equal(rq.cpu().numpy(), wq)
                assert np.array_equal(rs.cpu().numpy().view(np.uint32), ws.view(np.uint32))
            st = r.stats()
            assert st["device_error"] == 0 and st["cmds"] == 0
    finally:
        oracle.set_threads(1)


@pytest.mark.parametrize("cid,mode", [(4, "per_token"), (4, "chunk32"), (4, "chunk32_ordered"), (5, "per_token"),
                                      (5, "chunk32"), (5, "chunk32_ordered")])
def test_full_size_proxy_performed_writes(epmod, oracle, cid, mode):
    """Registered heaps at the workload's full size, in the shape the timing suite launches (4 proxy threads,
    8 channels x 4096 slots, no logs): the kernel only pushes commands (per token, straight out of x) or packs a
    send heap (chunks), the proxy threads move every row; the receive heap equals the oracle's element by element."""
    from paper_2512_19849_amd.runner import EPRunner, bits_to_bf16, bf16_to_bits
    cfg = g.config(cid, S=1)
    idx, _ = g.routing_all(cfg)
    x = g.activations(cfg)
    rows = idx.size
    oracle.set_threads(min(16, oracle.max_threads()))
    try:
        want = oracle.layout(idx, cfg.E, cfg.R)
        wrecv, _ = oracle.dispatch_bf16(x, idx[0], want["dst_row"][0], cfg.E_loc, rows)
    finally:
        oracle.set_threads(1)
    with EPRunner(cfg.R, cfg.E, cfg.K, cfg.H, cfg.T, num_proxy_threads=4, spin_timeout_ms=10000) as r:
        d_idx, d_x = _dev(idx), bits_to_bf16(x)
        lay = r.layout(d_idx)
        recv = torch.full((rows, cfg.H), -1.5, dtype=torch.bfloat16, device="cuda")
        if mode == "per_token":
            r.register_heaps(d_x, recv)
            target, cm = recv, epmod.EP_CMD_PER_TOKEN | epmod.EP_CMD_NO_PLACEMENT
        else:
            target = torch.full((rows, cfg.H), 2.5, dtype=torch.bfloat16, device="cuda")
            r.register_heaps(target, recv)
            cm = epmod.CMD_MODES[mode]
        for rep in range(2):                                   # the second dispatch overwrites the sentinel again
            recv.fill_(-1.5)
            r.dispatch(d_x, d_idx[0], lay, target, cmd_mode=cm)
            r.wait()
            torch.cuda.synchronize()
            assert np.array_equal(bf16_to_bits(recv), wrecv), rep
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert st["copied_bytes"] == st["write_bytes"] == 2 * rows * cfg.H * 2 and st["write_rows"] == 2 * rows
        if mode != "chunk32_ordered":
            assert np.array_equal(r.counters()[0], want["count"][0])
        r.register_heaps(None, None)


def test_full_size_decode_share_32_sources(epmod, oracle):
    """Config 2: this rank sends its 128 tokens to all 32 ranks, and receives in
    its own partition what the routing of all 32 source ranks sends to rank 0."""
    from paper_2512_19849_amd.runner import EPRunner, bits_to_bf16, bf16_to_bits
    cfg = g.config(2)
    idx, w = g.routing_all(cfg)
    rows = idx.size
    want = oracle.layout(idx, cfg.E, cfg.R)
    xs = [g.activations(cfg, s) for s in range(cfg.S)]
    with EPRunner(cfg.R, cfg.E, cfg.K, cfg.H, cfg.T, S=cfg.S, spin_timeout_ms=10000,
                  flags=epmod.EP_FLAG_LOG_EVENTS) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        recv = torch.full((rows, cfg.H), -1.5, dtype=torch.bfloat16, device="cuda")
        r.dispatch(bits_to_bf16(xs[0]), d_idx[0], lay, recv, src=0, cmd_mode=epmod.EP_CMD_PER_TOKEN)   # send share
        for s in range(1, cfg.S):                                                                        # inbound share
            r.dispatch(bits_to_bf16(xs[s]), d_idx[s], lay, recv, src=s, rank_filter=0,
                       cmd_mode=epmod.EP_CMD_PER_TOKEN)
        out = torch.zeros((cfg.T, cfg.H), dtype=torch.bfloat16, device="cuda")
        r.combine(recv, _dev(w[0]), lay.dst_row[0], out)
        r.wait()
        torch.cuda.synchronize()
        got = lay.numpy()
        for name, v in want.items():
            assert np.array_equal(got[name], v), name
        wrecv = np.full((rows, cfg.H), 0xBFC0, np.uint16)
        oracle.dispatch_bf16(xs[0], idx[0], want["dst_row"][0], cfg.E_loc, rows, recv=wrecv)
        for s in range(1, cfg.S):
            oracle.dispatch_bf16(xs[s], idx[s], want["dst_row"][s], cfg.E_loc, rows, rank_filter=0, recv=wrecv)
        assert np.array_equal(bf16_to_bits(recv), wrecv)
        assert np.array_equal(bf16_to_bits(out), oracle.combine(wrecv, w[0], want["dst_row"][0]))
        cnt = r.counters()
        assert np.array_equal(cnt[0], want["count"][0])
        assert np.array_equal(cnt[1:, :cfg.E_loc], want["count"][1:, :cfg.E_loc])       # rank 0's experts
        assert (cnt[1:, cfg.E_loc:] == 0).all()
        oracle.check_fence_trace(epmod.ep_event_log(r.h), want["count"])
        st = r.stats()
        assert st["atomics_applied"] == cfg.E + (cfg.S - 1) * cfg.E_loc


# ------------------------------------------------------- GPU-side receive wait
def test_recv_wait_orders_combine_after_the_counters_on_the_gpu(epmod, oracle):
    """dispatch -> ep_recv_wait -> combine in one stream, no host wait in between:
    the wait kernel polls the pinned-host counters the proxy posts, returns the
    counts and clears the flags; three rounds reuse the same flags."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.config(4, S=1)
    T = 512
    idx, w = g.routing_all(cfg, T)
    x = g.activations(cfg, 0, T=T)
    want = oracle.layout(idx, cfg.E, cfg.R)
    wrecv, _ = oracle.dispatch_bf16(x, idx[0], want["dst_row"][0], cfg.E_loc, idx.size)
    wout = oracle.combine(wrecv, w[0], want["dst_row"][0])
    with _runner(epmod, cfg, T) as r:
        d_idx, d_x, d_w = _dev(idx), bits_to_bf16(x), _dev(w[0])
        for rnd, mode in enumerate((epmod.EP_CMD_PER_TOKEN, epmod.EP_CMD_CHUNK32, epmod.EP_CMD_PER_TOKEN)):
            lay = r.layout(d_idx)
            recv = torch.zeros((idx.size, cfg.H), dtype=torch.bfloat16, device="cuda")
            out = torch.zeros((T, cfg.H), dtype=torch.bfloat16, device="cuda")
            counts = torch.full((cfg.E,), -7, dtype=torch.int32, device="cuda")
            r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=mode)
            r.recv_wait(counts)
            r.combine(recv, d_w, lay.dst_row[0], out)
            torch.cuda.synchronize()
            assert np.array_equal(counts.cpu().numpy(), want["count"][0])
            assert np.array_equal(bf16_to_bits(out), wout)
            r.wait()                                             # already satisfied
            assert r.stats()["device_error"] == 0


def test_recv_wait_with_rank_filter_and_other_source(epmod, oracle):
    from paper_2512_19849_amd.runner import bits_to_bf16
    cfg = g.config(2)
    idx, _ = g.routing_all(cfg, 64)
    want = oracle.layout(idx, cfg.E, cfg.R)
    x = g.activations(cfg, 5, T=64)
    with _runner(epmod, cfg, 64) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        recv = torch.zeros((idx.size, cfg.H), dtype=torch.bfloat16, device="cuda")
        counts = torch.full((cfg.E,), -7, dtype=torch.int32, device="cuda")
        r.dispatch(bits_to_bf16(x), d_idx[5], lay, recv, src=5, rank_filter=3, cmd_mode=epmod.EP_CMD_PER_TOKEN)
        r.recv_wait(counts, src=5, rank_filter=3)
        torch.cuda.synchronize()
        got = counts.cpu().numpy()
        lo, hi = 3 * cfg.E_loc, 4 * cfg.E_loc
        assert np.array_equal(got[lo:hi], want["count"][5, lo:hi])
        assert (got[:lo] == -1).all() and (got[hi:] == -1).all()


def test_recv_wait_times_out_when_nothing_was_dispatched(epmod):
    """No dispatch, so no counter is ever posted: the host never satisfies the
    kernel's bounded wait, which expires, reports EP_ETIMEOUT and exits."""
    cfg = g.config(1)
    with _runner(epmod, cfg, spin_timeout_ms=100) as r:
        counts = torch.zeros((cfg.E,), dtype=torch.int32, device="cuda")
        r.recv_wait(counts)
        torch.cuda.synchronize()
        assert r.stats()["device_error"] == epmod.EP_ETIMEOUT
        assert (counts.cpu().numpy() == -1).all()


# ------------------------------------------------- high-throughput mode (dedup + hierarchical reduce)
@pytest.mark.parametrize("cid,G,T,mask", [(1, 1, None, 0.0), (1, 2, 50, 0.3), (2, 8, 128, 0.0), (4, 1, 4096, 0.0),
                                          (4, 8, 1000, 0.1), (5, 2, 8192, 0.0)])
def test_ht_dedup_parity(epmod, oracle, cid, G, T, mask):
    cfg = g.config(cid)
    idx, _ = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=43)
    wg, wf = oracle.dedup(idx, cfg.E_loc, G)
    with _runner(epmod, cfg, idx.shape[1], num_proxy_threads=0) as r:
        d_idx = _dev(idx)
        gi = torch.full_like(d_idx, -9)
        fk = torch.full_like(d_idx, -9)
        epmod.ep_dedup(r.h, d_idx, idx.shape[1], G, gi, fk)
        torch.cuda.synchronize()
        assert np.array_equal(gi.cpu().numpy(), wg) and np.array_equal(fk.cpu().numpy(), wf)
        assert r.stats()["device_error"] == 0


# a top-k with an instance of its own (7), and without: a remainder of one and of three rows per batch of four
@pytest.mark.parametrize("K,E,R,G,H", [(3, 12, 4, 2, 640), (5, 16, 8, 4, 1024), (7, 24, 6, 1, 512), (9, 32, 4, 4, 640),
                                       (13, 48, 2, 2, 1536), (33, 48, 3, 1, 256)])
def test_partial_reduce_top_k_edges(epmod, oracle, K, E, R, G, H):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("partial", T=61, H=H, E=E, K=K, R=R, seed=K)
    idx, w = g.routing_all(cfg)
    idx = g.mask_random(idx, 0.15, seed=K)
    idx[0, 7, :] = -1
    wg, wf = oracle.dedup(idx, cfg.E_loc, G)
    lay, lay_g = oracle.layout(idx, E, R), oracle.layout(wg, R // G, R // G)
    rows, rows_g = int((idx >= 0).sum()), int((wg >= 0).sum())
    y = g.activations(cfg, 0, tid=g.TID_Y, T=rows)
    want = oracle.combine_partial(y, w[0], lay["dst_row"][0], wf[0], lay_g["dst_row"][0], rows_g)
    with _runner(epmod, cfg, num_proxy_threads=0) as r:
        partial = torch.zeros((rows_g, H), dtype=torch.bfloat16, device="cuda")
        epmod.ep_combine_partial(r.h, bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0]), _dev(wf[0]),
                                 _dev(lay_g["dst_row"][0]), cfg.T, rows, rows_g, partial)
        out = torch.full((cfg.T, H), 7.0, dtype=torch.bfloat16, device="cuda")
        r.combine(bits_to_bf16(y), _dev(w[0]), _dev(lay["dst_row"][0]), out)
        torch.cuda.synchronize()
        assert np.array_equal(bf16_to_bits(partial), want)
        assert _combine_check(oracle, bf16_to_bits(out), y, w[0], lay["dst_row"][0], K) == 0


# top-k that does not divide a workgroup's 256 threads, the largest, a single entry; tokens that leave a remainder
@pytest.mark.parametrize("S,T,K,E,R,G", [(1, 1, 1, 8, 4, 2), (2, 129, 3, 12, 6, 3), (1, 52, 5, 16, 8, 1),
                                         (3, 37, 7, 64, 16, 4), (1, 29, 33, 96, 12, 6), (2, 9, 64, 128, 8, 2)])
def test_ht_dedup_top_k_edges(epmod, oracle, S, T, K, E, R, G):
    rng = np.random.default_rng(K)
    idx = np.stack([np.stack([rng.permutation(E)[:K] for _ in range(T)]) for _ in range(S)]).astype(np.int32)
    idx = g.mask_random(idx, 0.15, seed=K)
    wg, wf = oracle.dedup(idx, E // R, G)
    cfg = g.EPConfig("dedup", T=T, H=128, E=E, K=K, R=R, S=S)
    with _runner(epmod, cfg, num_proxy_threads=0) as r:
        gi, fk = torch.full(idx.shape, -9, dtype=torch.int32, device="cuda"), torch.full(idx.shape, -9, dtype=torch.int32,
                                                                                         device="cuda")
        epmod.ep_dedup(r.h, _dev(idx), T, G, gi, fk)
        torch.cuda.synchronize()
        assert np.array_equal(gi.cpu().numpy(), wg) and np.array_equal(fk.cpu().numpy(), wf)
        assert r.stats()["device_error"] == 0


@pytest.mark.parametrize("cid,G,T,mask,mode", [(1, 1, None, 0.0, "per_token"), (1, 2, None, 0.25, "chunk32"),
                                               (4, 1, 600, 0.0, "chunk32"), (4, 8, 600, 0.1, "chunk32"),
                                               (5, 4, 500, 0.0, "per_token"), (4, 1, 4096, 0.0, "chunk32"),
                                               (4, 8, 600, 0.1, "ring"), (4, 1, 4096, 0.0, "ring"),
                                               (1, 2, None, 0.25, "ring"), (4, 8, 4096, 0.0, "chunk32"),
                                               (5, 1, 8192, 0.0, "chunk32")])
def test_ht_round_trip(epmod, oracle, cid, G, T, mask, mode):
    """dedup -> group-level layout and dispatch (second handle) -> per-expert index
    list -> expert outputs -> partial reduce per group -> final reduce."""
    from paper_2512_19849_amd.runner import EPRunner, bits_to_bf16, bf16_to_bits
    cfg = g.config(cid, S=1)
    idx, w = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=47)
    T = idx.shape[1]
    NG = cfg.R // G
    x = g.activations(cfg, 0, T=T)
    # oracle side
    wg, wf = oracle.dedup(idx, cfg.E_loc, G)
    lay = oracle.layout(idx, cfg.E, cfg.R)
    lay_g = oracle.layout(wg, NG, NG)
    rows, rows_g = int((idx >= 0).sum()), int((wg >= 0).sum())
    wrecv_g, _ = oracle.dispatch_bf16(x, wg[0], lay_g["dst_row"][0], 1, rows_g)
    windex = oracle.gather_index(lay["dst_row"][0], lay_g["dst_row"][0], wf[0], rows)
    y = g.activations(cfg, 0, tid=g.TID_Y, T=max(rows, 1))
    wpartial = oracle.combine_partial(y, w[0], lay["dst_row"][0], wf[0], lay_g["dst_row"][0], rows_g, fill=0x3F80)
    wout = oracle.combine(wpartial, np.ones_like(w[0]), lay_g["dst_row"][0])

    flags = epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS
    ring_kw = dict(ht_slices=16, ht_ring_slots=2, reorder_window=8) if mode == "ring" else {}
    with EPRunner(cfg.R, cfg.E, cfg.K, cfg.H, T, num_proxy_threads=0, spin_timeout_ms=3000) as r, \
            EPRunner(NG, NG, cfg.K, cfg.H, T, spin_timeout_ms=3000, flags=flags, **ring_kw) as rg:
        d_idx, d_x, d_w = _dev(idx), bits_to_bf16(x), _dev(w[0])
        gi, fk = torch.empty_like(d_idx), torch.empty_like(d_idx)
        epmod.ep_dedup(r.h, d_idx, T, G, gi, fk)
        L = r.layout(d_idx)
        Lg = rg.layout(gi)
        recv_g = torch.full((rows_g + 1, cfg.H), -1.5, dtype=torch.bfloat16, device="cuda")
        if mode == "ring":      # the deduplicated rows travel through the ring-buffer channels
            ring = torch.zeros(rg.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
            rg.ht_dispatch(d_x, gi[0], Lg, ring, recv_g)
        else:
            rg.dispatch(d_x, gi[0], Lg, recv_g, cmd_mode=epmod.CMD_MODES[mode])
        index = torch.full((rows,), -1, dtype=torch.int32, device="cuda")
        epmod.ep_gather_index(r.h, L.dst_row[0], Lg.dst_row[0], fk[0], T, rows, index)
        partial = torch.ones((rows_g, cfg.H), dtype=torch.bfloat16, device="cuda")
        epmod.ep_combine_partial(r.h, bits_to_bf16(y), d_w, L.dst_row[0], fk[0], Lg.dst_row[0], T, y.shape[0],
                                 rows_g, partial)
        out = torch.zeros((T, cfg.H), dtype=torch.bfloat16, device="cuda")
        rg.combine(partial, torch.ones_like(d_w), Lg.dst_row[0], out)
        rg.wait()
        torch.cuda.synchronize()
        got_g = Lg.numpy()
        for name, v in lay_g.items():
            assert np.array_equal(got_g[name], v), name
        assert np.array_equal(bf16_to_bits(recv_g)[:rows_g], wrecv_g)
        assert (bf16_to_bits(recv_g)[rows_g:] == 0xBFC0).all()
        assert np.array_equal(index.cpu().numpy(), windex)
        assert np.array_equal(bf16_to_bits(partial), wpartial)
        assert np.array_equal(bf16_to_bits(out), wout)
        # the wire: commands of the group-level dispatch, fewer rows than one per (token, expert)
        if mode == "ring":
            assert oracle.ring_cmd_multiset(epmod.ep_cmd_log(rg.h)) == \
                oracle.expected_ring_cmds(wg[0], 0, 1, NG, cfg.H, 16, 2)
            oracle.check_ring_trace(epmod.ep_event_log(rg.h), 2)
        else:
            want_cmds = oracle.expected_cmds(wg[0], lay_g, 0, 1, cfg.H, "bf16", mode)
            assert oracle.cmd_multiset(epmod.ep_cmd_log(rg.h)) == want_cmds
            oracle.check_fence_trace(epmod.ep_event_log(rg.h), lay_g["count"])
        st = rg.stats()
        assert st["write_rows"] == rows_g <= rows and st["device_error"] == 0 and r.stats()["device_error"] == 0


# --------------------------------- high-throughput style commands: per-channel sequence order
@pytest.mark.parametrize("cid,T,mask,window,payload", [(1, None, 0.0, 0, "bf16"), (1, None, 0.2, 6, "bf16"),
                                                       (4, 700, 0.0, 32, "bf16"), (5, 600, 0.1, 3, "fp8"),
                                                       (4, 4096, 0.0, 100, "bf16")])
def test_dispatch_ordered_chunks(epmod, oracle, cid, T, mask, window, payload):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.config(cid, S=1)
    idx, _ = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=53)
    T = idx.shape[1]
    x = g.activations(cfg, 0, T=T)
    rows = int((idx >= 0).sum())
    want = oracle.layout(idx, cfg.E, cfg.R)
    rb = oracle.row_bytes(cfg.H, payload)
    flags = epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS
    with _runner(epmod, cfg, T, flags=flags, reorder_window=window, reorder_seed=2) as r:
        d_idx, d_x = _dev(idx), bits_to_bf16(x)
        lay = r.layout(d_idx)
        first_cmd, first_ev = None, None
        ncmd = nev = 0
        for rnd in range(2):                                    # the second dispatch continues the numbering
            if payload == "bf16":
                recv = torch.zeros((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
                r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=epmod.EP_CMD_CHUNK32_ORDERED)
            else:
                recv = torch.zeros((rows, cfg.H), dtype=torch.uint8, device="cuda")
                rs = torch.zeros((rows, cfg.H // 128), dtype=torch.float32, device="cuda")
                r.dispatch(d_x, d_idx[0], lay, recv, rs, payload=epmod.EP_FP8_E4M3,
                           cmd_mode=epmod.EP_CMD_CHUNK32_ORDERED)
            r.wait()
            torch.cuda.synchronize()
            if payload == "bf16":
                wrecv, _ = oracle.dispatch_bf16(x, idx[0], want["dst_row"][0], cfg.E_loc, rows, fill=0)
                assert np.array_equal(bf16_to_bits(recv), wrecv)
            else:
                wq, ws, _ = oracle.dispatch_fp8(x, idx[0], want["dst_row"][0], cfg.E_loc, rows, fill=0)
                assert np.array_equal(recv.cpu().numpy(), wq) and np.array_equal(rs.cpu().numpy(), ws)
            cmds, evs = epmod.ep_cmd_log(r.h), epmod.ep_event_log(r.h)
            # logs are kept thread by thread: split each thread's part into this round's tail
            st = r.stats()
            nchunks = int(np.ceil(want["count"][0] / 32).sum())
            assert st["writes"] == nchunks * (rnd + 1) and st["atomics"] == nchunks * (rnd + 1)
            assert st["drains"] == 8 * (rnd + 1) and st["rejected"] == 0 and st["proxy_error"] == 0
            assert st["atomics_applied"] == 0                   # no per-expert count atomics in this mode
            per_rank = want["count"][0].reshape(cfg.R, cfg.E_loc).sum(1)
            assert np.array_equal(epmod.ep_tail_counters(r.h, 1, cfg.R)[0], per_rank * (rnd + 1))
            res = oracle.check_order_trace(evs)                 # both rounds together: one run per channel
            assert res["applied"] == 2 * nchunks * (rnd + 1) and res["waited"] == st["ordered_parked"]
            if rnd == 0:
                nxt = oracle.check_ordered_cmds(cmds, want, 0, cfg.E_loc, rb)
            else:
                seqs = cmds[np.isin((cmds[:, 0] >> 28) & 7, (5, 6))]
                second = seqs[[int(w[2]) >= nxt[int((w[0] >> 12) & 0xFF)] for w in seqs]]
                oracle.check_ordered_cmds(second, want, 0, cfg.E_loc, rb, first_seq=nxt)
        assert st["device_error"] == 0


# ------------------------------------------------------------- limits of the configuration
@pytest.mark.parametrize("S,T,K,E,R,H", [(1, 100, 64, 1024, 256, 128),      # widest routing the handle accepts
                                         (2, 37, 16, 1024, 4, 256),
                                         (1, 5, 2, 4, 2, 65536),            # widest row
                                         (1, 3, 1, 1, 1, 128),              # smallest everything
                                         (1, 300000, 1, 8, 8, 128),         # many tokens (4688 tiles)
                                         (3, 1, 3, 6, 3, 1152)])
def test_limits_round_trip(epmod, oracle, S, T, K, E, R, H):
    """Extreme shapes through layout, bf16 and FP8 dispatch (per-token commands), combine."""
    from paper_2512_19849_amd.runner import EPRunner, bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("limits", T=T, H=H, E=E, K=K, R=R, S=S, seed=777)
    rng = np.random.default_rng(S * 1000 + K)
    if K * 4 > E or T > 10000:
        keys = rng.random((S, T, E)) if T * E < 5e7 else None
        if keys is None:
            idx = rng.integers(0, E, size=(S, T, K)).astype(np.int32)         # K = 1: any draw is distinct
        else:
            idx = np.argsort(keys, axis=2)[:, :, :K].astype(np.int32)
        w = rng.random((S, T, K)).astype(np.float32)
    else:
        idx, w = g.routing_all(cfg)
    idx = g.mask_random(idx, 0.05, seed=9)
    g.validate_routing(idx, E)
    rows = int((idx >= 0).sum())
    x = g.f32_to_bf16_bits(rng.normal(0, 1, (T, H)).astype(np.float32))
    want = oracle.layout(idx, E, R)
    oracle.set_threads(min(16, oracle.max_threads()))
    try:
        with EPRunner(R, E, K, H, T, S=S, spin_timeout_ms=10000, num_channels=64 if T > 10000 else 8,
                      heap_rows=S * T * K + 1) as r:
            d_idx, d_x = _dev(idx), bits_to_bf16(x)
            lay = r.layout(d_idx)
            recv = torch.zeros((rows + 1, H), dtype=torch.bfloat16, device="cuda")
            rq = torch.zeros((rows + 1, H), dtype=torch.uint8, device="cuda")
            rs = torch.zeros((rows + 1, H // 128), dtype=torch.float32, device="cuda")
            src = S - 1
            r.dispatch(d_x, d_idx[src], lay, recv, src=src, cmd_mode=epmod.EP_CMD_PER_TOKEN)
            r.dispatch(d_x, d_idx[src], lay, rq, rs, src=src, payload=epmod.EP_FP8_E4M3,
                       cmd_mode=epmod.EP_CMD_CHUNK32)
            out = torch.zeros((T, H), dtype=torch.bfloat16, device="cuda")
            r.combine(recv, _dev(w[src]), lay.dst_row[src], out)
            r.wait()
            torch.cuda.synchronize()
            got = lay.numpy()
            for name, v in want.items():
                assert np.array_equal(got[name], v), name
            wrecv, _ = oracle.dispatch_bf16(x, idx[src], want["dst_row"][src], E // R, rows + 1, fill=0)
            assert np.array_equal(bf16_to_bits(recv), wrecv)
            wq, ws, _ = oracle.dispatch_fp8(x, idx[src], want["dst_row"][src], E // R, rows + 1, fill=0,
                                            recv_scale=np.zeros((rows + 1, H // 128), np.float32))
            assert np.array_equal(rq.cpu().numpy(), wq) and np.array_equal(rs.cpu().numpy(), ws)
            wout = oracle.combine(wrecv, w[src], want["dst_row"][src])
            assert np.array_equal(bf16_to_bits(out), wout)
            st = r.stats()
            assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
            assert st["atomics_applied"] == 2 * E
            assert np.array_equal(r.counters()[src], want["count"][src])
    finally:
        oracle.set_threads(1)


# ---------------------------------------------------------------------------- Barrier
# ------------------------------------- ring-buffer channels (HT mode storage)
@pytest.mark.parametrize("cid,T,mask,slices,W,window,threads", [
    (1, None, 0.0, 4, 2, 0, 2), (1, 50, 0.3, 7, 1, 5, 1), (4, 700, 0.0, 16, 2, 16, 4), (5, 1000, 0.1, 8, 3, 0, 4),
    (4, 700, 0.05, 2, 1, 0, 4),       # ~175 rows per channel through a single slot: every chunk waits for a release
    (2, 128, 0.0, 3, 1, 3, 4), (1, 3, 0.0, 8, 2, 0, 2),
    (4, 2000, 0.0, 2, 2, 0, 4),       # 8000 entries per slice: beyond the sender's order list, token by token
    (5, 1500, 0.1, 1, 1, 5, 2),       # one slice, one slot
    ("wide", 100, 0.0, 4, 2, 0, 4),   # 64 experts per token over 256 ranks: the widest routing the handle accepts
    ("long", 40, 0.0, 3, 1, 0, 2)])   # rows of 128 KiB: a row is many pieces, a slot 4 MiB
def test_ht_ring_dispatch(epmod, oracle, cid, T, mask, slices, W, window, threads):
    """Rows travel sending step -> ring slot -> receiving step -> packed receive buffer, slots are
    reused under head/tail flow control, and all three message kinds pass through the proxy.  The receive
    buffer must equal the plain definition of dispatch; the messages the oracle's expected multiset; the
    proxy's trace the ring protocol (in-sequence application, no overwrite, no stale read)."""
    if cid == "wide":
        cfg = g.EPConfig("wide", T=T, H=128, E=1024, K=64, R=256, S=1)
        rng = np.random.default_rng(1)
        idx = np.stack([rng.permutation(1024)[:64] for _ in range(T)]).astype(np.int32)[None]
    elif cid == "long":
        cfg = g.EPConfig("long", T=T, H=65536, E=8, K=2, R=4, S=1)
        rng = np.random.default_rng(2)
        idx = np.stack([rng.permutation(8)[:2] for _ in range(T)]).astype(np.int32)[None]
    else:
        cfg = g.config(cid, S=1)
        idx, _ = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=29)
    T = idx.shape[1]
    rows = int((idx >= 0).sum()) + 2
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    flags = epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    per_channel = oracle.ring_channel_rows(idx[0], cfg.E_loc, cfg.R, slices)
    nch = -(-per_channel // 32)
    with _runner(epmod, cfg, T, flags=flags, heap_rows=rows, ht_slices=slices, ht_ring_slots=W,
                 reorder_window=window, reorder_seed=2, num_proxy_threads=threads) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        assert r.ht_ring_bytes() == oracle.ring_bytes(cfg.H, cfg.R, slices, W)
        recv = torch.empty((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
        want_cmds = None
        for it in range(2):                      # the second call continues the channels' numbering and counters
            x = g.activations(cfg, it, T=T)
            recv.fill_(-1.5)
            r.ht_dispatch(bits_to_bf16(x), d_idx[0], lay, ring, recv)
            r.wait()
            torch.cuda.synchronize()
            want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
            assert np.array_equal(bf16_to_bits(recv), want), it
            exp = oracle.expected_ring_cmds(idx[0], 0, cfg.E_loc, cfg.R, cfg.H, slices, W, 2 * nch * it, nch * it)
            want_cmds = exp if want_cmds is None else want_cmds + exp
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert st["drains"] == 2 * 8 and st["writes"] == 2 * int(nch.sum()) and st["atomics"] == 4 * int(nch.sum())
        assert oracle.ring_cmd_multiset(epmod.ep_cmd_log(r.h)) == want_cmds
        res = oracle.check_ring_trace(epmod.ep_event_log(r.h), W)
        assert res["applied"] == 6 * int(nch.sum())
        tail, head = epmod.ep_ring_counters(r.h, 1, slices, cfg.R)
        assert np.array_equal(tail[0], 2 * per_channel) and np.array_equal(head[0], 2 * per_channel)


# a Write and its Atomic pushed as a pair: channels far too small for a wave's commands (every lane then publishes for itself),
# and rings whose ends a pair straddles
@pytest.mark.parametrize("entries,channels,threads", [(8, 1, 1), (8, 3, 2), (16, 8, 4), (4096, 1, 1)])
def test_pairs_of_commands_through_small_channels(epmod, oracle, entries, channels, threads):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    cfg = g.EPConfig("pairs", T=333, H=256, E=128, K=32, R=16, S=1)
    rng = np.random.default_rng(entries + channels)
    idx = g.mask_random(np.argsort(rng.random((1, cfg.T, cfg.E)), axis=-1)[..., :cfg.K].astype(np.int32), 0.1, seed=5)
    rows = int((idx >= 0).sum())
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    with _runner(epmod, cfg, flags=epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS, heap_rows=rows, ring_entries=entries,
                 num_channels=channels, num_proxy_threads=threads, ht_slices=3, ht_ring_slots=2, spin_timeout_ms=10000) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        for it in range(4):
            x = g.activations(cfg, it)
            recv = torch.full((rows, cfg.H), -1.5, dtype=torch.bfloat16, device="cuda")
            if it % 2:
                r.ht_dispatch(bits_to_bf16(x), d_idx[0], lay, ring, recv)
            else:
                r.dispatch(bits_to_bf16(x), d_idx[0], lay, recv, cmd_mode=epmod.EP_CMD_CHUNK32_ORDERED)
            r.wait()
            torch.cuda.synchronize()
            want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
            assert np.array_equal(bf16_to_bits(recv), want), it
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        if channels == 1 and entries == 8:
            assert st["gpu_ring_full"] > 0


# workgroups of a slice: 2 (rows of half a megabyte each, and one row less: one), 4 of 6 ranks, 8 of 9 ranks, 4 with a rank
# each and most rows for one of them, 16 with a slot per channel
@pytest.mark.parametrize("T,H,E,K,R,slices,W,mask", [
    (245, 2048, 6, 2, 3, 2, 2, 0.0), (244, 2048, 6, 2, 3, 2, 2, 0.0), (700, 2048, 48, 5, 6, 3, 2, 0.2),
    (520, 4096, 45, 7, 9, 7, 1, 0.0), (1100, 2048, 4, 1, 4, 2, 3, 0.1), (600, 8192, 64, 8, 16, 9, 1, 0.05)])
def test_ht_ring_dispatch_slices_shared_by_workgroups(epmod, oracle, T, H, E, K, R, slices, W, mask):
    rng = np.random.default_rng(T)
    score = rng.random((1, T, E))
    if K == 1:
        score[:, :, 1] -= rng.random((1, T)) < 0.9
    idx = g.mask_random(np.argsort(score, axis=-1)[..., :K].astype(np.int32), mask, seed=T)
    rows = int((idx >= 0).sum())
    cfg = g.EPConfig("shared", T=T, H=H, E=E, K=K, R=R, S=1)
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    want_lay = oracle.layout(idx, E, R)
    per_channel = oracle.ring_channel_rows(idx[0], cfg.E_loc, R, slices)
    nch = -(-per_channel // 32)
    with _runner(epmod, cfg, T, flags=epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS, heap_rows=rows,
                 ht_slices=slices, ht_ring_slots=W) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        recv = torch.empty((rows, H), dtype=torch.bfloat16, device="cuda")
        want_cmds = None
        for it in range(2):
            x = g.activations(cfg, it, T=T)
            recv.fill_(-1.5)
            r.ht_dispatch(bits_to_bf16(x), d_idx[0], lay, ring, recv)
            r.wait()
            torch.cuda.synchronize()
            want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
            assert np.array_equal(bf16_to_bits(recv), want), it
            exp = oracle.expected_ring_cmds(idx[0], 0, cfg.E_loc, R, H, slices, W, 2 * nch * it, nch * it)
            want_cmds = exp if want_cmds is None else want_cmds + exp
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert oracle.ring_cmd_multiset(epmod.ep_cmd_log(r.h)) == want_cmds
        oracle.check_ring_trace(epmod.ep_event_log(r.h), W)
        tail, head = epmod.ep_ring_counters(r.h, 1, slices, R)
        assert np.array_equal(tail[0], 2 * per_channel) and np.array_equal(head[0], 2 * per_channel)


# the workgroups of a slice take other ranks' channels in every dispatch (the hot rank moves on), 2 of 3 and 4 of 5 ranks
@pytest.mark.parametrize("T,R,slices", [(300, 3, 2), (600, 5, 3)])
def test_ht_ring_channels_change_hands_between_dispatches(epmod, oracle, T, R, slices):
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    H, E, K = 4096, 4 * R, 3
    cfg = g.EPConfig("hands", T=T, H=H, E=E, K=K, R=R, S=1)
    rows = T * K
    carried = np.zeros((slices, R), np.int64)
    with _runner(epmod, cfg, T, heap_rows=rows, ht_slices=slices, ht_ring_slots=2) as r:
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        recv = torch.empty((rows, H), dtype=torch.bfloat16, device="cuda")
        for it in range(4):
            score = np.random.default_rng(it).random((1, T, E))
            score[:, :, 4 * (it % R):4 * (it % R) + 2] -= 0.8
            idx = np.argsort(score, axis=-1)[..., :K].astype(np.int32)
            x = g.activations(cfg, it, T=T)
            d_idx = _dev(idx)
            lay = r.layout(d_idx)
            recv.fill_(-1.5)
            r.ht_dispatch(bits_to_bf16(x), d_idx[0], lay, ring, recv)
            r.wait()
            torch.cuda.synchronize()
            want_lay = oracle.layout(idx, E, R)
            want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
            assert np.array_equal(bf16_to_bits(recv), want), it
            carried += oracle.ring_channel_rows(idx[0], cfg.E_loc, R, slices)
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        tail, head = epmod.ep_ring_counters(r.h, 1, slices, R)
        assert np.array_equal(tail[0], carried) and np.array_equal(head[0], carried)


@pytest.mark.parametrize("cid,T,mask,slices,W,window", [(3, None, 0.0, 4, 2, 0), (3, 50, 0.3, 3, 1, 4),
                                                        (5, 700, 0.0, 8, 2, 8), (4, 300, 0.1, 2, 1, 0),
                                                        ("h128", 90, 0.0, 3, 2, 0)])
def test_ht_ring_dispatch_fp8(epmod, oracle, cid, T, mask, slices, W, window):
    """FP8 tokens through the rings: the sender quantises, a slot row is codes + scales, the receiver splits
    it into the two receive arrays.  Codes and scales must equal the oracle's bit for bit; the messages carry
    the FP8 row length."""
    if cid == "h128":                                          # one block per row: the row is padded to 16 bytes
        cfg = g.EPConfig("h128", T=T, H=128, E=8, K=2, R=4, S=1)
        rng = np.random.default_rng(3)
        idx = np.stack([rng.permutation(8)[:2] for _ in range(T)]).astype(np.int32)[None]
    else:
        cfg = g.config(cid, S=1)
        idx, _ = g.routing_all(cfg, T)
    if mask:
        idx = g.mask_random(idx, mask, seed=31)
    T = idx.shape[1]
    rows = int((idx >= 0).sum()) + 2
    from paper_2512_19849_amd.runner import bits_to_bf16
    flags = epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    nch = -(-oracle.ring_channel_rows(idx[0], cfg.E_loc, cfg.R, slices) // 32)
    with _runner(epmod, cfg, T, flags=flags, heap_rows=rows, ht_slices=slices, ht_ring_slots=W,
                 reorder_window=window, reorder_seed=6) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        rq = torch.empty((rows, cfg.H), dtype=torch.uint8, device="cuda")
        rs = torch.empty((rows, cfg.H // 128), dtype=torch.float32, device="cuda")
        want_cmds = None
        for it in range(2):
            x = g.activations(cfg, it, T=T)
            rq.fill_(0xA5)
            rs.fill_(-1.0)
            r.ht_dispatch(bits_to_bf16(x), d_idx[0], lay, ring, rq, recv_scale=rs)
            r.wait()
            torch.cuda.synchronize()
            wq, ws, _ = oracle.dispatch_fp8(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
            assert np.array_equal(rs.cpu().numpy().view(np.uint32), ws.view(np.uint32)), "scales differ"
            assert np.array_equal(rq.cpu().numpy(), wq), "codes differ"
            exp = oracle.expected_ring_cmds(idx[0], 0, cfg.E_loc, cfg.R, cfg.H, slices, W, 2 * nch * it, nch * it,
                                            payload="fp8")
            want_cmds = exp if want_cmds is None else want_cmds + exp
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert oracle.ring_cmd_multiset(epmod.ep_cmd_log(r.h)) == want_cmds
        oracle.check_ring_trace(epmod.ep_event_log(r.h), W)
        assert st["write_bytes"] == 2 * (128 * int(nch.sum()) + (rows - 2) * oracle.row_bytes(cfg.H, "fp8"))


# rows of the groups that a lane quantises in one go (8192 channels), and of one block more; 64 blocks and 65 in the receiving step
@pytest.mark.parametrize("H", [1024, 2176, 8192, 8320, 16512])
def test_ht_ring_dispatch_fp8_row_widths(epmod, oracle, H):
    from paper_2512_19849_amd.runner import bits_to_bf16
    T, E, K, R = 70, 8, 3, 4
    cfg = g.EPConfig("widths", T=T, H=H, E=E, K=K, R=R, S=1, seed=H)
    idx, _ = g.routing_all(cfg)
    rows = T * K
    lay_want = oracle.layout(idx, E, R)
    with _runner(epmod, cfg, T, heap_rows=rows, ht_slices=2, ht_ring_slots=2) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        rq = torch.full((rows, H), 0xA5, dtype=torch.uint8, device="cuda")
        rs = torch.full((rows, H // 128), -1.0, dtype=torch.float32, device="cuda")
        for it in range(2):
            x = g.activations(cfg, it, T=T)
            r.ht_dispatch(bits_to_bf16(x), d_idx[0], lay, ring, rq, recv_scale=rs)
            r.wait()
            torch.cuda.synchronize()
            wq, ws, _ = oracle.dispatch_fp8(x, idx[0], lay_want["dst_row"][0], cfg.E_loc, rows)
            assert np.array_equal(rs.cpu().numpy().view(np.uint32), ws.view(np.uint32)), "scales differ"
            assert np.array_equal(rq.cpu().numpy(), wq), "codes differ"
        assert r.stats()["device_error"] == 0


def test_ht_ring_dispatch_of_several_sources(epmod, oracle):
    """Config 2's 32 routing tables: sources 0, 7 and 31 each send their tokens through their own set of
    channels (counters, sequence numbers and proxy state are per source) into the one receive buffer."""
    cfg = g.config(2)
    idx, _ = g.routing_all(cfg)
    rows = idx.size
    slices, W = 5, 2
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    flags = epmod.EP_FLAG_LOG_CMDS | epmod.EP_FLAG_LOG_EVENTS
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    want = np.full((rows, cfg.H), 0xBFC0, np.uint16)
    with _runner(epmod, cfg, flags=flags, ht_slices=slices, ht_ring_slots=W, reorder_window=5) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        recv = torch.full((rows, cfg.H), -1.5, dtype=torch.bfloat16, device="cuda")
        want_cmds = None
        for s in (0, 7, 31):
            x = g.activations(cfg, s)
            epmod.ep_ht_dispatch(r.h, bits_to_bf16(x), d_idx[s], lay.dst_row[s], cfg.T, s, ring, recv, rows)
            r.wait()
            part, wc = oracle.dispatch_bf16(x, idx[s], want_lay["dst_row"][s], cfg.E_loc, rows, -1, fill=0xBFC0)
            want[wc > 0] = part[wc > 0]
            exp = oracle.expected_ring_cmds(idx[s], s, cfg.E_loc, cfg.R, cfg.H, slices, W)
            want_cmds = exp if want_cmds is None else want_cmds + exp
        torch.cuda.synchronize()
        assert np.array_equal(bf16_to_bits(recv), want)
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert oracle.ring_cmd_multiset(epmod.ep_cmd_log(r.h)) == want_cmds
        oracle.check_ring_trace(epmod.ep_event_log(r.h), W)
        tail, head = epmod.ep_ring_counters(r.h, cfg.S, slices, cfg.R)
        for s in range(cfg.S):
            per = oracle.ring_channel_rows(idx[s], cfg.E_loc, cfg.R, slices) if s in (0, 7, 31) else 0
            assert np.array_equal(tail[s], per + np.zeros_like(tail[s])) and np.array_equal(head[s], tail[s])


@pytest.mark.parametrize("cid,slices,W", [(4, 128, 2), (5, 64, 4), (4, 1024, 1), (4, 128, 4), (4, 256, 2), (5, 128, 2),
                                          (5, 128, 4), (5, 256, 2)])
def test_ht_ring_dispatch_full_size(epmod, oracle, cid, slices, W):
    """The full prefill-sized workloads through the rings, in the shape the timing suite launches; the last case
    has four times more workgroups than the chip holds at once (a workgroup depends on no other workgroup)."""
    cfg = g.config(cid, S=1)
    idx, _ = g.routing_all(cfg)
    x = g.activations(cfg)
    rows = idx.size
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    oracle.set_threads(oracle.max_threads())
    try:
        want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
    finally:
        oracle.set_threads(1)
    per_channel = oracle.ring_channel_rows(idx[0], cfg.E_loc, cfg.R, slices)
    with _runner(epmod, cfg, ht_slices=slices, ht_ring_slots=W, spin_timeout_ms=10000) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        recv = torch.zeros((rows, cfg.H), dtype=torch.bfloat16, device="cuda")
        r.ht_dispatch(bits_to_bf16(x), d_idx[0], lay, ring, recv)
        r.wait()
        torch.cuda.synchronize()
        assert np.array_equal(bf16_to_bits(recv), want)
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert st["write_rows"] == rows and st["writes"] == int((-(-per_channel // 32)).sum())
        tail, head = epmod.ep_ring_counters(r.h, 1, slices, cfg.R)
        assert np.array_equal(tail[0], per_channel) and np.array_equal(head[0], per_channel)


def test_ht_ring_dispatch_full_size_fp8(epmod, oracle):
    """The 8192-token workload with FP8 rows through the rings, in the shape the timing suite launches (128
    slices, rings of 2 slots): codes and scales equal the oracle's quantiser bit for bit at every row."""
    cfg = g.config(5, S=1)
    idx, _ = g.routing_all(cfg)
    x = g.activations(cfg)
    rows = idx.size
    slices, W = 128, 2
    from paper_2512_19849_amd.runner import bits_to_bf16
    want_lay = oracle.layout(idx, cfg.E, cfg.R)
    oracle.set_threads(oracle.max_threads())
    try:
        wq, ws, _ = oracle.dispatch_fp8(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
    finally:
        oracle.set_threads(1)
    per_channel = oracle.ring_channel_rows(idx[0], cfg.E_loc, cfg.R, slices)
    with _runner(epmod, cfg, ht_slices=slices, ht_ring_slots=W, spin_timeout_ms=10000) as r:
        d_idx = _dev(idx)
        lay = r.layout(d_idx)
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        rq = torch.full((rows, cfg.H), 0xA5, dtype=torch.uint8, device="cuda")
        rs = torch.full((rows, cfg.H // 128), -1.0, dtype=torch.float32, device="cuda")
        r.ht_dispatch(bits_to_bf16(x), d_idx[0], lay, ring, rq, recv_scale=rs)
        r.wait()
        torch.cuda.synchronize()
        assert np.array_equal(rs.cpu().numpy().view(np.uint32), ws.view(np.uint32)), "scales differ"
        assert np.array_equal(rq.cpu().numpy(), wq), "codes differ"
        st = r.stats()
        assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0
        assert st["write_rows"] == rows and st["writes"] == int((-(-per_channel // 32)).sum())
        tail, head = epmod.ep_ring_counters(r.h, 1, slices, cfg.R)
        assert np.array_equal(tail[0], per_channel) and np.array_equal(head[0], per_channel)


def test_ht_ring_dispatch_argument_errors(epmod):
    cfg = g.config(1)
    x = torch.zeros((cfg.T, cfg.H), dtype=torch.bfloat16, device="cuda")
    recv = torch.zeros((cfg.T * cfg.K, cfg.H), dtype=torch.bfloat16, device="cuda")
    idx = _dev(g.routing_all(cfg)[0])

    def rc_of(fn):
        with pytest.raises(epmod.EPError) as ei:
            fn()
        return ei.value.rc
    with _runner(epmod, cfg) as r:                                   # no ring channels configured
        lay = r.layout(idx)
        ring = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
        assert rc_of(lambda: r.ht_dispatch(x, idx[0], lay, ring, recv)) == epmod.EP_ESTATE
    with _runner(epmod, cfg, ht_slices=2, ht_ring_slots=2) as r:
        lay = r.layout(idx)
        small = torch.zeros(r.ht_ring_bytes() - 16, dtype=torch.uint8, device="cuda")
        assert rc_of(lambda: r.ht_dispatch(x, idx[0], lay, small, recv)) == epmod.EP_EINVAL
        ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
        assert rc_of(lambda: epmod.ep_ht_dispatch(r.h, x, idx[0], lay.dst_row[0], cfg.T, 1, ring, recv,
                                                  recv.shape[0])) == epmod.EP_EINVAL      # source 1 of 1
        assert rc_of(lambda: epmod.ep_ht_dispatch(r.h, x, idx[0], lay.dst_row[0], cfg.T + 1, 0, ring, recv,
                                                  recv.shape[0])) == epmod.EP_EINVAL      # beyond max_tokens
        sc = torch.zeros((recv.shape[0], cfg.H // 128), dtype=torch.float32, device="cuda")
        assert rc_of(lambda: epmod.ep_ht_dispatch(r.h, x, idx[0], lay.dst_row[0], cfg.T, 0, ring, recv, recv.shape[0],
                                                  payload=epmod.EP_FP8_E4M3)) == epmod.EP_EINVAL   # FP8 needs the scales
        assert rc_of(lambda: epmod.ep_ht_dispatch(r.h, x, idx[0], lay.dst_row[0], cfg.T, 0, ring, recv, recv.shape[0],
                                                  recv_scale=sc)) == epmod.EP_EINVAL                # bf16 must not have them
        # T = 0: nothing travels, the drains still do
        epmod.ep_ht_dispatch(r.h, x, idx[0], lay.dst_row[0], 0, 0, ring, recv, recv.shape[0])
        r.wait()
        assert r.stats()["drains"] == 8 and r.stats()["writes"] == 0


def test_fifo_stress_closed_loop(epmod):
    """Every pusher gets every command popped (Check-completion), the proxy sees exactly pushers x commands,
    spread over the channels, and each round trip takes a plausible time."""
    cfg = g.config(1)
    for pushers, per, ring_entries in ((1, 50, 4096), (64, 40, 4096), (1000, 10, 16)):
        with _runner(epmod, cfg, num_channels=8, num_proxy_threads=4, ring_entries=ring_entries) as r:
            s = torch.zeros(pushers, dtype=torch.int64, device="cuda")
            m = torch.zeros(pushers, dtype=torch.int64, device="cuda")
            epmod.ep_fifo_stress(r.h, pushers, per, s, m)
            r.wait()
            torch.cuda.synchronize()
            st = r.stats()
            assert st["cmds"] == pushers * per == st["atomics_applied"] and st["device_error"] == 0
            assert sum(st["per_thread_cmds"]) == pushers * per
            mean_us = s.cpu().numpy() / per / 100.0
            assert (mean_us > 0.5).all() and (mean_us < 5000).all()           # a PCIe round trip at least
            assert (m.cpu().numpy() >= s.cpu().numpy() / per).all()
    with _runner(epmod, cfg, num_proxy_threads=0) as r:                       # nobody would pop
        with pytest.raises(epmod.EPError):
            epmod.ep_fifo_stress(r.h, 1, 1, s, m)


def test_seeded_sweep_of_small_shapes_through_every_dispatch_mode(epmod, oracle):
    """Twenty seeded shapes (ranks, experts, top-k, hidden, tokens, masking, threads, channels, ring sizes,
    reordering, pacing, packing drawn at random within the documented limits), each sent through every way
    of dispatching - ring off, per token, chunks, sequenced chunks, ring-buffer channels, and the
    proxy-performed forms - into one handle; every receive buffer must equal the plain definition."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    rng = np.random.default_rng(20251219)
    for case in range(20):
        R = int(rng.choice([1, 2, 4, 8, 16]))
        E = R * int(rng.choice([1, 2, 3, 8]))
        K = int(rng.integers(1, min(E, 9) + 1))
        H = 128 * int(rng.choice([1, 2, 5, 8, 24]))
        T = int(rng.integers(1, 400))
        cfg = g.EPConfig(f"sweep{case}", T=T, H=H, E=E, K=K, R=R, S=1, seed=1000 + case)
        idx = np.stack([rng.permutation(E)[:K] for _ in range(T)]).astype(np.int32)[None]
        if rng.random() < 0.5:
            idx = g.mask_random(idx, float(rng.choice([0.05, 0.5])), seed=case)
        x = g.activations(cfg)
        rows = int((idx >= 0).sum()) + 1
        slices, W = int(rng.integers(1, 9)), int(rng.integers(1, 4))
        kw = dict(num_proxy_threads=int(rng.integers(1, 5)), num_channels=int(rng.choice([1, 3, 8, 16])),
                  ring_entries=int(rng.choice([8, 64, 4096])), reorder_window=int(rng.choice([0, 3, 50])),
                  reorder_seed=case, max_outstanding=int(rng.choice([0, 2, 16])), pack_rows=int(rng.choice([0, 4])),
                  ht_slices=slices, ht_ring_slots=W, heap_rows=rows)
        want_lay = oracle.layout(idx, E, R)
        want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
        tag = f"case {case}: R={R} E={E} K={K} H={H} T={T} {kw}"
        with _runner(epmod, cfg, **kw) as r:
            d_idx, d_x = _dev(idx), bits_to_bf16(x)
            lay = r.layout(d_idx)
            recv = torch.empty((rows, H), dtype=torch.bfloat16, device="cuda")
            ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
            send = torch.empty((rows, H), dtype=torch.bfloat16, device="cuda")

            def check(what):
                torch.cuda.synchronize()
                assert np.array_equal(bf16_to_bits(recv), want), f"{what}; {tag}"
                st = r.stats()
                assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0, f"{what}; {tag}"

            for name in ("none", "per_token", "chunk32", "chunk32_ordered"):
                recv.fill_(-1.5)
                r.dispatch(d_x, d_idx[0], lay, recv, cmd_mode=epmod.CMD_MODES[name])
                if name != "none":
                    try:
                        r.wait()
                    except epmod.EPError as err:
                        raise AssertionError(f"{name}: {err}; {tag}")
                check(name)
            recv.fill_(-1.5)
            r.ht_dispatch(d_x, d_idx[0], lay, ring, recv)
            r.wait()
            check("ring-buffer channels")
            for name, src_heap, target, flag in (("per_token", d_x, recv, epmod.EP_CMD_NO_PLACEMENT),
                                                 ("chunk32", send, send, 0), ("chunk32_ordered", send, send, 0)):
                recv.fill_(-1.5)
                r.register_heaps(src_heap, recv)
                r.dispatch(d_x, d_idx[0], lay, target, cmd_mode=epmod.CMD_MODES[name] | flag)
                r.wait()
                check("proxy-performed " + name)
            r.register_heaps(None, None)
            assert np.array_equal(lay.numpy()["dst_row"], want_lay["dst_row"]), tag


def test_seeded_sweep_of_ring_buffer_channels(epmod, oracle):
    """Forty seeded shapes through ep_ht_dispatch alone, three dispatches per handle (the second with fewer
    tokens; sequence numbers, tails and heads carry over), with what the other sweeps do not reach: top-k up to
    48 (one lane per destination of a token), rows longer than one register piece (hidden 9216), FP8 rows,
    64 to 1024 threads per workgroup, rings of one to three slots, every entry masked."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    import os
    rng = np.random.default_rng(20251220)
    old_threads = os.environ.get("EP_HT_THREADS")
    try:
        for case in range(40):
            R = int(rng.choice([1, 2, 4, 8, 16, 32]))
            E = R * int(rng.choice([1, 2, 3, 8]))
            K = int(rng.integers(1, min(E, 48) + 1)) if rng.random() < 0.3 else int(rng.integers(1, min(E, 9) + 1))
            H = 128 * int(rng.choice([1, 2, 5, 8, 24, 56, 72]))
            T = int(rng.integers(1, 500))
            os.environ["EP_HT_THREADS"] = str(int(rng.choice([64, 256, 512, 1024])))
            cfg = g.EPConfig(f"rsweep{case}", T=T, H=H, E=E, K=K, R=R, S=1, seed=3000 + case)
            kw = dict(num_proxy_threads=int(rng.integers(1, 5)), num_channels=int(rng.choice([1, 3, 8, 16])),
                      ring_entries=int(rng.choice([8, 64, 4096])), reorder_window=int(rng.choice([0, 3, 50])),
                      reorder_seed=case, ht_slices=int(rng.integers(1, 12)), ht_ring_slots=int(rng.integers(1, 4)),
                      heap_rows=T * K + 1, spin_timeout_ms=5000)
            tag = f"case {case}: R={R} E={E} K={K} H={H} T={T} threads={os.environ['EP_HT_THREADS']} {kw}"
            with _runner(epmod, cfg, **kw) as r:
                ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
                for rep in range(3):
                    Tr = T if rep != 1 else int(rng.integers(1, T + 1))
                    idx = np.stack([rng.permutation(E)[:K] for _ in range(Tr)]).astype(np.int32)[None]
                    if rng.random() < 0.5:
                        idx = g.mask_random(idx, float(rng.choice([0.05, 0.5, 1.0])), seed=case * 7 + rep)
                    x = g.activations(cfg, 0, T=Tr)
                    rows = int((idx >= 0).sum()) + 1
                    want_lay = oracle.layout(idx, E, R)
                    d_idx, d_x = _dev(idx), bits_to_bf16(x)
                    lay = r.layout(d_idx)
                    if rng.random() < 0.6:
                        want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows, -1,
                                                       fill=0xBFC0)
                        recv = torch.full((rows, H), -1.5, dtype=torch.bfloat16, device="cuda")
                        r.ht_dispatch(d_x, d_idx[0], lay, ring, recv)
                        r.wait()
                        torch.cuda.synchronize()
                        assert np.array_equal(bf16_to_bits(recv), want), f"bf16, dispatch {rep}; {tag}"
                    else:
                        wq, ws, _ = oracle.dispatch_fp8(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows)
                        rq = torch.zeros((rows, H), dtype=torch.uint8, device="cuda")
                        rs = torch.zeros((rows, H // 128), dtype=torch.float32, device="cuda")
                        r.ht_dispatch(d_x, d_idx[0], lay, ring, rq, recv_scale=rs)
                        r.wait()
                        torch.cuda.synchronize()
                        dr = want_lay["dst_row"][0]
                        hit = np.zeros(rows, bool)
                        hit[dr[dr >= 0]] = True
                        assert np.array_equal(rq.cpu().numpy()[hit], wq[hit]), f"FP8 codes, dispatch {rep}; {tag}"
                        assert np.array_equal(rs.cpu().numpy()[hit], ws[hit]), f"FP8 scales, dispatch {rep}; {tag}"
                        assert not rq.cpu().numpy()[~hit].any(), f"FP8 rows nobody owns, dispatch {rep}; {tag}"
                    st = r.stats()
                    assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0, tag
    finally:
        if old_threads is None:
            os.environ.pop("EP_HT_THREADS", None)
        else:
            os.environ["EP_HT_THREADS"] = old_threads


def test_seeded_sweep_of_sources_payloads_and_the_way_back(epmod, oracle):
    """Twenty-five seeded shapes with several sources: the layout over all of them, then for a random
    source and (sometimes) a single destination rank: FP8 dispatch in a random command mode, FP8 through
    the ring-buffer channels, the GPU-side wait for the counters, and combine over random expert outputs -
    each against the oracle."""
    from paper_2512_19849_amd.runner import bits_to_bf16, bf16_to_bits
    rng = np.random.default_rng(77)
    for case in range(25):
        R = int(rng.choice([1, 2, 4, 8, 32]))
        E = R * int(rng.choice([1, 2, 4]))
        K = int(rng.integers(1, min(E, 8) + 1))
        H = 128 * int(rng.choice([1, 3, 8, 16, 56]))
        S = int(rng.choice([1, 2, 3]))
        T = int(rng.integers(1, 300))
        cfg = g.EPConfig(f"sweepb{case}", T=T, H=H, E=E, K=K, R=R, S=S, seed=5000 + case)
        idx = np.stack([np.stack([rng.permutation(E)[:K] for _ in range(T)]) for _ in range(S)]).astype(np.int32)
        if rng.random() < 0.5:
            idx = g.mask_random(idx, float(rng.choice([0.1, 0.6])), seed=case)
        w = rng.standard_normal((T, K)).astype(np.float32)
        s = int(rng.integers(S))
        filt = int(rng.integers(R)) if rng.random() < 0.4 else -1
        x = g.activations(cfg, s)
        rows = int((idx >= 0).sum()) + 1
        mode = str(rng.choice(["none", "per_token", "chunk32", "chunk32_ordered"]))
        slices, W = int(rng.integers(1, 6)), int(rng.integers(1, 4))
        kw = dict(num_proxy_threads=int(rng.integers(1, 5)), num_channels=int(rng.choice([2, 8, 32])),
                  ring_entries=int(rng.choice([16, 256, 4096])), reorder_window=int(rng.choice([0, 5, 40])),
                  reorder_seed=case, ht_slices=slices, ht_ring_slots=W, heap_rows=rows)
        tag = f"case {case}: R={R} E={E} K={K} H={H} S={S} T={T} src={s} filter={filt} mode={mode} {kw}"
        want_lay = oracle.layout(idx, E, R)
        wq, ws, _ = oracle.dispatch_fp8(x, idx[s], want_lay["dst_row"][s], cfg.E_loc, rows, filt)
        y = g.activations(cfg, s, tid=g.TID_Y, T=rows)
        wout = oracle.combine(y, w, want_lay["dst_row"][s])
        with _runner(epmod, cfg, **kw) as r:
            d_idx, d_x = _dev(idx), bits_to_bf16(x)
            lay = r.layout(d_idx)
            torch.cuda.synchronize()
            got = lay.numpy()
            for name, v in want_lay.items():
                assert np.array_equal(got[name], v), f"layout {name}; {tag}"
            rq = torch.full((rows, H), 0xA5, dtype=torch.uint8, device="cuda")
            rs = torch.full((rows, H // 128), -1.0, dtype=torch.float32, device="cuda")
            counts = torch.full((E,), -7, dtype=torch.int32, device="cuda")
            try:
                r.dispatch(d_x, d_idx[s], lay, rq, rs, src=s, rank_filter=filt, payload=epmod.EP_FP8_E4M3,
                           cmd_mode=epmod.CMD_MODES[mode])
                if mode in ("per_token", "chunk32"):
                    r.recv_wait(counts, src=s, rank_filter=filt)
                if mode != "none":
                    r.wait()
                torch.cuda.synchronize()
            except epmod.EPError as err:
                raise AssertionError(f"{err}; {tag}")
            assert np.array_equal(rs.cpu().numpy().view(np.uint32), ws.view(np.uint32)), f"scales; {tag}"
            assert np.array_equal(rq.cpu().numpy(), wq), f"codes; {tag}"
            if mode in ("per_token", "chunk32"):
                sel = np.arange(E) // cfg.E_loc == filt if filt >= 0 else np.ones(E, bool)
                wc = np.where(sel, want_lay["count"][s], -1)
                assert np.array_equal(counts.cpu().numpy(), wc), f"counts; {tag}"
            # the same source through the ring-buffer channels (all ranks)
            wq2, ws2, _ = oracle.dispatch_fp8(x, idx[s], want_lay["dst_row"][s], cfg.E_loc, rows)
            rq.fill_(0xA5)
            rs.fill_(-1.0)
            ring = torch.zeros(r.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
            try:
                r.ht_dispatch(d_x, d_idx[s], lay, ring, rq, src=s, recv_scale=rs)
                r.wait()
                torch.cuda.synchronize()
            except epmod.EPError as err:
                raise AssertionError(f"rings: {err}; {tag}")
            assert np.array_equal(rs.cpu().numpy().view(np.uint32), ws2.view(np.uint32)), f"ring scales; {tag}"
            assert np.array_equal(rq.cpu().numpy(), wq2), f"ring codes; {tag}"
            out = torch.full((T, H), 7.0, dtype=torch.bfloat16, device="cuda")
            r.combine(bits_to_bf16(y), _dev(w), lay.dst_row[s], out)
            torch.cuda.synchronize()
            assert int(oracle.bf16_ulp_distance(bf16_to_bits(out), wout).max()) <= 1, f"combine; {tag}"
            st = r.stats()
            assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0, tag


def test_seeded_sweep_of_the_deduplicating_mode(epmod, oracle):
    """Twenty seeded shapes of the high-throughput pipeline with random group sizes: dedup, group-level layout
    and dispatch (per token, chunks or ring-buffer channels), per-expert index list, partial reduce per group
    and final reduce, each stage against the oracle."""
    from paper_2512_19849_amd.runner import EPRunner, bits_to_bf16, bf16_to_bits
    rng = np.random.default_rng(5)
    for case in range(20):
        G = int(rng.choice([1, 2, 4, 8]))
        NG = int(rng.choice([1, 2, 4]))
        R = G * NG
        E = R * int(rng.choice([1, 2, 4]))
        K = int(rng.integers(1, min(E, 8) + 1))
        H = 128 * int(rng.choice([1, 2, 8, 56]))
        T = int(rng.integers(1, 300))
        cfg = g.EPConfig(f"s3_{case}", T=T, H=H, E=E, K=K, R=R, S=1, seed=9000 + case)
        idx = np.stack([rng.permutation(E)[:K] for _ in range(T)]).astype(np.int32)[None]
        if rng.random() < 0.5:
            idx = g.mask_random(idx, float(rng.choice([0.1, 0.5])), seed=case)
        w = rng.standard_normal((1, T, K)).astype(np.float32)
        x = g.activations(cfg, 0)
        tag = f"case {case}: G={G} NG={NG} E={E} K={K} H={H} T={T}"
        wg, wf = oracle.dedup(idx, cfg.E_loc, G)
        lay = oracle.layout(idx, E, R)
        lay_g = oracle.layout(wg, NG, NG)
        rows, rows_g = int((idx >= 0).sum()), int((wg >= 0).sum())
        if rows == 0:
            continue
        windex = oracle.gather_index(lay["dst_row"][0], lay_g["dst_row"][0], wf[0], rows)
        y = g.activations(cfg, 0, tid=g.TID_Y, T=max(rows, 1))
        wpartial = oracle.combine_partial(y, w[0], lay["dst_row"][0], wf[0], lay_g["dst_row"][0], rows_g, fill=0x3F80)
        wout = oracle.combine(wpartial, np.ones_like(w[0]), lay_g["dst_row"][0])
        wrecv_g, _ = oracle.dispatch_bf16(x, wg[0], lay_g["dst_row"][0], 1, rows_g)
        mode = str(rng.choice(["per_token", "chunk32", "ring"]))
        ring_kw = dict(ht_slices=int(rng.integers(1, 5)), ht_ring_slots=int(rng.integers(1, 3)))
        with EPRunner(R, E, K, H, T, num_proxy_threads=0, spin_timeout_ms=3000) as r, \
                EPRunner(NG, NG, K, H, T, spin_timeout_ms=3000, reorder_window=int(rng.choice([0, 6])),
                         heap_rows=max(rows_g, 1), **ring_kw) as rg:
            d_idx, d_x, d_w = _dev(idx), bits_to_bf16(x), _dev(w[0])
            gi, fk = torch.empty_like(d_idx), torch.empty_like(d_idx)
            epmod.ep_dedup(r.h, d_idx, T, G, gi, fk)
            L = r.layout(d_idx)
            Lg = rg.layout(gi)
            recv_g = torch.zeros((max(rows_g,1), H), dtype=torch.bfloat16, device="cuda")
            if mode == "ring":
                ring = torch.zeros(rg.ht_ring_bytes(), dtype=torch.uint8, device="cuda")
                rg.ht_dispatch(d_x, gi[0], Lg, ring, recv_g)
            else:
                rg.dispatch(d_x, gi[0], Lg, recv_g, cmd_mode=epmod.CMD_MODES[mode])
            index = torch.full((rows,), -1, dtype=torch.int32, device="cuda")
            epmod.ep_gather_index(r.h, L.dst_row[0], Lg.dst_row[0], fk[0], T, rows, index)
            partial = torch.ones((max(rows_g,1), H), dtype=torch.bfloat16, device="cuda")
            epmod.ep_combine_partial(r.h, bits_to_bf16(y), d_w, L.dst_row[0], fk[0], Lg.dst_row[0], T, y.shape[0],
                                     rows_g, partial)
            out = torch.zeros((T, H), dtype=torch.bfloat16, device="cuda")
            rg.combine(partial, torch.ones_like(d_w), Lg.dst_row[0], out)
            rg.wait()
            torch.cuda.synchronize()
            assert np.array_equal(gi.cpu().numpy(), wg) and np.array_equal(fk.cpu().numpy(), wf), tag
            assert np.array_equal(bf16_to_bits(recv_g)[:rows_g], wrecv_g), tag
            assert np.array_equal(index.cpu().numpy(), windex), tag
            assert np.array_equal(bf16_to_bits(partial)[:rows_g], wpartial[:rows_g]), tag
            assert np.array_equal(bf16_to_bits(out), wout), tag
            assert rg.stats()["device_error"] == 0 and r.stats()["device_error"] == 0 and rg.stats()["proxy_error"] == 0, tag


def test_seeded_sweep_of_proxy_options_and_dispatch_flags(epmod, oracle):
    """Fifteen seeded shapes, three dispatches each on one handle, with the proxy's options (threads, channels,
    ring size down to 8 slots, reordering, pacing, packing with and without hold time, fence at the sender or
    at the receiver) and the dispatch flags (count Atomics first, Drain, proxy-performed writes) drawn at
    random: buffer, counters, fence trace and pacing trace must hold in every combination."""
    from paper_2512_19849_amd.runner import EPRunner, bits_to_bf16, bf16_to_bits
    rng = np.random.default_rng(11)
    for case in range(15):
        R = int(rng.choice([1, 2, 4, 8, 16]))
        E = R * int(rng.choice([1, 2, 3, 8]))
        K = int(rng.integers(1, min(E, 8) + 1))
        H = 128 * int(rng.choice([1, 2, 5, 8, 24]))
        T = int(rng.integers(1, 500))
        cfg = g.EPConfig(f"s4_{case}", T=T, H=H, E=E, K=K, R=R, S=1, seed=3000 + case)
        idx = np.stack([rng.permutation(E)[:K] for _ in range(T)]).astype(np.int32)[None]
        if rng.random() < 0.5:
            idx = g.mask_random(idx, float(rng.choice([0.05, 0.5])), seed=case)
        x = g.activations(cfg)
        rows = int((idx >= 0).sum()) + 1
        flags = epmod.EP_FLAG_LOG_EVENTS | (epmod.EP_FLAG_SENDER_FENCE if rng.random() < 0.5 else 0)
        kw = dict(num_proxy_threads=int(rng.integers(1, 5)), num_channels=int(rng.choice([1, 2, 8, 16])),
                  ring_entries=int(rng.choice([8, 32, 4096])), reorder_window=int(rng.choice([0, 3, 50])),
                  reorder_seed=case, max_outstanding=int(rng.choice([0, 1, 4])), pack_rows=int(rng.choice([0, 2, 16])),
                  pack_hold_us=int(rng.choice([0, 30])), heap_rows=rows, flags=flags)
        want_lay = oracle.layout(idx, E, R)
        want, _ = oracle.dispatch_bf16(x, idx[0], want_lay["dst_row"][0], cfg.E_loc, rows, -1, fill=0xBFC0)
        with EPRunner(R, E, K, H, T, spin_timeout_ms=3000, **kw) as r:
            d_idx, d_x = _dev(idx), bits_to_bf16(x)
            lay = r.layout(d_idx)
            recv = torch.empty((rows, H), dtype=torch.bfloat16, device="cuda")
            send = torch.empty((rows, H), dtype=torch.bfloat16, device="cuda")
            for rep in range(3):
                base = str(rng.choice(["per_token", "chunk32"]))
                cm = epmod.CMD_MODES[base]
                if rng.random() < 0.4:
                    cm |= epmod.EP_CMD_ATOMICS_FIRST
                if rng.random() < 0.4:
                    cm |= epmod.EP_CMD_DRAIN
                pw = rng.random() < 0.4
                tag = (f"case {case}.{rep}: R={R} E={E} K={K} H={H} T={T} mode={base} cm={cm:#x} pw={pw} "
                       f"flags={flags} {kw}")
                recv.fill_(-1.5)
                target = recv
                if pw:
                    if base == "per_token":
                        cm |= epmod.EP_CMD_NO_PLACEMENT
                        r.register_heaps(d_x, recv)
                    else:
                        target = send
                        r.register_heaps(send, recv)
                r.dispatch(d_x, d_idx[0], lay, target, cmd_mode=cm)
                r.wait()
                torch.cuda.synchronize()
                if pw:
                    r.register_heaps(None, None)
                assert np.array_equal(bf16_to_bits(recv), want), tag
                st = r.stats()
                assert st["device_error"] == 0 and st["proxy_error"] == 0 and st["rejected"] == 0, tag
                assert np.array_equal(r.counters()[0], want_lay["count"][0]), tag
            ev = epmod.ep_event_log(r.h)
            oracle.check_fence_trace(ev, want_lay["count"])
            oracle.check_pacing_trace(ev, kw["max_outstanding"], cfg.E_loc)
            if flags & epmod.EP_FLAG_SENDER_FENCE:
                assert st["atomics_deferred"] == 0, tag


def _cpu_barrier_peer(name, delay, q):
    import time as _t
    import paper_2512_19849_amd as ep_
    h = ep_.ep_proxy_start(4, 16, 2, 1024, 64, num_channels=1, ring_entries=8, num_proxy_threads=1,
                           spin_timeout_ms=20000, flags=ep_.EP_FLAG_HOST_ONLY, barrier_peers=2, barrier_name=name)
    try:
        q.put("ready")
        _t.sleep(delay)
        t_push = _t.time()
        i = ep_.ep_host_push(h, 0, 4 << 28, 0, 0, 0)
        while not ep_.ep_host_check_completion(h, 0, i):
            _t.sleep(0.0005)
        q.put((t_push, _t.time(), ep_.ep_stats(h)["proxy_error"]))
    finally:
        ep_.ep_proxy_stop(h)


def test_barrier_kernel_waits_for_a_peer_process(epmod):
    """ep_barrier on the GPU: the stream is held until a second process (a CPU-side
    peer with its own proxy) has pushed its Barrier too."""
    import multiprocessing as mp
    import os
    import time
    from paper_2512_19849_amd.runner import EPRunner
    with EPRunner(4, 16, 2, 1024, 64, spin_timeout_ms=3000) as r:         # alone: completes at once
        epmod.ep_barrier(r.h)
        torch.cuda.synchronize()
        st = r.stats()
        assert st["barriers"] == 1 and st["device_error"] == 0 and st["proxy_error"] == 0
    ctx = mp.get_context("spawn")
    name = f"g{os.getpid()}"
    q = ctx.Queue()
    child = ctx.Process(target=_cpu_barrier_peer, args=(name, 0.3, q))
    child.start()
    try:
        with EPRunner(4, 16, 2, 1024, 64, spin_timeout_ms=20000, barrier_peers=2, barrier_name=name) as r:
            assert q.get(timeout=60) == "ready"
            torch.cuda.synchronize()
            t0 = time.time()
            epmod.ep_barrier(r.h)
            torch.cuda.synchronize()
            t1 = time.time()
            p_push, p_done, p_err = q.get(timeout=30)
            assert p_err == 0 and t1 >= p_push - 1e-3 and t1 - t0 > 0.15   # held until the peer arrived
            st = r.stats()
            assert st["barriers"] == 1 and st["device_error"] == 0 and st["proxy_error"] == 0
        child.join(timeout=30)
        assert child.exitcode == 0
    finally:
        if child.is_alive():
            child.terminate()
