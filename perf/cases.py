"""The work a program built on this library has it do, as cases that can be timed.

A case names one of five uses and its sizes:

  decode        one decode step: the new token of every sequence of a batch through the layers of a
                model (cache update, probe, scores, cut-off, attention), budgets handed from layer to layer
  decode_heads  a layer of a decode step with retrieval per KV head
  prefill       one layer's pass over a whole context whose inputs exist (a model that runs layer by
                layer over groups of windows)
  stream        windows that arrive one at a time on top of a cached context: append, retrieve, attend
  host_cache    a layer's pass with the key-value cache in pinned host memory

Shapes, windows, contexts and batches are those of the library's workloads and tests.
"""
import math

import torch

from paper_2502_13542_amd import binding as B
from paper_2502_13542_amd import harness as H
from paper_2502_13542_amd import synth
from paper_2502_13542_amd.synth import LayerShape

DEV = "cuda"

# (query heads, KV heads, channels per head, storage, local span) of the layers that are in use
LAYERS = [(32, 8, 128, "bf16", 512), (28, 4, 128, "bf16", 512), (8, 2, 128, "bf16", 256), (8, 2, 64, "bf16", 256),
          (8, 2, 64, "fp32", 256)]


def _case(kind, layer, n_ctx, k_cap, cutoff, window=1, batch=1, layers=1, ragged=False, graph=False, windows=0, name=None):
    hq, hkv, d, dtype, n_local = layer
    c = dict(kind=kind, hq=hq, hkv=hkv, d=d, dtype=dtype, n_local=n_local, n_ctx=n_ctx, window=window, k_cap=k_cap,
             cutoff=cutoff, batch=batch, layers=layers, ragged=ragged, graph=graph, windows=windows)
    return c if name is None else dict(c, name=name)


def listed():
    llama, g7, small, small64, fp32 = LAYERS
    return [
        # the smallest call: one layer for one sequence with a short context, called eagerly from a model
        _case("decode", llama, 8192, 32, True, name="decode_b1_8k"),
        # a served batch at 64K cached tokens, the step's launches in a graph; 4 of a model's 32 layers
        _case("decode", llama, 65536, 32, True, batch=16, layers=4, graph=True, name="decode_b16_64k"),
        # a larger batch whose sequences differ in length, seven query heads per KV head, fixed top-k
        _case("decode", g7, 20480, 16, False, batch=48, layers=2, ragged=True, graph=True, name="decode_b48_ragged_g7"),
        # the fp32 mode, for checking a model against its reference
        _case("decode", fp32, 8192, 8, True, batch=4, layers=4, name="decode_b4_8k_fp32"),
        # every KV head retrieves for itself
        _case("decode_heads", llama, 32768, 32, True, batch=8, name="decode_heads_b8_32k"),
        # a layer's pass over a short, an ordinary ragged and a long context
        _case("prefill", fp32, 8192, 8, False, window=256, name="prefill_8k_fp32"),
        _case("prefill", g7, 50001, 32, True, window=512, name="prefill_50k_g7_ragged"),
        _case("prefill", llama, 131072, 32, True, window=512, name="prefill_128k"),
        # four windows of a chat turn on top of a cached context, the last one ragged
        _case("stream", llama, 65536, 32, True, window=512, windows=4, ragged=True, name="stream_512_at_64k"),
        # long windows: a prompt taken in few large pieces
        _case("stream", small, 12288, 6, True, window=4096, windows=2, ragged=True, name="stream_4096"),
        # 64 channels per head in bf16, short windows
        _case("stream", small64, 16384, 8, False, window=256, windows=4, name="stream_256_d64"),
        # the cache kept in CPU memory, blocks brought in as they are selected and written back as they fill
        _case("host_cache", llama, 32768, 16, False, window=512, name="host_cache_32k"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "decode_heads", "prefill", "prefill", "prefill", "stream",
                       "stream", "stream", "host_cache"])
    k_cap = rng.choice([6, 8, 16, 32])
    cutoff = rng.random() < 0.7
    layer = rng.choice(LAYERS[:2] + LAYERS)              # the two large layers twice as often
    small = layer[0] * layer[2] <= 1024
    if kind == "decode":
        batch = _log(rng, 1, 48)
        most = min(65536, 1 << 20 >> int(math.log2(batch)))
        return _case(kind, layer, _log(rng, 2048, most), k_cap, cutoff, batch=batch, layers=rng.choice([1, 2, 4]),
                     ragged=rng.random() < 0.5, graph=rng.random() < 0.5)
    if kind == "decode_heads":
        return _case(kind, layer, _log(rng, 4096, 49152), k_cap, cutoff, batch=_log(rng, 1, 16), ragged=rng.random() < 0.5)
    if kind == "prefill":
        return _case(kind, layer, _log(rng, 4096, 32768 if small else 120000), k_cap, cutoff,
                     window=rng.choice([256, 512] if small else [256, 384, 512, 512, 1024]))
    if kind == "stream":
        window = _log(rng, 128, 4096)
        return _case(kind, layer, _log(rng, 4096, 32768 if small else 98304), k_cap, cutoff, window=window,
                     windows=2 if window > 1024 else rng.choice([2, 4]), ragged=rng.random() < 0.5)
    return _case(kind, rng.choice(LAYERS[:2]), 128 * _log(rng, 64, 256) + rng.choice([0, 0, 77]), k_cap, cutoff,
                 window=rng.choice([256, 512]))


# ---------------------------------------------------------------- sizes of a case
def _shape(c):
    return LayerShape(c["hq"], c["hkv"], c["d"], 128, 4, 128, c["n_local"], c["dtype"])


def _workload(c, seed, n_ctx):
    return synth.Workload("case", _shape(c), n_ctx, c["window"], c["k_cap"], c["cutoff"], seed,
                          n_planted=max(4, min(32, n_ctx // 4096)), n_layers=c["layers"])


def _lengths(c):
    """Cached tokens of every sequence of a decode batch, the step's token included."""
    if not c["ragged"]:
        return [c["n_ctx"] + 1] * c["batch"]
    return [1 + int(c["n_ctx"] * (0.1 + 0.9 * ((0.37 + 0.618034 * s) % 1.0))) for s in range(c["batch"])]


def _stream_rows(c):
    rows = [c["window"]] * c["windows"]
    if c["ragged"]:
        rows[-1] = max(2, c["window"] * 5 // 8 + 3)
    return rows


# ---------------------------------------------------------------- prepare
def _decode_caches(sh, w, c, nb, gen, layer):
    bt, hk, d = c["batch"], sh.n_kv_heads, sh.head_dim
    kc = torch.empty(bt, nb, hk, 128, d, dtype=sh.torch_dtype, device=DEV).normal_(generator=gen)
    vc = torch.empty(bt, nb, hk, d, 128, dtype=sh.torch_dtype, device=DEV).normal_(generator=gen)
    u = synth.direction(w, 0, 0, DEV)
    # (sequences of a ragged batch may all be shorter than the context the blocks are drawn for)
    planted = torch.tensor([b for b in synth.planted_blocks(w, layer, 0) if b < nb], dtype=torch.int64, device=DEV)
    kc[:, planted] += (w.shift * u)[None, None, :, None, :].to(kc.dtype)
    return kc, vc, synth.pick_rep_keys_blocked(kc, sh.n_rep)


def _prepare_decode(c, seed):
    sh, bt, L = _shape(c), c["batch"], c["layers"]
    w = _workload(c, seed, c["n_ctx"])
    lens = _lengths(c)
    nb = (max(lens) + 127) // 128
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    hk, d = sh.n_kv_heads, sh.head_dim
    u_hat = synth.direction(w, 0, 0, DEV).repeat_interleave(sh.group, dim=0)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV)  # noqa: E731
    ends = [H.eligible_range(sh, n - 1)[1] for n in lens]
    n_elig = max(max(ends) - 1, 1)
    i32, f32 = dict(dtype=torch.int32, device=DEV), dict(dtype=torch.float32, device=DEV)
    st = dict(c=c, cs=B.c_shape(sh), sh=sh, n_ctx=torch.tensor(lens, **i32), pos0=torch.tensor([n - 1 for n in lens], **i32),
              nb_end=torch.tensor(ends, **i32), nb_end_max=max(ends))
    layers = [_decode_caches(sh, w, c, nb, gen, l) for l in range(L)]
    st["kc"], st["vc"], st["rep"] = ([x[i] for x in layers] for i in range(3))
    q = [(rnd(bt, 1, sh.n_q_heads, d) + w.alpha * u_hat).to(sh.torch_dtype) for _ in range(L)]
    st["q"] = q
    st["k_new"] = [rnd(bt, 1, hk, d).to(sh.torch_dtype) for _ in range(L)]
    st["v_new"] = [rnd(bt, 1, hk, d).to(sh.torch_dtype) for _ in range(L)]
    st["out"] = [torch.zeros_like(x) for x in q]
    b0, _ = synth.decode_cutoff_profile(w, n_elig)
    st["k_mean"], st["prior"] = b0 / L, math.log(max(n_elig, 2))
    if c["kind"] == "decode_heads":
        rows = bt * hk
        stride = (nb + 3) // 4 * 4
        st.update(nb=nb, stride=stride, probe=torch.empty(bt, sh.d_model, **f32), probe_kv=torch.empty(bt, hk * d, **f32),
                  probe_norm=torch.empty(bt, **f32), scores=torch.zeros(bt, hk, stride, **f32),
                  nb_end_h=st["nb_end"][:, None].expand(bt, hk).contiguous().view(rows),
                  idx=torch.full((bt, hk, c["k_cap"]), -1, **i32), n_sel=torch.zeros(bt, hk, **i32),
                  theta=torch.zeros(bt, hk, **f32), budget0=torch.full((rows,), b0, **f32),
                  rest=torch.full((rows,), st["prior"] * 0.5, **f32), budget=torch.zeros(rows, **f32),
                  ws=torch.zeros(B.workspace_bytes(st["cs"], bt, 1, nb, c["k_cap"]), dtype=torch.uint8, device=DEV))
        return st
    st["runners"] = [H.LayerRunner(sh, bt, 1, nb, c["k_cap"], DEV) for _ in range(L)]
    st["theta"] = torch.full((L, bt), st["prior"], **f32)        # the densities of the step before
    for l, r in enumerate(st["runners"]):
        r.theta = st["theta"][l]
    st["theta_sum"], st["steps"] = torch.zeros(bt, L, **f32), torch.zeros(bt, **f32)
    st["rest"] = torch.zeros(L, bt, **f32)
    st["budgets"] = [torch.zeros(bt, **f32), torch.zeros(bt, **f32)]
    if c["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _step_decode(st)                                     # everything has been called once before the capture
        torch.cuda.current_stream().wait_stream(side)
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            _step_decode(st)
    return st


def _prepare_layer(c, seed):
    """One layer of one sequence: a whole context, or the context and the windows behind it."""
    sh, m = _shape(c), c["window"]
    rows = _stream_rows(c) if c["kind"] == "stream" else []
    n = c["n_ctx"] + sum(rows)
    w = _workload(c, seed, n)
    q, k, v = synth.gen_layer(w, DEV)
    rep = synth.pick_rep_keys(k[:c["n_ctx"]] if rows else k, 128, sh.n_rep)
    nb = w.n_blocks
    repd = torch.zeros(nb, sh.n_rep, sh.n_kv_heads, sh.head_dim, dtype=rep.dtype, device=DEV)
    repd[: rep.shape[0]] = rep
    w0s = [c["n_ctx"] + sum(rows[:i]) for i in range(len(rows))] if rows else list(range(0, n, m))
    cut = None
    if c["cutoff"]:
        cut = []
        for t, w0 in enumerate(w0s):
            b, e = H.eligible_range(sh, w0)
            cut.append(synth.cutoff_state(w, e - b, t, 0))
    st = dict(c=c, sh=sh, rep=repd, w0s=w0s, rows=rows)
    if c["kind"] == "stream":
        st["cs"] = B.c_shape(sh)
        st["runner"] = r = H.LayerRunner(sh, 1, m, nb, c["k_cap"], DEV)
        old = k[:c["n_ctx"]], v[:c["n_ctx"]]
        st["kc"], st["vc"] = H.blocked_k(old[0], sh, nb), H.blocked_vt(old[1], sh, nb)
        i32 = dict(dtype=torch.int32, device=DEV)
        one = lambda xs: [torch.tensor([x], **i32) for x in xs]  # noqa: E731
        st["pos0"], st["n_ctx"] = one(w0s), one([a + b for a, b in zip(w0s, rows)])
        st["ends"] = [H.eligible_range(sh, a)[1] for a in w0s]
        st["nb_end"] = one(st["ends"])
        cutt = None if cut is None else torch.tensor(cut, dtype=torch.float32, device=DEV)
        st["bud0"] = None if cutt is None else cutt[:, 0].contiguous()
        st["bud"] = None if cutt is None else st["bud0"].clone()
        st["rest"] = None if cutt is None else cutt[:, 1].contiguous()
        a = c["n_ctx"]
        st["q"], st["k"], st["v"] = (x[a:].contiguous() for x in (q, k, v))
        # the statistics of the queries before the windows
        h = min(a, 1024)
        B.build_probe(st["cs"], 1, min(h, m), q[a - min(h, m):a], r.stats, True, r.probe, r.probe_kv, r.probe_norm, None,
                      r.workspace)
        st["stats0"] = r.stats.clone()
        st["out"] = torch.zeros_like(st["q"])
        st["idx"] = [torch.full((1, c["k_cap"]), -1, **i32) for _ in rows]
        st["n_sel"] = [torch.zeros(1, **i32) for _ in rows]
        return st
    st["q"], st["out"] = q, torch.zeros_like(q)
    st["runner"] = H.LayerRunner(sh, 1, m, nb, c["k_cap"], DEV)
    st["plan"] = H.make_prefill_plan(sh, n, m, cut, DEV)
    st["bud0"] = None if cut is None else st["plan"].budget.clone()
    if c["kind"] == "host_cache":
        st["k"], st["v"] = k, v
        full = lambda *s: torch.zeros(*s, dtype=sh.torch_dtype, pin_memory=True)  # noqa: E731
        st["ks"] = full(nb, sh.n_kv_heads, 128, sh.head_dim)
        st["vs"] = full(nb, sh.n_kv_heads, sh.head_dim, 128)
        st["host"] = H.HostCachePrefill(st["runner"], st["plan"])
    else:
        st["kc"], st["vc"] = H.blocked_k(k, sh, nb), H.blocked_vt(v, sh, nb)
        st["pipe"] = H.PrefillPipeline(st["runner"], st["plan"])
    return st


def prepare(case, seed):
    return (_prepare_decode if case["kind"].startswith("decode") else _prepare_layer)(case, seed)


# ---------------------------------------------------------------- run
def _step_decode(st):
    c = st["c"]
    B.cutoff_next_step(c["batch"], c["layers"], st["k_mean"], st["prior"], st["theta"], st["theta_sum"], st["steps"],
                       st["budgets"][0], st["rest"])
    bud, rest = st["budgets"], st["rest"]
    two = c["dtype"] == "bf16" and c["d"] == 128
    for l, r in enumerate(st["runners"]):
        if two:
            b = (bud[l % 2], rest[l], bud[(l + 1) % 2]) if c["cutoff"] else (None, None, None)
            r.decode_step_two_launches(st["q"][l], st["kc"][l], st["vc"][l], st["rep"][l], st["n_ctx"], st["nb_end"],
                                       st["out"][l], *b, st["k_new"][l], st["v_new"][l], st["pos0"])
        else:
            b = (bud[0], rest[l]) if c["cutoff"] else (None, None)
            r.decode_step(st["q"][l], st["kc"][l], st["vc"][l], st["rep"][l], st["n_ctx"], st["nb_end"],
                          st["nb_end_max"], st["out"][l], *b, st["k_new"][l], st["v_new"][l], st["pos0"])


def _run_decode(st):
    if st["c"]["graph"]:
        st["graph"].replay()
    else:
        _step_decode(st)
    got = dict(out=st["out"], theta=st["theta"], idx=[r.idx for r in st["runners"]], n_sel=[r.n_sel for r in st["runners"]])
    if sum(x.numel() for x in st["kc"]) <= 1 << 26:              # larger caches would take longer to compare than to make
        got.update(k_cache=st["kc"], v_cache=st["vc"], rep_keys=st["rep"])
    return got


def _run_heads(st):
    c, sh, cs = st["c"], st["sh"], st["cs"]
    bt, nb = c["batch"], st["nb"]
    kc, vc, rep = st["kc"][0], st["vc"][0], st["rep"][0]
    bud = None
    if c["cutoff"]:
        bud = st["budget"]
        bud.copy_(st["budget0"])
    B.append_kv_probe(cs, bt, st["q"][0], st["k_new"][0], st["v_new"][0], st["pos0"], kc, vc, kc.stride(0), rep,
                      rep.stride(0), nb, st["probe"], st["probe_kv"], st["probe_norm"])
    B.score_blocks_per_head(cs, bt, st["probe"], rep, rep.stride(0), st["nb_end_max"], 1, st["nb_end_h"], st["scores"],
                            st["stride"])
    B.select(bt * sh.n_kv_heads, st["scores"], st["stride"], st["nb_end_max"], 1, st["nb_end_h"], c["k_cap"], bud,
             st["rest"] if c["cutoff"] else None, st["idx"], st["n_sel"], st["theta"])
    B.retrieval_attention(cs, bt, 1, st["q"][0], kc, vc, kc.stride(0), nb, st["n_ctx"], st["idx"], st["n_sel"],
                          c["k_cap"], st["out"][0], None, st["ws"], per_head=True)
    return dict(out=st["out"], theta=st["theta"], idx=st["idx"], n_sel=st["n_sel"])


def _run_prefill(st):
    r, plan = st["runner"], st["plan"]
    r.stats.zero_()
    if st["bud0"] is not None:
        plan.budget.copy_(st["bud0"])
    if st["c"]["kind"] == "host_cache":
        h = st["host"]
        h.run_overlapped(st["q"], st["k"], st["v"], st["ks"], st["vs"], st["rep"], st["out"])
        return dict(out=st["out"], stats=r.stats, idx=h.idx_all, n_sel=h.n_sel_all)
    p = st["pipe"]
    p.run(st["q"], st["kc"], st["vc"], st["rep"], st["out"], True, chunk=32, batched=True, late_cus=32,
          attention_cus=224)
    return dict(out=st["out"], stats=r.stats, idx=p.idx, n_sel=p.n_sel)


def _run_stream(st):
    r, cs, rows = st["runner"], st["cs"], st["rows"]
    r.stats.copy_(st["stats0"])
    if st["bud"] is not None:
        st["bud"].copy_(st["bud0"])
    at = 0
    for t, m in enumerate(rows):
        q = st["q"][at:at + m]
        B.append_kv(cs, 1, m, st["k"][at:at + m], st["v"][at:at + m], st["pos0"][t], st["kc"], st["vc"], 0, st["rep"], 0,
                    r.nb_capacity)
        r.idx, r.n_sel = st["idx"][t], st["n_sel"][t]
        bud, rest = (None, None) if st["bud"] is None else (st["bud"][t:t + 1], st["rest"][t:t + 1])
        r.step(q, st["kc"], st["vc"], st["rep"], st["n_ctx"][t], st["nb_end"][t], st["ends"][t], st["out"][at:at + m],
               bud, rest, True, m)
        at += m
    return dict(out=st["out"], k_cache=st["kc"], v_cache=st["vc"], rep_keys=st["rep"], stats=r.stats, idx=st["idx"],
                n_sel=st["n_sel"])


def run(state):
    kind = state["c"]["kind"]
    return {"decode": _run_decode, "decode_heads": _run_heads, "stream": _run_stream}.get(kind, _run_prefill)(state)


# ---------------------------------------------------------------- work and tolerance
def _selected(c, sh, w0):
    """Blocks retrieved at position w0: the cut-off's inputs let about a third of k_cap pass."""
    b, e = H.eligible_range(sh, w0)
    return min(max(e - b, 0), max(1.0, 0.325 * c["k_cap"]) if c["cutoff"] else c["k_cap"])


def work(case):
    c, sh = case, _shape(case)
    e = 4 if c["dtype"] == "fp32" else 2
    hk, d, hq = sh.n_kv_heads, sh.head_dim, sh.n_q_heads
    byt = flops = 0.0
    if c["kind"].startswith("decode"):
        for n in _lengths(c):
            lo, hi = H.eligible_range(sh, n - 1)
            keys = min(128, n - 1) + 128 * _selected(c, sh, n - 1) + n - H.local_start(sh, n - 1)
            byt += (2 * keys * hk + (hi - lo) * sh.n_rep * hk + 2 * hq + 2 * hk) * d * e
            flops += 4 * d * hq * keys + 2 * (hi - lo) * sh.n_rep * hk * d
        return {"bytes": byt * c["layers"], "flops": flops * c["layers"]}
    rows = _stream_rows(c) if c["kind"] == "stream" else None
    w0s = range(0, c["n_ctx"], c["window"]) if rows is None else [c["n_ctx"] + sum(rows[:i]) for i in range(len(rows))]
    selected = 0.0
    for t, w0 in enumerate(w0s):
        m = min(c["window"], c["n_ctx"] - w0) if rows is None else rows[t]
        sel = _selected(c, sh, w0)
        selected += sel
        past = min(128, w0) + 128 * sel + w0 - H.local_start(sh, w0)
        lo, hi = H.eligible_range(sh, w0)
        flops += 4.0 * d * hq * (m * past + m * (m + 1) / 2) + 8.0 * m * hq * d + 2.0 * (hi - lo) * sh.n_rep * hk * d
        byt += 2 * m * hq * d * e                                # queries in, outputs out
        if rows is not None:                                     # new keys and values in and into the cache, what is seen
            byt += (2 * (2 * m + past) + (hi - lo) * sh.n_rep) * hk * d * e
    if rows is None:                                             # the cache and the representatives once
        byt += (2 * c["n_ctx"] + c["n_ctx"] / 128 * sh.n_rep) * hk * d * e
    if c["kind"] == "host_cache":                                # selected blocks over the link, new blocks into the store
        byt += (2 * 128 * selected + 2 * c["n_ctx"]) * hk * d * e
    return {"bytes": byt, "flops": flops}


def tolerance(case):
    # differ: two blocks whose scores are equal up to fp32 rounding may change places
    return {"rel": 1e-5 if case["dtype"] == "fp32" else 1e-2, "differ": 0.005}
