"""The calls whose speed is watched: what programs that use this library have
it do, through its public entry points, with inputs of the shapes and
distributions of the workloads in ``synth/configs.py``.

A case is a dict of plain values; its "kind" names the work:

  linattn     one layer's chunked linear-attention prefill
  gdn         one layer's gated delta-rule prefill
  resume      a session resumed from its capsule: restore, then one decode
              token (append of K/V rows and conv inputs, one decode step per
              linear layer)
  checkpoint  a capsule taken of a running session and restored into another
  fork        one capsule restored into several sessions at once
  gather      batched episode reset: every environment receives a capsule of
              a gallery
  fp8         new K/V rows enter the FP8 region, then the bf16 working stage
              of all its rows is rebuilt (first read after a restore into
              another session)

``listed`` gives the fixed cases, ``draw`` more of the same ranges, ``prepare``
what the program holds before the call, ``run`` one pass, ``work`` the bytes
and operations it cannot do without, ``exact`` its results in 64 bits from the
token recurrences, ``tolerance`` how far a correct result may differ.
"""
import math

import torch

import paper_2606_20537_amd as cap

CHUNK = 64


# ------------------------------------------------------------------ cases --
def listed():
    return [
        # one linear layer of the 48-layer stack over its 16k prefix, keeping
        # every chunk-boundary state (any boundary can become a capsule)
        _linattn("linattn_16k_states", T=16384, H=32, states=True),
        # the same layer when only the state after the prefix is kept (a cold
        # prefill for a first token)
        _linattn("linattn_16k_final", T=16384, H=32),
        # one layer of the 8-layer stack over its 2k prefix, from a state
        _linattn("linattn_2k_final", T=2048, H=16, state_in=True),
        # an unaligned prefix of the same stack (a partial last chunk), with
        # chunk states
        _linattn("linattn_4159_states", T=4159, H=16, states=True, state_in=True),
        # the smallest model: 2 heads of 64, fp32 inputs, 256 tokens
        _linattn("linattn_256_f32", T=256, H=2, dk=64, dv=64, dtype="f32", states=True),
        # one delta-rule layer of the 48-layer stack
        _gdn("gdn_16k_states", T=16384, H=32, states=True),
        # a delta-rule layer of the 8-layer stack, unaligned prefix
        _gdn("gdn_2111_final", T=2111, H=16, state_in=True),
        # the 8-layer session resumed at 2048 and decoding its first token:
        # small copies and short launches
        _resume("resume_8_layers", layers=6, full=2, H=16, kv_row=1024, prefix=2048, rows=8448, channels=2048),
        # the 48-layer session checkpointed and restored (882 MB each way)
        _checkpoint("checkpoint_48_layers", layers=36, full=12, H=32, kv_row=2048, prefix=16384, rows=16448,
                    channels=4096),
        # the same capsule forked into four sessions
        _fork("fork4_48_layers", n=4, layers=36, full=12, H=32, kv_row=2048, prefix=16384, rows=16448, channels=4096),
        # robot episode reset: 32 environments, a gallery of 8 capsules of 17 MB
        _gather("gather_32_of_8", envs=32, gallery=8, full=18, kv_row=512, prefix=816, fixed=2 << 20),
        # FP8 K/V of 12 full-attention layers over the 16k prefix
        _fp8("fp8_kv_16k", bufs=24, rows=16384, row=1024),
    ]


def _linattn(name, T, H, dk=128, dv=128, dtype="bf16", states=False, state_in=False):
    return {"name": name, "kind": "linattn", "T": T, "H": H, "dk": dk, "dv": dv, "dtype": dtype, "states": states,
            "state_in": state_in}


def _gdn(name, T, H, dk=128, dv=128, states=False, state_in=False, noalloc=False):
    return {"name": name, "kind": "gdn", "T": T, "H": H, "dk": dk, "dv": dv, "states": states,
            "state_in": state_in, "noalloc": noalloc}


def _resume(name, layers, full, H, kv_row, prefix, rows, channels, mixer="linattn"):
    return {"name": name, "kind": "resume", "layers": layers, "full": full, "H": H, "kv_row": kv_row,
            "prefix": prefix, "rows": rows, "channels": channels, "mixer": mixer}


def _checkpoint(name, layers, full, H, kv_row, prefix, rows, channels):
    return {"name": name, "kind": "checkpoint", "layers": layers, "full": full, "H": H, "kv_row": kv_row,
            "prefix": prefix, "rows": rows, "channels": channels}


def _fork(name, n, **kw):
    return {**_checkpoint(name, **kw), "kind": "fork", "n": n}


def _gather(name, envs, gallery, full, kv_row, prefix, fixed):
    return {"name": name, "kind": "gather", "envs": envs, "gallery": gallery, "full": full, "kv_row": kv_row,
            "prefix": prefix, "fixed": fixed}


def _fp8(name, bufs, rows, row):
    return {"name": name, "kind": "fp8", "bufs": bufs, "rows": rows, "row": row}


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: token counts 1 to 16384, 1 to 32 heads, key width 64 or
    128, value widths 16 to 256, capsules from about 100 KB to those of the
    listed stacks; odd and ragged sizes throughout."""
    kind = rng.choice(["linattn", "linattn", "linattn", "gdn", "gdn", "resume", "checkpoint", "fork", "gather", "fp8"])
    if kind in ("linattn", "gdn"):
        dk, dv, H = rng.choice([64, 128, 128]), 16 * rng.choice([1, 2, 3, 4, 4, 6, 8, 8, 8, 8, 11, 16]), _log_int(rng, 1, 32)
        T = _log_int(rng, 1, 16384)
        T = max(1, min(T, 16384 * 32 * 128 // (H * dv)))  # no more than the largest listed call
        if kind == "linattn":
            dtype = rng.choice(["bf16", "f32"]) if dk == 64 else "bf16"
            c = _linattn("", T, H, dk, dv, dtype, rng.random() < 0.5, rng.random() < 0.5)
        else:
            c = _gdn("", T, H, dk, dv, rng.random() < 0.5, rng.random() < 0.5, rng.random() < 0.25)
    elif kind == "gather":
        c = _gather("", rng.randint(2, 48), rng.randint(1, 8), rng.randint(1, 18), 16 * rng.randint(4, 32),
                    _log_int(rng, 32, 816), 16 * _log_int(rng, 64, 1 << 17))
    elif kind == "fp8":
        c = _fp8("", rng.randint(2, 24), _log_int(rng, 1, 16384), 16 * rng.randint(8, 64))
    else:
        full = rng.randint(1, 12 if kind != "resume" else 6)
        prefix = CHUNK * _log_int(rng, 4, 256 if kind != "resume" else 64)
        kw = dict(layers=rng.randint(1, 3 * full), full=full, H=_log_int(rng, 2, 32), kv_row=256 * rng.randint(1, 8),
                  prefix=prefix, rows=prefix + rng.randint(1, 500), channels=8 * rng.randint(32, 512))
        if kind == "resume":
            c = _resume("", mixer=rng.choice(["linattn", "gdn"]), **kw)
        else:
            c = _fork("", rng.randint(2, 4), **kw) if kind == "fork" else _checkpoint("", **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------- prepare --
def _gen(seed, stream=0):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + stream)


def _randn(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)


def _tokens(gen, T, H, dk, dv, dtype, beta):
    """q and k of unit length per token and head, v ~ N(0, 1), log-gates
    log(sigmoid(N(3, 0.5))), write strengths sigmoid(N(0, 1))."""
    el = torch.float32 if dtype == "f32" else torch.bfloat16
    d = {n: torch.nn.functional.normalize(_randn(gen, T, H, dk), dim=-1).to(el) for n in ("q", "k")}
    d["v"] = _randn(gen, T, H, dv).to(el)
    d["g"] = torch.nn.functional.logsigmoid(3.0 + 0.5 * _randn(gen, T, H))
    if beta:
        d["beta"] = torch.sigmoid(_randn(gen, T, H))
    return d


def _prefill_state(case, seed):
    T, H, dk, dv = case["T"], case["H"], case["dk"], case["dv"]
    gen = _gen(seed)
    s = {"case": case, **_tokens(gen, T, H, dk, dv, case.get("dtype", "bf16"), case["kind"] == "gdn")}
    s["state_in"] = _randn(gen, H, dk, dv) if case["state_in"] else None
    s["o"] = torch.zeros((T, H, dv), device="cuda")
    s["cs"] = torch.zeros(((T + CHUNK - 1) // CHUNK, H, dk, dv), device="cuda") if case["states"] else None
    s["final"] = torch.zeros((H, dk, dv), device="cuda")
    if case["kind"] == "gdn" and not case["noalloc"]:
        s["ws"] = torch.empty(cap.gdn_workspace_bytes(T, H), dtype=torch.uint8, device="cuda")
    return s


def _layout(case):
    """(name, row bytes, rows, kind) of a session's live buffers: three linear
    layers (fp32 state, conv window of 4 inputs) to one full-attention layer
    (K and V rows), in model order."""
    if case["kind"] == "gather":
        kv = [("kv%d%s" % (i, x), case["kv_row"], case["prefix"], cap.CAP_KIND_POSITIONAL)
              for i in range(case["full"]) for x in "kv"]
        return kv + [("denoiser", case["fixed"], 1, cap.CAP_KIND_FIXED)]
    out, lin, full = [], 0, 0
    while lin < case["layers"] or full < case["full"]:
        if (lin + full) % 4 == 3 and full < case["full"] or lin == case["layers"]:
            out += [("kv%d%s" % (full, x), case["kv_row"], case["rows"], cap.CAP_KIND_POSITIONAL) for x in "kv"]
            full += 1
        else:
            out.append(("state%d" % lin, case["H"] * 128 * 128 * 4, 1, cap.CAP_KIND_FIXED))
            out.append(("conv%d" % lin, case["channels"] * 2, 4, cap.CAP_KIND_FIXED))
            lin += 1
    return out


def _group(name):
    return "kv" if name.startswith("kv") else name.rstrip("0123456789")


def _sessions(layout, gen, n, chunk):
    """n live sets whose buffers lie in one tensor per group, as a model
    allocates them: states and denoiser buffers fp32, conv windows and K/V
    rows bf16, all N(0, 1).  Returns the sets and the groups [n, bytes / size]."""
    groups, size = {}, {}
    for name, rb, rows, _ in layout:
        grp = _group(name)
        groups.setdefault(grp, []).append(name)
        size[grp] = size.get(grp, 0) + rb * rows
    pool = {grp: _randn(gen, n, size[grp] // 4) if grp in ("state", "denoiser") else
            _randn(gen, n, size[grp] // 2).to(torch.bfloat16) for grp in groups}
    sets = []
    for i in range(n):
        at, bufs = dict.fromkeys(groups, 0), []
        for name, rb, rows, kind in layout:
            grp = _group(name)
            es = pool[grp].element_size()
            bufs.append((name, pool[grp][i, at[grp] // es:(at[grp] + rb * rows) // es], rb, rows, kind))
            at[grp] += rb * rows
        sets.append(cap.cap_set_create(bufs, chunk, 7))
    return sets, list(pool.values())


def _capsules(case, layout, gen, n, chunk):
    sets, pool = _sessions(layout, gen, n, chunk)
    out = []
    for x in sets:
        cap.cap_set_set_position(x, case["prefix"])
        arena = torch.empty(cap.capsule_bytes(x, case["prefix"]), dtype=torch.uint8, device="cuda")
        out.append(cap.capsule_snapshot(x, case["prefix"], 5, arena))
    return out, sets, pool


def prepare(case, seed):
    kind, gen = case["kind"], _gen(seed, 1)
    if kind in ("linattn", "gdn"):
        return _prefill_state(case, seed)
    s = {"case": case}
    if kind == "fp8":
        n = case["rows"] * case["row"]
        s["new"] = [_randn(gen, n).to(torch.bfloat16) for _ in range(case["bufs"])]
        s["fp8"] = [torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(case["bufs"])]
        s["stage"] = [torch.zeros(n, dtype=torch.bfloat16, device="cuda") for _ in range(case["bufs"])]
        s["set"] = cap.cap_set_create([("kv%d" % i, t, case["row"], case["rows"], cap.CAP_KIND_POSITIONAL)
                                       for i, t in enumerate(s["fp8"])], 1, 7)
        s["scale"] = 0.0125
        for i, t in enumerate(s["stage"]):
            cap.cap_set_bind_stage(s["set"], i, t, s["scale"])
        cap.cap_set_set_position(s["set"], case["rows"])
        return s
    layout = _layout(case)
    if kind == "gather":
        s["gallery"] = _capsules(case, layout, gen, case["gallery"], 1)[0]
        s["ids"] = torch.randint(0, case["gallery"], (case["envs"],), generator=torch.Generator().manual_seed(seed)).tolist()
        s["sets"], s["bufs"] = _sessions(layout, gen, case["envs"], 1)
        return s
    if kind == "checkpoint":
        (s["from"],), s["from_bufs"] = _sessions(layout, gen, 1, CHUNK)
        cap.cap_set_set_position(s["from"], case["prefix"])
        s["arena"] = torch.zeros(cap.capsule_bytes(s["from"], case["prefix"]), dtype=torch.uint8, device="cuda")
        (s["to"],), s["bufs"] = _sessions(layout, gen, 1, CHUNK)
        return s
    (s["capsule"],), (live,), bufs = _capsules(case, layout, gen, 1, CHUNK)
    if kind == "fork":
        del live, bufs
        s["sets"], s["bufs"] = _sessions(layout, gen, case["n"], CHUNK)
        return s
    # resume: the session goes on where the capsule was taken
    s["set"], s["bufs"], s["names"] = live, bufs, [x[0] for x in layout]
    H, L = case["H"], case["layers"]
    s["tok"] = [_tokens(gen, 1, H, 128, 128, "bf16", case["mixer"] == "gdn") for _ in range(L)]
    s["o"] = torch.zeros((L, 1, H, 128), device="cuda")
    s["states"] = bufs[0].view(L, H, 128, 128)
    s["new_kv"] = _randn(gen, 2 * case["full"], case["kv_row"] // 2).to(torch.bfloat16)
    s["new_conv"] = _randn(gen, L, case["channels"]).to(torch.bfloat16)
    kv, conv = iter(s["new_kv"]), iter(s["new_conv"])
    s["rows"] = [None if n.startswith("state") else next(kv if n.startswith("kv") else conv) for n in s["names"]]
    return s


# -------------------------------------------------------------------- run --
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "linattn":
        cap.linattn_chunked_prefill(s["q"], s["k"], s["v"], s["g"], s["o"], state_in=s["state_in"],
                                    chunk_states=s["cs"], final_state=s["final"])
        return (s["o"], s["final"]) + ((s["cs"],) if case["states"] else ())
    if kind == "gdn":
        if case["noalloc"]:
            cap.gdn_chunked_prefill_noalloc(s["q"], s["k"], s["v"], s["g"], s["beta"], s["o"], state_in=s["state_in"],
                                            chunk_states=s["cs"], final_state=s["final"])
        else:
            cap.gdn_chunked_prefill(s["q"], s["k"], s["v"], s["g"], s["beta"], s["o"], state_in=s["state_in"],
                                    chunk_states=s["cs"], final_state=s["final"], workspace=s["ws"])
        return (s["o"], s["final"]) + ((s["cs"],) if case["states"] else ())
    if kind == "checkpoint":
        c = cap.capsule_snapshot(s["from"], case["prefix"], 5, s["arena"])
        cap.capsule_restore(c, s["to"], 5)
        return [s["arena"]] + s["bufs"]
    if kind == "fork":
        cap.capsule_fork(s["capsule"], s["sets"], 5)
        return s["bufs"]
    if kind == "gather":
        cap.capsule_gather_restore(s["gallery"], s["ids"], s["sets"])
        return s["bufs"]
    if kind == "fp8":
        cap.kv_fp8_quantize([(x, y, x.numel(), s["scale"]) for x, y in zip(s["new"], s["fp8"])])
        cap.cap_stage_invalidate(s["set"])
        cap.cap_stage_acquire(s["set"], case["rows"])
        return s["fp8"] + s["stage"]
    cap.capsule_restore(s["capsule"], s["set"], 5)
    cap.cap_set_append(s["set"], s["rows"], 1)
    for d, o, st in zip(s["tok"], s["o"], s["states"]):
        if case["mixer"] == "gdn":
            cap.gdn_decode_step(d["q"], d["k"], d["v"], d["g"], d["beta"], o, state_in=st, final_state=st)
        else:
            cap.linattn_decode_step(d["q"], d["k"], d["v"], d["g"], o, state_in=st, final_state=st)
    return [s["o"]] + s["bufs"]


# ------------------------------------------------------------------- work --
def _capsule_bytes(case):
    return sum(rb * (case["prefix"] if kind == cap.CAP_KIND_POSITIONAL else rows)
               for _, rb, rows, kind in _layout(case))


def work(case):
    kind = case["kind"]
    if kind in ("linattn", "gdn"):
        T, H, dk, dv = case["T"], case["H"], case["dk"], case["dv"]
        state = H * dk * dv * 4
        nbytes = T * H * ((2 * dk + dv) * (4 if case.get("dtype") == "f32" else 2) + 4 + 4 * dv) + state
        nbytes += state * ((T + CHUNK - 1) // CHUNK) * case["states"] + state * case["state_in"]
        if kind == "linattn":  # causal scores and values of half a chunk, the entering state, the fold
            flops = T * H * ((CHUNK + 1) * (dk + dv) + 4 * dk * dv)
        else:                  # k S, the fold and q S
            nbytes += T * H * 4
            flops = T * H * 6 * dk * dv
        return {"bytes": nbytes, "flops": flops}
    if kind == "fp8":
        n = case["bufs"] * case["rows"] * case["row"]
        return {"bytes": 5 * n, "flops": 2 * n}
    n = _capsule_bytes(case)
    if kind == "checkpoint":
        return {"bytes": 3 * n, "flops": 0}
    if kind == "fork":
        return {"bytes": (1 + case["n"]) * n, "flops": 0}
    if kind == "gather":
        return {"bytes": (min(case["gallery"], case["envs"]) + case["envs"]) * n, "flops": 0}
    one = 2 * case["full"] * case["kv_row"] + case["layers"] * case["H"] * 128 * (3 * 2 + 4)
    return {"bytes": 2 * n + 2 * one, "flops": case["layers"] * case["H"] * 6 * 128 * 128}


# -------------------------------------------------------------- tolerance --
def tolerance(case):
    # about four times the error against the 64-bit results, measured over the
    # ranges of draw(): products of bf16 operands in hi and lo parts (prefill:
    # 2.6e-6 with bf16 inputs, 6.2e-6 with fp32 inputs, 5.1e-6 for the delta
    # rule), 32-bit sums and products (decode step: 1e-7)
    if case["kind"] == "linattn":
        return {"rel": 2.5e-5 if case["dtype"] == "f32" else 1e-5}
    if case["kind"] == "gdn":
        return {"rel": 2e-5}
    if case["kind"] == "resume":
        return {"rel": 4e-7}
    return "exact"


# ------------------------------------------------------------------ exact --
def _recurrence(d, S, states_every=0):
    """Token by token in 64 bits: o [T, H, dv], the states entering tokens 0,
    states_every, ..., and the last state."""
    q, k, v, g = (d[n].double() for n in ("q", "k", "v", "g"))
    gamma, beta = torch.exp(g), d["beta"].double() if "beta" in d else None
    T = q.shape[0]
    o, cs = torch.empty(v.shape, dtype=torch.float64, device="cuda"), []
    for t in range(T):
        if states_every and t % states_every == 0:
            cs.append(S.float())
        S = S * gamma[t][:, None, None]
        kt, vt = k[t][:, :, None], v[t][:, None, :]
        if beta is not None:
            vt = beta[t][:, None, None] * (vt - torch.bmm(kt.transpose(1, 2).contiguous(), S))
        S = torch.baddbmm(S, kt, vt.contiguous())
        o[t] = torch.bmm(q[t][:, None, :], S)[:, 0]
    return o, cs, S


def exact(case, seed):
    kind = case["kind"]
    if kind in ("linattn", "gdn"):
        d = _prefill_state(case, seed)
        S = d["state_in"].double() if case["state_in"] else torch.zeros(
            (case["H"], case["dk"], case["dv"]), dtype=torch.float64, device="cuda")
        o, cs, S = _recurrence(d, S, CHUNK if case["states"] else 0)
        return (o, S) + ((torch.stack(cs),) if case["states"] else ())
    if kind == "resume":
        s = prepare(case, seed)
        state, conv, kv = s["bufs"]
        steps = [_recurrence(d, x.double()) for d, x in zip(s["tok"], s["states"])]
        conv = torch.cat([conv.view(case["layers"], 4, -1)[:, 1:], s["new_conv"][:, None]], dim=1)
        kv = kv.view(2 * case["full"], case["rows"], -1).clone()
        kv[:, case["prefix"]] = s["new_kv"]
        return [torch.stack([x[0] for x in steps]), torch.stack([x[2] for x in steps]).view(1, -1),
                conv.double().view(1, -1), kv.double().view(1, -1)]
    return None
