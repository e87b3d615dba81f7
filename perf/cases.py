"""Performance cases of the S^4R decode path: what is timed, on which inputs.

Each case is one pass of a program that decodes with a compressed KV cache:

  step         one fused decode step (`decode_step`), the token appended or not
  windowed     one step with a query window kept in a window state
               (`decode_step_windowed`)
  ragged       one step over sequences of different lengths
               (`decode_step_ragged`)
  stages       the step as its four separate calls (`score_latent`,
               `select_topk`, `reconstruct`, `sparse_attn`), for a program that
               needs the scores, the selection or the reconstructed rows
  project      the bulk projection of a prompt (`prefill_project`)
  first_token  a prompt's whole way to its first decoded token: `prefill`
               (bases and projection), `project_queries`, `window_state_init`,
               one windowed step

listed() names the cases, draw() gives more of the same ranges, prepare()
makes what such a program holds on the GPU, run() is the pass, work() what it
cannot do without, exact() the same results in 64 bits by plain torch.

The state is drawn in latent coordinates: orthonormal bases, coefficient rows
with a decaying spectrum plus noise, queries with latent logits of standard
deviation about 1.5, a few needles, sinks ten times larger; prompts are raw
low-rank keys and values with noise and a few outlier channels.
"""

import math

import torch

import paper_2608_00528_amd as s4r

# name: query heads, KV heads, head dim, RoPE base
SHAPES = {
    "llama8b": (32, 8, 128, 5e5),     # Llama-3.1-8B layer, also Qwen3-4B's head counts
    "qwen7b": (28, 4, 128, 1e6),      # Qwen2.5-7B layer
    "small": (8, 2, 64, 1e4),         # a small layer with 64-wide heads
    "wide64": (16, 4, 64, 1e4),       # 64-wide heads, four per KV head
    "mha": (8, 8, 128, 1e4),          # no grouping
    "gqa2": (16, 8, 128, 1e6),        # two query heads per KV head
    "gqa8": (32, 4, 128, 1e6),        # eight query heads per KV head
}


def _case(kind, shape, batch, length, rank, window, topk, **more):
    c = {"kind": kind, "shape": shape, "batch": batch, "length": length, "rank": rank, "rank_v": 0, "groups": 1,
         "window": window, "topk": topk, "q_window": 1, "dtype": "bf16", "append": False, "pool_kernel": 7,
         "pool_mode": "max", "group_agg": "mean"}
    c.update(more)
    return c


def listed():
    cases = [
        # the smallest layer, fp32 storage, two basis groups: latency of the chain of calls
        ("step_small_fp32_4k", _case("step", "small", 1, 4092, 32, 64, 128, dtype="fp32", groups=2)),
        # a single user's chat at 32k
        ("step_llama8b_32k", _case("step", "llama8b", 1, 32764, 160, 64, 1024)),
        # fp32 storage at an ordinary size and odd length, four query rows scored in every step
        ("step_llama8b_fp32_wq4_16k", _case("step", "llama8b", 1, 16381, 160, 32, 700, dtype="fp32", q_window=4)),
        # the headline: four sequences at 128k
        ("step_llama8b_128k", _case("step", "llama8b", 4, 131068, 160, 128, 2048)),
        # eight sequences at 128k, seven query heads per KV head
        ("step_qwen7b_128k", _case("step", "qwen7b", 8, 131068, 96, 64, 1024)),
        # a serving batch in steady decode: every step appends its token
        ("step_llama8b_b32_append", _case("step", "llama8b", 32, 32765, 160, 64, 1024, append=True)),
        # a fifth of a 120k context kept, window of 4: the paper's efficiency setting
        ("window4_llama8b_120k", _case("windowed", "llama8b", 1, 120001, 204, 4, 23996, q_window=4, append=True)),
        # the same with the paper's default window of 32
        ("window32_llama8b_120k", _case("windowed", "llama8b", 1, 120001, 204, 32, 23968, q_window=32, append=True)),
        # a serving batch of unequal conversations, 9k to 60k tokens, value-heavy ranks
        ("ragged_llama8b_6x60k", _case("ragged", "llama8b", 6, 60013, 128, 64, 1500, rank_v=192, append=True)),
        # the separate calls
        ("stages_llama8b_32k", _case("stages", "llama8b", 1, 32764, 160, 64, 1024)),
        # four 128k prompts into their caches
        ("project_llama8b_4x128k", _case("project", "llama8b", 4, 131068, 160, 128, 2048)),
        # a 32k prompt's way to its first token
        ("first_token_llama8b_32k", _case("first_token", "llama8b", 1, 32765, 160, 64, 1024, q_window=4,
                                          append=True)),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["windowed"] * 2 + ["ragged"] * 2 + ["stages", "project", "first_token"])
    shape = rng.choice(["llama8b", "llama8b", "qwen7b", "small", "wide64", "mha", "gqa2", "gqa8"])
    hq, hkv, dh, _ = SHAPES[shape]
    dp, g = hkv * dh, hq // hkv
    rank = rng.choice([32, 64, 96, 100, 128, 160, 160, 192, 204, 224, 256])
    rank = min(rank, dp)
    window = rng.choice([0, 4, 8, 32, 64, 128])
    more = {"pool_kernel": rng.choice([1, 5, 7, 7, 7]), "pool_mode": rng.choice(["max", "max", "avg"]),
            "group_agg": rng.choice(["mean", "mean", "max"])}
    if kind == "project":
        batch = rng.choice([1, 2, 4])
        length = _log(rng, 1000, 131068)
        return _case(kind, shape, batch, length, min(rank, 192), window, 256, **more)
    if kind == "first_token":
        shape = rng.choice(["llama8b", "qwen7b", "gqa8"])
        length = _log(rng, 2500, 32765)
        return _case(kind, shape, 1, length, min(rank, 192), window, max(16, length // 20), q_window=4, append=True,
                     **more)
    batch = rng.choice([1, 1, 2, 3, 4, 8]) if kind != "ragged" else rng.choice([2, 3, 5, 8])
    length = _log(rng, 1000, min(131068, 1048576 // batch))
    if kind != "stages":
        more["append"] = rng.random() < 0.6
    share = rng.choice([0.01, 0.02, 0.05, 0.2] if batch == 1 else [0.01, 0.02, 0.05])
    topk = max(16, int(length * share))
    if kind in ("step", "stages"):
        if rng.random() < 0.2:
            more["dtype"] = "fp32"
            length = min(length, 40009)
            topk = max(16, int(length * min(share, 0.05)))
            rank = min(rank, 192)
        if g <= 4 and rng.random() < 0.3:
            more["q_window"] = rng.choice([2, 4])
    if kind == "stages":
        batch = min(batch, 2)
        length = min(length, 65537)
        topk = max(16, int(length * min(share, 0.03)))
    if kind == "windowed":
        more["q_window"] = rng.choice([2, 4, 8, 32 if g <= 4 else 16])
    if kind == "ragged":
        length = max(length, 2500)
        topk = max(16, min(topk, length // 12))
        if rng.random() < 0.4 and g <= 8 and dp >= 512:
            rank, more["rank_v"] = rng.choice([(96, 160), (128, 192), (160, 224)])
    return _case(kind, shape, batch, length, rank, window, topk, **more)


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------

def _stride(rank):
    return (rank + 31) // 32 * 32


def _dims(case):
    hq, hkv, dh, theta = SHAPES[case["shape"]]
    rv = case["rank_v"] or case["rank"]
    return {"hq": hq, "hkv": hkv, "dh": dh, "theta": theta, "G": hq // hkv, "Dp": hkv * dh, "Dg": hkv * dh // case["groups"],
            "s": 4, "rs": _stride(case["rank"]), "rvs": _stride(rv), "R": _stride(case["rank"]) * case["groups"],
            "Rv": _stride(rv) * case["groups"], "rv": rv, "es": 2 if case["dtype"] == "bf16" else 4,
            # room for the tokens that a conversation still appends
            "cap": (case["length"] + 15) // 16 * 16 + (256 if case["append"] else 0)}


def _lengths(case):
    """The sequences' lengths of a ragged batch: the longest first, down to 0.15 of it."""
    n, longest = case["batch"], case["length"]
    return [longest - int(0.85 * longest * b / max(n - 1, 1)) - 3 * b for b in range(n)]


def _config(case):
    d = _dims(case)
    return s4r.make_config(batch=case["batch"], n_q_heads=d["hq"], n_kv_heads=d["hkv"], head_dim=d["dh"],
                           rank=case["rank"], rank_v=case["rank_v"], capacity=d["cap"], basis_groups=case["groups"],
                           n_sink=d["s"], window=case["window"], q_window=case["q_window"], topk=case["topk"],
                           pool_kernel=case["pool_kernel"], pool_mode=case["pool_mode"],
                           group_agg=case["group_agg"], rope_theta=d["theta"], dtype=case["dtype"])


def _selected(case, length):
    return min(case["topk"], max(length - case["window"], 0)) + min(case["window"], length)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _orthonormal(gen, n, rows, cols, stride):
    """n matrices [rows, stride] with `cols` orthonormal columns (then zeros):
    Newton's iteration for the polar factor of a Gaussian matrix."""
    x = torch.randn((n, rows, cols), generator=gen, device="cuda")
    x /= math.sqrt(rows) + math.sqrt(cols)
    for _ in range(40 if cols * 4 > rows else 12):
        xtx = torch.bmm(x.transpose(1, 2).contiguous(), x)
        x = 1.5 * x - 0.5 * torch.bmm(x, xtx)
    out = torch.zeros((n, rows, stride), device="cuda")
    out[:, :, :cols] = x
    return out


def _tile(x):
    """[B, n, R] row-major (n a multiple of 16) to the caches' tiles of 16 rows x 32 columns."""
    b, n, r = x.shape
    return x.reshape(b, n // 16, 16, r // 32, 32).transpose(2, 3).contiguous().reshape(b, n, r)


def _untile(x):
    b, n, r = x.shape
    return x.reshape(b, n // 16, r // 32, 16, 32).transpose(2, 3).reshape(b, n, r)


def _heads(group_queries, d):
    """[..., G, Dp] group queries to [..., h_q, d_h] heads (head j G + g)."""
    lead = group_queries.shape[:-2]
    x = group_queries.reshape(*lead, d["G"], d["hkv"], d["dh"])
    return x.transpose(-3, -2).reshape(*lead, d["hq"], d["dh"])


def _columns(case, d, side):
    """Storage columns that hold latent data (the rest of each group's stride is zero)."""
    rank, stride = (case["rank"], d["rs"]) if side == "k" else (d["rv"], d["rvs"])
    return torch.cat([torch.arange(rank) + g * stride for g in range(case["groups"])]).cuda()


def _decode_inputs(case, seed):
    d = _dims(case)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    B, L, Dp, nb = case["batch"], case["length"], d["Dp"], case["groups"]
    randn = lambda *shape: torch.randn(shape, generator=gen, device="cuda")  # noqa: E731
    out = {}
    out["bases_k"] = _orthonormal(gen, B * nb, d["Dg"], case["rank"], d["rs"]).reshape(B, nb, d["Dg"], d["rs"]).to(dt)
    out["bases_v"] = _orthonormal(gen, B * nb, d["Dg"], d["rv"], d["rvs"]).reshape(B, nb, d["Dg"], d["rvs"]).to(dt)
    r_true = max(16, min(128, case["rank"] * nb * 4 // 5))
    latent = {}
    for side, width in (("k", case["rank"] * nb), ("v", d["rv"] * nb)):
        spectrum = 1.0 / (1.0 + torch.arange(width, device="cuda") / 16.0)
        scale = math.sqrt(Dp) / float(spectrum.square().sum().sqrt())
        mix = randn(B, r_true, width) * spectrum * (scale / math.sqrt(r_true))
        latent[side] = (spectrum * scale, mix, _columns(case, d, side))
    qnorm = 1.5 * math.sqrt(case["rank"] * nb) / (2.0 * math.sqrt(Dp) / math.sqrt(r_true))
    u = torch.bmm(randn(B, d["G"] * case["q_window"], r_true), latent["k"][1])
    u /= u.norm(dim=-1, keepdim=True)
    u = u.reshape(B, d["G"], case["q_window"], -1)
    noise = randn(*u.shape)
    noise /= noise.norm(dim=-1, keepdim=True)
    full = torch.zeros((B, d["G"], case["q_window"], d["R"]), device="cuda")
    full[..., latent["k"][2]] = (0.9 * u + 0.1 * noise) * qnorm
    # the newest query through the bases, the older ones as the coefficient rows a program keeps
    lat = full[:, :, -1].reshape(B, d["G"], nb, d["rs"]).permute(0, 2, 1, 3).reshape(B * nb, d["G"], d["rs"])
    back = out["bases_k"].float().reshape(B * nb, d["Dg"], d["rs"]).transpose(1, 2).contiguous()
    q = torch.bmm(lat.contiguous(), back).reshape(B, nb, d["G"], d["Dg"]).permute(0, 2, 1, 3).reshape(B, d["G"], Dp)
    q = q + randn(B, d["G"], Dp) * (0.1 * qnorm / math.sqrt(Dp))
    out["q"] = _heads(q, d).to(dt).contiguous()
    if case["q_window"] > 1:
        out["qwin_prev"] = full[:, :, :-1].contiguous()
    needle = u[:, :, -1].mean(dim=1)
    needle /= needle.norm(dim=-1, keepdim=True)
    lengths = _lengths(case) if case["kind"] == "ragged" else [L] * B
    for side, (columns, mix, at) in latent.items():
        width = d["R"] if side == "k" else d["Rv"]
        cache = torch.zeros((B, d["cap"], width), dtype=dt, device="cuda")
        for b in range(B):
            rows = torch.mm(randn(lengths[b], r_true), mix[b]) + 0.05 * randn(lengths[b], mix.shape[2]) * columns
            if side == "k":
                count = 32 if L > 8192 else 5
                where = torch.randint(0, max(lengths[b] - case["window"], 1), (count,), generator=gen, device="cuda")
                lift = (10.0 + 4.0 * torch.rand((count, 1), generator=gen, device="cuda"))
                rows[where] = rows[where] + lift * (math.sqrt(case["rank"] * nb) / qnorm) * needle[b]
            row_major = torch.zeros((1, (lengths[b] + 15) // 16 * 16, width), dtype=dt, device="cuda")
            row_major[0, :lengths[b], at] = rows.to(dt)
            cache[b, :row_major.shape[1]] = _tile(row_major)[0]
        out["coef_" + side] = cache
    for side in "kv":
        out["sink_" + side] = (10.0 * randn(B, d["s"], Dp)).to(dt)
        if case["append"]:
            out[side + "_new"] = randn(B, Dp).to(dt)
    return out


def _prompt_inputs(case, seed):
    """A prompt's raw keys and values (sinks first), its last queries, and the first decoded token."""
    d = _dims(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    randn = lambda *shape: torch.randn(shape, generator=gen, device="cuda")  # noqa: E731
    B, Dp, n = case["batch"], d["Dp"], case["length"] - (1 if case["append"] else 0)
    r_true = max(16, case["rank"] * 4 // 5)
    raw = {}
    for side in "kv":
        raw["s_" + side] = torch.empty((B, d["s"] + n, Dp), dtype=torch.bfloat16, device="cuda")
    q = torch.empty((B, case["q_window"], d["G"], Dp), device="cuda")
    for b in range(B):
        for side in "kv":
            mix = randn(r_true, Dp) / math.sqrt(r_true)
            if side == "k":
                mix[:, torch.randperm(Dp, generator=gen, device="cuda")[:4]] *= 8.0
                dirs = torch.mm(randn(case["q_window"] * d["G"], r_true), mix)
                dirs = dirs / dirs.norm(dim=-1, keepdim=True)
                noise = randn(*dirs.shape)
                dirs = 0.9 * dirs + 0.1 * noise / noise.norm(dim=-1, keepdim=True)
                q[b] = dirs.reshape(case["q_window"], d["G"], Dp) * (1.5 * math.sqrt(case["rank"]) / math.sqrt(Dp / r_true))
            rows = torch.mm(randn(d["s"] + n, r_true), mix) + 0.05 * randn(d["s"] + n, Dp)
            rows[:d["s"]] *= 10.0
            raw["s_" + side][b] = rows.to(torch.bfloat16)
    raw["q_rows"] = _heads(q, d).to(torch.bfloat16).contiguous()
    raw["k_new"], raw["v_new"] = randn(B, Dp).to(torch.bfloat16), randn(B, Dp).to(torch.bfloat16)
    return raw


def prepare(case, seed):
    cfg, d = _config(case), _dims(case)
    state = {"case": case, "cfg": cfg, "ws": s4r.alloc_workspace(cfg)}
    if case["kind"] == "first_token":
        raw = _prompt_inputs(case, seed)
        state.update(raw, q=raw["q_rows"][:, -1].contiguous(), q_prev=raw["q_rows"][:, :-1].contiguous())
        return state
    if case["kind"] == "project":
        raw = _prompt_inputs(case, seed)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed) + 1)
        for side in "kv":
            state["s_" + side] = raw["s_" + side][:, d["s"]:].contiguous()
            state["bases_" + side] = _orthonormal(gen, case["batch"], d["Dp"], case["rank"],
                                                  d["rs"])[:, None].to(torch.bfloat16).contiguous()
            state["coef_" + side] = torch.zeros((case["batch"], d["cap"], d["R"]), dtype=torch.bfloat16, device="cuda")
        return state
    state.update(_decode_inputs(case, seed))
    if case["kind"] == "windowed":
        state["state"] = s4r.alloc_window_state(cfg)
        s4r.window_state_init(cfg, case["length"], state["qwin_prev"], state["coef_k"], state["state"], state["ws"])
    if case["kind"] == "ragged":
        state["lengths"] = _lengths(case)
    return state


# ---------------------------------------------------------------------------
# the pass
# ---------------------------------------------------------------------------

def run(st):
    case, cfg, length, kind = st["case"], st["cfg"], st["case"]["length"], st["case"]["kind"]
    if kind == "project":
        s4r.prefill_project(cfg, length, st["s_k"], st["s_v"], st["bases_k"], st["bases_v"], st["coef_k"],
                            st["coef_v"], st["ws"])
        return {"coef_k": st["coef_k"], "coef_v": st["coef_v"]}
    if kind == "first_token":
        kv = s4r.prefill(cfg, st["s_k"], st["s_v"], ws=st["ws"])
        older = s4r.project_queries(cfg, st["q_prev"], kv["bases_k"], st["ws"])
        window = s4r.alloc_window_state(cfg)
        s4r.window_state_init(cfg, length, older, kv["coef_k"], window, st["ws"])
        scores = torch.empty((case["batch"], length), dtype=torch.float32, device=older.device)
        # the bases' signs are arbitrary, so the coefficients are judged by what is decoded from them
        out = s4r.decode_step_windowed(cfg, length, st["q"], window, kv["sink_k"], kv["sink_v"], kv["bases_k"],
                                       kv["bases_v"], kv["coef_k"], kv["coef_v"], st["ws"], k_new=st["k_new"],
                                       v_new=st["v_new"], scores_out=scores)
        return {"out": out, "scores": scores}
    if kind == "stages":
        scores = s4r.score_latent(cfg, length, st["q"], st["bases_k"], st["coef_k"], st["ws"],
                                  qwin_prev=st.get("qwin_prev"))
        idx = s4r.select_topk(cfg, length, scores, st["ws"])
        k_hat, v_hat = s4r.reconstruct(cfg, length, idx, st["bases_k"], st["bases_v"], st["coef_k"], st["coef_v"])
        out = s4r.sparse_attn(cfg, length, st["q"], st["sink_k"], st["sink_v"], idx, k_hat, v_hat, st["ws"])
        return {"scores": scores, "idx": idx, "k_hat": k_hat, "v_hat": v_hat, "out": out}
    args = (st["sink_k"], st["sink_v"], st["bases_k"], st["bases_v"], st["coef_k"], st["coef_v"], st["ws"])
    new = {"k_new": st["k_new"], "v_new": st["v_new"]} if case["append"] else {}
    if kind == "windowed":
        out = s4r.decode_step_windowed(cfg, length, st["q"], st["state"], *args, **new)
    elif kind == "ragged":
        out = s4r.decode_step_ragged(cfg, st["lengths"], st["q"], *args, qwin_prev=st.get("qwin_prev"), **new)
    else:
        out = s4r.decode_step(cfg, length, st["q"], *args, qwin_prev=st.get("qwin_prev"), **new)
    if case["append"]:
        return {"out": out, "coef_k": st["coef_k"], "coef_v": st["coef_v"]}
    return {"out": out}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    d = _dims(case)
    B, es = case["batch"], d["es"]
    bases = B * d["Dp"] * (d["rs"] + d["rvs"]) * es

    def step(length, rows):
        """One sequence's step with `rows` query rows scored: C^K once, the selected rows of C^V, sinks, query, output."""
        m = _selected(case, length)
        n_bytes = (length * d["R"] + m * d["Rv"] + 2 * d["s"] * d["Dp"] + d["hq"] * d["dh"]) * es + d["hq"] * d["dh"] * 4
        n_flops = 2.0 * length * d["R"] * d["G"] * rows + 2.0 * d["hq"] * d["dh"] * d["R"]
        n_flops += 2.0 * m * d["Dp"] * (d["rs"] + d["rvs"]) + 4.0 * (m + d["s"]) * d["hq"] * d["dh"]
        if case["append"]:
            n_bytes += (2 * d["Dp"] + d["R"] + d["Rv"]) * es
            n_flops += 2.0 * d["Dp"] * (d["rs"] + d["rvs"])
        if rows > 1:
            n_bytes += d["G"] * (rows - 1) * d["R"] * 4
        return n_bytes, n_flops

    def project(n):
        return (B * n * (2 * d["Dp"] + d["R"] + d["Rv"]) * es + bases, 2.0 * B * n * d["Dp"] * (d["rs"] + d["rvs"]))

    if case["kind"] == "project":
        n_bytes, n_flops = project(case["length"])
        return {"bytes": n_bytes, "flops": n_flops}
    if case["kind"] == "first_token":
        n = case["length"] - 1
        n_bytes, n_flops = project(n)
        sampled = int(s4r.num_samples(n, 0.2))
        # Gram matrices of the sample (half of each), their eigenvectors at the rank's share of a full reduction
        n_flops += 2 * B * (1.0 * sampled * d["Dp"] ** 2 + 4.0 / 3.0 * d["Dp"] ** 3 + 4.0 * d["Dp"] ** 2 * d["rs"])
        b1, f1 = step(case["length"], case["q_window"])
        return {"bytes": n_bytes + bases + B * b1, "flops": n_flops + B * f1}
    rows = 1 if case["kind"] == "windowed" else case["q_window"]
    n_bytes, n_flops = bases, 0.0
    for length in _lengths(case) if case["kind"] == "ragged" else [case["length"]] * B:
        b1, f1 = step(length, rows)
        n_bytes, n_flops = n_bytes + b1, n_flops + f1
    if case["kind"] == "windowed":
        # the newest row's softmax stored, the older rows' sum read
        n_bytes += B * case["length"] * d["G"] * 8
    if case["kind"] == "stages":
        m = _selected(case, case["length"])
        # scores and indices written, the selected rows written out in fp32
        n_bytes += B * (case["length"] * 4 + m * 4 + 2 * m * d["Dp"] * 4)
    return {"bytes": n_bytes, "flops": n_flops}


def tolerance(case):
    if case["kind"] == "project":
        return {"rel": 5e-4, "max": 0.05}       # sums rounded once to bf16: a few values one step apart
    if case["kind"] == "stages" or case["dtype"] == "fp32":
        # fp32 results of exactly read inputs (off by 1e-7 to 8e-7 from 64 bits)
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.01}
    if case["kind"] == "first_token":
        # a rounding of a basis or coefficient entry may fall the other way (off by 2e-5 from 64 bits)
        return {"rel": 1e-3, "max": 0.1}
    # reconstructed values and weights rounded once to bf16 (off by 1e-3 to 2e-3 from 64 bits)
    return {"rel": 8e-3, "max": 0.1}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _rope(x, pos, theta):
    """x [n, heads, d_h] at positions pos [n], rotate-half."""
    half = x.shape[-1] // 2
    freq = float(theta) ** (-torch.arange(half, dtype=torch.float64, device=x.device) * 2.0 / x.shape[-1])
    ang = pos.to(torch.float64)[:, None, None] * freq
    c, s = torch.cos(ang), torch.sin(ang)
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)


def _by_group(x, bases):
    """x [n, Dp] times one sequence's bases [nb, Dg, stride]: [n, nb * stride]."""
    nb, dg, rs = bases.shape
    return torch.cat([torch.mm(x[:, g * dg:(g + 1) * dg], bases[g]) for g in range(nb)], dim=1)


def _rebuild(rows, bases):
    nb, dg, rs = bases.shape
    return torch.cat([torch.mm(rows[:, g * rs:(g + 1) * rs], bases[g].t()) for g in range(nb)], dim=1)


def _exact_sequence(case, d, length, q, older, sink_k, sink_v, bk, bv, ck, cv):
    """One sequence's step from fp64 rows ck / cv [>= length, R]: scores, indices, rows, output."""
    groups = q.reshape(d["hkv"], d["G"], d["dh"]).transpose(0, 1).reshape(d["G"], d["Dp"])
    cq = _by_group(groups, bk)[:, None]
    if older is not None:
        cq = torch.cat([older, cq], dim=1)
    n_rows = cq.shape[1]
    keys = torch.arange(length, device=q.device)
    prob = torch.zeros((d["G"], length), dtype=torch.float64, device=q.device)
    for i in range(n_rows):
        z = torch.mm(cq[:, i], ck[:length].t()) / math.sqrt(case["rank"] * case["groups"])
        z = z.masked_fill(keys[None] > length - n_rows + i, -math.inf)
        prob += torch.softmax(z, dim=1)
    prob /= n_rows
    kap = case["pool_kernel"]
    if case["pool_mode"] == "max":
        pooled = torch.nn.functional.max_pool1d(prob[None], kap, stride=1, padding=kap // 2)[0]
    else:
        pooled = torch.nn.functional.avg_pool1d(prob[None], kap, stride=1, padding=kap // 2)[0]
    scores = pooled.mean(dim=0) if case["group_agg"] == "mean" else pooled.amax(dim=0)
    n_hist = max(length - case["window"], 0)
    top = torch.sort(scores[:n_hist], descending=True, stable=True).indices[:min(case["topk"], n_hist)]
    idx = torch.cat([torch.sort(top).values, torch.arange(n_hist, length, device=q.device)])
    k_hat, v_hat = _rebuild(ck[idx], bk), _rebuild(cv[idx], bv)
    pos = torch.cat([torch.arange(d["s"], device=q.device), idx + d["s"]])
    keys_all = _rope(torch.cat([sink_k, k_hat]).reshape(-1, d["hkv"], d["dh"]), pos, d["theta"])
    vals = torch.cat([sink_v, v_hat]).reshape(-1, d["hkv"], d["dh"])
    at = torch.full((1,), d["s"] + length - 1, device=q.device)
    qr = _rope(q[None], at, d["theta"])[0].reshape(d["hkv"], d["G"], d["dh"])
    logits = torch.bmm(qr, keys_all.permute(1, 2, 0).contiguous()) / math.sqrt(d["dh"])
    out = torch.bmm(torch.softmax(logits, dim=-1), vals.transpose(0, 1).contiguous()).reshape(d["hq"], d["dh"])
    return {"scores": scores, "idx": idx, "k_hat": k_hat, "v_hat": v_hat, "out": out}


def _exact_step(case, d, st):
    """All sequences' steps from a prepared state; also the caches with the appended rows (fp64, tiled)."""
    lengths = _lengths(case) if case["kind"] == "ragged" else [case["length"]] * case["batch"]
    got = []
    caches = {"coef_k": [], "coef_v": []}
    for b, length in enumerate(lengths):
        bk, bv = st["bases_k"][b].double(), st["bases_v"][b].double()
        ck, cv = _untile(st["coef_k"][b:b + 1])[0].double(), _untile(st["coef_v"][b:b + 1])[0].double()
        if case["append"]:
            for c, new, basis in ((ck, st["k_new"], bk), (cv, st["v_new"], bv)):
                c[length - 1] = _by_group(new[b:b + 1].double(), basis)[0].to(st["coef_k"].dtype).double()
            caches["coef_k"].append(_tile(ck[None]))
            caches["coef_v"].append(_tile(cv[None]))
        older = st["qwin_prev"][b].double() if st.get("qwin_prev") is not None else None
        got.append(_exact_sequence(case, d, length, st["q"][b].double(), older, st["sink_k"][b].double(),
                                   st["sink_v"][b].double(), bk, bv, ck, cv))
    want = {k: torch.stack([g[k] for g in got]) for k in (got[0] if case["kind"] != "ragged" else ["out"])}
    if case["append"]:
        want.update({k: torch.cat(v) for k, v in caches.items()})
    return want


def _exact_bases(rows, rank, stride, eta=0.2):
    """The `rank` leading right singular vectors of the sampled, normalised rows [n, Dp], in storage precision."""
    n = rows.shape[0]
    total = max(1, int(math.floor(eta * n)))
    recent = int(round(0.7 * total))
    early = total - recent
    at = torch.arange(n - recent, n)
    if early:
        spread = torch.linspace(0, n - recent - 1, early, dtype=torch.float64)
        at = torch.cat([torch.round(spread).long(), at])
    x = rows[at.to(rows.device)].double()
    x = x / x.norm(dim=1, keepdim=True)
    vec = torch.linalg.eigh(torch.mm(x.t(), x).cpu()).eigenvectors.flip(1)[:, :rank]
    out = torch.zeros((1, rows.shape[1], stride), dtype=torch.float64, device=rows.device)
    out[0, :, :rank] = vec.to(torch.bfloat16).double().to(rows.device)
    return out


def exact(case, seed):
    d = _dims(case)
    if case["kind"] == "project":
        st = prepare(case, seed)
        want = {}
        for side in "kv":
            full = torch.zeros((case["batch"], d["cap"], d["R"]), dtype=torch.float64, device="cuda")
            for b in range(case["batch"]):
                full[b, :case["length"]] = torch.mm(st["s_" + side][b].double(), st["bases_" + side][b, 0].double())
            want["coef_" + side] = _tile(full)
        return want
    if case["kind"] == "first_token":
        raw = _prompt_inputs(case, seed)
        n, got = case["length"] - 1, []
        for b in range(case["batch"]):
            rows = {side: raw["s_" + side][b] for side in "kv"}
            bases = {side: _exact_bases(rows[side][d["s"]:], case["rank"], d["rs"]) for side in "kv"}
            cache = {}
            for side in "kv":
                x = torch.cat([rows[side][d["s"]:].double(), raw[side + "_new"][b:b + 1].double()])
                cache[side] = _by_group(x, bases[side]).to(torch.bfloat16).double()
            q = raw["q_rows"][b].double()
            prev = q[:-1].reshape(-1, d["hkv"], d["G"], d["dh"]).transpose(1, 2).reshape(-1, d["Dp"])
            older = _by_group(prev, bases["k"]).reshape(-1, d["G"], d["R"]).transpose(0, 1)
            got.append(_exact_sequence(case, d, n + 1, q[-1], older, rows["k"][:d["s"]].double(),
                                       rows["v"][:d["s"]].double(), bases["k"], bases["v"], cache["k"], cache["v"]))
        return {k: torch.stack([g[k] for g in got]) for k in ("out", "scores")}
    want = _exact_step(case, d, prepare(case, seed))
    if case["kind"] == "stages":
        return {k: want[k] for k in ("scores", "idx", "k_hat", "v_hat", "out")}
    return {k: v for k, v in want.items() if k in ("out", "coef_k", "coef_v")}
