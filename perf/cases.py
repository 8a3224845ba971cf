"""The work that is timed and compared: calls a decode loop makes through the library's public entry points.

A case is a dict of plain values.  `op` names the calls of one pass:
  round   one decode round as one call (Tapout.round); truncate: only the tokens up to the stop position are verified
          (Algorithm 1 as written), else all k_len drafted tokens
  calls   one decode round as four calls (bandit_select, draft_stats, verify, bandit_update)
  draft   draft_stats that also draws the draft tokens (u_draft): one step of the draft loop (K = 1) or a drafted block
  shard   one GPU's share of a round with a tensor-parallel lm_head of G shards: shard_stats and draft_stats_sharded on the
          draft side, shard_stats, verify_accept_sharded, shard_final_sums and shard_final_token on the target side (the
          records and sums of the other shards are in hand, as after an all-gather)

Inputs are the synthetic logits of paper_2511_02017_amd.synth, whose laws stand for a diffuse model ("normal"), rows that are
peaked or flat ("regime") and Zipf-like next-token distributions ("zipf").
"""
import math

import torch

from paper_2511_02017_amd import binding, synth

DEV = "cuda" if torch.cuda.is_available() else "cpu"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
ESZ = {"f32": 4, "bf16": 2}
THREE = ((binding.RULE_SVIP, 0.6), (binding.RULE_MAXCONF, 0.8), (binding.RULE_MARGIN, 0.2))
FIVE = THREE + ((binding.RULE_SVIP_DIFF, 0.2), (binding.RULE_ADAEDL, 0.4))
ADAEDL_GAMMA = 0.5
LAWS = {"normal": dict(sigma_draft=2.0, sigma_target=(1.0, 1.0)), "regime": dict(sigma_draft=3.0, sigma_target=(1.2, 1.2)),
        "zipf": dict(sigma_draft=0.3, sigma_target=(0.6, 0.6))}
POLICY = {"ucb1": binding.UCB1, "ucb_tuned": binding.UCB_TUNED, "ts": binding.TS_BETA}


def _case(op, V, B, K, draft, target, law, **kw):
    c = dict(op=op, V=V, B=B, K=K, draft=draft, target=target, law=law, policy="ucb1", arms=3, truncate=False, ragged=False,
             token_level=False, G=1)
    c.update(kw)
    return c


def listed():
    return [
        # one user, a small vocabulary, binary32 logits, Algorithm 1 as written: the smallest call there is
        dict(_case("round", 32000, 1, 5, "f32", "f32", "normal", truncate=True), name="one_32k_alg1"),
        # one user at a 128k vocabulary with the paper's pool of five stop rules (the paper's own setting is batch 1)
        dict(_case("round", 128256, 1, 8, "bf16", "bf16", "regime", arms=5, truncate=True), name="one_128k_five_alg1"),
        # a small batch at a small vocabulary, every drafted token verified
        dict(_case("round", 32000, 32, 8, "bf16", "bf16", "normal"), name="small_round"),
        # the headline workload: a serving batch at a 128k vocabulary
        dict(_case("round", 128256, 64, 8, "bf16", "bf16", "regime"), name="batch_128k_round"),
        # the same batch, verifying only up to the stop position
        dict(_case("round", 128256, 64, 8, "bf16", "bf16", "regime", truncate=True), name="batch_128k_alg1"),
        # the same batch with the five-rule pool (two rules carry state from draft to draft) and UCB-Tuned
        dict(_case("round", 128256, 64, 8, "bf16", "bf16", "regime", arms=5, policy="ucb_tuned"), name="batch_128k_five"),
        # a large batch, long drafts, Zipf-like rows, Thompson Sampling
        dict(_case("round", 151936, 256, 16, "bf16", "bf16", "zipf", policy="ts"), name="large_zipf_ts"),
        # the largest: ragged draft lengths, a quarter of the sequences greedy, binary32 target logits
        dict(_case("round", 256000, 512, 16, "bf16", "f32", "normal", ragged=True), name="largest_ragged"),
        # one step of the draft loop for a serving batch: signals, stop decision and the sampled token of one row each
        dict(_case("draft", 128256, 64, 1, "bf16", "bf16", "regime"), name="draft_step_sampled"),
        # a drafted block (all K rows at hand, as a parallel-drafting head gives them), tokens sampled by the library
        dict(_case("draft", 128256, 64, 8, "bf16", "bf16", "regime"), name="draft_block_sampled"),
        # a vocabulary of odd size (rows start at every alignment), four calls, one bandit per draft position
        dict(_case("calls", 50257, 48, 7, "bf16", "f32", "normal", policy="ts", token_level=True), name="odd_vocab_token_level"),
        # one of eight vocabulary shards of the serving batch
        dict(_case("shard", 128256, 64, 8, "bf16", "bf16", "regime", G=8), name="shard_of_eight"),
    ]


def draw(rng):
    while True:
        V = int(round(math.exp(rng.uniform(math.log(8000), math.log(256000)))))
        V += rng.choice((0, 1, -V % 8, -V % 64, -V % 128))
        B = int(round(math.exp(rng.uniform(0.0, math.log(512)))))
        K = rng.randint(1, 16)
        draft = rng.choice(("bf16", "bf16", "f32"))
        target = rng.choice((draft, draft, "f32"))
        op = rng.choice(("round", "round", "round", "calls", "draft", "shard"))
        if V * B * ((K * ESZ[draft] + (K + 1) * ESZ[target])) <= 3e9:
            break
    return _case(op, V, B, 1 if op == "draft" and rng.random() < 0.5 else K, draft, target, rng.choice(("normal", "regime", "zipf")),
                 policy=rng.choice(("ucb1", "ucb_tuned", "ts")), arms=rng.choice((3, 3, 5)), truncate=rng.random() < 0.4,
                 ragged=rng.random() < 0.3, token_level=op == "calls" and rng.random() < 0.5, G=rng.choice((2, 4, 8)) if op == "shard" else 1)


def _arms(c):
    return FIVE if c["arms"] == 5 else THREE


def _inputs(c, seed):
    """Logits, tokens, uniforms, lengths and this round's arms."""
    K = c["K"]
    w = synth.Workload("case", 100 + seed, c["V"], c["B"], K, DTYPES[c["draft"]], DTYPES[c["target"]], c["law"], rounds=1,
                       policy="ucb1", n_arms=c["arms"], **LAWS[c["law"]])
    gen = synth.RoundGenerator(w, DEV, chunk_rows=512)
    g = torch.Generator(device=DEV)
    g.manual_seed(977 * seed + 5)
    if c["ragged"]:
        gen.k_len = torch.randint(max(1, K // 4), K + 1, (c["B"],), generator=g, device=DEV, dtype=torch.int32)
        gen.greedy = (torch.rand(c["B"], generator=g, device=DEV) < 0.25).to(torch.uint8)
    rnd = gen.round(seed)
    P = K if c["token_level"] else 1
    shape = (c["B"],) if P == 1 else (c["B"], P)
    arm = torch.randint(0, c["arms"], shape, generator=g, device=DEV, dtype=torch.int32)
    u_ts = torch.rand((*shape, c["arms"], synth.TS_UNIFORMS_PER_ARM), generator=g, device=DEV, dtype=torch.float32)
    u_draft = torch.rand(c["B"], K, generator=g, device=DEV, dtype=torch.float32)
    return rnd, arm, u_ts, u_draft


def _bounds(c):
    return [c["V"] * g // c["G"] for g in range(c["G"] + 1)]


def prepare(case, seed):
    c = case
    B, K, V = c["B"], c["K"], c["V"]
    rnd, arm, u_ts, u_draft = _inputs(c, seed)
    rules, thresholds = zip(*_arms(c))
    tp = binding.Tapout(B, K, V, policy=POLICY[c["policy"]], rules=rules, thresholds=thresholds, token_level=c["token_level"],
                        draft_sampling=c["op"] == "draft")
    s = dict(case=c, tp=tp, rnd=rnd, arm=arm, u_ts=u_ts, u_draft=u_draft)
    if c["op"] == "round":
        s["args"], outs = tp.round_args(rnd, arm, c["truncate"], u_ts_next=u_ts if c["policy"] == "ts" else None)
        s["out"] = dict(arm=arm, draft=outs["draft"], verify=outs["verify"], select_flags=outs["select_flags"])
    elif c["op"] == "calls":
        s["draft"], s["verify"] = tp.alloc_draft_outputs(B, K), tp.alloc_verify_outputs(B, K)
    elif c["op"] == "draft":
        s["draft"] = tp.alloc_draft_outputs(B, K)
        s["draft"]["sampled_tok"] = torch.full((B, K), -1, dtype=torch.int32, device=DEV)
        rnd["target"] = None
    else:
        # the middle shard is this GPU's; the others' records and sums come from the same calls on their columns
        at, G = _bounds(c), c["G"]
        mine = G // 2
        cut = lambda t, g: t[:, :, at[g]:at[g + 1]].contiguous()  # noqa: E731
        s.update(at=at, mine=mine, shard_draft=cut(rnd["draft"], mine), shard_target=cut(rnd["target"], mine))
        dst = torch.zeros((G, B * K, 8), dtype=torch.int32, device=DEV)
        tst = torch.zeros((G, B * (K + 1), 8), dtype=torch.int32, device=DEV)
        for g in range(G):
            tp.shard_stats(cut(rnd["draft"], g), at[g], rnd["k_len"], 0, rnd["draft_tok"], out=dst[g])
            tp.shard_stats(cut(rnd["target"], g), at[g], rnd["k_len"], 1, rnd["draft_tok"], out=tst[g])
        do = tp.draft_stats_sharded(dst, B, K, V, draft_tok=rnd["draft_tok"], k_len=rnd["k_len"], arm=arm)
        vo = tp.verify_accept_sharded(tst, B, K, V, do["logq_tok"], rnd["draft_tok"], rnd["k_len"], rnd["u_accept"],
                                      greedy=rnd["greedy"], draft_lse=do["lse"])
        s["sums_all"] = torch.stack([tp.shard_final_sums(cut(rnd["target"], g), cut(rnd["draft"], g), vo["final_jobs"]) for g in range(G)])
        rnd["draft"] = rnd["target"] = None
        s.update(dst=dst, tst=tst, draft=tp.alloc_draft_outputs(B, K), verify=tp.alloc_verify_outputs(B, K))
    return s


def run(state):
    s, c, tp, rnd = state, state["case"], state["tp"], state["rnd"]
    if c["op"] == "round":
        tp.round(s["args"])
        return s["out"]
    if c["op"] == "calls":
        arm = tp.bandit_select(c["B"], u_ts=s["u_ts"] if c["policy"] == "ts" else None, arm_out=s["arm"])
        do = tp.draft_stats(rnd["draft"], rnd["draft_tok"], rnd["k_len"], arm, out=s["draft"])
        n = do["n_stop"] if c["truncate"] else rnd["k_len"]
        vo = tp.verify(rnd["target"], rnd["draft"], do["lse"], do["logq_tok"], rnd["draft_tok"], n, rnd["u_accept"], rnd["u_sample"],
                       greedy=rnd["greedy"], out=s["verify"])
        tp.bandit_update(arm, vo["accept_len"], n, rnd["k_len"])
        return dict(arm=arm, draft=do, verify=vo)
    if c["op"] == "draft":
        return tp.draft_stats(rnd["draft"], None, rnd["k_len"], s["arm"], u_draft=s["u_draft"], out=s["draft"])
    B, K, V, g, at = c["B"], c["K"], c["V"], s["mine"], s["at"]
    tok, n = rnd["draft_tok"], rnd["k_len"]
    tp.shard_stats(s["shard_draft"], at[g], n, 0, tok, out=s["dst"][g])
    do = tp.draft_stats_sharded(s["dst"], B, K, V, draft_tok=tok, k_len=n, arm=s["arm"], out=s["draft"])
    tp.shard_stats(s["shard_target"], at[g], n, 1, tok, out=s["tst"][g])
    vo = tp.verify_accept_sharded(s["tst"], B, K, V, do["logq_tok"], tok, n, rnd["u_accept"], greedy=rnd["greedy"],
                                  draft_lse=do["lse"], out=s["verify"])
    sums = tp.shard_final_sums(s["shard_target"], s["shard_draft"], vo["final_jobs"])
    s["sums_all"][g].copy_(sums)
    token, _, _ = tp.shard_final_token(s["shard_target"], s["shard_draft"], at[g], c["G"], g, vo["final_jobs"], s["sums_all"], rnd["u_sample"])
    return dict(draft=do, verify={k: v for k, v in vo.items() if k != "final_jobs"}, sums=sums, token=token)


def work(case):
    """Live logits once.  Truncated rounds verify at least one token: two target rows.  Ragged lengths by their mean."""
    c = case
    V = c["V"] / c["G"]
    rows = c["B"] * ((max(1, c["K"] // 4) + c["K"]) / 2 if c["ragged"] else c["K"])
    t_rows = 0 if c["op"] == "draft" else c["B"] * 2 if c["truncate"] and c["op"] != "shard" else rows + c["B"]
    pair = rows if c["op"] == "draft" else c["B"]              # rows that an inverse CDF runs over
    return {"bytes": V * (rows * ESZ[c["draft"]] + t_rows * ESZ[c["target"]]), "flops": V * (6.0 * rows + 4.0 * t_rows + 10.0 * pair)}


def tolerance(case):
    # Binary32 sums over up to 256000 terms: 2e-8 to 1e-7 against double is what they show.  Integers differ only where a
    # uniform lies that close to a decision.
    return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}


def _stats(x, tok):
    """The signals of logits rows [n, V] in double."""
    x = x.double()
    lse = torch.logsumexp(x, -1)
    lp = x - lse[:, None]
    p = lp.exp()
    H = -torch.where(p > 0, p * lp, torch.zeros_like(p)).sum(-1)
    top = p.topk(2, -1).values
    lq = lp.gather(1, tok[:, None].long())[:, 0]
    return lse, H, top[:, 0], top[:, 1], top[:, 0] - top[:, 1], lq


def _draw_token(x, u):
    """Inverse CDF of softmax(x) at u, per row of [n, V], in double."""
    x = x.double()
    cum = torch.cumsum((x - x.max(-1, keepdim=True).values).exp(), -1)
    return torch.searchsorted(cum, (u.double() * cum[:, -1])[:, None], right=True)[:, 0].clamp_(max=x.shape[1] - 1)


def _n_stop(c, arm, k_len, H, p1, margin):
    """First firing position + 1 under Table 1's rules, no earlier draft; [B]."""
    B, K = H.shape
    rH = H.clamp(min=0).sqrt()
    prev = torch.cat([torch.full((B, 1), math.inf, dtype=H.dtype, device=H.device), rH[:, :-1]], 1)
    signal = {binding.RULE_SVIP: lambda h: rH > h, binding.RULE_MAXCONF: lambda h: p1 < h, binding.RULE_MARGIN: lambda h: margin < h,
              binding.RULE_SVIP_DIFF: lambda h: rH - prev > h, binding.RULE_ADAEDL: lambda h: 1 - (ADAEDL_GAMMA * H).sqrt() < h}
    f = lambda h: float(torch.tensor(h, dtype=torch.float32))  # noqa: E731
    fires = torch.stack([signal[r](f(h)) for r, h in _arms(c)], 0)[arm.long(), torch.arange(B, device=H.device)]
    k = torch.arange(K, device=H.device)[None]
    first = torch.where(fires & (k < k_len[:, None]), k + 1, torch.full_like(k, K + 1)).amin(1)
    return torch.minimum(first, k_len.long())


def exact(case, seed):
    c = case
    B, K, V = c["B"], c["K"], c["V"]
    rnd, arm, u_ts, u_draft = _inputs(c, seed)
    nan = lambda k: torch.full((B, k), math.nan, dtype=torch.float64, device=DEV)  # noqa: E731
    names = ("lse", "entropy", "p_top1", "p_top2", "margin", "logq_tok")
    d = {n: nan(K) for n in names}
    step = max(1, int(3e8 // ((K + 1) * V)))
    k = torch.arange(K + 1, device=DEV)[None]
    k_len = rnd["k_len"]
    for b in range(0, B, step):
        live = (k[:, :K] < k_len[b:b + step, None]).reshape(-1)
        x = rnd["draft"][b:b + step].reshape(-1, V)[live]
        tok = rnd["draft_tok"][b:b + step].reshape(-1)[live]
        if c["op"] == "draft":
            tok = _draw_token(x, u_draft[b:b + step].reshape(-1)[live])
        for n, v in zip(names, _stats(x, tok)):
            d[n][b:b + step].view(-1)[live] = v
    draft = dict(d, top1_id=None, n_stop=None, stop_fired=None, flags=None)
    if c["op"] == "draft":
        return dict(draft, sampled_tok=None)
    if c["op"] == "calls" and c["truncate"]:
        t_lse = lp = None                                     # the arms are the library's own draw
    else:
        n = _n_stop(c, arm, k_len, d["entropy"], d["p_top1"], d["margin"]) if c["truncate"] and c["op"] == "round" else k_len.long()
        t_lse, lp = nan(K + 1), nan(K)
        for b in range(0, B, step):
            live = (k <= n[b:b + step, None]).reshape(-1)
            x = rnd["target"][b:b + step].reshape(-1, V)[live].double()
            tok = torch.cat([rnd["draft_tok"][b:b + step], rnd["draft_tok"][b:b + step, :1] * 0], 1).reshape(-1)[live]
            v = torch.logsumexp(x, -1)
            both = torch.full((live.numel(), 2), math.nan, dtype=torch.float64, device=DEV)
            both[live] = torch.stack([v, x.gather(1, tok[:, None].long())[:, 0] - v], 1)
            both = both.view(-1, K + 1, 2)
            t_lse[b:b + step] = both[..., 0]
            has = k[:, :K] < n[b:b + step, None]
            lp[b:b + step] = torch.where(has, both[:, :K, 1], lp[b:b + step])
    verify = dict(accept_len=None, out_tok=None, n_out=None, target_lse=t_lse, logp_tok=lp, target_top1=None, flags=None)
    if c["op"] == "shard":
        return dict(draft=draft, verify=verify, sums=None, token=None)
    return dict(arm=None, draft=draft, verify=verify) if c["op"] == "calls" else dict(arm=None, draft=draft, verify=verify, select_flags=None)
