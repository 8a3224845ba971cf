"""The rules by which the library picks a launch shape or a kernel from sizes, types and alignment, at the sizes where each
rule turns, against the CPU oracle.  Tolerances are parity_util's."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2511_02017_amd import binding
from tests import parity_util as pu
from tests.test_gpu_parity import force_slices, random_arms, random_round, sharded_round

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def mixed_round(B, K, V, dt, tt, seed, **kw):
    rnd = random_round(B, K, V, torch.float32 if dt == tt == torch.float32 else torch.bfloat16, seed=seed, **kw)
    rnd["draft"], rnd["target"] = rnd["draft"].to(dt), rnd["target"].to(tt)
    return rnd


f32, bf16 = torch.float32, torch.bfloat16


@pytest.mark.parametrize("B,K,V,dt,tt", [
    (3, 2, 8192, bf16, bf16),        # one batch of 16 KB exactly: one slice
    (3, 2, 8193, bf16, bf16),        # one element more: still one, rows at every alignment
    (3, 2, 8199, bf16, bf16),        # no whole vector more: still one
    (3, 2, 8200, bf16, bf16),        # one vector more: two slices
    (2, 3, 8199, bf16, f32),         # two and a bit batches of binary32 rows beside one of bfloat16 rows
    (2, 3, 4096, f32, f32),
    (2, 3, 4101, f32, bf16),
    (1, 8, 131072, bf16, bf16),      # sixteen batches: as many slices as are merged across lanes
    (1, 8, 131080, bf16, bf16),      # one vector more: two batches per slice
    (1, 31, 70001, bf16, bf16),      # 32 target rows of nine slices in groups of sixteen lanes: the largest such shape
    (1, 32, 70001, bf16, bf16),      # 33 target rows: groups of eight lanes
    (1, 64, 40003, f32, f32),        # 65 target rows: the staged merge, as many slices as there are batches
    (300, 2, 12289, bf16, bf16),     # 1500 rows of both tensors together: a batch and a half
    (50, 5, 4100, f32, f32),         # a batch of binary32 and one vector: two slices for 250 draft rows, one for 300 target rows
    (55, 5, 5000, f32, bf16),
    (2, 33, 17000, f32, f32),        # four batches and a bit: three slices, not five in groups of eight lanes
    (2, 80, 8003, f32, f32),         # staged: one slice of nearly two batches
    (2, 80, 30522, bf16, f32),       # staged: four slices of two batches of binary32 rows, of one of bfloat16 rows
    (16, 70, 9001, bf16, bf16),
])
def test_slices_of_whole_batches(B, K, V, dt, tt):
    rnd = mixed_round(B, K, V, dt, tt, seed=V + K)
    tp = binding.Tapout(B, K, V)
    arm = random_arms(B, seed=K)
    c = [pu.check_round(tp, rnd), pu.check_round(tp, rnd, arm=arm),
         pu.check_round_call(tp, rnd, arm.clone(), truncate=False), pu.check_round_call(tp, rnd, arm.clone(), truncate=True)]
    # near ties: a few per thousand decisions at the tolerance of 1e-5
    assert sum(x["accept_flagged"] + x["icdf_flagged"] + x["stop_flagged"] for x in c) <= 2 + 4 * B * K // 500


@pytest.mark.parametrize("V,dt", [(32000, f32), (9001, bf16)])
def test_round_up_to_the_stop_position_reads_no_target_row_beyond_the_cap(V, dt):
    """Small rounds stream the target rows before the stop position is known: rows 0..k_len of each sequence and no other."""
    B, K = 5, 6
    rnd = mixed_round(B, K, V, dt, dt, seed=V, k_len=[1, 2, 4, 6, 3])
    for b, n in enumerate([1, 2, 4, 6, 3]):
        rnd["target"][b, n + 1:] = float("nan")
    for arm in range(3):
        for thresholds in ((0.6, 0.8, 0.2), (1e9, 0.0, -1.0)):             # the second: no rule fires, every row up to the cap counts
            tp = binding.Tapout(B, K, V, thresholds=thresholds)
            c = pu.check_round_call(tp, rnd, torch.full((B,), arm, dtype=torch.int32, device=DEV), truncate=True, thresholds=thresholds)
            assert c["accept_flagged"] + c["icdf_flagged"] + c["stop_flagged"] <= 1


@pytest.mark.parametrize("policy", [binding.UCB1, binding.UCB_TUNED, binding.TS_BETA, binding.TS_GAUSS])
@pytest.mark.parametrize("max_batch", [1, 3])
@pytest.mark.parametrize("five", [False, True])
def test_one_sequence_of_a_shared_bandit_is_its_own(policy, max_batch, five):
    """With one sequence a shared bandit takes the launches of a bandit of its own: same arms and state as the separate calls."""
    pool = dict(rules=(0, 1, 2, 3, 4), thresholds=(0.6, 0.8, 0.2, 0.2, 0.4)) if five else {}
    a, b = (binding.Tapout(max_batch, 4, 3000, policy=policy, shared_bandit=True, **pool) for _ in range(2))
    g = torch.Generator(device=DEV).manual_seed(1)
    arm_a = arm_b = torch.zeros(1, dtype=torch.int32, device=DEV)
    for t in range(8):
        rnd = mixed_round(1, 4, 3000, bf16, bf16, seed=t)
        u = torch.rand(1, a.cfg.n_arms, 48, generator=g, device=DEV)
        arm_a = arm_a.clone()
        args, out = a.round_args(rnd, arm_a, bool(t & 1), u_ts_next=u)
        a.round(args)
        ds = b.draft_stats(rnd["draft"], rnd["draft_tok"], rnd["k_len"], arm_b)
        n = ds["n_stop"] if t & 1 else rnd["k_len"]
        vf = b.verify(rnd["target"], rnd["draft"], ds["lse"], ds["logq_tok"], rnd["draft_tok"], n, rnd["u_accept"], rnd["u_sample"])
        b.bandit_update(arm_b, vf["accept_len"], n, rnd["k_len"])
        arm_b = b.bandit_select(1, u_ts=u)
        torch.cuda.synchronize()
        assert torch.equal(arm_a, arm_b) and torch.equal(out["verify"]["out_tok"], vf["out_tok"])
        for x, y in zip(a.bandit_get_state(moments=True), b.bandit_get_state(moments=True)):
            assert (x == y).all()
    if five:
        sa, sb = a.rule_state_get(), b.rule_state_get()
        assert all((sa[k][:1] == sb[k][:1]).all() for k in ("accept_rate", "lam"))


@pytest.mark.parametrize("V", [2047, 2049, 2055, 4097, 6150, 8191])
@pytest.mark.parametrize("dt,tt", [(bf16, bf16), (bf16, f32), (f32, f32), (f32, bf16)])
@pytest.mark.parametrize("fuse", [0, 1])
def test_final_token_on_rows_at_every_alignment(V, dt, tt, fuse):
    """Whole 2048-element slices, the last short one and the in-slice search on rows that start at any element."""
    B, K = 9, 3
    rnd = mixed_round(B, K, V, dt, tt, seed=V)
    tp = binding.Tapout(B, K, V)
    tp.set_option("fuse_head", fuse)
    # The first slice, a middle one, the row's last elements.  (Not u = 0: the target is then the edge of the first cell, a
    # near tie by definition in all B sequences; else a cell edge within 1e-9 of the target is a chance of about V 1e-9.)
    for u in (2.0 ** -12, 0.5, 1.0 - 2.0 ** -24):
        rnd["u_sample"] = torch.full((B,), u, device=DEV)
        assert pu.check_round(tp, rnd)["icdf_flagged"] <= 1


@pytest.mark.parametrize("V", [131072, 131073, 262144, 262145])
@pytest.mark.parametrize("dt,tt", [(bf16, bf16), (f32, bf16)])
def test_final_token_of_rows_of_several_slices_per_lane(V, dt, tt):
    """64 and 128 slices fill one and two per lane; one element more makes it two and three, with most lanes' last one empty."""
    B, K = 5, 2
    rnd = mixed_round(B, K, V, dt, tt, seed=V)
    rnd["target"][1, :, :-3] = float("-inf")                    # everything in the last slices: no weight before them
    rnd["draft"][2] = rnd["target"][2, :K].to(dt)               # equal distributions
    tp = binding.Tapout(B, K, V)
    for u in (2.0 ** -12, 0.5, 1.0 - 2.0 ** -24):
        rnd["u_sample"] = torch.full((B,), u, device=DEV)
        assert pu.check_round(tp, rnd)["icdf_flagged"] <= 1


@pytest.mark.parametrize("B,K,V,dt,tt", [
    (64, 6, 32001, bf16, bf16),      # the first two target rows beside the epilogue, the others behind them; rows at every alignment
    (32, 1, 256000, bf16, bf16),     # no others
    (341, 3, 32000, bf16, bf16), (342, 3, 32000, bf16, bf16),    # 3069 and 3078 workgroups
    (20, 16, 40000, bf16, f32),      # 16 rows of five slices in groups of eight: 128 pieces of two lanes, the most
    (20, 17, 40000, bf16, f32),      # 17 rows: too many
    (60, 4, 50257, f32, bf16), (25, 17, 32000, bf16, bf16),      # four lanes a piece; two
    (11, 8, 128256, bf16, bf16), (6, 8, 128256, f32, f32),       # 8 rows of sixteen slices
])
@pytest.mark.parametrize("five", [False, True])
def test_round_up_to_the_stop_position_beyond_the_small_targets(B, K, V, dt, tt, five):
    pool = dict(rules=(0, 1, 2, 3, 4), thresholds=(0.6, 0.8, 0.2, 0.2, 0.4)) if five else dict(rules=(0, 1, 2), thresholds=(0.6, 0.8, 0.2))
    rnd = mixed_round(B, K, V, dt, tt, seed=B + K)
    assert rnd["target"].numel() * rnd["target"].element_size() > 24 << 20
    rnd["draft"][::2] *= 3                                       # peaked rows beside flat ones: stop positions of 1 and more
    tp = binding.Tapout(B, K, V, **pool)
    arm = (torch.arange(B, device=DEV, dtype=torch.int32) % len(pool["rules"])).contiguous()
    if five:
        arm %= 3                                                 # (the stateful rules need a previous draft: played in the test below)
    c = pu.check_round_call(tp, rnd, arm, truncate=True, **pool)
    assert c["icdf_flagged"] <= 1 and c["accept_flagged"] + c["stop_flagged"] <= 2 + 4 * B * K // 500


@pytest.mark.parametrize("dt,tt", [(bf16, bf16), (f32, f32), (bf16, f32)])
def test_round_up_to_the_stop_position_with_stateful_rules(dt, tt):
    """The first two target rows beside the epilogue, with arms whose rules carry state from draft to draft: every output and the state of
    several rounds are the bits of the separate calls, and so are the rounds replayed from HIP graphs with eager work between them."""
    B, K, V = 64, 6, 32001
    pool = dict(rules=(0, 1, 2, 3, 4), thresholds=(0.6, 0.8, 0.2, 0.2, 0.4))
    rounds = []
    for i in range(3):
        rnd = mixed_round(B, K, V, dt, tt, seed=40 + i)
        rnd["draft"][i::2] *= 3                                  # peaked rows beside flat ones
        assert rnd["target"].numel() * rnd["target"].element_size() > 24 << 20
        rounds.append((rnd, torch.where(torch.arange(B, device=DEV) % 5 < 1, i, 3 + (torch.arange(B, device=DEV) + i) % 2).to(torch.int32)))
    order = [0, 1, 2, 2, 1, 0, 1]
    bits = lambda outs: {k: v.cpu().view(torch.int32) if v.dtype == f32 else v.cpu() for o in outs for k, v in o.items()}  # noqa: E731
    named = lambda d, v: ({"d_" + k: x for k, x in d.items()}, {"v_" + k: x for k, x in v.items()})  # noqa: E731
    state = lambda tp: (*(x.tobytes() for x in tp.bandit_get_state(moments=True)), *(tp.rule_state_get()[k].tobytes() for k in ("prev_entropy", "accept_rate", "lam")))  # noqa: E731

    ref, expect = binding.Tapout(B, K, V, **pool), []
    for i in order:
        rnd, arm = rounds[i]
        ds = ref.draft_stats(rnd["draft"], rnd["draft_tok"], rnd["k_len"], arm)
        vf = ref.verify(rnd["target"], rnd["draft"], ds["lse"], ds["logq_tok"], rnd["draft_tok"], ds["n_stop"], rnd["u_accept"], rnd["u_sample"], greedy=rnd["greedy"])
        ref.bandit_update(arm, vf["accept_len"], ds["n_stop"], rnd["k_len"])
        torch.cuda.synchronize()
        expect.append((bits(named(ds, vf)), state(ref)))
    stops = torch.cat([e[0]["d_n_stop"] for e in expect])
    assert (stops < K).any() and (stops > 1).any()

    for graphed in (False, True):
        tp = binding.Tapout(B, K, V, **pool)
        arm = torch.zeros(B, dtype=torch.int32, device=DEV)
        calls = [tp.prepare_round_call(rnd, arm, True) for rnd, _ in rounds]
        fresh = [[(t, t.clone()) for o in (c[1]["draft"], c[1]["verify"]) for t in o.values()] for c in calls]     # (rows behind the stop position stay as they are)
        stream, junk = torch.cuda.Stream(), torch.zeros(1 << 20, device=DEV)
        runs = [lambda c=c: c[0](stream.cuda_stream) for c in calls]
        if graphed:
            graphs = []
            for launch, _ in calls:
                graphs.append(torch.cuda.CUDAGraph())
                with torch.cuda.graph(graphs[-1], stream=stream):
                    launch(torch.cuda.current_stream().cuda_stream)
            runs = [g.replay for g in graphs]
        with torch.cuda.stream(stream):
            for step, i in enumerate(order):
                arm.copy_(rounds[i][1])
                for t, was in fresh[i]:
                    t.copy_(was)
                runs[i]()
                junk.add_(1.0)
                stream.synchronize()
                got = bits(named(calls[i][1]["draft"], calls[i][1]["verify"]))
                for k, v in expect[step][0].items():
                    assert torch.equal(got[k], v), (graphed, step, k)
                assert state(tp) == expect[step][1], (graphed, step)


@pytest.mark.parametrize("dt,vec", [(f32, 4), (bf16, 8)])
@pytest.mark.parametrize("off", [0, 3])
def test_maxima_met_by_several_threads(dt, vec, off):
    """The first maximum, its batch and the second maximum when a value is met twice: inside a vector, by neighbouring threads, by two
    wavefronts, in two batches of a thread, in two slices; and rows with no other finite element."""
    wave, batch = 64 * vec, 1024 * vec
    V = 3 * batch + 5
    pairs = [(0, 1), (vec, 2 * vec), (5, wave + 2), (7, 3 * wave), (6, batch + 6), (vec + 1, 2 * batch + vec), (V - 1, V - 2), (3, 70 * vec)]
    B = len(pairs)
    rnd = mixed_round(B, 2, V + off, dt, dt, seed=off)
    rnd["draft"], rnd["target"] = rnd["draft"][:, :, off:], rnd["target"][:, :, off:]          # rows that start off a vector
    for b, (i, j) in enumerate(pairs):
        for t in (rnd["draft"], rnd["target"]):
            t[b, 0, [i, j]] = 9.0
            t[b, 1] = float("-inf")
            t[b, 1, [i, j]] = torch.tensor([2.0, 2.0 if b & 1 else 1.5], dtype=dt, device=DEV)
        rnd["draft_tok"][b] = torch.tensor([i, j], dtype=torch.int32)
    rnd["u_accept"] = torch.full((B, 2), 0.3, device=DEV)                                      # p / q is about 1 at these tokens: no near tie
    c = pu.check_round(binding.Tapout(B, 2, V), rnd)
    assert c["accept_flagged"] == 0 and c["icdf_flagged"] <= 1


@pytest.mark.parametrize("dt", [f32, bf16])
def test_entropy_is_as_good_as_its_format(dt):
    """Whatever the four wavefronts of a slice add to the entropy's error stays, root mean square over many rows, below what a binary32 result
    may be off by from its own rounding (2^-24 / sqrt(3)); the rounding itself takes 2^-24 / sqrt(3) / 1.75 of that at an entropy near 7."""
    B, K, V = 2048, 2, 8000
    g = torch.Generator(device=DEV).manual_seed(11)
    x = (torch.randn(B, K, V, generator=g, device=DEV) * 2).to(dt)
    H = binding.Tapout(B, K, V).draft_stats(x)["entropy"].double()
    lp = torch.log_softmax(x.double(), -1)
    want = -(lp.exp() * lp).sum(-1)
    assert 6.5 < want.mean() < 7.5
    assert ((H - want) / want).pow(2).mean().sqrt() <= 2.0 ** -24 / 3 ** 0.5


@pytest.mark.parametrize("B,V", [
    (128, 8191), (129, 8191), (320, 8191), (321, 8191),          # four slices a row: four wavefronts share one, two, two, none
    (102, 8200), (103, 8200),                                    # five: the last workgroup of two-way sharing has half its wavefronts idle
    (16, 65536), (17, 65537), (17, 65535), (16, 66001),          # 32 and 33 slices
    (600, 2048), (600, 2049), (700, 4096),                       # one and two slices: shared wherever that adds no workgroup
])
@pytest.mark.parametrize("dt,tt", [(bf16, bf16), (bf16, f32), (f32, f32)])
def test_final_token_with_slices_shared_by_wavefronts(B, V, dt, tt):
    K = 2 if B < 200 else 1
    rnd = mixed_round(B, K, V, dt, tt, seed=B + V)
    rnd["u_sample"][:3] = torch.tensor([2.0 ** -12, 0.5, 1.0 - 2.0 ** -24], device=DEV)
    tp = binding.Tapout(B, K, V)
    for fuse in (0, 1):
        tp.set_option("fuse_head", fuse)
        c = pu.check_round(tp, rnd)
        # near ties: a few per thousand decisions at the tolerance of 1e-5; a cell edge within 1e-9 is a chance of about V 1e-9
        assert c["icdf_flagged"] <= 1 and c["accept_flagged"] + c["stop_flagged"] <= 2 + 4 * B * K // 500


@pytest.mark.parametrize("V", [2047, 2048, 8193, 10240, 133001])
@pytest.mark.parametrize("dt", [f32, bf16])
def test_exact_slice_weights_a_wavefront_per_slice(V, dt):
    """p = q to 1e-5 for every token but four, which hold the residual: the list of undecided elements overflows and all slices
    are weighed again, with fewer slices than wavefronts, one more than a multiple of them, and two or more per lane."""
    B, K = 5, 2
    g = torch.Generator().manual_seed(V)
    d = (torch.randn(B, K, V, generator=g) * 0.5).to(dt)
    tok = torch.randint(0, V, (B, K), generator=g, dtype=torch.int32)
    hot = torch.stack([torch.tensor([0, V // 3, V // 2 + 1, V - 1])] * B)
    for b in range(B):
        tok[b][(tok[b][:, None] == hot[b][None, :]).any(1)] += 2
        d[b, :, tok[b].long()] = -20.0                                    # q of the drafted tokens: below 1e-10
    t = torch.cat([d.float(), torch.randn(B, 1, V, generator=g)], 1)
    for b in range(B):
        t[b, :K, tok[b].long()] = -23.0                                   # p / q = 1 / 20: rejected, u is nearly 1
        t[b, :, hot[b]] += 1e-3                                           # L moves by less than 4e-3 e / V: inside the band of 1e-5
    rnd = dict(draft=d.to(DEV), target=t.to(DEV), draft_tok=tok.to(DEV), u_accept=torch.full((B, K), 1.0 - 2.0 ** -24, device=DEV),
               u_sample=torch.linspace(0.03, 0.97, B).to(DEV), k_len=torch.full((B,), K, dtype=torch.int32, device=DEV),
               greedy=torch.zeros(B, dtype=torch.uint8, device=DEV))
    tp = binding.Tapout(B, K, V)
    c = pu.check_round(tp, rnd)
    assert c["accept_flagged"] == 0 and c["icdf_flagged"] == 0
    _, vf, _ = pu.gpu_round(tp, rnd)
    assert (vf["accept_len"].cpu() == 0).all() and all(int(vf["out_tok"][b, 0]) in hot[b].tolist() for b in range(B))


@pytest.mark.parametrize("policy", [binding.TS_BETA, binding.UCB_TUNED])
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("B,K,A", [(3, 2, 8), (5, 16, 1), (67, 17, 3), (2, 65, 5)])
def test_token_level_bandit_at_the_edges_of_its_workgroups(policy, shared, B, K, A):
    """Sixteen positions per pass of the selection's workgroups, 64 positions per workgroup of the update."""
    tp = binding.Tapout(B, K, 100, policy=policy, shared_bandit=shared, token_level=True, rules=(0,) * A, thresholds=(0.5,) * A)
    ob = orc.Bandit(policy, 1 if shared else B, A, positions=K)
    g = torch.Generator().manual_seed(K)
    for r in range(12):
        u = torch.rand(B, K, A, 48, generator=g)
        if r == 5:
            u[B - 1, K - 1, :, ::3] = 0.0                       # every attempt of the last position's samplers is rejected
        fl = torch.full((B,), 7, dtype=torch.int32, device=DEV)
        arm = tp.bandit_select(B, u_ts=u.to(DEV) if policy == binding.TS_BETA else None, flags=fl)
        o_arm, o_fl = ob.select(B, u.numpy())
        assert (arm.cpu().numpy() == o_arm).all() and (fl.cpu().numpy().astype(np.uint32) == o_fl).all(), f"round {r}"
        n = torch.randint(0, K + 2, (B,), generator=g, dtype=torch.int32).clamp_(max=K)
        m = (torch.rand(B, generator=g) * (n + 1)).floor().clamp(max=n).to(torch.int32)
        gamma = torch.full((B,), K, dtype=torch.int32)
        arm[0, 0] = A if r == 7 else arm[0, 0]                  # an arm out of range is not played
        tp.bandit_update(arm, m.to(DEV), n.to(DEV), gamma.to(DEV))
        ob.update(arm.cpu().numpy(), m.numpy(), n.numpy(), gamma.numpy())
    s, q, c = tp.bandit_get_state(moments=True)
    assert (c == ob.count).all() and (s == ob.sum_r).all() and (q == ob.sum_r2).all()


@pytest.mark.parametrize("B,K,V,dt", [
    (1, 1, 5, bf16),                  # one short slice
    (1, 1, 2048, f32), (1, 3, 2049, bf16),
    (3, 7, 4099, bf16),               # rows at every alignment
    (64, 1, 131072, bf16), (65, 1, 131080, f32), (9, 16, 70001, bf16),       # rows of many slices, one slice to a workgroup's half
    (2047, 1, 3000, bf16), (2048, 1, 3000, bf16), (683, 3, 3000, bf16),      # 2047, 2048 slices: one for every half that is resident; 2049: two
    (1535, 1, 2500, f32), (1536, 1, 2500, f32), (1537, 1, 2500, f32),        # the same of binary32 rows, 1536 workgroups
    (300, 7, 9001, bf16), (150, 16, 20001, bf16),                            # three turns of two slices a row and of three
    (1400, 3, 2500, f32), (700, 3, 9001, f32),
    (1535, 1, 3001, bf16), (1536, 1, 3001, bf16), (1537, 1, 3001, bf16),     # 768 workgroups whose first batch travels with the table, 769 whose doesn't
    (96, 7, 5001, bf16), (110, 6, 5001, bf16),                               # 768 and 770 workgroups with the epilogue's: in one launch, in two
    (96, 7, 5001, f32), (110, 6, 5001, f32),
])
@pytest.mark.parametrize("ragged", [False, True])
def test_draft_token_draw_over_resident_workgroups(B, K, V, dt, ragged):
    """The draft pass of a draw has as many workgroups as are resident, each of which takes a slice (bfloat16: two side by side) and goes on by
    a fixed step to slices of other rows, sequences and positions; the launch behind it carries the epilogue where few rows are drawn."""
    rnd = random_round(B, K, V, dt, seed=V + B)
    tp = binding.Tapout(B, K, V, draft_sampling=True)
    g = torch.Generator().manual_seed(V)
    u = torch.rand(B, K, generator=g)
    k_len = torch.randint(0, K + 1, (B,), generator=g, dtype=torch.int32) if ragged else None
    n = np.full(B, K) if k_len is None else k_len.numpy()
    rnd["draft"][B // 2, K - 1] = float("-inf")                 # a row without a finite maximum: no token
    if dt == bf16 and V > 2048:
        rnd["draft"][0, 0] = 90.0 + (rnd["draft"][0, 0].float() % 3)    # beyond the table of exponentials: computed
        rnd["draft"][0, 0, 7::11] = 1e-6                        # and magnitudes below it
        rnd["draft"][B - 1, 0, 5::13] = 0.0
    out = tp.draft_stats(rnd["draft"], k_len=None if k_len is None else k_len.to(DEV), u_draft=u.to(DEV))
    live = np.arange(K)[None, :] < n[:, None]
    ref = orc.draft_sample(pu.host_logits(rnd["draft"]), u.numpy(), k_len=n.astype(np.int32), nthreads=16)
    tok = out["sampled_tok"].cpu().numpy()
    near = ref["icdf_margin"] <= pu.TAU_S
    assert near[live].sum() <= 2                                # a cell edge within 1e-9 of the target: V 1e-9 per row
    assert (tok[live & ~near] == ref["tok"][live & ~near]).all() and (tok[~live] == -1).all()
    # log q of the token and the flags as for tokens that the caller hands in
    given = tp.draft_stats(rnd["draft"], draft_tok=out["sampled_tok"], k_len=None if k_len is None else k_len.to(DEV))
    a, b = (torch.nan_to_num(x["logq_tok"][torch.from_numpy(live).to(DEV)], nan=7.0) for x in (out, given))
    assert torch.equal(a, b) and torch.equal(out["flags"], given["flags"])


@pytest.mark.parametrize("V,K,off,options", [
    (9001, 2, 0, {}), (9001, 2, 3, {"exp_lookup": 0}),
    (2055, 70, 1, {}), (2055, 80, 1, {}),                                           # 70 rows: the staged epilogue beside the draw; 80: in a launch of its own
    (7, 2, 1, {}), (40000, 2, 0, {"wgs_target": 1, "slice_bytes": 1 << 22}),        # no whole vector in some rows; slices of many batches
    (150001, 1, 5, {"wgs_target": 1, "slice_bytes": 1 << 22}),                      # more than sixteen of them
    (9001, 2, 0, {"min_slice": 256}),                                               # draw slices shorter than their batch
])
@pytest.mark.parametrize("dt", [f32, bf16])
def test_draft_token_draw_at_every_magnitude(V, K, off, options, dt):
    """The sums of the draw are kept in the logits' own scale: inside its range, beyond the table of bfloat16 exponentials, beyond the
    range on either side, and with values too small for the table; every other output as without a draw."""
    g = torch.Generator().manual_seed(V + K)
    moves = [lambda x: x, lambda x: x + 70, lambda x: x - 40, lambda x: x * 40, lambda x: x + 800, lambda x: x - 900, lambda x: x * 1e-4, lambda x: x * 0,
             lambda x: torch.where(x > 0, x * 1e-5, -torch.inf), lambda x: torch.where(x > 3, x + 62, torch.finfo(torch.float32).min)]
    B = len(moves)
    x = torch.randn(B, K, V + off, generator=g) * 2
    x[:, :, off + V // 2] = 4.0
    draft = torch.stack([m(x[b]) for b, m in enumerate(moves)]).to(dt).to(DEV)[:, :, off:]
    u = torch.rand(B, K, generator=g)
    tp = binding.Tapout(B, K, V, draft_sampling=True)
    for name, value in options.items():
        tp.set_option(name, value)
    arm = random_arms(B, seed=V)
    o = tp.draft_stats(draft, arm=arm, u_draft=u.to(DEV))
    osm = orc.draft_sample(pu.host_logits(draft), u.numpy(), nthreads=16)
    tok, near = o["sampled_tok"].cpu().numpy(), osm["icdf_margin"] <= pu.TAU_S
    # cell edges lie 1/V apart: a uniform within 1e-9 of one is a chance of about V 1e-9, more where few tokens hold all the mass
    assert near.sum() <= 1 and (tok[~near] == osm["tok"][~near]).all()
    again = tp.draft_stats(draft, draft_tok=o["sampled_tok"], arm=arm)
    for key in (*pu.STAT_KEYS, "top1_id", "n_stop", "flags"):
        assert torch.equal(o[key], again[key]), key


def _launch_time(tp, kind, call, n=8, groups=6):
    """Milliseconds of n launches of one kernel: the least of several groups (a single launch now and then takes twenty times as long)."""
    took = []
    for _ in range(groups + 1):
        tp.profile_enable((kind,), n)
        for _ in range(n):
            call()
        torch.cuda.synchronize()
        ms, launches = tp.profile_read(kind)
        assert launches == n
        took.append(ms)
    return min(took[1:])


@pytest.mark.parametrize("B,K,V", [(1, 1, 128256), (16, 2, 50257)])
@pytest.mark.parametrize("shift", [-17, -22, -40, -500, 60, 75, 600])
def test_draft_tokens_of_rows_off_the_table_are_found_in_the_draft_pass_sums(B, K, V, shift):
    """Rows of bfloat16 logits that the table of exponentials does not hold: the sums come from the draft pass all the same, and the launch
    that finds the tokens takes what it takes for any row (to sum a row of this size again it took eight times as long)."""
    g = torch.Generator(device=DEV).manual_seed(V + shift)
    x = torch.randn(B, K, V, generator=g, device=DEV) * 2
    x[0, 0, V // 3:] = float("-inf")
    u = torch.rand(B, K, generator=g, device=DEV)
    tp = binding.Tapout(B, K, V, draft_sampling=True)
    took = []
    for d in (x.to(bf16), (x + shift).to(bf16)):
        o = tp.draft_stats(d, u_draft=u)
        ref = orc.draft_sample(pu.host_logits(d), u.cpu().numpy(), nthreads=16)
        near = ref["icdf_margin"] <= pu.TAU_S
        assert near.sum() <= 1 and (o["sampled_tok"].cpu().numpy()[~near] == ref["tok"][~near]).all()
        took.append(_launch_time(tp, "sample_locate", lambda: tp.draft_stats(d, u_draft=u)))
    assert took[1] < 2 * took[0]


def _context_bytes(*a, **kw):
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    tp = binding.Tapout(*a, **kw)
    return tp, free - torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("B,K,V,most", [
    (1, 1, 100, 1 << 20), (64, 8, 128256, 4 << 20), (512, 16, 256000, 96 << 20),
    (65535, 16, 32000, 256 << 20),                              # (8 KB a row would be 8 GB)
])
def test_draft_sampling_takes_little_memory(B, K, V, most):
    """The sums of a draw: 128 bytes for every 16 KB of binary32 logits, a third more at most, up to 256 MB, and 1 MB; a row's lse."""
    a, plain = _context_bytes(B, K, V)
    b, drawing = _context_bytes(B, K, V, draft_sampling=True)
    a.close(), b.close()
    assert drawing - plain <= most + B * K * 8 + (4 << 20)      # (device memory is given out in pieces of up to 2 MB)


@pytest.mark.parametrize("B,K,V,dt", [(48, 8, 40003, bf16), (40, 8, 40000, f32), (13, 70, 40001, bf16), (200, 8, 20000, bf16)])
def test_draft_token_draw_without_room_for_its_sums(B, K, V, dt):
    """Slices so fine that their sums find no room: the tokens are found all the same, from the rows read again, and every other output is the
    one without a draw."""
    rnd = random_round(B, K, V, dt, seed=V)
    rnd["draft"][0, 0] += 80.0
    rnd["draft"][1, 0] = float("-inf")
    g = torch.Generator().manual_seed(V)
    u = torch.rand(B, K, generator=g)
    k_len = torch.randint(0, K + 1, (B,), generator=g, dtype=torch.int32)
    k_len[:2] = K
    tp = binding.Tapout(B, K, V, draft_sampling=True)
    tp.set_option("min_slice", 256)
    tp.set_option("wgs_target", 65536)
    out = tp.draft_stats(rnd["draft"], k_len=k_len.to(DEV), u_draft=u.to(DEV), arm=random_arms(B, seed=1))
    live = np.arange(K)[None, :] < k_len.numpy()[:, None]
    ref = orc.draft_sample(pu.host_logits(rnd["draft"]), u.numpy(), k_len=k_len.numpy(), nthreads=16)
    tok, near = out["sampled_tok"].cpu().numpy(), ref["icdf_margin"] <= pu.TAU_S
    assert near[live].sum() <= 2 and (tok[live & ~near] == ref["tok"][live & ~near]).all() and (tok[~live] == -1).all()
    given = tp.draft_stats(rnd["draft"], draft_tok=out["sampled_tok"], k_len=k_len.to(DEV), arm=random_arms(B, seed=1))
    on = torch.from_numpy(live).to(DEV)
    for key in (*pu.STAT_KEYS, "top1_id"):
        assert torch.equal(torch.nan_to_num(out[key][on].float(), nan=7.0), torch.nan_to_num(given[key][on].float(), nan=7.0)), key
    assert torch.equal(out["n_stop"], given["n_stop"]) and torch.equal(out["flags"], given["flags"])


@pytest.mark.parametrize("B,K,V,dt", [(64, 8, 128256, bf16), (64, 8, 128256, f32), (512, 16, 32000, bf16)])
def test_short_drafts_with_drawn_tokens_take_less_of_the_draft_pass(B, K, V, dt):
    """Where a quarter of the rows is live every compute unit has its share of them: half the time of the full block, at most three quarters
    with what a launch costs by itself.  (All of a workgroup's slices at the same draft position: as long as the full block.)"""
    x = torch.randn(1, K, V, device=DEV).to(dt).expand(B, K, V).contiguous()
    u = torch.rand(B, K, device=DEV)
    tp = binding.Tapout(B, K, V, draft_sampling=True)
    took = []
    for n in (K, K // 4):
        k_len = torch.full((B,), n, dtype=torch.int32, device=DEV)
        took.append(_launch_time(tp, "draft_pass", lambda: tp.draft_stats(x, k_len=k_len, u_draft=u)))
    assert took[1] < 0.75 * took[0]


@pytest.mark.parametrize("G,V", [(1, 3000), (3, 9001), (16, 20000), (17, 20011), (64, 40000), (70, 33000)])
@pytest.mark.parametrize("dt", [f32, bf16])
def test_vocabulary_shards_merged_across_lanes(G, V, dt):
    """Up to sixteen shards the records of a row are merged across lanes, beyond that one after the other; the final token's
    shard is found 64 shards at a time."""
    B, K = 6, 5
    rnd = mixed_round(B, K, V, dt, dt, seed=G)
    rnd["greedy"][1] = 1
    for u in (2.0 ** -12, 0.5, 1.0 - 2.0 ** -24):
        rnd["u_sample"] = torch.full((B,), u, device=DEV)
        acc, out, _ = sharded_round(rnd, G, V)
        _, ref, nd = pu.oracle_round(rnd)
        ok = ~((ref["accept_margin"] <= pu.TAU) & (np.arange(K)[None, :] < nd[:, None])).any(1) & ~(ref["icdf_margin"] <= pu.TAU_S)
        assert ok.sum() >= B - 1
        assert (acc.cpu().numpy()[ok] == ref["accept_len"][ok]).all() and (out.cpu().numpy()[ok] == ref["out_tok"][ok]).all()


@pytest.mark.parametrize("B,K,V,G,dt", [
    (5, 3, 65536, 2, bf16), (5, 3, 65538, 2, bf16), (5, 3, 32768, 2, f32), (5, 3, 32771, 2, f32),      # four batches a row and one element more
    (7, 4, 13, 3, bf16), (7, 4, 30, 2, f32),                    # rows without a whole vector, rows that start off one
    (191, 1, 8200, 2, bf16), (192, 1, 8200, 2, bf16),           # three slices of a sequence in workgroups of their own, in one
    (192, 1, 65560, 2, f32), (200, 1, 65600, 2, bf16),          # seventeen and sixteen slices
    (200, 2, 20000, 3, f32), (65, 2, 4000, 2, bf16),            # four, one
    (64, 4, 32770, 2, bf16), (43, 6, 32770, 2, bf16),           # 256 rows of two batches, shared by eight wavefronts; 258, by four
    (32, 8, 24000, 2, f32), (26, 10, 24000, 2, f32),            # 256 and 260 of three
    (64, 8, 65530, 2, bf16), (57, 9, 32760, 2, f32),            # 512 and 513 of four
    (5, 3, 98300, 2, bf16), (5, 3, 98310, 2, bf16),             # six batches a row, and one element more: slices again
    (16, 4, 65536, 2, f32), (21, 3, 65536, 2, f32),             # eight: 64 rows whole, 63 in slices
    (64, 4, 131050, 2, f32), (130, 4, 49100, 2, f32),           # in slices: sixteen batches; 520 rows of six
])
def test_shard_rows_and_sums_by_one_workgroup(B, K, V, G, dt):
    rnd = mixed_round(B, K, V, dt, dt, seed=V)
    rnd["greedy"][1] = 1
    rnd["u_sample"][2:5] = torch.tensor([2.0 ** -12, 0.5, 1.0 - 2.0 ** -24], device=DEV)
    for t in (rnd["draft"], rnd["target"]):                     # a maximum met twice, in one shard and in two; a shard without a finite logit
        t[0, 0, [1, V // 4]] = 12.0
        t[3, 0, [2, V - 2]] = 12.0
        t[4, 0, :(V + G - 1) // G] = float("-inf")
    acc, out, _ = sharded_round(rnd, G, V)
    _, ref, nd = pu.oracle_round(rnd)
    ok = ~((ref["accept_margin"] <= pu.TAU) & (np.arange(K)[None, :] < nd[:, None])).any(1) & ~(ref["icdf_margin"] <= pu.TAU_S)
    assert ok.sum() >= B - 1 - B * K // 100                      # near ties: a few per thousand decisions; two planted maxima
    assert (acc.cpu().numpy()[ok] == ref["accept_len"][ok]).all() and (out.cpu().numpy()[ok] == ref["out_tok"][ok]).all()
    tps = binding.Tapout(B, K, V)
    rec = torch.stack([tps.shard_stats(rnd["draft"][:, :, round(g * V / G):round((g + 1) * V / G)], round(g * V / G), length=rnd["k_len"],
                                       tok=rnd["draft_tok"]).clone() for g in range(G)])
    got = tps.draft_stats_sharded(rec, B, K, V, draft_tok=rnd["draft_tok"], k_len=rnd["k_len"])
    ods, _, _ = pu.oracle_round(rnd)
    live = np.arange(K)[None, :] < rnd["k_len"].cpu().numpy()[:, None]
    for key in pu.STAT_KEYS:
        pu.assert_stats_close(key, got[key].cpu().numpy(), ods[key], live)
    assert (got["top1_id"].cpu().numpy()[live] == ods["top1_id"][live]).all()


@pytest.mark.parametrize("batches", [1, 2, 3, 4])
@pytest.mark.parametrize("dt", [f32, bf16])
def test_shard_records_keep_the_precision_of_their_format(batches, dt):
    """The sums of a record are binary32 numbers, off by 2^-24 / sqrt(3) of themselves (root mean square) at worst from that rounding alone.
    What comes before it has to stay below: terms good to about 2^-23 and a thread's sums of up to 128 of them, both averaged over 256 threads
    (2^-23 / 16), and no binary32 reduction over the threads, which by itself is as much again: a fifth is allowed on top."""
    B, K, V = 512, 4, batches * 1024 * (4 if dt == f32 else 8)
    g = torch.Generator(device=DEV).manual_seed(V)
    x = (torch.randn(B, K, V, generator=g, device=DEV) * 0.5).to(dt)
    rec = binding.Tapout(B, K, V).shard_stats(x, 0, torch.full((B,), K, dtype=torch.int32, device=DEV)).reshape(B * K, 8)
    M, S, T = (rec[:, i].view(f32).double() for i in range(3))
    y = x.reshape(B * K, V).double() * 1.4426950408889634
    first = y.argmax(-1, keepdim=True)
    assert torch.equal(rec[:, 4].long(), first[:, 0]) and torch.equal(M, x.reshape(B * K, V).double().amax(-1))
    rest = lambda e: e.scatter(1, first, 0.0).sum(-1)  # noqa: E731
    R = torch.ceil(M * 1.4426950408889634)
    e = torch.exp2(y - R[:, None])
    assert torch.allclose(S, rest(e), rtol=1e-5, atol=0.0)     # (the reference is the integer above the maximum)
    for got, want in ((S, rest(e)), (T, rest(e * (y - R[:, None])))):
        assert ((got - want) / want).pow(2).mean().sqrt() <= 1.2 * 2.0 ** -24 / 3 ** 0.5


def _records_as_if_cut_into(B, K, V, dt, P, opts=()):
    """A context with these options leaves the records, bit by bit, of one that is asked for P slices by the smallest slice."""
    x = (torch.randn(B, K, V, generator=torch.Generator(device=DEV).manual_seed(V), device=DEV) * 2).to(dt)
    a, b = binding.Tapout(B, K, V), binding.Tapout(B, K, V)
    for name, v in opts:
        a.set_option(name, v)
    b.set_option("slice_bytes", 1 << 22)
    force_slices(b, B * K, P, min_slice=1000)
    k_len = torch.full((B,), K, dtype=torch.int32, device=DEV)
    return torch.equal(a.shard_stats(x, 7, k_len), b.shard_stats(x, 7, k_len))


@pytest.mark.parametrize("B,K,V,dt,P", [
    (64, 4, 32756, f32, 1), (43, 6, 32756, f32, 8),             # 256 rows of eight batches whole, 258 in slices
    (16, 4, 32756, f32, 1), (21, 3, 32756, f32, 8),             # 64 and 63 of them
    (32, 8, 49100, bf16, 1), (43, 6, 49100, bf16, 6),           # 256 and 258 rows of six
    (96, 8, 64128, f32, 6), (192, 8, 48000, bf16, 3),           # more rows: few are live in short drafts, a workgroup each would leave the chip idle
])
def test_long_shard_rows_are_read_whole_up_to_a_workgroup_per_compute_unit(B, K, V, dt, P):
    assert _records_as_if_cut_into(B, K, V, dt, P)


@pytest.mark.parametrize("name,value,P", [("slice_bytes", 16384, 8), ("wgs_target", 8192, 8), ("wgs_target", 512, 2), ("wgs_target", 65536, 8)])
def test_shard_rows_are_cut_as_the_options_say(name, value, P):
    assert _records_as_if_cut_into(64, 4, 32756, f32, P, ((name, value),))


@pytest.mark.parametrize("P", [1, 2, 3, 16, 17])
def test_shard_records_from_any_number_of_slices(P):
    """Sixteen slices of a shard's row are merged across lanes, seventeen one after the other: the same record."""
    B, K, V = 3, 4, 17 * 256 + 5
    rnd = mixed_round(B, K, V, bf16, bf16, seed=P, k_len=[4, 2, 3])
    tp = binding.Tapout(B, K, V)
    force_slices(tp, B * K, P)
    rec = tp.shard_stats(rnd["draft"], 0, length=rnd["k_len"], tok=rnd["draft_tok"])
    out = tp.draft_stats_sharded(rec[None], B, K, V, draft_tok=rnd["draft_tok"], k_len=rnd["k_len"])
    ref, _, _ = pu.oracle_round(rnd)
    live = np.arange(K)[None, :] < rnd["k_len"].cpu().numpy()[:, None]
    for key in pu.STAT_KEYS:
        pu.assert_stats_close(key, out[key].cpu().numpy(), ref[key], live)
    assert (out["top1_id"].cpu().numpy()[live] == ref["top1_id"][live]).all()


@pytest.mark.parametrize("K", [5, 70])
@pytest.mark.parametrize("dt", [f32, bf16])
@pytest.mark.parametrize("fuse", [0, 1])
def test_uniform_of_zero_accepts_no_token_of_probability_zero(K, dt, fuse):
    """u_accept = 0 < p/q as the oracle has it, in double: never where p = 0 (masked target logit, or a ratio below half the
    smallest double), always where the ratio is a number above that, however small.  K = 5 merges rows across lanes, 70 staged."""
    B, V, at = 4, 3000, 3
    rnd = mixed_round(B, K, V, dt, dt, seed=K)
    rnd["target"][:, :at] = rnd["draft"][:, :at]
    rnd["u_accept"][:] = 0.0
    bidx, tok = torch.arange(B, device=DEV), rnd["draft_tok"][:, at].long()
    rnd["target"][bidx, at, tok] = torch.tensor([float("-inf"), -720.0, -1000.0, -100.0], device=DEV).to(dt)    # p/q: 0, e^-720 or so, 0, e^-100
    rnd["u_accept"][:, at + 1:] = 0.5                                # the next position is rejected by an ordinary ratio
    rnd["target"][bidx, at + 1, rnd["draft_tok"][:, at + 1].long()] = -30.0
    want = [at, at + 1, at, at + 1]
    _, ref, _ = pu.oracle_round(rnd)
    assert ref["accept_len"].tolist() == want
    tp = binding.Tapout(B, K, V)
    tp.set_option("fuse_head", fuse)
    ds, vf, nd = pu.gpu_round(tp, rnd)
    assert vf["accept_len"].cpu().tolist() == want
    ds["logq_tok"][:, 1] = float("nan")                              # a ratio that is no number accepts nothing either
    vf = tp.verify(rnd["target"], rnd["draft"], ds["lse"], ds["logq_tok"], rnd["draft_tok"], nd, rnd["u_accept"], rnd["u_sample"])
    assert vf["accept_len"].cpu().tolist() == [1] * B
    args, out = tp.round_args(rnd, torch.zeros(B, dtype=torch.int32, device=DEV), False)
    tp.round(args)
    assert out["verify"]["accept_len"].cpu().tolist() == want
    for G in (2, 17):                                               # records merged across lanes, and one after the other
        acc, _, _ = sharded_round(rnd, G, V)
        assert acc.cpu().tolist() == want


@pytest.mark.parametrize("shared", [False, True])
def test_ucb_tuned_of_a_restored_state_without_a_variance(shared):
    """A restored state may hold sums of squares that no rewards have (sum_r2 = 0 beside sum_r > 0): the bonus of such an arm is
    the root of a negative number.  tapout_round chooses what the separate calls and the oracle choose: an index that is no
    number is never larger, but stays if it is the first."""
    g = torch.Generator().manual_seed(5)
    for trial in range(24):
        A = 3 + trial % 6
        N = torch.randint(200, 3000, (1, A), generator=g).numpy().astype(np.int64)
        S = np.round(N * (0.3 + 0.6 * torch.rand(1, A, generator=g).double().numpy()), 1)
        Q = S * S / N
        for a in range(A):
            if torch.rand(1, generator=g).item() < 0.5:
                Q[0, a] = 0.0
        rnd = mixed_round(1, 4, 3000, bf16, bf16, seed=trial)
        rnd["draft_tok"][0, 0] = 3000                                # nothing accepted
        tps = [binding.Tapout(1, 4, 3000, policy=binding.UCB_TUNED, shared_bandit=shared, rules=(0,) * A, thresholds=(0.6,) * A) for _ in range(2)]
        for tp in tps:
            tp.bandit_set_state(S, N, sum_r2=Q)
        arm = torch.zeros(1, dtype=torch.int32, device=DEV)
        inactive = torch.zeros(1, dtype=torch.uint8, device=DEV)     # no reward: the state as it was restored decides
        args, _ = tps[0].round_args(rnd, arm, False, active=inactive)
        tps[0].round(args)
        want = orc.ucb_tuned_select(S[0], Q[0], N[0])[0]
        assert tps[1].bandit_select(1).item() == want
        assert arm.item() == want, f"trial {trial}"


@pytest.mark.parametrize("B,K,V,dt", [(1, 8, 128256, bf16), (3, 5, 9001, f32), (40, 2, 20000, bf16)])
def test_default_slices_can_be_had_back(B, K, V, dt):
    """"min_slice" 0 is the default rule: after any other value the same bits as a context on which it was never set."""
    rnd = mixed_round(B, K, V, dt, dt, seed=V)
    fresh, tp = binding.Tapout(B, K, V), binding.Tapout(B, K, V)
    for v in (256, 4096, 0):
        tp.set_option("min_slice", v)
    for bad in (-1, 1, 255):
        with pytest.raises(binding.TapoutError, match="min_slice"):
            tp.set_option("min_slice", bad)
    (da, va, _), (db, vb, _) = pu.gpu_round(fresh, rnd), pu.gpu_round(tp, rnd)
    for a, b in ((da, db), (va, vb)):
        for k in a:
            assert torch.equal(torch.nan_to_num(a[k].float(), nan=7.0), torch.nan_to_num(b[k].float(), nan=7.0)), k


@pytest.mark.parametrize("B,V,dt", [(5, 32000, f32), (5, 9001, bf16), (64, 50257, f32)])       # the last: beyond 24 MB, a pass of its own
def test_round_up_to_the_stop_position_ignores_target_rows_beyond_it(B, V, dt):
    """Target rows between the stop position and k_len may be read before the stop position is known: whatever they hold (NaN
    here), the results are those of the separate calls, bit for bit, which read rows up to the stop position only."""
    K = 6
    rnd = mixed_round(B, K, V, dt, dt, seed=V, k_len=[1 + b % K for b in range(B)])
    for arm in range(3):
        tp = binding.Tapout(B, K, V, thresholds=(2.0, 0.3, 0.1))
        arms = torch.full((B,), arm, dtype=torch.int32, device=DEV)
        n = tp.draft_stats(rnd["draft"], draft_tok=rnd["draft_tok"], k_len=rnd["k_len"], arm=arms)["n_stop"]
        poisoned = dict(rnd, target=rnd["target"].clone())
        rows = torch.arange(K + 1, device=DEV)[None, :] > n[:, None]
        poisoned["target"][rows] = float("nan")
        _, want, _ = pu.gpu_round(tp, rnd, arm=arms)
        args, out = tp.round_args(poisoned, arms.clone(), True)
        tp.round(args)
        got = out["verify"]
        assert torch.equal(out["n_draft"], n) and not got["flags"].any()
        for k in ("accept_len", "out_tok", "n_out", "target_lse", "logp_tok", "target_top1", "flags"):
            a, b = (torch.nan_to_num(x[k].float(), nan=7.0) for x in (got, want))
            assert torch.equal(a, b), k
        assert (rows & (torch.arange(K + 1, device=DEV)[None, :] <= rnd["k_len"][:, None])).sum() >= B      # (some of them up to k_len)


@pytest.mark.parametrize("P,Ks", [
    (1, (1, 63, 64)),                 # a lane or more for every slice of a row: 1, 2, 4, 8, 16 of them, and four, two
    (2, (32, 33, 64)),                # or one lane for a slice up to 64, 128 and 256 slices of a sequence; beyond 256 two passes
    (3, (16, 17, 32, 33, 64)),
    (8, (8, 9, 16, 17, 32, 33)),
    (13, (1, 4, 5, 8, 9, 16, 17)),
])
@pytest.mark.parametrize("dt", [f32, bf16])
def test_draft_epilogue_at_every_arrangement_of_its_lanes(P, Ks, dt):
    for K in Ks:
        B, V = 2, P * 256 + 37 * K
        rnd = mixed_round(B, K, V, dt, dt, seed=P * 100 + K)
        tp = binding.Tapout(B, K, V, draft_sampling=True)
        force_slices(tp, B * K, P)
        c = pu.check_round(tp, rnd, arm=random_arms(B, seed=K))
        assert c["accept_flagged"] + c["icdf_flagged"] + c["stop_flagged"] <= 1
        # the tokens' launch forms a row's lse on the same lanes
        out = tp.draft_stats(rnd["draft"], u_draft=torch.rand(B, K, generator=torch.Generator().manual_seed(K)).to(DEV))
        given = tp.draft_stats(rnd["draft"], draft_tok=out["sampled_tok"])
        for n in ("lse", "entropy", "p_top1", "p_top2", "margin", "top1_id", "logq_tok", "flags"):
            assert torch.equal(out[n], given[n]), (P, K, n)


def test_entropy_rule_beside_its_threshold():
    """sqrt(H) > h is decided without the root: at thresholds next to the root of the entropy that the library returns, on either side, and at
    thresholds whose square it is."""
    V, K = 4096, 8
    g = torch.Generator().manual_seed(5)
    x = (torch.randn(1, K, V, generator=g) * torch.linspace(0.0, 9.0, K)[None, :, None]).to(DEV)
    H = binding.Tapout(1, K, V).draft_stats(x)["entropy"].cpu().numpy()[0]
    near = []
    for r in np.sqrt(H.astype(np.float64)).astype(np.float32):
        near += [r, np.nextafter(r, np.float32(0)), np.nextafter(r, np.float32(99))]
    near += [np.float32(0.0), np.float32(-1.0), np.float32(1e-30)]
    for h in near:
        tp = binding.Tapout(1, K, V, rules=(binding.RULE_SVIP,), thresholds=(float(h),))
        out = tp.draft_stats(x, arm=torch.zeros(1, dtype=torch.int32, device=DEV))
        assert np.array_equal(out["entropy"].cpu().numpy()[0], H)
        assert np.array_equal(out["stop_fired"].cpu().numpy()[0].astype(bool), np.sqrt(H.astype(np.float64)) > np.float64(h)), h


@pytest.mark.parametrize("B,K,V,dt,tt", [
    (12, 8, 128256, bf16, bf16), (11, 8, 128256, bf16, bf16),        # sixteen slices of a batch: two lanes each in the epilogue
    (16, 16, 128259, bf16, bf16),                                    # one lane each; rows at every alignment
    (16, 8, 151936, bf16, bf16),                                     # ten of two batches
    (16, 8, 151936, f32, f32), (20, 5, 128256, f32, bf16),           # sixteen of two batches and a third, of two
])
def test_draft_pass_of_a_mid_sized_batch(B, K, V, dt, tt):
    rnd = mixed_round(B, K, V, dt, tt, seed=V + K)
    tp = binding.Tapout(B, K, V)
    arm = random_arms(B, seed=K)
    c = [pu.check_round(tp, rnd, arm=arm), pu.check_round_call(tp, rnd, arm.clone(), truncate=True)]
    assert sum(x["accept_flagged"] + x["icdf_flagged"] + x["stop_flagged"] for x in c) <= 2 + 4 * B * K // 500
    u = torch.rand(B, K, generator=torch.Generator().manual_seed(V))
    out = binding.Tapout(B, K, V, draft_sampling=True).draft_stats(rnd["draft"], u_draft=u.to(DEV))
    ref = orc.draft_sample(pu.host_logits(rnd["draft"]), u.numpy(), k_len=np.full(B, K, dtype=np.int32), nthreads=16)
    near = ref["icdf_margin"] <= pu.TAU_S
    assert near.sum() <= 1 and (out["sampled_tok"].cpu().numpy()[~near] == ref["tok"][~near]).all()


STATS = ("lse", "entropy", "p_top1", "p_top2", "margin", "top1_id", "logq_tok", "flags")


def _same_bits(a, b, names=STATS):
    return [n for n in names if not torch.equal(a[n], b[n])]


@pytest.mark.parametrize("B,K,V,dt", [(12, 8, 128256, bf16), (14, 15, 47000, f32), (18, 14, 160000, bf16)])
def test_statistics_do_not_depend_on_who_may_draw_tokens(B, K, V, dt):
    """The same bits from a context that draws tokens, with a draw and without, from one that does not, and from the entry point without one."""
    x = (torch.randn(B, K, V, generator=torch.Generator(device=DEV).manual_seed(V), device=DEV) * 2).to(dt)
    draws, plain = binding.Tapout(B, K, V, draft_sampling=True), binding.Tapout(B, K, V)
    first = draws.draft_stats(x, u_draft=torch.rand(B, K, generator=torch.Generator().manual_seed(K)).to(DEV))
    for other in (draws.draft_stats(x, draft_tok=first["sampled_tok"]), plain.draft_stats(x, draft_tok=first["sampled_tok"]),
                  binding.draft_stats_static(x, draft_tok=first["sampled_tok"])):
        assert not _same_bits(first, other)


@pytest.mark.parametrize("B,K,V,dt,opts,P", [
    (24, 16, 128256, bf16, {}, 16),                                  # slices of one batch also where rows are many: in short drafts few are live
    (64, 8, 128256, bf16, {"slice_bytes": 16384}, 16), (64, 8, 128256, bf16, {"wgs_target": 8192}, 16),
    (24, 16, 128256, bf16, {"wgs_target": 65536}, 16),
    (64, 8, 128256, bf16, {"wgs_target": 1, "slice_bytes": 131072}, 1),
])
def test_draft_pass_is_cut_as_its_options_say(B, K, V, dt, opts, P):
    """The bits of the same cut asked for by the smallest slice."""
    x = (torch.randn(B, K, V, generator=torch.Generator(device=DEV).manual_seed(V), device=DEV) * 2).to(dt)
    tok = torch.randint(0, V, (B, K), generator=torch.Generator().manual_seed(K)).to(torch.int32).to(DEV)
    a, b = binding.Tapout(B, K, V), binding.Tapout(B, K, V)
    for name, v in opts.items():
        a.set_option(name, v)
    b.set_option("slice_bytes", 1 << 22)
    force_slices(b, B * K, P, min_slice=8000)
    assert not _same_bits(a.draft_stats(x, draft_tok=tok), b.draft_stats(x, draft_tok=tok))


@pytest.mark.parametrize("B,batches", [(64, 2), (64, 3), (64, 4), (64, 6), (64, 8), (64, 16), (256, 8), (256, 16), (384, 6)])
@pytest.mark.parametrize("dt", [f32, bf16])
def test_records_of_long_rows_keep_the_precision_of_their_format(B, batches, dt):
    """Rows shared by eight and sixteen wavefronts, and rows in slices: the bound of the test above."""
    K, V = 4, batches * 1024 * (4 if dt == f32 else 8)
    x = (torch.randn(B, K, V, generator=torch.Generator(device=DEV).manual_seed(V), device=DEV) * 0.5).to(dt)
    rec = binding.Tapout(B, K, V).shard_stats(x, 0, torch.full((B,), K, dtype=torch.int32, device=DEV)).reshape(B * K, 8)
    M, S, T = (rec[:, i].view(f32).double() for i in range(3))
    err = []
    for b in range(0, B * K, 128):
        y = x.reshape(B * K, V)[b:b + 128].double() * 1.4426950408889634
        first = y.argmax(-1, keepdim=True)
        assert torch.equal(rec[b:b + 128, 4].long(), first[:, 0])
        R = torch.ceil(M[b:b + 128] * 1.4426950408889634)[:, None]
        e = torch.exp2(y - R)
        for got, term in ((S, e), (T, e * (y - R))):
            want = term.scatter(1, first, 0.0).sum(-1)
            err.append((got[b:b + 128] - want) / want)
    s, t = torch.cat(err[::2]), torch.cat(err[1::2])
    assert s.pow(2).mean().sqrt() <= 1.2 * 2.0 ** -24 / 3 ** 0.5 and t.pow(2).mean().sqrt() <= 1.2 * 2.0 ** -24 / 3 ** 0.5


@pytest.mark.parametrize("K,P", [(24, 3), (24, 13), (70, 3), (24, 0)])      # lanes in one pass and in two, one slice after the other; shard records
@pytest.mark.parametrize("at", [0, 1])
@pytest.mark.parametrize("dt", [f32, bf16])
def test_second_maximum_wherever_it_lies(K, P, at, dt):
    """The second largest value in the vector, the batch, the thread, the slice of the largest and outside of them, before and behind it, and as
    large as it: probabilities and margin within the 1e-5 max(|value|, 1e-3) of all statistics."""
    vec = 8 if dt == bf16 else 4
    batch = 4 * 256 * vec
    # the largest value in thread 7's second vector of batch `at` of a slice of two batches, or of a shard of four: that slice or shard starts at
    # element `start` of what a row of `length` elements is cut from, whose first whole vector lies where 16 bytes are aligned
    V = (2047 * P if P else 8 * 1024) * vec - 3
    cut = [0, V] if P else [0, 4 * batch - 1000, V]
    start, length = cut[-2], V - cut[-2]
    slices = 2 * batch * (P // 2)
    off = [1, -1, vec, -vec, 256 * vec, -256 * vec, 512 * vec, batch, batch + 1, -batch, 2 * batch - 300 * vec, 0]
    x = torch.randn(1, K, V, generator=torch.Generator().manual_seed(P)).to(dt)
    largest, second = [], []
    for k in range(K):
        p = start + -(k * length) % vec + slices + at * batch + (256 + 7) * vec + 2
        q = p + off[k % 12] if k % 12 < 11 else V - 1
        x[0, k, p] = 9.0
        x[0, k, q] = 9.0 if k % 24 >= 12 else 8.5
        largest.append(p)
        second.append(q)
    tp = binding.Tapout(1, K, V)
    if P:
        force_slices(tp, K, P)                                        # of (2047 P + P) / P = 2048 vectors
        out = tp.draft_stats(x.to(DEV))
    else:
        rec = torch.stack([tp.shard_stats(x[:, :, i:j].contiguous().to(DEV), i).clone() for i, j in zip(cut, cut[1:])])
        out = tp.draft_stats_sharded(rec, 1, K, V)
    two = torch.softmax(x.double(), -1).topk(2, -1).values
    for n, w in {"p_top1": two[..., 0], "p_top2": two[..., 1], "margin": two[..., 0] - two[..., 1]}.items():
        assert ((out[n].cpu().double() - w).abs() <= 1e-5 * w.abs().clamp(min=1e-3)).all(), n
    assert out["top1_id"][0].tolist() == [min(p, q) if k % 24 >= 12 else p for k, (p, q) in enumerate(zip(largest, second))]
