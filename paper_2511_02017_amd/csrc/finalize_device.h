// Device code of the draft epilogue (see finalize.hip), in a header because several kernels run it: the epilogue kernel
// of its own, and the final-token locate kernel of a whole-round call, whose launch carries the epilogue's
// workgroups beside its own (as do the token search of the draft-token draw, and the launch that streams the first target rows
// of a round up to the stop position).
#pragma once
#include <type_traits>

#include "common.h"

namespace tapout {

constexpr int kFinalBlock = 256;
static_assert(kFinalBlock == kBlock, "stage_partials strides by kBlock");

__device__ inline bool rule_fires(int rule, float h, float H, float p1, float margin)
{
    // decisions on the returned binary32 signals, widened to double (strict inequalities of Table 1)
    switch (rule) {
    // sqrt(H) > h as H > h^2: H and h have 24 significant bits, h^2 is exact in double, and where H differs from it, it does by 2^-48 of
    // itself or more, the root by 2^-49: more than the rounding of a square root moves it
    case TAPOUT_RULE_SVIP:    return h < 0.0f ? H >= 0.0f : (double)H > (double)h * (double)h;
    case TAPOUT_RULE_MAXCONF: return (double)p1 < (double)h;
    default:                  return (double)margin < (double)h;
    }
}

// SVIP-Difference (Table 1): sqrt(H_t) - sqrt(H_{t-1}) > h; no previous entropy (NaN) or a bad row: no stop.
__device__ inline bool svip_diff_fires(float h, float H, float H_prev)
{
    if (H != H || H_prev != H_prev) return false;
    return sqrt((double)H) - sqrt((double)H_prev) > (double)h;
}

// AdaEDL (Table 1): 1 - sqrt(g H) < lambda.
__device__ inline bool adaedl_fires(double g, double lambda, float H)
{
    if (H != H) return false;
    return 1.0 - sqrt(g * (double)H) < lambda;
}

// One row's results: the signals from its merged sums into the output arrays (i = b K + k), log q(tok) of its token t with
// logit xt (want_tok), and its flags.
struct RowOut { float H, p1, margin; uint32_t flags; };
__device__ inline RowOut emit_row(const DraftFinalArgs &a, int64_t i, const RowTotal &r, bool want_tok, int32_t t, float xt)
{
    RowOut o;
    o.flags = 0;
    float lse, p2;
    double lse_d = NAN;
    if (__builtin_expect(r.bad, 0)) {
        o.flags = TAPOUT_FLAG_BAD_ROW | (a.sampling ? TAPOUT_FLAG_BAD_TOKEN : 0u);
        lse = o.H = o.p1 = p2 = o.margin = NAN;
    } else {
        const RowSignals g = row_signals(r, a.V > 1);
        lse_d = g.lse;
        lse = (float)g.lse; o.H = (float)g.H;
        o.p1 = (float)g.p1; p2 = (float)g.p2; o.margin = (float)g.margin;
    }
    if (a.sampled_lse) a.sampled_lse[i] = lse_d;
    if (a.lse) a.lse[i] = lse;
    if (a.entropy) a.entropy[i] = o.H;
    if (a.p_top1) a.p_top1[i] = o.p1;
    if (a.p_top2) a.p_top2[i] = p2;
    if (a.margin) a.margin[i] = o.margin;
    if (a.top1_id) a.top1_id[i] = (r.cand >= 0 && r.cand < a.V) ? r.cand : 0;      // exact: the pieces carry the index of their first maximum
    if (want_tok) {
        if (__builtin_expect(t < 0 || t >= a.V, 0)) { o.flags |= TAPOUT_FLAG_BAD_TOKEN; a.logq_tok[i] = NAN; }
        else a.logq_tok[i] = (float)((double)xt - lse_d);
    }
    if (a.round_entropy) a.round_entropy[i] = o.H;
    return o;
}

// Decision of a rule that looks beyond the row's own signals; H_prev: the previous row's entropy (the carried one for row 0).
__device__ inline bool stateful_fires(const DraftFinalArgs &a, int b, int arm, int rule, float threshold, float H, float H_prev)
{
    if (rule == TAPOUT_RULE_SVIP_DIFF) return svip_diff_fires(threshold, H, H_prev);
    return adaedl_fires(a.adaedl_gamma, a.lambda ? a.lambda[(int64_t)b * a.n_arms + arm] : (double)threshold, H);
}

// A row on its lanes: from the partial (w0, w1) of this lane's piece, if it has one (mine), to the statistics of the row, the
// same bits in every one of the row's 2^gsh lanes.  u: which of the piece's lanes this is, g: the piece's place in its row.  The
// second memory round trip: token_logit() and this lane's vectors of the left-out batch.
// meanwhile() is called once those are under way.
// dtype and gsh are constants wherever the caller knows them: what depends on them is then no branch on the way.
struct Idle { __device__ void operator()() const {} };
template <bool SHARDED, int USH, class TokenLogit, class Meanwhile = Idle>
__device__ __forceinline__ Piece row_on_lanes(const DraftFinalArgs &a, const int dtype, const BatchGeom &g, const u32x4 &w0, const u32x4 &w1, bool mine, int u, const int gsh, TokenLogit token_logit,
                                              Meanwhile meanwhile = Meanwhile())
{
    constexpr int NV = kStreamU >> USH;                               // vectors per lane
    const float v1 = mine ? __uint_as_float(w0.x) : -INFINITY;
    float S = __uint_as_float(w0.y), T = __uint_as_float(w0.z), v2 = __uint_as_float(w0.w);
    int32_t cand = (int32_t)w1.x;
    if (!mine || (v1 == -INFINITY && !(S != S))) { S = 0.0f; T = 0.0f; v2 = -INFINITY; cand = 0x7fffffff; }     // nothing in it
    float xt = token_logit();
    BatchVecs<NV> bt{};
    if constexpr (!SHARDED) bt = batch_issue_vecs<NV>(g, dtype, a.V, cand, u * NV, a.part);
    meanwhile();
    // the row's maximum and the piece that holds the first of it
    const float M = lanes_max(v1, USH, gsh);
    const bool holds = v1 == M && cand != 0x7fffffff;
    const int32_t first = lanes_min(holds ? cand : 0x7fffffff, USH, gsh);
    const bool wins = holds && cand == first;
    const float R = ref_of_max(M);
    const float d = R - ref_of_max(v1);                           // an integer, >= 0 for a piece that holds anything
    const int di = (int)fminf(fmaxf(d, -4000.0f), 4000.0f);       // 2^-4000 underflows to 0 as it should
    double Sd = u == 0 ? ldexp((double)S, -di) : 0.0;             // exact power-of-two scaling
    double Td = u == 0 ? ldexp((double)T - (double)d * (double)S, -di) : 0.0;
    if (S == 0.0f && T == 0.0f) { Sd = 0.0; Td = 0.0; }           // (0 * inf)
    int32_t idx = 0x7fffffff;
    v2 = wins ? v2 : v1;                                          // the second maximum: outside the winner's batch, of the others the maximum
    if constexpr (SHARDED) {
        // a record leaves its maximum out: an ordinary term here unless it is the row's first maximum
        idx = wins ? cand : 0x7fffffff;
        if (!wins && v1 > -INFINITY) {
            const float y = __builtin_fmaf(v1, kLog2e, -R), e = __builtin_amdgcn_exp2f(y);
            Sd += (double)e;
            Td += (double)e * (double)fmaxf(y, -200.0f);
        }
        xt = lanes_max(xt, USH, gsh);
    } else {
        // the batch's elements in the row's reference, all but the row's first maximum
        const BatchExtra x = dtype == TAPOUT_F32 ? batch_sum<TAPOUT_F32>(R, M, wins, bt, u * NV) : batch_sum<TAPOUT_BF16>(R, M, wins, bt, u * NV);
        Sd += (double)x.sa; Td += (double)x.ta; idx = x.idx;
        v2 = fmaxf(v2, x.m2);                                     // ... or in it
    }
    Piece t;
    t.M = M; t.v2 = lanes_max(v2, 0, gsh); t.xt = xt;
    t.idx = lanes_min(idx, 0, gsh);
    lanes_sum2(Sd, Td, 0, gsh);
    t.S = Sd; t.T = Td;
    return t;
}

// log2 of the lanes per piece of a sequence of so many (row, slice) pieces.
__device__ inline int draft_lanes_shift(int pieces) { return pieces > kFinalBlock / 2 ? 0 : (pieces > kFinalBlock / 4 ? 1 : 2); }

// f(msh, ush) with the lanes of a row's pieces (lane_merge_shift, not negative) and of a piece as constants, for pieces that fit one pass (K << msh
// <= kFinalBlock, K <= 64).  USH: what ush is, or -1.  TWO: two lanes a piece or four.
template <int USH, bool TWO = false, class F>
__device__ __forceinline__ void on_lanes(int msh, int ush, F f)
{
    auto with = [&](auto m) __attribute__((always_inline)) {
        constexpr int M = decltype(m)::value;
        if constexpr (USH >= 0) f(m, std::integral_constant<int, USH>{});
        else if constexpr (M == 0) f(m, std::integral_constant<int, 2>{});
        else if (ush == 2) f(m, std::integral_constant<int, 2>{});
        else if constexpr (M == 1 || TWO) f(m, std::integral_constant<int, 1>{});
        else if (ush == 1) f(m, std::integral_constant<int, 1>{});
        else f(m, std::integral_constant<int, 0>{});
    };
    if (msh <= 1) {
        if (msh == 0) with(std::integral_constant<int, 0>{}); else with(std::integral_constant<int, 1>{});
    } else if (msh == 2) with(std::integral_constant<int, 2>{});
    else if (msh == 3) with(std::integral_constant<int, 3>{});
    else with(std::integral_constant<int, 4>{});
}

// ---- lane path: few rows and slices (see lane_merge_shift) -----------------------------------------
// A wavefront of these small kernels executes an instruction about every nine cycles whatever it is, so what counts is
// the number of instructions from the first request to the last store.  Every (row, slice) piece has 2^USH lanes of its
// own, each of which takes 4 >> USH vectors of the piece's left-out batch; a row's lanes find the row's maximum first (one
// instruction per exchange), bring every piece to the row's reference once, add the batch's elements in that reference
// and then only sum.  Two or four lanes per piece where the workgroup has that many to spare.  No LDS between a row's
// lanes and its signals.  (Pairwise merges of whole records, the batch by one lane, and the row totals handed to a
// thread per row through LDS: launch 8.4 us at V = 128256, B = 64, K = 8, this 6.5; one sequence at V = 32000 6.2 / 4.7.)
//
// ONCE: the pieces have their lanes in one pass, and there is no loop: the compiler formed everything that stays the same from pass to
// pass (addresses and checks of ten outputs, constants) ahead of it, two hundred instructions in front of the first request.
// The row's reductions run with their lanes as constants then (on_lanes): a step that may or may not be wanted is a branch.
// (With the loop, and the lanes as variables: launch of its own, V = 32000, one sequence, binary32 4.8 us, now 4.4; rounds up to the stop position
// V = 32000, one sequence 18.7 / 18.3 us, V = 128256, one sequence 20.8 / 20.2, drawn tokens of 64 rows 15.65 / 15.5.)
// FEW: few_pieces holds, and with it two or four lanes a piece.
template <bool SHARDED, bool ONCE, bool FEW = false>
__device__ __forceinline__ void draft_finalize_lanes(const DraftFinalArgs &a, const int b, unsigned char *lds, const int dtype, const int msh)
{
    const int ush = SHARDED || !ONCE ? 0 : draft_lanes_shift(a.K << msh), U = 1 << ush;      // lanes per piece
    float *sh_H = (float *)lds;                                       // [64] entropies of the sequence (stateful rules)
    uint8_t *sh_dec = lds + 4 * kWave, *sh_flag = sh_dec + kWave;     // [64] each: decisions, flags
    const int K = a.K, tid = threadIdx.x, gsh = msh + ush;            // 2^gsh lanes per row
    const int u = tid & (U - 1), sl = (tid >> ush) & ((1 << msh) - 1), per_pass = kFinalBlock >> gsh;
    const bool want_tok = a.draft_tok && a.logq_tok, tok_mode = a.arm_stride > 0;
    int kb = a.k_len ? a.k_len[b] : K;
    int arm = (a.arm && !tok_mode) ? a.arm[b] : -1;                   // sequence-level bandit: one arm for all steps
    float H_carry = a.prev_entropy ? a.prev_entropy[b] : NAN;
    int row0 = 0;
    do {
        const int row = row0 + (tid >> gsh), row_c = min(row, K - 1);
        const int64_t i = (int64_t)b * K + row;
        // First memory round trip: the partial, the row's token and arm (and above the sequence's values).  A lane without a
        // piece asks for one all the same: a request under a condition is waited for where the branches meet.
        const Partial *pp = SHARDED ? a.part + (int64_t)min(sl, a.nsplit - 1) * a.B * K + (int64_t)b * K + row_c
                                    : a.part + ((int64_t)b * K + row_c) * a.nsplit + min(sl, a.nsplit - 1);
        const u32x4 w0 = ((const u32x4 *)pp)[0], w1 = ((const u32x4 *)pp)[1];
        int32_t tok = -1, arm_k = -1;
        if (want_tok) tok = a.draft_tok[(int64_t)b * K + row_c];
        if (tok_mode && a.arm) arm_k = a.arm[(int64_t)b * a.arm_stride + row_c];
        // while they travel: the row's geometry
        BatchGeom g{};
        const char *row_p = nullptr;
        if constexpr (!SHARDED) {
            row_p = (const char *)row_address(a.base, dtype, a.stride_b, a.stride_k, b, row_c);
            g = batch_geom(row_p, dtype, a.V, sl, a.per);
            asm volatile("" :: "v"(g.row), "v"(g.head), "v"(g.nvec), "v"(g.v0), "v"(g.v1e));
        }
        asm volatile("" :: "v"(w0), "v"(w1), "v"(tok), "v"(arm_k), "v"(kb), "v"(arm), "v"(H_carry));
        if (row0 == 0) { kb = kb > K ? K : (kb < 0 ? 0 : kb); arm = __builtin_amdgcn_readfirstlane(arm); }
        const bool live = row < kb, mine = live && sl < a.nsplit;     // rows beyond k_len hold stale partials
        auto token_logit = [&]() __attribute__((always_inline)) {
            if constexpr (SHARDED) return mine ? __uint_as_float(w1.y) : NAN;     // the shard that owns the token sent its logit, the others NaN
            else return want_tok && live && tok >= 0 && tok < a.V ? load_elem_rt(row_p, dtype, tok) : NAN;
        };
        // The sequence's rule (sequence-level bandits: one arm for all rows), looked up while the batch's vectors are under way instead of
        // behind them, where the two selections took 0.2 us of every call: draft pass with its epilogue 10.65 -> 10.36 us for 256 rows of
        // 32000 bf16 logits, 14.9 -> 14.3 for 336 of 50257, 8.0 -> 7.85 for 8 of 32000.
        int rule_seq = -1;
        float threshold_seq = 0.0f;
        auto pick_rule = [&]() __attribute__((always_inline)) {
            if (tok_mode || !a.arm) return;
            const int one = __builtin_amdgcn_readfirstlane(arm);
            const bool ok = one >= 0 && one < a.n_arms;
            rule_seq = ok ? pick8(a.rule, one) : -1;
            threshold_seq = pick8(a.threshold, ok ? one : 0);
            asm volatile("" : "+s"(rule_seq), "+s"(threshold_seq));
        };
        Piece t;
        if constexpr (!ONCE) t = row_on_lanes<SHARDED, 0>(a, dtype, g, w0, w1, mine, u, msh, token_logit, pick_rule);
        else on_lanes<SHARDED ? 0 : -1, FEW>(msh, ush, [&](auto m, auto us) __attribute__((always_inline)) {
            constexpr int USH = decltype(us)::value;
            t = row_on_lanes<SHARDED, USH>(a, dtype, g, w0, w1, mine, u, decltype(m)::value + USH, token_logit, pick_rule);
        });
        if (live && (tid & ((1 << gsh) - 1)) == 0) {
            const RowOut o = emit_row(a, i, row_total<true>(t), want_tok, tok, t.xt);
            sh_flag[row] = (uint8_t)o.flags;
            if (a.arm) {
                int rule = rule_seq;
                float threshold = threshold_seq;
                if (tok_mode) {
                    const bool ok = arm_k >= 0 && arm_k < a.n_arms;
                    rule = ok ? pick8(a.rule, arm_k) : -1;
                    threshold = pick8(a.threshold, arm_k);
                } else arm_k = arm;
                sh_H[row] = o.H;
                if (rule == TAPOUT_RULE_SVIP_DIFF || rule == TAPOUT_RULE_ADAEDL) sh_dec[row] = (uint8_t)(2 + arm_k);    // decided below
                else {
                    const bool fire = rule >= 0 && rule_fires(rule, threshold, o.H, o.p1, o.margin);
                    if (a.stop_fired) a.stop_fired[i] = fire ? 1 : 0;
                    sh_dec[row] = fire ? 1 : 0;
                }
            }
        }
        row0 += per_pass;
    } while (!ONCE && row0 < K);
    __syncthreads();
    // the sequence: rows are lanes of the first wavefront, ballots give the stop position and the flags
    if (tid < kWave) {
        const bool row = tid < kb;
        const uint32_t f = row ? sh_flag[tid] : 0u;
        uint32_t fa = 0;
        if (__builtin_amdgcn_ballot_w64((f & TAPOUT_FLAG_BAD_ROW) != 0)) fa |= TAPOUT_FLAG_BAD_ROW;
        if (__builtin_amdgcn_ballot_w64((f & TAPOUT_FLAG_BAD_TOKEN) != 0)) fa |= TAPOUT_FLAG_BAD_TOKEN;
        if (tid == 0 && a.flags) a.flags[b] = fa;
        if (a.arm) {
            const int dec = row ? sh_dec[tid] : 0;
            bool fire = dec == 1;
            if (dec >= 2) {
                const int ar = dec - 2;
                fire = stateful_fires(a, b, ar, pick8(a.rule, ar), pick8(a.threshold, ar), sh_H[tid], tid > 0 ? sh_H[tid - 1] : H_carry);
                if (a.stop_fired) a.stop_fired[(int64_t)b * K + tid] = fire ? 1 : 0;
            }
            const uint64_t fired = __builtin_amdgcn_ballot_w64(fire);
            if (tid == 0 && a.n_stop) a.n_stop[b] = fired ? __builtin_ctzll(fired) + 1 : kb;
        }
    }
}

// ---- staged path: any number of rows and pieces ------------------------------------------------------
template <bool SHARDED>
__device__ inline void draft_finalize_staged(const DraftFinalArgs &a, const int b, unsigned char *lds)
{
    Partial *sh_part = (Partial *)lds;
    float *sh_H = (float *)(lds + sizeof(Partial) * kStageCap);                 // entropies of the sequence (stateful rules only)
    uint8_t *sh_dec = lds + sizeof(Partial) * kStageCap + 4 * kScanCap;
    uint32_t &sh_flags = *(uint32_t *)(sh_dec + kScanCap);
    const int K = a.K;
    // kStageCap partials at a time (nsplit <= kStageCap is guaranteed by the host)
    const int rows_per_stage = kStageCap / a.nsplit;
    const bool want_tok = a.draft_tok && a.logq_tok;
    static_assert(kFinalBlock == 256, "stage_issue / stage_commit assume 256 threads");
    // First memory round trip: k_len, the arm, the carried entropy, the drafted tokens and the partials, all
    // requested before anything is waited for.  (Rows beyond k_len hold stale partials and unused tokens:
    // read, never used.)  The empty asm keeps the compiler from sinking the small loads below the barrier.
    const bool tok_mode = a.arm_stride > 0;
    int kb = a.k_len ? a.k_len[b] : K;
    const int arm = (a.arm && !tok_mode) ? a.arm[b] : -1;     // sequence-level bandit: one arm for all steps
    float H_carry = a.prev_entropy ? a.prev_entropy[b] : NAN;
    const int count0 = min(K, rows_per_stage) * a.nsplit;
    const StageRegs st0 = SHARDED ? stage_issue_shards(a.part, (int64_t)a.B * K, (int64_t)b * K, a.nsplit, count0)
                                  : stage_issue(a.part + (int64_t)b * K * a.nsplit, count0);
    asm volatile("" :: "v"(kb), "v"(arm), "v"(H_carry), "v"(st0.w0), "v"(st0.w1));
    kb = kb > K ? K : (kb < 0 ? 0 : kb);
    if (threadIdx.x == 0) sh_flags = 0;                       // ahead of the barrier in the commit: rows of other wavefronts OR into it
    // The `count` partials of rows k0.. lie in LDS; every thread completes some of them (left-out batch
    // back in, exact index of the first maximum into the cand slot) before the rows are merged one by one.
    auto complete_stage = [&](int k0, int count) {
        if constexpr (!SHARDED) {
            for (int i = threadIdx.x; i < count; i += kFinalBlock) {
                const int k = k0 + i / a.nsplit, sl = i % a.nsplit;
                if (k >= kb) continue;                          // stale partial of a row that was not drafted
                Piece e = piece_from_partial(sh_part[i]);
                const BatchRegs bt = batch_issue(row_address(a.base, a.dtype, a.stride_b, a.stride_k, b, k), a.dtype, a.V, e.idx, sl, a.per, a.part);
                batch_fix(e, bt, a.dtype);
                sh_part[i].S = (float)e.S; sh_part[i].T = (float)e.T; sh_part[i].cand = e.idx; sh_part[i].v2 = e.v2;
            }
            __syncthreads();
        }
    };
    stage_commit(sh_part, st0, count0);
    complete_stage(0, count0);
    const bool arm_ok = arm >= 0 && arm < a.n_arms;
    const int rule_b = arm_ok ? pick8(a.rule, arm) : -1;
    // rows whose rule looks beyond their own signals are decided in a second sweep (uniform over the workgroup);
    // token-level bandits: the arm of step k is arm[b, k]
    const bool sweep = tok_mode ? (a.round_entropy != nullptr)
                                : (rule_b == TAPOUT_RULE_SVIP_DIFF || rule_b == TAPOUT_RULE_ADAEDL);
    for (int k0 = 0; k0 < kb; k0 += rows_per_stage) {
        const int k1 = min(kb, k0 + rows_per_stage);
        if (k0 > 0) {
            __syncthreads();
            if constexpr (SHARDED) {
                stage_commit(sh_part, stage_issue_shards(a.part, (int64_t)a.B * K, (int64_t)b * K + k0, a.nsplit, (k1 - k0) * a.nsplit),
                             (k1 - k0) * a.nsplit);
            } else {
                stage_partials(sh_part, a.part + ((int64_t)b * K + k0) * a.nsplit, (k1 - k0) * a.nsplit);
                complete_stage(k0, (k1 - k0) * a.nsplit);
            }
        }
        for (int k = k0 + threadIdx.x; k < k1; k += kFinalBlock) {
            const int64_t i = (int64_t)b * K + k;
            const RowTotal r = merge_partials<true>(sh_part + (k - k0) * a.nsplit, a.nsplit);
            int32_t t = -1;
            float xt = NAN;
            if (want_tok) {
                t = a.draft_tok[i];
                if constexpr (SHARDED) {
                    // the shard that owns the token sent its logit; the others sent NaN
                    for (int g = 0; g < a.nsplit; ++g) {
                        const float v = __int_as_float(sh_part[(k - k0) * a.nsplit + g].pad[0]);
                        if (v == v) xt = v;
                    }
                } else if (t >= 0 && t < a.V) {
                    xt = load_elem_rt(row_address(a.base, a.dtype, a.stride_b, a.stride_k, b, k), a.dtype, t);
                }
            }
            const RowOut o = emit_row(a, i, r, want_tok, t, xt);
            if (a.arm) {
                const int arm_k = tok_mode ? a.arm[(int64_t)b * a.arm_stride + k] : arm;
                const bool ok_k = arm_k >= 0 && arm_k < a.n_arms;
                const int rule_k = ok_k ? pick8(a.rule, arm_k) : -1;
                if (sweep) sh_H[k] = o.H;
                if (rule_k == TAPOUT_RULE_SVIP_DIFF || rule_k == TAPOUT_RULE_ADAEDL) {
                    sh_dec[k] = 2;                             // decided below, once every row's entropy is known
                } else {
                    const bool fire = ok_k && rule_fires(rule_k, pick8(a.threshold, arm_k), o.H, o.p1, o.margin);
                    if (a.stop_fired) a.stop_fired[i] = fire ? 1 : 0;
                    sh_dec[k] = fire ? 1 : 0;                  // k < K <= kScanCap
                }
            }
            if (o.flags) atomicOr(&sh_flags, o.flags);
        }
    }
    __syncthreads();                       // orders the LDS / scratch writes above before the scan
    if (__builtin_expect(sweep, 0)) {
        for (int k = threadIdx.x; k < kb; k += kFinalBlock) {
            if (sh_dec[k] != 2) continue;
            const int arm_k = tok_mode ? a.arm[(int64_t)b * a.arm_stride + k] : arm;      // in range: checked when it was marked
            const bool fire = stateful_fires(a, b, arm_k, pick8(a.rule, arm_k), pick8(a.threshold, arm_k), sh_H[k], k > 0 ? sh_H[k - 1] : H_carry);
            if (a.stop_fired) a.stop_fired[(int64_t)b * K + k] = fire ? 1 : 0;
            sh_dec[k] = fire ? 1 : 0;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (a.flags) a.flags[b] = sh_flags;
        if (a.arm && a.n_stop) {
            int ns = kb;
            for (int k = 0; k < kb; ++k) {
                if (sh_dec[k] != 0) { ns = k + 1; break; }
            }
            a.n_stop[b] = ns;
        }
    }
}

constexpr size_t kLanesLds = 6 * kWave;

// The epilogue of sequence b where lane_merge_fits holds; called by all kFinalBlock threads of a workgroup.
template <bool SHARDED>
__device__ __forceinline__ void draft_finalize_on_lanes(const DraftFinalArgs &a, const int b, const int dtype)
{
    __shared__ __align__(16) unsigned char lds[kLanesLds];
    const int msh = lane_merge_shift(a.K, a.nsplit);
    if (__builtin_expect(a.K << msh > kFinalBlock, 0)) draft_finalize_lanes<SHARDED, false>(a, b, lds, dtype, msh);
    else draft_finalize_lanes<SHARDED, true>(a, b, lds, dtype, msh);
}
// The same where few_pieces holds, for a kernel that needs the registers for something else.
__device__ __forceinline__ void draft_finalize_few(const DraftFinalArgs &a, const int b, const int dtype)
{
    __shared__ __align__(16) unsigned char lds[kLanesLds];
    draft_finalize_lanes<false, true, true>(a, b, lds, dtype, lane_merge_shift(a.K, a.nsplit));
}
// The staged path's LDS.
constexpr size_t kStagedLds = sizeof(Partial) * kStageCap + 5 * kScanCap + 16;

}  // namespace tapout
