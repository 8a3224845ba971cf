// Sequence-level bandit over the stop rules (Section 3.3: UCB1, UCB-Tuned,
// Thompson Sampling with Beta or Gaussian posteriors) and the rewards of
// Section 3.2.  State: per bandit and arm the number of plays N, the summed
// reward S and the summed squared reward Q, in int64 / double.  The update also
// advances the carried state of the stateful stop rules of Appendix A.1
// (SVIP-Difference's previous entropy, AdaEDL's acceptance rate and thresholds).
// The work is O(B * arms) and never touches the vocabulary.  A thread per
// sequence, where a sequence's work is a short chain; the Gamma draws of Thompson
// Sampling take sixteen lanes per bandit, token-level updates a thread per
// position.
//
// This file is compiled without floating-point contraction: every product,
// quotient and sum below is a separately rounded IEEE double operation.
#include "common.h"
#include "bandit_device.h"

namespace tapout {

namespace {

// Sequence-level bandit: one thread per sequence.
__global__ void bandit_select_kernel(BanditArgs a, const float *u_ts, int32_t *arm_out, uint32_t *flags)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= a.B) return;
    arm_out[b] = select_arm(a, (size_t)(a.n_bandits == 1 ? 0 : b) * a.n_arms, u_ts);
    if (flags) flags[b] = 0u;
}

// Sequence-level Thompson Sampling with Beta posteriors, lane-parallel: the Marsaglia-Tsang loops of the 2 * arms
// Gamma variates of a sequence are long serial chains of double-precision log / sqrt / cos, so each gets a lane
// of its own (16 lanes per sequence: lane = 2 * arm + variate), the pair is combined with one lane exchange and
// the argmax runs over the sequence's 16 lanes.  Same operations per variate as the one-thread version, hence
// the same bits.
// `index`: the bandit's state and uniforms start at arm index * n_arms; !valid: idle group.  All 16 lanes must be active;
// every lane returns the arm, *exhausted is set in every lane if a sampler of the group ran out of attempts.
__device__ inline int ts_arm_lanes(const BanditArgs &a, bool valid, size_t index, int lane16, const float *u_ts, bool *exhausted)
{
    static_assert(TAPOUT_MAX_ARMS * 2 == 16, "16 lanes per bandit");
    const int arm = lane16 >> 1, which = lane16 & 1;
    const bool live = valid && arm < a.n_arms;
    double g = 1.0;
    bool ex = false;
    if (live) {
        const double S = a.sum_r[index * a.n_arms + arm], N = (double)a.count[index * a.n_arms + arm];
        const double shape = which == 0 ? 1.0 + S : 1.0 + (N - S);
        const float *ua = u_ts + (index * a.n_arms + arm) * TAPOUT_TS_UNIFORMS_PER_ARM + which * kAttempts * 3;
        g = gamma_draw(shape, ua, &ex);
    }
    // theta = g1 / (g1 + g2) on the even lane of each pair
    const double other = __shfl_xor(g, 1);
    double th = (live && which == 0) ? g / (g + other) : -INFINITY;
    int best = (live && which == 0) ? arm : 0x7fffffff;
    uint32_t exm = ex ? 1u : 0u;
    // argmax over the 16 lanes of the bandit; ties go to the lowest arm (the one-thread loop keeps the first maximum)
#pragma unroll
    for (int d = 2; d < 16; d <<= 1) {
        const double oth = __shfl_xor(th, d);
        const int ob = __shfl_xor(best, d);
        if (oth > th || (oth == th && ob < best)) { th = oth; best = ob; }
    }
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) exm |= __shfl_xor(exm, d);
    best = __shfl(best, (threadIdx.x & 63) & ~15);               // lanes 0 and 1 of the group hold the even lanes' argmax
    *exhausted = exm != 0;
    return best == 0x7fffffff ? 0 : best;
}

__global__ __launch_bounds__(64) void bandit_select_ts_kernel(BanditArgs a, const float *u_ts, int32_t *arm_out, uint32_t *flags)
{
    const int lane16 = threadIdx.x & 15;
    const int b = blockIdx.x * 4 + (threadIdx.x >> 4);
    bool ex;
    const size_t index = a.n_bandits == 1 ? 0 : b;
    const int arm = ts_arm_lanes(a, b < a.B, index, lane16, u_ts, &ex);
    if (b < a.B && lane16 == 0) {
        arm_out[b] = arm;
        if (flags) flags[b] = ex ? TAPOUT_FLAG_SAMPLER_EXHAUSTED : 0u;
    }
}

// The same for token-level bandits: one workgroup per sequence, sixteen lanes per draft position.  With a thread per
// position the Gamma variates of its arms were drawn one after the other: 48 sequences, K = 7, three arms 15.5 us, this 6.0.
__global__ __launch_bounds__(256) void bandit_select_token_ts_kernel(BanditArgs a, const float *u_ts, int32_t *arm_out, uint32_t *flags)
{
    __shared__ uint32_t sh_flag;
    const int b = blockIdx.x, lane16 = threadIdx.x & 15;
    if (threadIdx.x == 0) sh_flag = 0;
    __syncthreads();
    const size_t first = (size_t)(a.n_bandits == 1 ? 0 : b) * a.positions;
    for (int k0 = 0; k0 < a.positions; k0 += 16) {
        const int k = k0 + (int)(threadIdx.x >> 4);
        const bool valid = k < a.positions;
        bool ex;
        const size_t index = first + (valid ? k : 0);
        const int arm = ts_arm_lanes(a, valid, index, lane16, u_ts, &ex);
        if (valid && lane16 == 0) {
            arm_out[(size_t)b * a.positions + k] = arm;
            if (ex) atomicOr(&sh_flag, TAPOUT_FLAG_SAMPLER_EXHAUSTED);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && flags) flags[b] = sh_flag;
}

// Token-level bandits, the policies without Gamma draws: one workgroup per sequence, its threads take the positions.
__global__ void bandit_select_token_kernel(BanditArgs a, const float *u_ts, int32_t *arm_out, uint32_t *flags)
{
    const int b = blockIdx.x;
    for (int k = threadIdx.x; k < a.positions; k += blockDim.x)
        arm_out[(size_t)b * a.positions + k] = select_arm(a, ((size_t)(a.n_bandits == 1 ? 0 : b) * a.positions + k) * a.n_arms, u_ts);
    if (threadIdx.x == 0 && flags) flags[b] = 0u;
}

__global__ void bandit_update_kernel(BanditArgs a, const int32_t *arm, const int32_t *accept_len,
                                     const int32_t *n_draft, const int32_t *gamma, const uint8_t *active)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (a.n_bandits == 1) {
        // shared bandit: the B plays are applied in index order by one thread
        if (b == 0)
            for (int i = 0; i < a.B; ++i)
                if (playable(a, i, arm, n_draft, gamma, active)) apply_reward(a, 0, arm[i], accept_len[i], n_draft[i], gamma[i]);
    } else if (b < a.B && playable(a, b, arm, n_draft, gamma, active)) {
        apply_reward(a, b, arm[b], accept_len[b], n_draft[b], gamma[b]);
    }
    if (a.accept_rate && b < a.B && !(active && !active[b])) {
        const int n = n_draft[b];
        if (n >= 1 && (a.round_K == 0 || n <= a.round_K)) advance_rule_state(a, b, accept_len[b], n);
    }
}

// Token-level bandits: one thread per position.  With a bandit per sequence, thread b * positions + k plays position k of
// sequence b; with a shared one, thread k plays position k of every sequence, in index order.  A thread that took the
// positions of its sequence one after the other waited for memory at each: 48 sequences, K = 7 5.0 us, this 3.2.
__global__ __launch_bounds__(64) void bandit_update_token_kernel(BanditArgs a, const int32_t *arm, const int32_t *accept_len,
                                                                  const int32_t *n_draft, const int32_t *gamma, const uint8_t *active)
{
    const int P = a.positions, i = blockIdx.x * 64 + (int)threadIdx.x;
    const bool shared = a.n_bandits == 1;
    if (i < (shared ? 1 : a.B) * P) {
        const int k = i % P;
        for (int b = shared ? 0 : i / P, end = shared ? a.B : b + 1; b < end; ++b) {
            const int m = accept_len[b], n = n_draft[b], am = arm[(size_t)b * P + k];
            if (!playable(a, b, arm, n_draft, gamma, active) || k >= n || k > m || am < 0 || am >= a.n_arms) continue;
            const size_t at = (size_t)i * a.n_arms + am;          // [bandit, position, arm]
            const double r = k < m ? 1.0 : 0.0;                   // accepted, or the first rejected one; later positions were never evaluated
            a.count[at] += 1;
            a.sum_r[at] += r;
            a.sum_r2[at] += r;
        }
    }
    if (a.accept_rate && i < a.B && !(active && !active[i])) {
        const int n = n_draft[i];
        if (n >= 1 && (a.round_K == 0 || n <= a.round_K)) advance_rule_state(a, i, accept_len[i], n);
    }
}

// ---- update and next selection in one launch ---------------------------------------------------------
// Sequence-level bandits, one per sequence: the thread that applies sequence b's reward is the one that picks its
// next arm, so the selection reads the state it has just written (program order within a thread) and the round
// saves a launch.  Same operations as the two kernels: same bits.
__global__ void bandit_update_select_kernel(BanditArgs a, const int32_t *arm, const int32_t *accept_len,
                                            const int32_t *n_draft, const int32_t *gamma, const uint8_t *active,
                                            const float *u_ts, int32_t *arm_out, uint32_t *flags)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= a.B) return;
    update_select_one(a, b, arm, accept_len, n_draft, gamma, active, u_ts, arm_out, flags);
}

// The same for Thompson Sampling with Beta posteriors, lane-parallel (update_select_ts_lanes): four sequences per wavefront.
__global__ __launch_bounds__(64) void bandit_update_select_ts_kernel(BanditArgs a, const int32_t *arm_in, const int32_t *accept_len,
                                                                      const int32_t *n_draft, const int32_t *gamma, const uint8_t *active,
                                                                      const float *u_ts, int32_t *arm_out, uint32_t *flags)
{
    update_select_ts_lanes(a, blockIdx.x * 4 + (threadIdx.x >> 4), threadIdx.x & 15, arm_in, accept_len, n_draft, gamma, active, u_ts, arm_out, flags);
}

}  // namespace

// Update followed by the next selection.  One launch where every sequence has a sequence-level bandit of its own (or
// there is one sequence: bandit 0 either way); otherwise (shared bandit, token-level bandits) the two kernels one after the other.
hipError_t launch_bandit_update_select(const BanditArgs &a, const int32_t *arm, const int32_t *accept_len,
                                       const int32_t *n_draft, const int32_t *gamma, const uint8_t *active,
                                       const float *u_ts, int32_t *arm_out, uint32_t *flags, hipStream_t st, Timing tm)
{
    if (a.positions > 1 || (a.n_bandits == 1 && a.B > 1)) {
        hipError_t e = launch_bandit_update(a, arm, accept_len, n_draft, gamma, active, st, tm);
        if (e != hipSuccess) return e;
        return launch_bandit_select(a, u_ts, arm_out, flags, st, Timing{});
    }
    if (a.policy == TAPOUT_TS_BETA)
        launch_kernel(bandit_update_select_ts_kernel, dim3((a.B + 3) / 4), dim3(64), st, tm, a, arm, accept_len, n_draft, gamma, active, u_ts, arm_out, flags);
    else
        launch_kernel(bandit_update_select_kernel, dim3((a.B + 63) / 64), dim3(64), st, tm, a, arm, accept_len, n_draft, gamma, active, u_ts, arm_out, flags);
    return hipGetLastError();
}

hipError_t launch_bandit_select(const BanditArgs &a, const float *u_ts, int32_t *arm_out, uint32_t *flags, hipStream_t st, Timing tm)
{
    const int block = 64;
    if (a.positions > 1 && a.policy == TAPOUT_TS_BETA) launch_kernel(bandit_select_token_ts_kernel, dim3(a.B), dim3(256), st, tm, a, u_ts, arm_out, flags);
    else if (a.positions > 1) launch_kernel(bandit_select_token_kernel, dim3(a.B), dim3(block), st, tm, a, u_ts, arm_out, flags);
    else if (a.policy == TAPOUT_TS_BETA) launch_kernel(bandit_select_ts_kernel, dim3((a.B + 3) / 4), dim3(64), st, tm, a, u_ts, arm_out, flags);
    else launch_kernel(bandit_select_kernel, dim3((a.B + block - 1) / block), dim3(block), st, tm, a, u_ts, arm_out, flags);
    return hipGetLastError();
}

hipError_t launch_bandit_update(const BanditArgs &a, const int32_t *arm, const int32_t *accept_len,
                                const int32_t *n_draft, const int32_t *gamma, const uint8_t *active, hipStream_t st, Timing tm)
{
    const int block = 64;
    if (a.positions > 1) {
        const int plays = (a.n_bandits == 1 ? 1 : a.B) * a.positions, n = a.accept_rate && a.B > plays ? a.B : plays;
        launch_kernel(bandit_update_token_kernel, dim3((n + block - 1) / block), dim3(block), st, tm, a, arm, accept_len, n_draft, gamma, active);
        return hipGetLastError();
    }
    int grid = (a.n_bandits == 1 && !a.accept_rate) ? 1 : (a.B + block - 1) / block;
    launch_kernel(bandit_update_kernel, dim3(grid), dim3(block), st, tm, a, arm, accept_len, n_draft, gamma, active);
    return hipGetLastError();
}

}  // namespace tapout
