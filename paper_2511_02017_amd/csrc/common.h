// Internal declarations shared by the translation units of libtapout (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "tapout.h"

namespace tapout {

constexpr int kBlock = 256;          // threads per workgroup of the streaming kernels (4 wavefronts)
constexpr int kStreamU = 4;          // 16-byte vectors a thread of the streaming kernels has in flight (one batch)
constexpr int kWave = 64;
constexpr float kLog2e = 1.44269504088896340736f;   // binary32 nearest to log2(e); also used (widened) by the finalisers
constexpr double kLn2 = 0.693147180559945309417232121458;

// Partial statistics of one (row, split) slice, written by row_reduce and
// merged by the finalisers.  Sums are kept in the base-2 domain relative to an
// integer reference R = ceil(v1 * log2 e):  S = sum 2^(x*log2e - R),
// T = sum 2^(x*log2e - R) * (x*log2e - R).  Changing the reference by an
// integer is an exact power-of-two scaling, so merging loses nothing.
// Target rows: S runs over the whole slice.  Draft rows: S and T leave out the batch of vectors in which the
// slice's first maximum was met (see the streaming kernel); the epilogue adds that batch's elements back from the
// logits, the first maximum itself as an exact term.  Shard records: S and T leave out the first maximum element only.
struct Partial {
    float v1;        // slice maximum (NaN entries ignored), -inf for an empty slice
    float S;
    float T;         // draft rows only
    float v2;        // draft rows: the largest value outside the batch that S and T leave out (shard records: the second largest value, duplicates counted)
    int32_t cand;    // element index at which the 8- (bf16) / 4- (f32) element vector holding the first maximum starts
                     // (shard records: the global index of the first maximum itself)
    int32_t pad[3];  // pad[0]: bits of the logit of the row's token if the slice / shard holds it, else NaN
                     // pad[1]: draft rows: the left-out batch's own sum (binary32, same reference): S + it covers the slice
};
static_assert(sizeof(Partial) == 32, "Partial is one 32-byte record");
static_assert(sizeof(tapout_shard_stat) == sizeof(Partial), "shard records are staged and merged as partials");

// Final-token job of one sequence, produced by the verify finaliser and
// consumed by the residual sampler.
struct SampleJob {
    int32_t kind;    // 0: nothing to sample (greedy / flagged: token already written), 1: residual max(0,p-q), 2: target row only
    int32_t row;     // m: target row (and draft row for kind 1) to sample from
    float ref_p;     // exponent reference of the target row (its maximum)
    float ref_q;     // exponent reference of the draft row (its lse)
    double lam;      // binary32-grade estimate of S_p / S_q in those references (kind 1)
};


static_assert(sizeof(tapout_final_job) == sizeof(SampleJob), "the public job record is the internal one");

constexpr int kExpBf16Doubles = 4608;   // exp(x) of the bfloat16 values with 2^-12 <= |x| < 63.5, both signs, and two stand-in pairs (see the final-token slice kernel)

constexpr int kBandCap = 32;         // band elements per job the locate kernel settles one by one; more: exact slow path

// The job as it lies in memory, together with the list of elements of its row pair whose sign of a - L b is
// open until L is exact (appended by the slice kernel, read by the locate kernel).  One record, so that the
// locate kernel finds everything about its job in two neighbouring cache lines of one page.
struct JobRecord {
    SampleJob job;
    int32_t band_cnt;              // appended so far; entries beyond kBandCap are dropped (the count still grows)
    int32_t pad;
    int32_t band_idx[kBandCap];    // element indices, any order
};
static_assert(sizeof(JobRecord) == 160, "job record layout");

__host__ __device__ __forceinline__ float ref_of_max(float v1)
{
    // integer-valued reference >= v1*log2e; 0 for a slice without finite maximum
    return (v1 == -INFINITY) ? 0.0f : ceilf(v1 * kLog2e);
}

// Optional timing of one launch: when both events are set the kernel is launched through
// hipExtLaunchKernelGGL, which stamps them with the begin / end of the kernel's execution itself.
struct Timing {
    hipEvent_t start = nullptr, stop = nullptr;
};

struct RowReduceArgs {
    const void *base;
    int64_t stride_b, stride_k;   // elements
    int32_t V;
    int32_t KK;                   // rows per sequence in this tensor (K for draft, K+1 for target)
    int32_t nsplit;               // workgroups per row
    int32_t per;                  // 16-byte vectors per slice (multiple of 64; nsplit * per covers any row)
    int32_t n_rows;               // B * KK
    const int32_t *len;           // draft: k_len (or NULL); target: n_draft
    int32_t len_mode;             // 0: row k active iff k < len[b] (NULL: all); 1: iff k <= clamp(len[b], 1, KK-1)
    Partial *out;                 // [n_rows, nsplit]
    JobRecord *clear_jobs;        // NULL, or [B]: the first workgroup of sequence b empties the band list of its job record
    const int32_t *tok;           // NULL, or [B, tok_rows]: row k < tok_rows of sequence b has a token whose logit the
    int32_t tok_rows;             //   slice holding it puts into its partial (pad[0]; NaN bits in all other partials)
    const int32_t *arm_src;       // NULL, or [B] with arm_dst [B]: the first workgroup of sequence b copies the sequence's arm
    int32_t *arm_dst;             //   (a later launch overwrites the caller's array while another of its workgroups still wants the old value)
};
// Streaming pass: one Partial per (row, slice).  Returns hipGetLastError() after enqueueing.
hipError_t launch_row_reduce(const RowReduceArgs &a, int dtype, bool full, hipStream_t st, Timing tm);
// The records of a vocabulary shard's rows in one launch: `out` is [n_rows], nsplit 1; tok holds global indices, of which the shard's
// first is vocab_offset.
hipError_t launch_shard_records(const RowReduceArgs &a, int vocab_offset, int dtype, hipStream_t st, Timing tm);
// Wavefronts of a row's workgroup in that launch: four read its batches (kBlock * kStreamU vectors) one after the other, eight or sixteen share them.
// While there is no more than a workgroup to a compute unit they shorten the chain that the launch is (us per call, rows of 2 / 3 / 4 batches, 256
// rows, four wavefronts bfloat16 6.1 / 6.9 / 9.4, binary32 5.4 / 6.6 / 8.0, with more 5.3 / 6.2 / 7.2 and 4.5 / 5.8 / 6.2; 8 rows 5.45 / 6.3 / 7.6, 4.85 / 6.05 / 6.0); then
// their reductions get in each other's way (320 rows 6.5 / 8.2 / 10.2, 5.35 / 6.5 / 8.4, with more 6.6 / 8.8 / 9.8, 5.6 / 7.4 / 8.1), for long rows later: 512 rows of
// 4 batches 10.7 / 10.2, 576 rows 11.8 / 14.0.
inline int shard_record_waves(int64_t n_rows, int V, int vec)
{
    const int batch = kBlock * kStreamU, batches = (V / vec + batch - 1) / batch;
    if (batches <= 1) return 4;
    if (batches <= 3) return n_rows <= 256 ? (batches == 2 ? 8 : 16) : 4;
    return n_rows <= 512 ? 16 : 4;
}
// A shard's rows are read whole, by a workgroup each that writes the row's record; longer ones, and more of them, in slices that a launch behind the
// pass merges.  us per call, slices and merge / whole rows, bfloat16: 2 batches, 8 / 512 / 2048 rows 7.4 / 4.8, 9.9 / 7.1, 18.5 / 15.2; 4 batches 7.5 / 6.0, 12.9 / 10.1,
// 28.1 / 27.2.  Beyond 4 batches up to a workgroup to a compute unit: more rows gain where all of them are live, and lose in short drafts, whose
// few live rows then leave most of the chip idle (all live / a quarter: 8 batches, 8 rows a sequence, 256 rows 13.4 / 9.5 and 12.6 / 9.0, 512 rows 19.2 / 14.8 and
// 14.0 / 13.1, 1536 rows 43.4 / 36.7 and 20.7 / 27.2; 6 batches, 64 rows 8.8 / 7.8 and 8.1 / 7.6, 256 rows 11.8 / 8.5 and 9.2 / 8.2, 320 rows 13.3 / 11.6 and 10.1 / 11.1,
// 1024 rows 25.2 / 21.6 and 14.4 / 16.7; binary32, 8 batches, 256 rows 11.5 / 8.7 and 10.7 / 7.9, 1536 rows 37.0 / 33.1 and 18.5 / 23.7; 16 batches, 256 rows bfloat16 18.9 / 14.4 and
// 12.7 / 13.0, binary32 16.6 / 13.7 and 11.0 / 11.0, 320 rows 18.7 / 19.4 and 11.2 / 16.4).  One sequence of 8 batches 7.5 / 7.65.
inline bool shard_rows_whole(int64_t n_rows, int V, int vec)
{
    const int64_t batch = (int64_t)kBlock * kStreamU * vec;
    if (V <= 4 * batch) return true;
    return n_rows <= 256 && (V <= 6 * batch || (n_rows >= 64 && V <= 8 * batch));
}
// Draft pass (all statistics) and target pass of the same sequences in one launch.
hipError_t launch_row_reduce_pair(const RowReduceArgs &d, int d_dtype, const RowReduceArgs &t, int t_dtype, hipStream_t st, Timing tm);

struct DraftFinalArgs {
    const void *base; int32_t dtype; int64_t stride_b, stride_k;
    int32_t B, K, V, nsplit;
    int32_t per;                  // 16-byte vectors per slice of the streaming pass that wrote `part`
    const Partial *part;
    const int32_t *draft_tok, *k_len, *arm;
    int32_t arm_stride;           // 0: arm[b] decides every step; > 0 (token-level bandits): step k uses arm[b * arm_stride + k]
    int32_t n_arms; int32_t rule[TAPOUT_MAX_ARMS]; float threshold[TAPOUT_MAX_ARMS];
    float *lse, *entropy, *p_top1, *p_top2, *margin, *logq_tok;
    int32_t *top1_id, *n_stop; uint8_t *stop_fired; uint32_t *flags;
    // stateful rules (SVIP-Difference, AdaEDL); all NULL when the configuration has no such arm
    const float *prev_entropy;    // [B] entropy of the last drafted position of the previous draft, NaN = none
    const double *lambda;         // [B, n_arms] AdaEDL thresholds
    double adaedl_gamma;
    float *round_entropy;         // [B, K] entropies of this draft, kept for the state update
    // the library draws the draft tokens: a bad row gets none (BAD_TOKEN with BAD_ROW); sampled_lse, or NULL: where to leave each
    // row's lse, in double, for their log q
    int32_t sampling;
    double *sampled_lse;
    // vocabulary-sharded input: part holds the records of `shards` vocabulary shards, shard-major [shards, B*K], instead
    // of slice partials [B*K, nsplit] (then nsplit = shards; the argmax of a record is exact and global, the logit of
    // the drafted token travels in the record, and base is not used)
    int32_t shards;
};
hipError_t launch_draft_finalize(const DraftFinalArgs &a, hipStream_t st, Timing tm);

// The draft epilogue and the target pass up to the stop position it finds, in two launches: the first streams target rows 0 and 1, which
// are wanted whatever that position is, beside the epilogue, the second the rows behind them (not to be launched for K = 1).
constexpr int kFirstRows = 2;
hipError_t launch_epilogue_stream(const DraftFinalArgs &f, RowReduceArgs t, int t_dtype, hipStream_t st, Timing tm);
hipError_t launch_stream_rest(RowReduceArgs t, int t_dtype, hipStream_t st, Timing tm);

// A sequence's draft rows are so few pieces that the epilogue has two lanes for each or four (draft_lanes_shift): with one lane and four vectors each it
// takes 120 registers, with these 73 (binary32 57), which leave the streaming workgroups beside it their six wavefronts per SIMD.
inline bool few_pieces(int K, int nsplit)
{
    int p = 1;
    while (p < nsplit) p *= 2;
    return p <= 16 && K <= 64 && K * p <= 128;
}
// The epilogue streams the first target rows beside it while that is one or two rounds of workgroups (six or eight are resident per compute unit).
// us per round up to the stop position, V = 128256, bfloat16, 64 sequences, K = 8, apart / together 60.9 / 59.3 (92.0 / 89.1 diffuse rows,
// 57.6 / 54.1 Zipf-like ones), 24 sequences, K = 4 34.9 / 33.9 (36.4 / 33.9, 32.9 / 30.1); V = 256000, binary32, 32 sequences, K = 3
// 64.0 / 61.6 (63.4 / 56.6, 61.4 / 55.6); two lanes a piece, V = 128256, K = 8, bfloat16, 14 sequences 30.0 / 28.35, binary32, 8 sequences 29.7 / 26.75,
// V = 256000, bfloat16, 8 sequences 34.8 / 31.5, V = 50257, K = 16, bfloat16, 16 sequences 30.1 / 27.6; 1300 to
// 2000 workgroups, V = 32000, binary32, 90 sequences, K = 8 47.0 / 43.95, V = 100001, bfloat16, 90 sequences 66.5 / 63.8; 2700, 300 sequences, K = 3, V = 32000
// 55.3 / 51.8, V = 128256 124.1 / 117.0, binary32 190.5 / 184.9; 3600, 400 sequences, K = 2, V = 128256 127.9 / 129.2, V = 100001, binary32 165.1 / 166.5.
inline bool epilogue_streams(int B, int K, int d_nsplit, int t_nsplit) { return few_pieces(K, d_nsplit) && (int64_t)B * (1 + kFirstRows * t_nsplit) <= 3072; }

// One record per live row of a vocabulary shard from its slice partials (see tapout_shard_stats).
struct ShardMergeArgs {
    const void *base; int32_t dtype; int64_t stride_b, stride_k;
    int32_t B, KK, Vs, nsplit, per, vocab_offset, rows_mode;
    const Partial *part; const int32_t *len, *tok;
    Partial *out;
};
hipError_t launch_shard_merge(const ShardMergeArgs &a, hipStream_t st, Timing tm);

struct BanditArgs {
    int32_t policy, n_bandits, n_arms, B;
    int32_t positions;            // bandits per slot: 1 (sequence-level) or max_k (token-level, one per draft position)
    int32_t reward;               // tapout_reward
    double alpha;
    double *sum_r, *sum_r2; int64_t *count;
    // stateful stop rules (all NULL when the configuration has no such arm)
    int32_t rule[TAPOUT_MAX_ARMS];
    float *prev_entropy; double *accept_rate; double *lambda;
    const float *round_entropy; int32_t round_K;      // entropies of the last draft_stats call, [B, round_K]; round_K = 0: none
    double ad_alpha, ad_beta1, ad_beta2, ad_eps;
    int32_t ad_steer;             // tapout_config.adaedl_steer
};
// Kernel arguments sit in device memory and reach a wavefront through the scalar cache, one 64-byte line per miss,
// and the compiler loads a field where the code first wants it: a kernel that is a chain of round trips anyway takes
// a miss of this kind at several points along the chain (with the arguments in host memory instead, the final-token
// launches of a Llama-3-vocabulary round take 4.6 and 6.5 us longer).  Reading one word of every line first thing
// makes them one round trip; the later loads hit.  (The hidden arguments behind the declared ones, grid and
// workgroup sizes, are one more line: the kernels on the round's critical path do not read them.)
template <class T>
__device__ inline int32_t arg_lines(const T &a)
{
    const int32_t *w = reinterpret_cast<const int32_t *>(&a);
    int32_t acc = w[sizeof(T) / 4 - 1];
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; i += 16) acc |= w[i];
    return acc;
}
template <class... Ts>
__device__ inline void warm_args(const Ts &...as)
{
    const int32_t acc = (arg_lines(as) | ...);
    asm volatile("" :: "s"(acc));
}

// Verification + final token: the head kernel merges the target partials of each sequence, takes the
// accept decisions and describes the final-token draw (SampleJob); the slice kernel sums the row pair
// per slice; the locate kernel finds the token.
constexpr int32_t kVerifyOwnQ = 1;          // accept decisions form log q(tok) from the draft partials (see dpart)
constexpr int32_t kVerifyNoExpTable = 2;    // final-token slice kernel: computed exponentials also for bfloat16 row pairs
struct VerifyArgs {
    const void *tbase; int32_t t_dtype; int32_t vflags; int64_t t_stride_b, t_stride_k;   // vflags: kVerify* bits
    const void *dbase; int32_t d_dtype; int32_t d_nsplit; int64_t d_stride_b, d_stride_k;
    int32_t B, K, V, nsplit;      // nsplit: slices per row of the streaming pass
    int32_t nsl;                  // slices per row of the final-token passes (kSampleSlice elements each)
    int32_t shards;               // > 0: part holds records of vocabulary shards, shard-major [shards, B*(K+1)] (head kernel only)
    int32_t fused_head;           // 1: no head launch; every workgroup of the slice kernel works out its sequence's job itself
    SampleJob *final_jobs;        // sharded head: the job of every sequence for the caller (or NULL); sharded final token: the caller's jobs
    const Partial *part;
    const float *draft_lse, *logq_tok; const int32_t *draft_tok, *n_draft; const uint8_t *greedy;
    const float *u_accept, *u_sample;
    int32_t *accept_len, *out_tok, *n_out;
    float *target_lse, *logp_tok; int32_t *target_top1; uint32_t *flags;
    uint32_t *flags_ws;           // internal copy of the flags (always present)
    JobRecord *jobs;              // [B]
    double *part1;                // [B, nsl, 5]  A, B, R~, D, U of each slice
    double *part2;                // [B, nsl]     exact weight of each slice (slow path); slice launch of a shard: [B, 5] the sequences' sums
    const double *exp_table;      // 2^(k/256), k = 0..255, then the kExpBf16Doubles entries of the bfloat16 table
    // tapout_round: workgroups of the locate launch also end the round: rewards into the sequences' bandits
    // (arm b_arm_in[b], accept_len, n_draft, b_gamma, b_active as tapout_bandit_update) and the arms of the next round
    // (b_arm_out, b_flags as tapout_bandit_select).  Sequence-level bandits, one per sequence.
    int32_t bandit_tail;          // 0: no; 1: UCB1, UCB-Tuned; 2: Thompson Sampling with Beta posteriors
    BanditArgs bandit;
    const int32_t *b_arm_in, *b_gamma; const uint8_t *b_active; const float *b_u_ts; int32_t *b_arm_out; uint32_t *b_flags;
    // tapout_round with n_draft from the caller: the accept decisions form log q(tok) and the draft rows' lse themselves
    // from the draft pass's partials (kVerifyOwnQ; dpart [B*K, d_nsplit], whose token slots the draft pass filled), so the
    // draft epilogue can run beside the locate kernel, in the same launch (B more workgroups, ahead of the others).
    const Partial *dpart;
};
// fin: the draft epilogue's arguments when kVerifyOwnQ is set (pass 2 then runs it too), else NULL.
hipError_t launch_verify(const VerifyArgs &a, int pass /*0 head, 1 slices, 2 locate*/, hipStream_t st, Timing tm,
                         const DraftFinalArgs *fin = nullptr);
// The per-sequence kernels take their lane paths for `rows` rows of `nsplit` pieces (lane_merge_shift >= 0, for the host).
inline bool lane_merge_fits(int rows, int nsplit)
{
    if (nsplit > 16 || rows > 64) return false;
    int sh = 0;
    while ((1 << sh) < nsplit) ++sh;
    return (rows << sh) <= 512;
}
// ... and a workgroup has a lane for every piece.
inline bool lanes_in_one_pass(int rows, int nsplit)
{
    int sh = 0;
    while ((1 << sh) < nsplit) ++sh;
    return (rows << sh) <= kBlock;
}
// The accept decisions can take log q(tok) from the draft partials themselves (kVerifyOwnQ) for these shapes.
inline bool own_q_shape(int K, int nsplit_target, int nsplit_draft)
{
    return lane_merge_fits(K + 1, nsplit_target) && lane_merge_fits(K, nsplit_draft);
}

// Draft-token sampling (Algorithm 1, the sampling step of the draft loop): the inverse CDF of every live draft row.  The draft
// pass leaves the sums of exponentials it runs over beside its partials; a launch behind it finds the tokens.
// Sums of exp(x) in the logits' own scale are good for rows whose maximum lies between kDrawLow + 100 and kDrawHigh; others are summed again
// where their token is drawn.  bfloat16: the table holds values up to kTabEnd, and counts those from -kTabEnd down as 0, which is good
// beside a value of kDrawLowTab or more (each of them is below e^-43 of it; 256000 of them are 4e-14 of the sum, where a computed
// exponential is good to 2e-13).
constexpr float kDrawLow = -700.0f, kDrawHigh = 700.0f, kDrawLowTab = -20.0f, kTabEnd = 63.5f;
// Draw slices of a streaming slice of `per` vectors: kStreamU, of kBlock vectors each, in every batch it takes.
inline int draw_batches(int per) { return (per + kBlock * kStreamU - 1) / (kBlock * kStreamU); }
struct DrawArgs {
    double *sums;                 // [B * K, nsplit, nb, kStreamU, wavefronts of a workgroup]
    const double *exp_table;
    int32_t vflags;               // kVerifyNoExpTable
    int32_t nb;                   // batches per slice
    int32_t turns, step_b, step_k, step_s;      // (filled in by the launcher) slices per workgroup part, and the step from one to the next
};
// The draft pass (launch_row_reduce, full) with these sums.
hipError_t launch_stream_draw(const RowReduceArgs &a, int dtype, DrawArgs d, hipStream_t st, Timing tm);
struct SampleArgs {
    const void *base; int32_t dtype; int32_t vflags; int64_t stride_b, stride_k;
    int32_t B, K, V, nsplit, per, nb;      // how the draft pass cut the rows
    const Partial *part; const int32_t *k_len; const float *u;
    int32_t *tok; float *logq_tok;    // [B, K] token of each live row (-1: bad row) and its log q (or NULL)
    double *sums;                 // DrawArgs::sums; nb == 0: there are none, but room for a sum per kSampleSlice elements of every row
    const double *lse;            // [B * K] from the epilogue, or NULL: it runs beside this launch, and each row forms its own
    const double *exp_table;
};
// Tokens.  fin: the draft epilogue, to run in the same launch (a.lse NULL; where sample_own_lse holds), or NULL.
hipError_t launch_sample(const SampleArgs &a, const DraftFinalArgs *fin, hipStream_t st, Timing tm);
// Every row forms its lse itself while that costs no second round of workgroups (three are resident per compute unit: the epilogue's
// LDS and registers), and its pieces fit a wavefront.  (us per call, apart / in one launch, bfloat16, V = 32000: 576 workgroups 26.0 / 23.2, 765
// 33.6 / 29.7, 768 of one row a sequence 22.8 / 20.2; then 864 33.4 / 32.2, 1152 38.3 / 37.8, 1400 32.7 / 33.3, 2304 57.4 / 61.8; V = 128256 765
// 70.3 / 65.8, 864 73.0 / 71.6, 1152 83.0 / 86.3; binary32 765 99.8 / 97.1, 864 105.5 / 106.2, 1152 139.9 / 144.9.)
inline bool sample_own_lse(int B, int K, int nsplit) { return (int64_t)B * (K + 1) <= 768 && nsplit <= kWave; }

// Final token over vocabulary shards (see tapout_shard_final_sums / tapout_shard_final_token).  The VerifyArgs
// describe this shard's column slices (V = its width, nsl = its slices, jobs / part1 / part2 of the context).
struct ShardFinalArgs {
    VerifyArgs v;
    double *sums_out;             // [B, 5]                       (sums)
    const double *sums_all;       // [G, B, 5]                    (token)
    const double *exact_all;      // [G, B] or NULL               (token)
    int32_t G, g, vocab_offset;
    int32_t *tok_out; double *exact_mass; uint8_t *need_exact;
};
hipError_t launch_shard_final_sums(const ShardFinalArgs &a, hipStream_t st);
hipError_t launch_shard_final_token(const ShardFinalArgs &a, hipStream_t st);

constexpr int kSampleSlice = 2048;   // elements per slice of the final-token passes

hipError_t launch_bandit_select(const BanditArgs &a, const float *u_ts, int32_t *arm_out, uint32_t *flags, hipStream_t st, Timing tm);
hipError_t launch_bandit_update(const BanditArgs &a, const int32_t *arm, const int32_t *accept_len,
                                const int32_t *n_draft, const int32_t *gamma, const uint8_t *active, hipStream_t st, Timing tm);
hipError_t launch_bandit_update_select(const BanditArgs &a, const int32_t *arm, const int32_t *accept_len,
                                       const int32_t *n_draft, const int32_t *gamma, const uint8_t *active,
                                       const float *u_ts, int32_t *arm_out, uint32_t *flags, hipStream_t st, Timing tm);

// ---- device helpers --------------------------------------------------------
#ifdef __HIPCC__

template <class F, class... Args>
inline void launch_kernel(F kernel, dim3 grid, dim3 block, hipStream_t st, Timing tm, Args... args)
{
    if (tm.start && tm.stop) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, tm.start, tm.stop, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int DT> struct Elem;
template <> struct Elem<TAPOUT_F32>  { static constexpr int size = 4, vec = 4; };
template <> struct Elem<TAPOUT_BF16> { static constexpr int size = 2, vec = 8; };

__device__ inline float bf16_to_float(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

template <int DT>
__device__ inline float load_elem(const void *row, int64_t j)
{
    if constexpr (DT == TAPOUT_F32) return ((const float *)row)[j];
    else return bf16_to_float(((const uint16_t *)row)[j]);
}

__device__ inline float load_elem_rt(const void *row, int dtype, int64_t j)
{
    return dtype == TAPOUT_F32 ? ((const float *)row)[j] : bf16_to_float(((const uint16_t *)row)[j]);
}

// Split a row into an unaligned head, 16-byte vectors and a tail.
template <int DT>
__device__ inline void row_geometry(const void *row, int32_t V, int &head, int &nvec, int &tail)
{
    constexpr int VEC = Elem<DT>::vec;
    int mis = (int)(((uintptr_t)row & 15u) / Elem<DT>::size);
    head = (VEC - mis) % VEC;
    if (head > V) head = V;
    nvec = (V - head) / VEC;
    tail = V - head - nvec * VEC;
}

template <int DT>
__device__ inline void unpack(const u32x4 &w, float (&x)[Elem<DT>::vec])
{
    if constexpr (DT == TAPOUT_F32) {
        x[0] = __uint_as_float(w.x); x[1] = __uint_as_float(w.y);
        x[2] = __uint_as_float(w.z); x[3] = __uint_as_float(w.w);
    } else {
        x[0] = __uint_as_float(w.x << 16); x[1] = __uint_as_float(w.x & 0xffff0000u);
        x[2] = __uint_as_float(w.y << 16); x[3] = __uint_as_float(w.y & 0xffff0000u);
        x[4] = __uint_as_float(w.z << 16); x[5] = __uint_as_float(w.z & 0xffff0000u);
        x[6] = __uint_as_float(w.w << 16); x[7] = __uint_as_float(w.w & 0xffff0000u);
    }
}

__device__ inline const void *row_address(const void *base, int dtype, int64_t stride_b, int64_t stride_k, int b, int k)
{
    int64_t off = (int64_t)b * stride_b + (int64_t)k * stride_k;
    return (const char *)base + off * (dtype == TAPOUT_F32 ? 4 : 2);
}

// ---- reductions over the 2^(hi - lo) lanes that differ in bits lo .. hi - 1 of the lane number ---------------
// Commutative, every lane of a group ends with the same bits.  Steps 2 and 3 mirror half a row of sixteen lanes and a row:
// they also flip the lower bits, in which the lanes agree by then (already reduced, or copies of one piece).
// lo and hi are uniform.
template <int CTRL>
__device__ inline int dpp_mov(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }
template <int CTRL>
__device__ inline float dpp_mov(float v) { return __int_as_float(dpp_mov<CTRL>(__float_as_int(v))); }
template <int CTRL>
__device__ inline double dpp_mov(double v) { return __hiloint2double(dpp_mov<CTRL>(__double2hiint(v)), dpp_mov<CTRL>(__double2loint(v))); }
struct IntPair { int a, b; };
__device__ inline IntPair swap16(int v) { auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false); return {(int)r[0], (int)r[1]}; }
__device__ inline IntPair swap32(int v) { auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false); return {(int)r[0], (int)r[1]}; }
template <class F>
__device__ __forceinline__ int lanes_reduce_i(int v, int lo, int hi, F f)
{
    if (lo <= 0 && hi > 0) v = f(v, dpp_mov<0xB1>(v));
    if (lo <= 1 && hi > 1) v = f(v, dpp_mov<0x4E>(v));
    if (lo <= 2 && hi > 2) v = f(v, dpp_mov<0x141>(v));
    if (lo <= 3 && hi > 3) v = f(v, dpp_mov<0x140>(v));
    if (hi > 4) { const IntPair p = swap16(v); v = f(p.a, p.b); }          // the two values of a pair, in the same order in both lanes
    if (hi > 5) { const IntPair p = swap32(v); v = f(p.a, p.b); }
    return v;
}
__device__ __forceinline__ int lanes_min(int v, int lo, int hi) { return lanes_reduce_i(v, lo, hi, [](int x, int y) { return min(x, y); }); }
__device__ __forceinline__ float lanes_max(float v, int lo, int hi)                   // of the numbers: a NaN gives way
{
    return __int_as_float(lanes_reduce_i(__float_as_int(v), lo, hi, [](int x, int y) { return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(y))); }));
}
__device__ __forceinline__ double lanes_sum(double v, int lo, int hi)
{
    if (lo <= 0 && hi > 0) v += dpp_mov<0xB1>(v);
    if (lo <= 1 && hi > 1) v += dpp_mov<0x4E>(v);
    if (lo <= 2 && hi > 2) v += dpp_mov<0x141>(v);
    if (lo <= 3 && hi > 3) v += dpp_mov<0x140>(v);
    if (hi > 4) { const IntPair h = swap16(__double2hiint(v)), l = swap16(__double2loint(v)); v = __hiloint2double(h.a, l.a) + __hiloint2double(h.b, l.b); }
    if (hi > 5) { const IntPair h = swap32(__double2hiint(v)), l = swap32(__double2loint(v)); v = __hiloint2double(h.a, l.a) + __hiloint2double(h.b, l.b); }
    return v;
}
__device__ __forceinline__ void lanes_sum2(double &s, double &t, int lo, int hi)
{
    s = lanes_sum(s, lo, hi);
    t = lanes_sum(t, lo, hi);
}

constexpr int kStageCap = 256;     // partials staged in LDS at a time by an epilogue (8 KB)
constexpr int kScanCap = 4096;     // largest K: one stop / accept decision byte per draft position fits LDS

// All threads of the workgroup copy `count` partials (count <= kStageCap) into LDS; the loads of
// all threads are in flight together, so the copy costs one memory round trip.
__device__ inline void stage_partials(Partial *sh, const Partial *src, int count)
{
    const u32x4 *s = (const u32x4 *)src;
    u32x4 *d = (u32x4 *)sh;
    for (int i = threadIdx.x; i < 2 * count; i += kBlock) d[i] = s[i];      // (256-thread workgroups)
    __syncthreads();
}

// The same copy in two steps for a 256-thread workgroup, so that a caller can put other independent loads
// into the same memory round trip: stage_issue requests (at most two 16-byte words per thread, count <=
// kStageCap), stage_commit stores to LDS and synchronises.
struct StageRegs { u32x4 w0, w1; };
__device__ inline StageRegs stage_issue(const Partial *src, int count)
{
    const u32x4 *s = (const u32x4 *)src;
    StageRegs r;
    r.w0 = r.w1 = u32x4{0u, 0u, 0u, 0u};
    const int i = threadIdx.x;
    if (i < 2 * count) r.w0 = s[i];
    if (i + 256 < 2 * count) r.w1 = s[i + 256];
    return r;
}
__device__ inline void stage_commit(Partial *sh, const StageRegs &r, int count)
{
    u32x4 *d = (u32x4 *)sh;
    const int i = threadIdx.x;
    if (i < 2 * count) d[i] = r.w0;
    if (i + 256 < 2 * count) d[i + 256] = r.w1;
    __syncthreads();
}

// The same for records of vocabulary shards: src is shard-major [shards, rows_total]; the `count` = rows * shards
// records of rows row0 .. land in LDS row-major ([row][shard]), where merge_partials expects the slices of a row.
__device__ inline StageRegs stage_issue_shards(const Partial *src, int64_t rows_total, int64_t row0, int shards, int count)
{
    StageRegs r;
    r.w0 = r.w1 = u32x4{0u, 0u, 0u, 0u};
    const u32x4 *s = (const u32x4 *)src;
    const int i = threadIdx.x;                                 // 16-byte word i of the LDS image: record i/2, half i%2
    if (i < 2 * count) { const int rec = i >> 1; r.w0 = s[2 * ((int64_t)(rec % shards) * rows_total + row0 + rec / shards) + (i & 1)]; }
    if (i + 256 < 2 * count) { const int rec = (i + 256) >> 1; r.w1 = s[2 * ((int64_t)(rec % shards) * rows_total + row0 + rec / shards) + (i & 1)]; }
    return r;
}

// 2^f for |f| <= 1/2: the Taylor polynomial of exp(f ln 2) to the 13th power (remainder < 4e-18), evaluated in pairs so that
// the chain of dependent operations is six long.
__device__ inline double exp2_frac(double f)
{
    constexpr double c[14] = {1.0, 0.6931471805599453, 0.24022650695910072, 0.05550410866482158, 0.009618129107628477, 0.0013333558146428443, 0.0001540353039338161, 1.5252733804059841e-05, 1.321548679014431e-06, 1.01780860092397e-07, 7.054911620801123e-09, 4.4455382718708116e-10, 2.5678435993488206e-11, 1.3691488853904128e-12};
    const double f2 = f * f, f4 = f2 * f2;
    const double p0 = fma(c[1], f, c[0]), p1 = fma(c[3], f, c[2]), p2 = fma(c[5], f, c[4]), p3 = fma(c[7], f, c[6]);
    const double p4 = fma(c[9], f, c[8]), p5 = fma(c[11], f, c[10]), p6 = fma(c[13], f, c[12]);
    const double q0 = fma(p1, f2, p0), q1 = fma(p3, f2, p2), q2 = fma(p5, f2, p4);
    return fma(fma(fma(p6, f4, q2), f4, q1), f4, q0);
}
// 2^x for x <= 0 (also -inf; underflows to 0).
__device__ inline double exp2_neg(double x)
{
    x = fmax(x, -1100.0);
    const double n = rint(x);
    return ldexp(exp2_frac(x - n), (int)n);
}
// log2 x for x in the range of normal binary32 numbers: the hardware's binary32 logarithm y, then one step of Newton's method
// in double: log2 x = y + log2(1 + d), d = x 2^-y - 1, |d| < 4e-6.  Off by no more than 6e-16 and half a unit in the result's
// last place (exp2_frac is good to 1.3 units, and d carries that): an absolute bound, log2(1 + 1e-7) holds nine digits.  That is
// all its callers need: they add the result to an integer reference, or form it from 1 + eps, which is rounded to 1e-16
// itself.  The device library's functions, which are good to one unit and cover every argument, take several times the
// instructions, one after the other in a kernel that is nothing but latency.
__device__ inline double log2_pos(double x)
{
    const float y = __builtin_amdgcn_logf((float)x), n = rintf(y);
    const double d = fma(ldexp(x, -(int)n), exp2_frac((double)(n - y)), -1.0);
    constexpr double l = 1.4426950408889634;
    return (double)y + d * fma(d, fma(d, l / 3.0, -0.5 * l), l);
}
// 1 / x for normal x whose reciprocal is normal: the hardware's approximation (2^-24 or better) and two Newton steps.
__device__ inline double rcp_pos(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// v[i] for a small array that lives in scalar registers (kernel arguments): selects instead of a load from
// the argument buffer, which would be one more memory round trip.
template <class T>
__device__ inline T pick8(const T (&v)[TAPOUT_MAX_ARMS], int i)
{
    T r = v[0];
#pragma unroll
    for (int q = 1; q < TAPOUT_MAX_ARMS; ++q) r = (i == q) ? v[q] : r;
    return r;
}

// ---- merging the statistics of the pieces of a row ---------------------------------------------------
// A piece is one slice of a row (a Partial) or one vocabulary shard of it (a shard record).  Two kinds:
//   EXCL = false  S, T run over every element of the piece (target rows of the unsharded path);
//   EXCL = true   S, T leave the piece's first maximum element out (draft rows and all shard records): the entropy of a
//                 peaked row is made of small terms, and they must not share a binary32 sum with the dominant one.
//                 When two pieces meet, the maximum of the one that does not hold the row's maximum is an ordinary
//                 term again and is added in (binary32 exponential: it is either negligible or the row is not peaked);
//                 the row's own first maximum is added at the very end as an exact double term.
struct Piece {
    float M;          // maximum (-inf: no finite element)
    double S, T;      // base-2 sums relative to ref_of_max(M)
    float v2;         // second largest, duplicates counted
    int32_t idx;      // EXCL: index of the first maximum; else: start of the vector that holds it
    float xt;         // logit of the row's token if this piece holds it, else NaN
};

__device__ inline bool piece_empty(const Piece &e) { return e.M == -INFINITY && !(e.S != e.S); }

__device__ inline Piece empty_piece()
{
    Piece e;
    e.M = -INFINITY; e.S = 0.0; e.T = 0.0; e.v2 = -INFINITY; e.idx = 0x7fffffff; e.xt = NAN;
    return e;
}

__device__ inline Piece piece_from_words(const u32x4 &w0, const u32x4 &w1)
{
    Piece e;
    e.M = __uint_as_float(w0.x); e.S = (double)__uint_as_float(w0.y); e.T = (double)__uint_as_float(w0.z);
    e.v2 = __uint_as_float(w0.w); e.idx = (int32_t)w1.x; e.xt = __uint_as_float(w1.y);
    if (piece_empty(e)) { e.S = 0.0; e.T = 0.0; e.v2 = -INFINITY; e.idx = 0x7fffffff; }       // one image for every empty piece
    return e;
}
__device__ inline Piece piece_from_partial(const Partial &p)
{
    const u32x4 *w = (const u32x4 *)&p;
    return piece_from_words(w[0], w[1]);
}

// Commutative: both partners of an exchange compute the same bits.
template <bool EXCL>
__device__ inline Piece merge_pair(const Piece &a, const Piece &b)
{
    const bool a_wins = a.M > b.M || (a.M == b.M && a.idx <= b.idx);            // the piece with the row's first maximum
    const float Mw = a_wins ? a.M : b.M, Ml = a_wins ? b.M : a.M;
    const double Sw = a_wins ? a.S : b.S, Sl = a_wins ? b.S : a.S;
    const double Tw = a_wins ? a.T : b.T, Tl = a_wins ? b.T : a.T;
    const float Rw = ref_of_max(Mw);
    const double d = (double)Rw - (double)ref_of_max(Ml);                       // integer; >= 0 unless the other piece is empty
    const int di = d > 4000.0 ? 4000 : (d < -4000.0 ? -4000 : (int)d);          // 2^-4000 underflows to 0 as it should
    Piece o;
    o.M = Mw;
    o.S = Sw + ldexp(Sl, -di);                                                  // exact power-of-two scaling
    o.T = Tw + ldexp(Tl - d * Sl, -di);
    if constexpr (EXCL) {
        if (Ml > -INFINITY) {                                                   // the other piece's maximum: an ordinary term here
            const float y = __builtin_fmaf(Ml, kLog2e, -Rw);
            const float e = __builtin_amdgcn_exp2f(y);
            o.S += (double)e;
            o.T += (double)e * (double)fmaxf(y, -200.0f);
        }
    }
    o.v2 = fmaxf(fmaxf(fminf(a.M, b.M), a.v2), b.v2);                           // second largest of the union, duplicates counted
    o.idx = a_wins ? a.idx : b.idx;
    o.xt = (a.xt == a.xt) ? a.xt : b.xt;                                        // at most one piece holds the token
    return o;
}

// Merged statistics of a whole row, in double.
struct RowTotal {
    float M;          // row maximum
    double R;         // integer reference of M
    double Sx, Tx;    // the merged base-2 sums relative to R as the pieces carry them: EXCL: without the row's first maximum
    double yM;        // M log2e - R, in (-1, 0]
    double eM;        // EXCL: 2^yM to binary32 precision, the term of the first maximum; else 0
    double S;         // sum over ALL elements: Sx + eM
    float v2;
    int32_t cand;     // EXCL: index of the first maximum; else: start of the vector that holds it
    bool bad;
};

template <bool EXCL>
__device__ inline RowTotal row_total(const Piece &p)
{
    RowTotal r;
    r.M = p.M;
    r.R = (double)ref_of_max(p.M);
    const bool finite = p.M > -INFINITY && p.M < INFINITY;
    r.yM = finite ? (double)p.M * (double)kLog2e - r.R : 0.0;
    r.eM = (EXCL && finite) ? (double)__builtin_amdgcn_exp2f((float)r.yM) : 0.0;
    r.Sx = p.S; r.Tx = p.T;
    r.S = p.S + r.eM;
    r.v2 = p.v2; r.cand = p.idx;
    r.bad = !(r.S > 0.0) || !(r.S < INFINITY) || !finite;
    return r;
}

// Signals of a row whose sums leave the first maximum out (EXCL), written so that the binary32 error of eM and of the
// sums enters every result as a RELATIVE error, however peaked the row: with eps = Sx / eM (everything but the maximum,
// relative to it),
//   log2 sum_j 2^(x_j log2e) = R + yM + log2(1 + eps)          exactly: no eM in it
//   H / ln 2 = log2(1 + eps) + (yM eps - Tx / eM) / (1 + eps)
//   p_top1 = 1 / (1 + eps),  p_top2 = r2 p_top1,  margin = (1 - r2) p_top1,  r2 = 2^((v2 - M) log2e)  (double: a margin
//   between near-tied logits is the small difference 1 - r2)
// (log2(1 + eps) comes from the rounded 1 + eps: 6e-16 absolute, below binary32's relative rounding of H down to H = 1e-8.)
struct RowSignals { double lse, H, p1, p2, margin; };
__device__ inline RowSignals row_signals(const RowTotal &r, bool has_second)
{
    RowSignals o;
    const double inv = rcp_pos(r.eM), eps = r.Sx * inv;          // eM in (1/2, 1], eps below the vocabulary size
    const double l2 = log2_pos(1.0 + eps);
    o.p1 = rcp_pos(1.0 + eps);
    o.lse = (r.R + r.yM + l2) * kLn2;
    const double Hd = (l2 + (r.yM * eps - r.Tx * inv) * o.p1) * kLn2;
    o.H = Hd > 0.0 ? Hd : 0.0;
    const double r2 = has_second ? exp2_neg(((double)r.v2 - (double)r.M) * (double)kLog2e) : 0.0;
    o.p2 = r2 * o.p1;
    o.margin = (1.0 - r2) * o.p1;
    return o;
}

// The batch of vectors (or the single head / tail element) of the draft pass in which a slice met its first
// maximum, as the streaming kernel laid its work out: thread t of the slice's workgroup takes vectors
// v0 + t + q * kBlock, q = 0, 1, ..., in batches of kStreamU.  `cand` is the element index at which the vector with the
// first maximum starts (or the index of a head / tail element).  All addresses are checked against the slice.
struct BatchRegs {
    u32x4 w[kStreamU];
    uint32_t valid;       // bit u: vector u is wanted (the others hold stand-in data); bit 8: a single element, in `single`
    uint32_t single;      // bits of the single head / tail element
    int32_t first;        // element index of vector 0 (or of the single element)
    int32_t ucand;        // which vector of the batch the candidate is: the one that holds the first maximum
};

// Written so that the four requests are straight-line code at the end: where the branches above them only choose
// addresses (`safe`, any readable 16-byte aligned address, stands in for a vector that is not wanted; the valid bits
// tell), the compiler has no loaded registers to merge between branches.  With the requests inside the branches it
// merged them with the zeros of the other paths and waited for the data right there: a second memory round trip in a
// kernel that is nothing but round trips.
// What of it does not depend on the candidate comes apart (BatchGeom): a caller forms it while the partial travels.
struct BatchGeom {
    const char *row;
    int32_t head, nvec, v0, v1e;      // the row's unaligned elements and whole vectors; the slice's vectors [v0, v1e)
};
__device__ __forceinline__ BatchGeom batch_geom(const void *row, int dtype, int32_t V, int split, int per)
{
    const int esz = dtype == TAPOUT_F32 ? 4 : 2, vsh = dtype == TAPOUT_F32 ? 2 : 3, VEC = 1 << vsh;
    BatchGeom g;
    g.row = (const char *)row;
    const int mis = (int)(((uintptr_t)row & 15u) / (unsigned)esz);              // as row_geometry
    g.head = min((VEC - mis) & (VEC - 1), V);
    g.nvec = (V - g.head) >> vsh;
    g.v0 = min(split * per, g.nvec);
    g.v1e = min(g.v0 + per, g.nvec);
    return g;
}
__device__ inline BatchRegs batch_issue(const BatchGeom &g, int dtype, int32_t V, int32_t cand, const void *safe)
{
    const int esz = dtype == TAPOUT_F32 ? 4 : 2, vsh = dtype == TAPOUT_F32 ? 2 : 3;
    BatchRegs b;
    b.valid = 0; b.first = 0; b.ucand = 0; b.single = 0;
    // (device memory, and said so: chosen among several pointers the compiler would otherwise treat them as generic
    // addresses, whose loads also count as LDS traffic)
    typedef const __attribute__((address_space(1))) u32x4 *GlobalVec;
    GlobalVec p[kStreamU];
#pragma unroll
    for (int u = 0; u < kStreamU; ++u) p[u] = (GlobalVec)safe;
    if (cand >= 0 && cand < V) {
        if (cand < g.head || cand >= g.head + (g.nvec << vsh)) {
            b.single = __float_as_uint(load_elem_rt(g.row, dtype, cand));
            b.valid = 0x100u; b.first = cand;
        } else {
            const int i = (cand - g.head) >> vsh, rel = i - g.v0;
            if (rel >= 0 && i < g.v1e) {                                        // else: not a candidate of this slice: stale record
                constexpr int kSpan = kBlock * kStreamU;                        // vectors of a batch; thread t holds every kBlock-th
                static_assert((kSpan & (kSpan - 1)) == 0 && (kBlock & (kBlock - 1)) == 0, "masks below");
                const int i0 = g.v0 + (rel & ~(kSpan - 1)) + (rel & (kBlock - 1));      // the thread's vector 0 of the batch
                GlobalVec vp = (GlobalVec)(g.row + (int64_t)g.head * esz);
                b.first = g.head + (i0 << vsh);
                b.ucand = (rel & (kSpan - 1)) / kBlock;
#pragma unroll
                for (int u = 0; u < kStreamU; ++u) {
                    const int iu = i0 + u * kBlock;
                    p[u] = vp + min(iu, g.v1e - 1);                             // v0 <= i <= v1e - 1: inside the slice
                    b.valid |= iu < g.v1e ? 1u << u : 0u;
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < kStreamU; ++u) b.w[u] = *p[u];
    return b;
}

__device__ inline BatchRegs batch_issue(const void *row, int dtype, int32_t V, int32_t cand, int split, int per, const void *safe)
{
    return batch_issue(batch_geom(row, dtype, V, split, per), dtype, V, cand, safe);
}

// The same split over the lanes of a piece: NV of the batch's kStreamU vectors, from vector u0 on.
template <int NV>
struct BatchVecs {
    u32x4 w[NV];
    uint32_t valid;       // bit n: vector n is wanted; bit 8: a single head / tail element, in w[0].x (the lane with u0 == 0)
    int32_t first;        // element index of the lane's vector 0 (or of the single element)
    int32_t search;       // which of the lane's vectors the candidate is (else outside 0 .. NV - 1)
};
template <int NV>
__device__ __forceinline__ BatchVecs<NV> batch_issue_vecs(const BatchGeom &g, int dtype, int32_t V, int32_t cand, int u0, const void *safe)
{
    const int esz = dtype == TAPOUT_F32 ? 4 : 2, vsh = dtype == TAPOUT_F32 ? 2 : 3;
    BatchVecs<NV> b;
    b.valid = 0; b.first = 0; b.search = -1;
    typedef const __attribute__((address_space(1))) u32x4 *GlobalVec;          // (see batch_issue)
    GlobalVec p[NV];
#pragma unroll
    for (int n = 0; n < NV; ++n) p[n] = (GlobalVec)safe;
    uint32_t single = 0;
    if (cand >= 0 && cand < V) {
        const int i = (cand - g.head) >> vsh, rel = i - g.v0;
        if (__builtin_expect(cand < g.head || i >= g.nvec, 0)) {
            if (u0 == 0) { single = __float_as_uint(load_elem_rt(g.row, dtype, cand)); b.valid = 0x100u; b.first = cand; }
        } else if (rel >= 0 && i < g.v1e) {                                      // else: not a candidate of this slice: stale record
            constexpr int kSpan = kBlock * kStreamU;
            const int i0 = g.v0 + (rel & ~(kSpan - 1)) + (rel & (kBlock - 1)) + u0 * kBlock;
            GlobalVec vp = (GlobalVec)(g.row + (int64_t)g.head * esz);
            b.first = g.head + (i0 << vsh);
            b.search = (rel & (kSpan - 1)) / kBlock - u0;
#pragma unroll
            for (int n = 0; n < NV; ++n) {
                const int iu = i0 + n * kBlock;
                p[n] = vp + min(iu, g.v1e - 1);
                b.valid |= iu < g.v1e ? 1u << n : 0u;
            }
        }
    }
#pragma unroll
    for (int n = 0; n < NV; ++n) b.w[n] = *p[n];
    if (b.valid & 0x100u) b.w[0].x = single;
    return b;
}

// The elements of a piece's left-out batch, except the first one equal to the piece's maximum M: their two sums
// relative to ref_of_max(M) (binary32 terms as in the streaming pass: they are small, or the row is not peaked) and
// the index of that first maximum (0x7fffffff if the batch does not hold it).  m2: the largest of these elements (with the
// partial's v2, the largest value outside the batch, it makes the piece's second maximum).
struct BatchExtra { float sa, ta; int32_t idx; float m2; };

// The first maximum lies in the candidate vector (the thread's running maximum reached M there: the vectors before it
// in the batch are below M, equal values after it are duplicates and count as ordinary terms), so only that vector is
// searched.  The entropy terms are formed without looking at them; a masked (-inf) logit makes their sum NaN
// (0 * -inf), and only then they are formed again with the exponent clamped.
template <int DT>
__device__ inline BatchExtra batch_extra_t(float M, const BatchRegs &b)
{
    constexpr int VEC = Elem<DT>::vec;
    const float R = ref_of_max(M);
    BatchExtra o;
    o.sa = 0.0f; o.ta = 0.0f; o.idx = 0x7fffffff; o.m2 = -INFINITY;
    auto sums = [&](bool clamp) {
        float sa = 0.0f, ta = 0.0f, m2 = -INFINITY;
        int32_t idx = 0x7fffffff;
        if (b.valid & 0x100u) {
            const float x = __uint_as_float(b.single);
            if (x == M) idx = b.first;
            else {
                const float y = __builtin_fmaf(x, kLog2e, -R), e = __builtin_amdgcn_exp2f(y);
                sa = e; ta = e * (clamp ? fmaxf(y, -200.0f) : y);
                m2 = x;
            }
        }
#pragma unroll
        for (int u = 0; u < kStreamU; ++u) {
            if (!((b.valid >> u) & 1u)) continue;
            float x[VEC];
            unpack<DT>(b.w[u], x);
            const bool search = u == b.ucand;
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const bool first = search && x[j] == M && idx == 0x7fffffff;
                const float y = __builtin_fmaf(x[j], kLog2e, -R);
                const float e = first ? 0.0f : __builtin_amdgcn_exp2f(y);
                if (search) idx = first ? b.first + u * kBlock * VEC + j : idx;
                m2 = fmaxf(m2, first ? -INFINITY : x[j]);
                sa += e;
                ta = __builtin_fmaf(e, clamp ? fmaxf(y, -200.0f) : y, ta);
            }
        }
        o.sa = sa; o.ta = ta; o.idx = idx; o.m2 = m2;
    };
    sums(false);
    if (o.ta != o.ta) sums(true);
    return o;
}
__device__ inline BatchExtra batch_extra(const Piece &p, const BatchRegs &b, int dtype)
{
    if (piece_empty(p) || !b.valid) { BatchExtra o; o.sa = 0.0f; o.ta = 0.0f; o.idx = 0x7fffffff; o.m2 = -INFINITY; return o; }
    return dtype == TAPOUT_F32 ? batch_extra_t<TAPOUT_F32>(p.M, b) : batch_extra_t<TAPOUT_BF16>(p.M, b);
}

// A vector's maximum, and its second largest value, duplicates counted; NaN values are passed over (v_med3 of a NaN is the
// lesser of the other two).  Each is one block of instructions: a statement per instruction makes the compiler put a wait
// state after each.
__device__ __forceinline__ float vector_max(const float (&x)[1]) { return x[0]; }
__device__ __forceinline__ float vector_max(const float (&x)[4])
{
    float m;
    asm("v_max3_f32 %0, %1, %2, %3\n\tv_max_f32 %0, %0, %4" : "=&v"(m) : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]));
    return m;
}
__device__ __forceinline__ float vector_max(const float (&x)[8])
{
    float m;
    asm("v_max3_f32 %0, %1, %2, %3\n\tv_max3_f32 %0, %0, %4, %5\n\tv_max3_f32 %0, %0, %6, %7\n\tv_max_f32 %0, %0, %8"
        : "=&v"(m)
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
    return m;
}
__device__ __forceinline__ float vector_second(const float (&x)[4])
{
    float first, second, a;
    asm("v_max_f32 %0, %3, %4\n\tv_med3_f32 %1, %7, %3, %4\n\tv_med3_f32 %2, %0, %5, %6\n\tv_max_f32 %1, %1, %2"
        : "=&v"(first), "=&v"(second), "=&v"(a) : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(-INFINITY));
    return second;
}
__device__ __forceinline__ float vector_second(const float (&x)[8])
{
    float first, second, a;
    asm("v_max_f32 %0, %3, %4\n\tv_med3_f32 %1, %11, %3, %4\n\tv_med3_f32 %2, %0, %5, %6\n\tv_max_f32 %1, %1, %2\n\tv_max3_f32 %0, %0, %5, %6\n\t"
        "v_med3_f32 %2, %0, %7, %8\n\tv_max_f32 %1, %1, %2\n\tv_max3_f32 %0, %0, %7, %8\n\tv_med3_f32 %2, %0, %9, %10\n\tv_max_f32 %1, %1, %2"
        : "=&v"(first), "=&v"(second), "=&v"(a)
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]), "v"(-INFINITY));
    return second;
}

// Sums of a lane's vectors of a left-out batch in the row's reference R; excl: the piece holds the row's first maximum M,
// which stays out and whose index is idx.  (See batch_extra_t for the search and the masked logits.)
template <int DT, int NV>
__device__ __forceinline__ BatchExtra batch_sum(float R, float M, bool excl, const BatchVecs<NV> &b, int u0)
{
    constexpr int VEC = Elem<DT>::vec;
    BatchExtra o;
    // the candidate vector, if this lane has it: where its first maximum is, and what comes next
    u32x4 ws = b.w[0];
#pragma unroll
    for (int n = 1; n < NV; ++n) ws = b.search == n ? b.w[n] : ws;
    const bool search = excl && b.search >= 0 && ((b.valid >> (b.search & (NV - 1))) & 1u) != 0 && b.search < NV;
    int at = -1;
    {
        float x[VEC];
        unpack<DT>(ws, x);
#pragma unroll
        for (int j = VEC - 1; j >= 0; --j) at = x[j] == M ? j : at;            // the lowest one stays
        at = search ? at : -1;
        o.m2 = at >= 0 ? vector_second(x) : -INFINITY;
    }
    const int32_t found = at >= 0 ? b.first + b.search * (kBlock * VEC) + at : 0x7fffffff;
    // (the other vectors' maxima)
#pragma unroll
    for (int n = 0; n < NV; ++n) {
        float x[VEC];
        unpack<DT>(b.w[n], x);
        o.m2 = ((b.valid >> n) & 1u) != 0 && !(at >= 0 && n == b.search) ? fmaxf(o.m2, vector_max(x)) : o.m2;
    }
    asm volatile("" : "+v"(o.m2));
    auto sums = [&](bool clamp) {
        float sa[2] = {0.0f, 0.0f}, ta[2] = {0.0f, 0.0f};
        int32_t idx = found;
#pragma unroll
        for (int n = 0; n < NV; ++n) {
            const bool on = (b.valid >> n) & 1u;
            const u32x4 w = {on ? b.w[n].x : 0u, on ? b.w[n].y : 0u, on ? b.w[n].z : 0u, on ? b.w[n].w : 0u};   // stand-in data may be anything
            float x[VEC];
            unpack<DT>(w, x);
            const int skip = NV == 1 || n == b.search ? at : -1;
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const float y = __builtin_fmaf(x[j], kLog2e, -R);
                const float e = (on && j != skip) ? __builtin_amdgcn_exp2f(y) : 0.0f;
                sa[j & 1] += e;
                ta[j & 1] = __builtin_fmaf(e, clamp ? fmaxf(y, -200.0f) : y, ta[j & 1]);
            }
        }
        if (__builtin_expect(b.valid & 0x100u, 0)) {
            const float x = __uint_as_float(b.w[0].x);
            if (excl) idx = b.first;
            else {
                const float y = __builtin_fmaf(x, kLog2e, -R), e = __builtin_amdgcn_exp2f(y);
                sa[0] += e;
                ta[0] = __builtin_fmaf(e, clamp ? fmaxf(y, -200.0f) : y, ta[0]);
            }
        }
        o.sa = sa[0] + sa[1]; o.ta = ta[0] + ta[1]; o.idx = idx;
    };
    sums(false);
    if (o.ta != o.ta) sums(true);
    return o;
}

// Completes a piece of the draft pass: the left-out batch back in, all but the first maximum, whose index becomes idx.
__device__ inline void batch_fix(Piece &p, const BatchRegs &b, int dtype)
{
    const BatchExtra x = batch_extra(p, b, dtype);
    p.S += (double)x.sa; p.T += (double)x.ta;
    p.idx = x.idx; p.v2 = fmaxf(p.v2, x.m2);
}

// Sequential merge of the `n` pieces of one row held as Partials (LDS or memory) at stride `stride` records.
// EXCL pieces must have been completed (batch_fix) before: idx exact, only the first maximum left out.
template <bool EXCL>
__device__ inline RowTotal merge_partials(const Partial *p, int n, int stride = 1)
{
    Piece acc = empty_piece();
    for (int s = 0; s < n; ++s) acc = merge_pair<EXCL>(acc, piece_from_partial(p[(int64_t)s * stride]));
    return row_total<EXCL>(acc);
}

// ---- records of a row's pieces on neighbouring lanes -------------------------------------------------
template <int CTRL>
__device__ inline Piece piece_dpp(const Piece &e)
{
    auto mv = [](int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); };
    Piece o;
    o.M = __int_as_float(mv(__float_as_int(e.M)));
    o.S = __hiloint2double(mv(__double2hiint(e.S)), mv(__double2loint(e.S)));
    o.T = __hiloint2double(mv(__double2hiint(e.T)), mv(__double2loint(e.T)));
    o.v2 = __int_as_float(mv(__float_as_int(e.v2)));
    o.idx = mv(e.idx);
    o.xt = __int_as_float(mv(__float_as_int(e.xt)));
    return o;
}

// log2 of the lanes per row, one for each of its `nsplit` pieces (1, 2, 4, 8 or 16), that the per-sequence kernels' lane
// paths use for `rows` rows, or -1 where they do not apply (then partials are staged in LDS and merged one by one): the
// rows of a sequence fit two passes of one workgroup, and a wavefront's ballots.
__device__ inline int lane_merge_shift(int rows, int nsplit)
{
    if (nsplit > 16 || rows > 64) return -1;
    const int sh = nsplit <= 1 ? 0 : 32 - __clz(nsplit - 1);
    return (rows << sh) <= 512 ? sh : -1;
}

// The pieces of the 2^sh lanes of a group combined; every lane of the group returns the same bits.
template <bool EXCL>
__device__ inline Piece lane_group_merge(Piece e, int sh)
{
    // quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror: each pairs groups that already agree
    if (sh >= 1) e = merge_pair<EXCL>(e, piece_dpp<0xB1>(e));
    if (sh >= 2) e = merge_pair<EXCL>(e, piece_dpp<0x4E>(e));
    if (sh >= 3) e = merge_pair<EXCL>(e, piece_dpp<0x141>(e));
    if (sh >= 4) e = merge_pair<EXCL>(e, piece_dpp<0x140>(e));
    return e;
}

// First index j in [cand, cand + window) with x_j == M (the lowest argmax index of the row), in two steps so
// that a caller can put other work between the request and the use of the window.
struct ArgmaxProbe { u32x4 w; bool loaded; };
__device__ inline ArgmaxProbe argmax_issue(const void *row, int dtype, int32_t V, int32_t cand)
{
    ArgmaxProbe pr;
    pr.w = u32x4{0u, 0u, 0u, 0u};
    pr.loaded = false;
    if (cand < 0 || cand >= V) return pr;
    const int window = dtype == TAPOUT_F32 ? 4 : 8;
    const char *p = (const char *)row + (int64_t)cand * (dtype == TAPOUT_F32 ? 4 : 2);
    if ((((uintptr_t)p) & 15u) == 0 && cand + window <= V) {
        // the usual case: the window is one of the 16-byte vectors the streaming pass loaded; one load
        pr.w = *(const u32x4 *)p;
        pr.loaded = true;
    }
    return pr;
}
__device__ inline int32_t argmax_finish(const ArgmaxProbe &pr, const void *row, int dtype, int32_t V, int32_t cand, float M)
{
    if (cand < 0 || cand >= V) return 0;
    const int window = dtype == TAPOUT_F32 ? 4 : 8;
    float x[8];
    if (pr.loaded) {
        const u32x4 w = pr.w;
        const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (dtype == TAPOUT_F32) { x[i] = __uint_as_float(ww[i]); x[4 + i] = NAN; }
            else { x[2 * i] = __uint_as_float(ww[i] << 16); x[2 * i + 1] = __uint_as_float(ww[i] & 0xffff0000u); }
        }
    } else {
        // unaligned head / tail elements of a row
#pragma unroll
        for (int i = 0; i < 8; ++i)
            x[i] = (i < window && cand + i < V) ? load_elem_rt(row, dtype, cand + i) : NAN;
    }
    int32_t hit = cand;
#pragma unroll
    for (int i = 7; i >= 0; --i)
        if (x[i] == M) hit = cand + i;
    return hit;
}
__device__ inline int32_t resolve_argmax(const void *row, int dtype, int32_t V, int32_t cand, float M)
{
    return argmax_finish(argmax_issue(row, dtype, V, cand), row, dtype, V, cand, M);
}

#endif  // __HIPCC__

}  // namespace tapout
