// Verification of the drafted tokens and the final token (Algorithm 1, lines
// 10-11; "verify" = speculative sampling as in the works the paper cites).
//
// After the streaming pass over the target rows (row_reduce.hip) three small
// launches finish the job:
//
//   head    one workgroup per sequence merges the target partials, forms
//           log p(tok), takes the accept decisions u < p(tok)/q(tok), finds the
//           first rejection m, emits the accepted tokens and describes the draw
//           of the final token (row pair (m, m), or target row n alone)
//   slices  per 2048-element slice of the row pair, in double: A = sum a_j,
//           B = sum b_j (a = exp(t - ref_p), b = exp(d - ref_q)) and, with the
//           head's binary32-grade estimate L~ of L = S_p / S_q:
//           R~ = sum max(0, a_j - L~ b_j), D = sum of b_j over a_j > L~ b_j,
//           U = sum of b_j over the band |a_j - L~ b_j| <= eta L~ b_j; the
//           indices of the band elements (a handful: the band is 1e-5 wide) go
//           to a short per-sequence list
//   locate  one workgroup per sequence: exact L = sum A / sum B; the slice
//           weights of the residual max(0, a - L b) are R~ - (L - L~) D, which
//           is exact for every element whose sign of a - L b is the same at L~
//           and at L; an element can change sign only inside the band (given
//           |L - L~| <= eta L~, which is checked), where it is off by at most
//           |L - L~| b_j: in total at most |L - L~| * sum U.  If that bound is
//           below 2e-10 of the total weight (typically it is 1e-12) the sums
//           are used as they are.  If a heavy token sits in the band, the
//           listed elements are evaluated one by one with the exact L and
//           their slices corrected.  Then the slice holding u * Z is found
//           from the slice weights and the token by an exact scan inside it.
//           If the list overflowed (ratios tied inside the band, p == q), L~ is
//           off or Z vanishes, the slice weights are recomputed exactly first
//           (slow path).
//
// token = smallest j whose inclusive prefix sum exceeds u * Z.  Everything is
// double precision: with ~1e5 CDF cell edges in [0,1) a binary32 evaluation
// would move an edge across u for about one draw in a hundred; in double the
// chance is ~1e-10, so the token agrees with a sequential fp64 evaluation.
// Only one row pair per sequence is touched (2/(2K+1) of the round's logits),
// with two exponentials per element.  exp() is 2^(n/256) * (1 + r + r^2/2 +
// r^3/6), |r| <= ln2/512, with a 256-entry table in LDS: relative error
// < 2e-13, far inside what the 1e-9 decision margin needs, at a third of the
// instructions of a correctly rounded exp; row pairs of bfloat16 logits take
// exp(x) itself from a table of all bfloat16 values a softmax row can hold.
#include "common.h"
#include "bandit_device.h"
#include "exp_device.h"
#include "finalize_device.h"

namespace tapout {

// Per-workgroup time stamps (a build with -DTAPOUT_WG_STAMPS only: `python -m paper_2511_02017_amd.build --stamps`
// makes libtapout_stamps.so beside the library proper, `python -m paper_2511_02017_amd.wg_stamps` runs it).  The first
// thread of a workgroup stores the 100 MHz wall clock at a few points of the final-token kernels; the table a stamp goes
// to and its slots are listed with the reader at the end of this file.  Stamps stretch what they measure (each is a scalar
// memory instruction the wavefront waits for: a few tenths of a microsecond); the library proper has none of this.
#ifdef TAPOUT_WG_STAMPS
constexpr int kStampWgs = 1 << 16;
__device__ unsigned long long g_stamps_slices[kStampWgs * 8];      // slice kernel, by linear workgroup index
__device__ unsigned long long g_stamps_head[kStampWgs * 4];        // accept decisions inside it, same index
__device__ unsigned long long g_stamps_locate[4096 * 8];           // locate kernel (and the draft epilogue's workgroups in its launch)
#define HEAD_STAMP_BY(who, slot) do { if (who) g_stamps_head[WG_LINEAR() * 4 + (slot)] = wall_clock64(); } while (0)
#define WG_LINEAR() ((int)(((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) & (kStampWgs - 1)))
#define WG_STAMP(table, per, wg, slot) do { if (threadIdx.x == 0) table[(wg) * (per) + (slot)] = wall_clock64(); } while (0)
#define WG_STAMP_LANE0(table, per, wg, slot) do { if ((threadIdx.x & (kWave - 1)) == 0) table[(wg) * (per) + (slot)] = wall_clock64(); } while (0)
#else
#define WG_LINEAR() 0
#define HEAD_STAMP_BY(who, slot) do {} while (0)
#define WG_STAMP(table, per, wg, slot) do {} while (0)
#define WG_STAMP_LANE0(table, per, wg, slot) do {} while (0)
#endif
#define HEAD_STAMP(slot) HEAD_STAMP_BY(threadIdx.x == 0, slot)
#define LOCATE_STAMP(slot) WG_STAMP(g_stamps_locate, 8, (int)(blockIdx.x & 4095), slot)

namespace {

constexpr int kVBlock = 256;
static_assert(kVBlock == kBlock, "stage_partials strides by kBlock");
constexpr int kPer = 8;                       // elements per 16-byte (bf16) / 32-byte (f32) run



// Eight consecutive elements j .. j+7 of a row as they lie in memory (one 16-byte vector of bfloat16, two of binary32;
// -inf beyond V), so that a kernel can hold several requests in flight in few registers and widen them, exactly, when
// their turn comes.
template <int DT> struct Raw8 { u32x4 w[DT == TAPOUT_F32 ? 2 : 1]; };
// Sixteen bytes at an element's address: one request whatever the alignment (the target's memory mode allows it; a
// vector across two cache lines costs a second access).  Rows of an odd vocabulary size start at every alignment, and
// element loads there made the slice kernel wait for memory several times per vector (V = 50257, 48 sequences, bfloat16
// draft and binary32 target rows: 22.6 us with element loads, 14.4 with these; locate kernel 8.0 / 6.9).
typedef uint32_t u32x4_at2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_at4 __attribute__((ext_vector_type(4), aligned(4)));
template <int DT>
__device__ inline u32x4 load16(const char *p)
{
    if constexpr (DT == TAPOUT_F32) return *(const u32x4_at4 *)p;
    else return *(const u32x4_at2 *)p;
}
template <int DT>
__device__ inline Raw8<DT> load_raw8(const char *rowp, int j, int V)
{
    Raw8<DT> r;
    if (j + kPer <= V) {
        r.w[0] = load16<DT>(rowp + (int64_t)j * Elem<DT>::size);
        if constexpr (DT == TAPOUT_F32) r.w[1] = load16<DT>(rowp + (int64_t)j * 4 + 16);
    } else if (j >= V) {
        // beyond the row: nothing to load (the usual case in a row's last slice)
        constexpr uint32_t ninf = DT == TAPOUT_BF16 ? 0xff80ff80u : 0xff800000u;
#pragma unroll
        for (int h = 0; h < (DT == TAPOUT_F32 ? 2 : 1); ++h) r.w[h] = u32x4{ninf, ninf, ninf, ninf};
    } else {
        uint32_t e[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) e[i] = __float_as_uint((j + i < V) ? load_elem<DT>(rowp, j + i) : -INFINITY);
        if constexpr (DT == TAPOUT_BF16) {
            r.w[0] = u32x4{(e[0] >> 16) | (e[1] & 0xffff0000u), (e[2] >> 16) | (e[3] & 0xffff0000u),
                           (e[4] >> 16) | (e[5] & 0xffff0000u), (e[6] >> 16) | (e[7] & 0xffff0000u)};
        } else {
            r.w[0] = u32x4{e[0], e[1], e[2], e[3]}; r.w[1] = u32x4{e[4], e[5], e[6], e[7]};
        }
    }
    return r;
}
template <int DT>
__device__ inline void widen8(const Raw8<DT> &r, float (&x)[kPer])
{
    if constexpr (DT == TAPOUT_BF16) {
        unpack<TAPOUT_BF16>(r.w[0], x);
    } else {
        float lo[4], hi[4];
        unpack<TAPOUT_F32>(r.w[0], lo); unpack<TAPOUT_F32>(r.w[1], hi);
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[i] = lo[i]; x[4 + i] = hi[i]; }
    }
}

// ---- head: accept decisions of one sequence -----------------------------------------
// verify_head_lanes and verify_head_staged are called by all 256 threads of a workgroup.  They return the sequence's job
// (identical in every workgroup of the sequence); with `writer` they also write the sequence's outputs.
//
// kVerifyOwnQ (whole-round calls, lane-path shapes only): log q(tok) and the draft rows' lse are not read from the draft
// epilogue's outputs, which then need not exist yet, but formed here from the draft pass's partials: a draft partial's S
// leaves out the batch with the slice's first maximum, pad[1] holds that batch's own sum in the same reference, so S +
// pad[1] is the sum over the whole slice (binary32 precision, which a ratio p/q compared with a uniform needs no more
// than); the token's logit was left in pad[0] of the slice that holds it.
//
// shT: 256 doubles of LDS for the table of exp_fast, which this function fills (each thread requests its entry with the
// first requests and stores it ahead of the first barrier): the two exponentials on the critical path take 13
// instructions each instead of a call into the device library.
//
// request_table(): called once, where the caller's copy of its table to LDS may start (the slice kernel's; it may lie over
// `stg`): on the lane path right behind this function's own first requests (loads return in order).  The copy is complete
// and published when this function returns.
struct NoTable { __device__ void operator()() const {} };
constexpr uint32_t kFatal = TAPOUT_FLAG_BAD_NDRAFT | TAPOUT_FLAG_BAD_TOKEN | TAPOUT_FLAG_BAD_ROW;

// LDS of the decisions on either path.
struct HeadRow { double lse; float M, dl; int32_t top1, tok; };             // what the job and the outputs want of a target row
struct HeadLanes { HeadRow rows[kWave]; uint8_t dec[kWave], flag[kWave]; };
struct HeadStaged {
    Partial part[kStageCap];
    uint8_t dec[kScanCap];                  // accept decisions exist for rows k < n <= K <= kScanCap
    uint32_t flags;
    int32_t bcast[8];
    double lse;
};

// One row's decision: t the drafted token, u its uniform, lq its log q, xt its target logit.
struct Accept { bool yes; float lp; uint32_t flags; };
__device__ inline Accept accept_row(const VerifyArgs &a, bool bad, double lse, bool greedy, int32_t t, float u, float lq, float xt, int32_t top1, const double *shT)
{
    Accept o{false, NAN, 0u};
    if (__builtin_expect(t < 0 || t >= a.V, 0)) o.flags = TAPOUT_FLAG_BAD_TOKEN;
    else if (!bad) {
        o.lp = (float)((double)xt - lse);
        if (greedy) o.yes = t == top1;
        else {
            // (NaN: the ratio is then 0, which no uniform is below)
            o.yes = (double)u < exp_fast_d((double)o.lp - (double)lq, shT);
        }
    }
    return o;
}

// The sequence's job: row m, its maximum Mm and lse, the draft row's lse dl.
__device__ inline SampleJob head_job(bool draws, int m, int n, float Mm, double lse_m, float dl_m, bool have_dl, const double *shT)
{
    SampleJob job;
    job.kind = 0; job.row = 0; job.ref_p = 0.0f; job.ref_q = 0.0f; job.lam = 0.0;
    if (draws) {
        job.kind = m < n ? 1 : 2;
        job.row = m;
        job.ref_p = Mm;                          // exponent references: the target row's maximum, the draft row's lse
        job.ref_q = (m < n && have_dl) ? dl_m : 0.0f;
        // binary32-grade estimate of S_p / S_q in these references (S_q = sum exp(d - lse_q) = 1): lets the
        // slice pass form the residual before the exact normalisers exist
        job.lam = exp_fast_d(lse_m - (double)Mm, shT);
    }
    return job;
}

// The sequence's outputs but for the rows'; tok(k): the drafted token of row k.
template <bool SHARDED, class Tok>
__device__ inline void head_outputs(const VerifyArgs &a, int b, const SampleJob &job, int m, int n, bool flagged, bool greedy, uint32_t f, int32_t top1m, Tok tok)
{
    const int K = a.K;
    const int32_t final_tok = (flagged || greedy) ? top1m : -1;   // sampled sequences: written by pass 3
    if (threadIdx.x == 0) {
        a.accept_len[b] = m;
        a.n_out[b] = m + 1;
        if constexpr (!SHARDED) {
            a.jobs[b].job = job;
            // the slice kernel appends to the sequence's band list; fused into that kernel, this workgroup
            // cannot empty the list under the others' appends: the target pass has done it
            if (!a.fused_head) a.jobs[b].band_cnt = 0;
            a.flags_ws[b] = f;
        } else if (a.final_jobs) {
            a.final_jobs[b] = job;
        }
        if (a.flags) a.flags[b] = f;
    }
    int32_t *o = a.out_tok + (int64_t)b * (K + 1);
    for (int k = threadIdx.x; k <= K; k += kVBlock) {
        o[k] = k < m ? tok(k) : (k == m ? final_tok : -1);
        if (flagged && a.logp_tok && k < n) a.logp_tok[(int64_t)b * K + k] = NAN;
    }
}

// Few rows and slices (lane_merge_shift): 2^msh lanes per target row, one piece each; they find the row's maximum, bring
// their sums to its reference and add them up, the draft row of the same position beside it (kVerifyOwnQ), and every
// lane takes the row's decision: no LDS on the way to it, and one barrier behind it, after which every wavefront finds
// the first rejection for itself.  An instruction costs a wavefront here about nine cycles whatever it is: see
// draft_finalize_lanes.  (Pairwise merges of whole records, rows and draft rows handed to a thread per row through LDS, the
// first rejection published by a second barrier, and the table through registers: slice kernel with the decisions, V = 128256,
// 64 sequences, up to the stop position 17.4 us, this 15.9; head launch at 256 sequences, K = 16 7.0 / 5.6.)
template <bool SHARDED, class Table>
__device__ inline SampleJob verify_head_lanes(const VerifyArgs &a, int b, bool writer, HeadLanes *sh, double *shT, Table request_table, const int msh, const int turn)
{
    const int K = a.K, tid = threadIdx.x, lane = tid & (kWave - 1), sl = tid & ((1 << msh) - 1), per_pass = kVBlock >> msh;
    // The rows go to the wavefronts from the `turn`-th on, and a wavefront without a row waits at the barrier: the workgroups of a compute
    // unit put their wavefronts on the same four SIMDs, and one wavefront or two is all that most drafts need.  (us per round, rows clamped to the
    // last one in all wavefronts / this: V = 32000, 32 sequences 24.06 / 23.81, V = 128256, 64 sequences 68.4 / 68.2.)
    const int wave0 = __builtin_amdgcn_readfirstlane(((tid / kWave - turn) & (kVBlock / kWave - 1)) * kWave), vt = wave0 + lane;
    // Everything whose address does not depend on n_draft is requested before n_draft is looked at, so that
    // the first memory round trip carries n_draft, the tokens, the uniforms and the partials together.
    // (Rows beyond n_draft hold stale partials and unused tokens: read, never used.)
    // n_draft and greedy are requested as vector loads (the index carries a zero the compiler cannot
    // see through): a scalar load would share its counter with the loads of kernel arguments, and the first wait
    // for one of those would wait for memory.
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    int n = a.n_draft[b + zero];
    uint8_t greedy_raw = a.greedy ? a.greedy[b + zero] : (uint8_t)0;
    const double tv = a.exp_table[tid];
    const bool own_q = !SHARDED && (a.vflags & kVerifyOwnQ) != 0;          // (the host offers it for shapes that take this path on both sides)
    bool greedy = false;
    uint32_t f0 = 0;
    for (int row0 = 0; row0 <= K; row0 += per_pass) {                      // one pass but for long drafts of many slices
        const bool busy = row0 + (wave0 >> msh) <= K;
        const int row = row0 + (vt >> msh), row_t = min(row, K), row_d = min(row, K - 1);
        const int64_t it = (int64_t)b * (K + 1) + row_t, i = (int64_t)b * K + row_d;
        u32x4 w0{}, w1{};
        float qv1 = -INFINITY, qS = 0.0f, qx = NAN, qh = 0.0f, u = 0.0f, lq = 0.0f, dl = 0.0f;
        int32_t tok = -1;
        if (busy) {
            const u32x4 *pt = (const u32x4 *)(SHARDED ? a.part + (int64_t)min(sl, a.nsplit - 1) * a.B * (K + 1) + it : a.part + it * a.nsplit + min(sl, a.nsplit - 1));
            w0 = pt[0]; w1 = pt[1];
            tok = a.draft_tok[i];
            u = a.u_accept[i];
            if (own_q) {
                const Partial *pd = a.dpart + i * a.d_nsplit + min(sl, a.d_nsplit - 1);
                qv1 = pd->v1; qS = pd->S; qx = __int_as_float(pd->pad[0]); qh = __int_as_float(pd->pad[1]);
            } else {
                lq = a.logq_tok[i];
                if (a.draft_lse) dl = a.draft_lse[i];                      // the final token's job wants it for row m: no dependent load later
            }
        }
        if (row0 == 0) request_table();
        asm volatile("" :: "v"(w0), "v"(w1), "v"(tok), "v"(u), "v"(qv1), "v"(qS), "v"(qx), "v"(qh));     // every request is out before the first wait
        HEAD_STAMP_BY(vt == 0, 0);                                        // first requests answered
        if (row0 == 0) {
            shT[tid] = tv;
            n = __builtin_amdgcn_readfirstlane(n);
            if (__builtin_expect(n < 1 || n > K, 0)) { f0 = TAPOUT_FLAG_BAD_NDRAFT; n = n < 1 ? 1 : K; }
            greedy = __builtin_amdgcn_readfirstlane((int)greedy_raw) != 0;
            __syncthreads();                                               // the table: every row's decision reads it
        }
        if (!busy) continue;
        // target row: maximum, sum and (start of the vector that holds) its first maximum.  Slice partials run over every
        // element of their slice; shard records leave their maximum out.
        const bool mine = sl < a.nsplit;
        const float v1 = mine ? __uint_as_float(w0.x) : -INFINITY;
        float S = mine ? __uint_as_float(w0.y) : 0.0f;
        if (v1 == -INFINITY && !(S != S)) S = 0.0f;
        Piece p;
        p.M = lanes_max(v1, 0, msh);
        const float R = ref_of_max(p.M);
        p.S = ldexp((double)S, -(int)fminf(fmaxf(R - ref_of_max(v1), -4000.0f), 4000.0f));
        if (S == 0.0f) p.S = 0.0;                                          // (0 * inf)
        const bool holds = mine && v1 == p.M;
        p.idx = lanes_min(holds ? (int32_t)w1.x : 0x7fffffff, 0, msh);
        if constexpr (SHARDED)
            if (!(holds && (int32_t)w1.x == p.idx) && v1 > -INFINITY) p.S += (double)__builtin_amdgcn_exp2f(__builtin_fmaf(v1, kLog2e, -R));
        p.S = lanes_sum(p.S, 0, msh);
        p.T = 0.0; p.v2 = 0.0f;
        p.xt = lanes_max(mine ? __uint_as_float(w1.y) : NAN, 0, msh);      // the piece that holds the token put its logit there, the others NaN
        const RowTotal r = row_total<SHARDED>(p);
        double lse = NAN;
        uint32_t f = 0;
        if (__builtin_expect(r.bad, 0)) f = TAPOUT_FLAG_BAD_ROW;
        else lse = (r.R + log2_pos(r.S)) * kLn2;
        if (own_q) {
            const bool has = sl < a.d_nsplit;
            qv1 = has ? qv1 : -INFINITY;
            float s = has ? qS + qh : 0.0f;
            if (qv1 == -INFINITY && !(s != s)) s = 0.0f;
            const float qM = lanes_max(qv1, 0, msh), qR = ref_of_max(qM);
            double qs = ldexp(has ? (double)qS + (double)qh : 0.0, -(int)fminf(fmaxf(qR - ref_of_max(qv1), -4000.0f), 4000.0f));
            if (s == 0.0f) qs = 0.0;
            qs = lanes_sum(qs, 0, msh);
            const float x = lanes_max(has ? qx : NAN, 0, msh);
            const bool bad = !(qs > 0.0) || !(qs < INFINITY) || !(qM > -INFINITY && qM < INFINITY);
            const double lse_q = bad ? (double)NAN : ((double)qR + log2_pos(qs)) * kLn2;
            lq = (float)((double)x - lse_q);
            dl = (float)lse_q;
        }
        HEAD_STAMP_BY(vt == 0, 1);                                        // row merged
        const bool lead = sl == 0 && row <= n;
        int32_t top1 = (SHARDED && r.cand >= 0 && r.cand < a.V) ? r.cand : 0;      // a shard's argmax is exact and global
        // Greedy sequences decide on the argmax; the others only report it: their leading lane looks at the window last.
        const void *row_p = SHARDED ? nullptr : row_address(a.tbase, a.t_dtype, a.t_stride_b, a.t_stride_k, b, row_t);
        ArgmaxProbe probe;
        if constexpr (!SHARDED) {
            if (lead && (writer || greedy)) {
                probe = argmax_issue(row_p, a.t_dtype, a.V, r.cand);
                if (greedy) top1 = argmax_finish(probe, row_p, a.t_dtype, a.V, r.cand, r.M);
            }
        }
        Accept acc{false, NAN, 0u};
        if (row < n) acc = accept_row(a, r.bad, lse, greedy, tok, u, lq, p.xt, top1, shT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                   // (the table's copy, before this wavefront's first stores)
        if (lead) {
            if constexpr (!SHARDED)
                if (writer && !greedy) top1 = argmax_finish(probe, row_p, a.t_dtype, a.V, r.cand, r.M);
            sh->dec[row] = acc.yes ? 1 : 0;
            sh->flag[row] = (uint8_t)(f | acc.flags);
            HeadRow h;
            h.lse = lse; h.M = r.M; h.dl = dl; h.top1 = top1; h.tok = tok;
            sh->rows[row] = h;
            if (writer) {
                if (row < n && a.logp_tok) a.logp_tok[i] = acc.lp;
                if (a.target_lse) a.target_lse[it] = (float)lse;
                if (a.target_top1) a.target_top1[it] = top1;
            }
        }
        HEAD_STAMP_BY(vt == 0, 2);                                        // lse, log p(tok), accept decision
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                       // the table's copy
    __syncthreads();
    // rows are lanes of every wavefront: ballots give the first rejection and the flags
    const uint64_t acc_mask = __builtin_amdgcn_ballot_w64(lane < n && sh->dec[lane] != 0);
    const uint32_t fl = lane <= n ? sh->flag[lane] : 0u;
    uint32_t f = f0;
    if (__builtin_amdgcn_ballot_w64((fl & TAPOUT_FLAG_BAD_TOKEN) != 0)) f |= TAPOUT_FLAG_BAD_TOKEN;
    if (__builtin_amdgcn_ballot_w64((fl & TAPOUT_FLAG_BAD_ROW) != 0)) f |= TAPOUT_FLAG_BAD_ROW;
    const bool flagged = (f & kFatal) != 0;
    const int m = flagged ? 0 : __builtin_ctzll(~acc_mask | (1ull << n));  // first draft position that was not accepted, n if there is none (n <= 63 here)
    const HeadRow h = sh->rows[m];                                         // a flagged sequence has m = 0 and emits the argmax of row 0
    HEAD_STAMP(3);                                                         // first rejection known
    const SampleJob job = head_job(!flagged && !greedy, m, n, h.M, h.lse, h.dl, a.draft_lse || own_q, shT);
    if (writer) head_outputs<SHARDED>(a, b, job, m, n, flagged, greedy, f, h.top1, [&](int k) { return sh->rows[k].tok; });
    return job;
}

// Any number of rows and pieces: kStageCap partials at a time in LDS, one row per thread.  In a launch of its own the first memory
// round trip carries, as on the lane path, all that does not depend on n_draft: the first stage's partials, and token, uniform,
// log q and lse of the thread's first row; further stages ask for these ahead of their partials, and the argmax window travels
// while the logarithm is formed.  (Asked for row by row behind the merge, as the slice kernel does: V = 50257, 200 sequences,
// K = 66 6.2 us, this 5.5; in the slice kernel itself the early requests' registers cost the lane path scalar spills: one
// sequence, V = 32000, round 20.0 us without them, 20.5 with them.)
template <bool SHARDED, class Table>
__device__ inline SampleJob verify_head_staged(const VerifyArgs &a, int b, bool writer, HeadStaged *sh, double *shT, Table request_table)
{
    constexpr bool kOwnLaunch = std::is_same_v<Table, NoTable>;
    const int K = a.K, rows_per_stage = kStageCap / a.nsplit;
    int zero = 0;
    if constexpr (kOwnLaunch) asm volatile("v_mov_b32 %0, 0" : "=v"(zero));          // (vector loads: see verify_head_lanes)
    int n = a.n_draft[b + zero];
    const uint8_t greedy_raw = a.greedy ? a.greedy[b + zero] : (uint8_t)0;
    const double tv = a.exp_table[threadIdx.x];
    int32_t tok0 = -1;                                                               // kOwnLaunch: of row k0 + threadIdx.x of the stage in LDS
    float u0 = 0.0f, lq0 = 0.0f, dl0 = 0.0f;
    auto request_row = [&](int k) {
        if (k >= K) return;
        const int64_t i = (int64_t)b * K + k;
        tok0 = a.draft_tok[i]; u0 = a.u_accept[i]; lq0 = a.logq_tok[i];
        if (a.draft_lse) dl0 = a.draft_lse[i];
    };
    auto stage = [&](int k0, int count) {
        if constexpr (SHARDED) return stage_issue_shards(a.part, (int64_t)a.B * (K + 1), (int64_t)b * (K + 1) + k0, a.nsplit, count);
        else return stage_issue(a.part + ((int64_t)b * (K + 1) + k0) * a.nsplit, count);
    };
    {
        const int c0 = min(K + 1, rows_per_stage) * a.nsplit;
        if constexpr (kOwnLaunch) request_row(threadIdx.x);
        const StageRegs st = stage(0, c0);
        shT[threadIdx.x] = tv;
        if (threadIdx.x == 0) { sh->flags = 0; sh->bcast[4] = 0; }         // ahead of the barrier: rows of other wavefronts OR into the flags
        stage_commit(sh->part, st, c0);
    }
    if constexpr (kOwnLaunch) n = __builtin_amdgcn_readfirstlane(n);
    const bool greedy = kOwnLaunch ? __builtin_amdgcn_readfirstlane((int)greedy_raw) != 0 : greedy_raw != 0;
    if (n < 1 || n > K) {
        if (threadIdx.x == 0) atomicOr(&sh->flags, TAPOUT_FLAG_BAD_NDRAFT);
        n = n < 1 ? 1 : K;
    }
    const bool need_top1 = writer || greedy;
    int last_k = -1; float last_M = 0.0f, last_dl = 0.0f; int32_t last_top1 = 0; double last_lse = 0.0;   // the last row this thread merged
    for (int k0 = 0; k0 <= n; k0 += rows_per_stage) {
        const int k1 = min(n + 1, k0 + rows_per_stage);
        if (k0 > 0) {
            if constexpr (kOwnLaunch) request_row(k0 + threadIdx.x);
            __syncthreads();
            stage_commit(sh->part, stage(k0, (k1 - k0) * a.nsplit), (k1 - k0) * a.nsplit);
        }
        for (int k = k0 + threadIdx.x; k < k1; k += kVBlock) {
            const int64_t it = (int64_t)b * (K + 1) + k, i = (int64_t)b * K + k;
            // shard records leave their first maximum out of the sums (and carry its exact index), slice partials of
            // target rows do not
            const RowTotal r = merge_partials<SHARDED>(sh->part + (k - k0) * a.nsplit, a.nsplit);
            const void *row_p = SHARDED ? nullptr : row_address(a.tbase, a.t_dtype, a.t_stride_b, a.t_stride_k, b, k);
            int32_t top1 = 0;
            ArgmaxProbe probe;
            if constexpr (SHARDED) top1 = (r.cand >= 0 && r.cand < a.V) ? r.cand : 0;
            else if (need_top1) {
                if constexpr (kOwnLaunch) probe = argmax_issue(row_p, a.t_dtype, a.V, r.cand);
                else top1 = resolve_argmax(row_p, a.t_dtype, a.V, r.cand, r.M);
            }
            double lse = NAN;
            uint32_t f = 0;
            if (r.bad) f |= TAPOUT_FLAG_BAD_ROW;
            else lse = (r.R + log2_pos(r.S)) * kLn2;
            if constexpr (!SHARDED && kOwnLaunch)                                    // greedy sequences decide on it, the others only report it
                if (greedy) top1 = argmax_finish(probe, row_p, a.t_dtype, a.V, r.cand, r.M);
            if (k < n) {
                float xt = NAN;
                for (int g = 0; g < a.nsplit; ++g) {
                    const float v = __int_as_float(sh->part[(k - k0) * a.nsplit + g].pad[0]);
                    if (v == v) xt = v;
                }
                Accept acc;
                if constexpr (kOwnLaunch) {
                    if (__builtin_expect(k != k0 + (int)threadIdx.x, 0)) request_row(k);      // more rows than threads
                    acc = accept_row(a, r.bad, lse, greedy, tok0, u0, lq0, xt, top1, shT);
                } else acc = accept_row(a, r.bad, lse, greedy, a.draft_tok[i], a.u_accept[i], a.logq_tok[i], xt, top1, shT);
                f |= acc.flags;
                if (writer && a.logp_tok) a.logp_tok[i] = acc.lp;
                sh->dec[k] = acc.yes ? 1 : 0;
                if constexpr (kOwnLaunch) last_dl = dl0; else last_dl = a.draft_lse ? a.draft_lse[i] : 0.0f;
            }
            if constexpr (!SHARDED && kOwnLaunch)
                if (!greedy) top1 = argmax_finish(probe, row_p, a.t_dtype, a.V, r.cand, r.M);
            if (writer) {
                if (a.target_lse) a.target_lse[it] = (float)lse;
                if (a.target_top1) a.target_top1[it] = top1;
            }
            last_k = k; last_M = r.M; last_top1 = top1; last_lse = lse;
            if (f) atomicOr(&sh->flags, f);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t f = sh->flags;
        int m = 0;
        if (!(f & kFatal))
            while (m < n && sh->dec[m] != 0) ++m;
        sh->bcast[0] = m;
    }
    __syncthreads();
    const int m = sh->bcast[0];                  // a flagged sequence has m = 0 and emits the argmax of row 0
    const uint32_t f = sh->flags;
    const bool flagged = (f & kFatal) != 0;
    // maximum and argmax of row m: from the thread that merged it, if it still holds them
    if (last_k == m) { sh->bcast[4] = 1; sh->bcast[5] = __float_as_int(last_M); sh->bcast[6] = last_top1; sh->bcast[7] = __float_as_int(last_dl); sh->lse = last_lse; }
    __syncthreads();
    float Mm, dl_m = 0.0f; int32_t top1m; double lse_m;
    if (sh->bcast[4] != 0) {
        Mm = __int_as_float(sh->bcast[5]); top1m = sh->bcast[6]; dl_m = __int_as_float(sh->bcast[7]); lse_m = sh->lse;
    } else {                                     // more rows than threads: merge row m once more
        __syncthreads();
        stage_commit(sh->part, stage(m, a.nsplit), a.nsplit);
        const RowTotal r = merge_partials<SHARDED>(sh->part, a.nsplit);
        Mm = r.M;
        lse_m = (r.R + log2_pos(r.S)) * kLn2;
        if constexpr (SHARDED) top1m = (r.cand >= 0 && r.cand < a.V) ? r.cand : 0;
        else top1m = need_top1 ? resolve_argmax(row_address(a.tbase, a.t_dtype, a.t_stride_b, a.t_stride_k, b, m), a.t_dtype, a.V, r.cand, r.M) : 0;
        if (m < n && a.draft_lse) dl_m = a.draft_lse[(int64_t)b * K + m];
    }
    const SampleJob job = head_job(!flagged && !greedy, m, n, Mm, lse_m, dl_m, a.draft_lse != nullptr, shT);
    if (writer) head_outputs<SHARDED>(a, b, job, m, n, flagged, greedy, f, top1m, [&](int k) { return a.draft_tok[(int64_t)b * K + k]; });
    if constexpr (!kOwnLaunch) {
        __syncthreads();                         // every thread is done with `sh`
        request_table();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    return job;
}

// Lanes per target row (log2): both tensors' slices on the same lanes where the draft rows are merged too.
template <bool SHARDED>
__device__ inline int head_lanes_shift(const VerifyArgs &a)
{
    const int msh = lane_merge_shift(a.K + 1, a.nsplit);
    return !SHARDED && (a.vflags & kVerifyOwnQ) ? max(msh, lane_merge_shift(a.K, a.d_nsplit)) : msh;
}
// In the slice kernel: either path.
template <class Table>
__device__ inline SampleJob verify_head(const VerifyArgs &a, int b, bool writer, HeadStaged *stg, HeadLanes *lanes, double *shT, Table request_table, int wgs)
{
    if (__builtin_expect(lane_merge_shift(a.K + 1, a.nsplit) < 0, 0)) return verify_head_staged<false>(a, b, writer, stg, shT, request_table);
    // (a compute unit's workgroups follow each other by about the number of units)
    return verify_head_lanes<false>(a, b, writer, lanes, shT, request_table, head_lanes_shift<false>(a), (int)((blockIdx.y * (unsigned)wgs + blockIdx.x) >> 8));
}

struct Rows {
    const char *trow, *drow;
};

template <int TD, int DD>
__device__ inline Rows job_rows(const VerifyArgs &a, int b, const SampleJob &job)
{
    Rows r;
    r.trow = (const char *)row_address(a.tbase, TD, a.t_stride_b, a.t_stride_k, b, job.row);
    r.drow = (const char *)row_address(a.dbase, DD, a.d_stride_b, a.d_stride_k, b, job.kind == 1 ? job.row : 0);
    return r;
}

// ---- head kernel: one workgroup per sequence ------------------------------------------
// A kernel for each path: compiled as the unlikely side of the lane path the staged one kept its values in spilled scalars
// (64 shard records a row, 8 sequences, K = 4: 48.7 us, apart 47.1; V = 32000, one sequence, K = 100, slice kernel with the decisions 14.0 / 13.7).
template <bool SHARDED, bool STAGED>
__global__ __launch_bounds__(kVBlock) void verify_head_kernel(VerifyArgs a)
{
    warm_args(a);
    __shared__ std::conditional_t<STAGED, HeadStaged, HeadLanes> sh;
    __shared__ double shT[256];
    static_assert(kVBlock == 256, "one table entry per thread");
    if constexpr (STAGED) verify_head_staged<SHARDED>(a, blockIdx.x, true, &sh, shT, NoTable());
    else verify_head_lanes<SHARDED>(a, blockIdx.x, true, &sh, shT, NoTable(), head_lanes_shift<SHARDED>(a), 0);
}

// ---- slice kernel -----------------------------------------------------------------------
// A slice is kSampleSlice = 2048 elements.
constexpr double kEta = 1.0e-5;        // half-width (relative) of the band around L~ in which a sign may be wrong
constexpr int kSliceVals = 5;          // A, B, R~, D, U

constexpr int kWavesPerWG = kVBlock / kWave;                    // 4 slices per workgroup, one per wavefront
constexpr int kChunks = kSampleSlice / (kWave * kPer);          // a wavefront takes its slice in 4 chunks of 512 elements

__device__ inline bool tab_job_ok(const SampleJob &job)
{
    // ref_p: the target row's maximum; ref_q: the draft row's lse, at most ln V above its maximum
    return job.ref_p >= -14.0f && job.ref_p < 63.0f && (job.kind != 1 || (job.ref_q >= 0.0f && job.ref_q < 63.0f));
}
// Scales of a job's two rows (see above); identical code, hence identical bits, in the slice and the locate kernel.
struct TabScale { double ct, cd, Lp; };
__device__ inline TabScale tab_scale(const SampleJob &job, bool tab_t, bool tab_d, const double *shT)
{
    TabScale o;
    const double st = tab_t ? -(double)job.ref_p : 0.0, sd = tab_d ? -(double)job.ref_q : 0.0;
    o.ct = tab_t ? exp_fast_d(st, shT) : 1.0;
    o.cd = tab_d ? exp_fast_d(sd, shT) : 1.0;
    o.Lp = (tab_t || tab_d) ? job.lam * exp_fast_d(sd - st, shT) : job.lam;
    return o;
}

// Adds the sums of one chunk (8 elements per lane) of a row pair to cA .. cDs.  TABT / TABD: that row's exponentials come from the
// table, through tab_exp_any (the chunks that chunk_pair_tab cannot take: tiny magnitudes; band elements).
template <bool TABT, bool TABD>
__device__ inline void chunk_pair(const float (&ct)[kPer], const float (&cd)[kPer], const ExpRef &rp, const ExpRef &rq,
                                  const double *shT, const double *shE, double c2, float top, double Lp, double band,
                                  double &cA, double &cB, double &cR, double &cDs, uint64_t &any_band)
{
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        double av, bv;
        if constexpr (!TABT) av = exp_fast(ct[i], rp.neg_ref_c, rp.lo, shT, c2, top);
        else av = tab_exp_any(ct[i], shE);
        if constexpr (!TABD) bv = exp_fast(cd[i], rq.neg_ref_c, rq.lo, shT, c2, top);
        else bv = tab_exp_any(cd[i], shE);
        const double diff = fma(-Lp, bv, av);
        cA += av;
        cB += bv;
        cR += fmax(diff, 0.0);
        cDs += copysign(bv, diff);
        // band test: the comparison's lane mask is ORed up over the chunk in scalar registers; one branch
        // per chunk instead of one per element (a branch on a fresh vector comparison stalls the wavefront)
        any_band |= __builtin_amdgcn_ballot_w64(fabs(diff) < band * bv);      // strict: an entry with b = 0 (masked, beyond V) is no band element
    }
}
// The same sums for a chunk of two bfloat16 rows as it lies in memory (four words of two values each), every
// exponential straight from the table in LDS; same order of additions.  A value below the table's range makes
// the sums NaN (entry 0).
__device__ inline void chunk_pair_tab(const u32x4 &wt, const u32x4 &wd, const double *shE, double Lp, double band,
                                      double &cA, double &cB, double &cR, double &cDs, uint64_t &any_band)
{
    const char *E = (const char *)shE;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const TabOffsets ot = tab_offsets2(wt[k]), od = tab_offsets2(wd[k]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double av = *(const double *)(E + (h ? ot.hi : ot.lo));
            const double bv = *(const double *)(E + (h ? od.hi : od.lo));
            const double diff = fma(-Lp, bv, av);
            cA += av;
            cB += bv;
            cR += fmax(diff, 0.0);
            cDs += copysign(bv, diff);
            any_band |= __builtin_amdgcn_ballot_w64(fabs(diff) < band * bv);
        }
    }
}
// One wavefront per slice, four slices per workgroup; in small launches two or four wavefronts per slice (SPLIT; see
// slice_split), whose sums meet in LDS.  A wavefront takes its slice in chunks of one 8-element run per
// lane; its five sums need no LDS and no barrier of their own.  The requests run ahead of the arithmetic (see kAhead): with one
// chunk ahead the launch was bound by memory latency.  Four wavefronts per SIMD: the bfloat16 table limits a CU to
// four workgroups anyway, and under a tighter register limit the loop spills.  Pairs of one bfloat16 and one binary32 row
// have no table and fit five (96 registers, no spills; two binary32 rows spill).  Launch at five / four, V = 256000, 512
// sequences, K = 4: binary32 draft rows 164.8 / 167.7 us, bfloat16 draft rows the same within its spread of 3; V = 128256, 128
// sequences 27.7 / 27.3.
// WAVES: four, or in the sums of a vocabulary shard sixteen, a workgroup for all slices of a sequence, which leaves the sequence's
// sums too (a.part2).
template <int TD, int DD, bool FUSED, int SPLIT, int WAVES = kWavesPerWG>
__global__ __launch_bounds__(WAVES * kWave) __attribute__((amdgpu_waves_per_eu(TD != DD && !FUSED && WAVES == kWavesPerWG ? 5 : 4))) void verify_slices(VerifyArgs a)
{
    constexpr bool kTotals = WAVES > kWavesPerWG;                // one workgroup per sequence
    static_assert(!kTotals || !FUSED, "the accept decisions are taken by 256 threads");
    constexpr int kSliceChunks = kChunks / SPLIT;                // of a wavefront

    // The table serves row pairs of bfloat16 only: with one row computed and one looked up the compiler's schedule
    // of the mixed loop wants 160-170 registers (two wavefronts per SIMD), and held to four wavefronts it spills
    // inside the loop (V = 256000, 512 sequences, binary32 target rows: 210 us against 139 us all computed; at three
    // wavefronts per SIMD, 154 registers and no spills, 147 us).
    constexpr bool kTabT = TD == TAPOUT_BF16 && DD == TAPOUT_BF16, kTabD = kTabT;
    // LDS: the table lies over the staged accept decisions' buffers (FUSED), which are dead once the job is known
    constexpr size_t kTabBytes = kTabT ? sizeof(double) * kTabDoubles : 16;
    constexpr size_t kRaw = (FUSED && sizeof(HeadStaged) > kTabBytes) ? sizeof(HeadStaged) : kTabBytes;
    __shared__ double shT[256];
    __shared__ __align__(16) unsigned char sh_raw[kRaw];
    __shared__ HeadLanes sh_lanes[1];
    __shared__ double sh_sums[SPLIT > 1 || kTotals ? WAVES : 1][kSliceVals];        // (see kMeet)
    static_assert(kTotals || sizeof shT + sizeof sh_raw + sizeof sh_lanes + sizeof sh_sums <= 32 * 1280, "four workgroups' LDS per compute unit");
    warm_args(a);
    [[maybe_unused]] const int wg = WG_LINEAR();
    WG_STAMP(g_stamps_slices, 8, wg, 0);                         // entry
    const int b = blockIdx.y;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    // FUSED: the sequence's last workgroup writes the sequence's outputs, from its first wavefront, which therefore
    // takes the group's last slice: most often none at all, or the row's short last one
    const bool writer = FUSED && (int)blockIdx.x == (a.nsl * SPLIT + WAVES - 1) / WAVES - 1;
    const int piece = blockIdx.x * WAVES + (writer ? WAVES - 1 - wave : wave);
    const int s = piece / SPLIT, part = piece % SPLIT;
    // The table goes from memory to LDS directly, no registers in between, while the accept decisions are taken (FUSED) or the
    // job's record travels.  (Through registers it held 36 of them over the decisions: spills, and the wait for the table
    // in front of the decisions; 20.5 us where this takes 15.9.)
    static_assert(kVBlock == 256, "one entry of the small table per thread");
    auto request_table = [&]() {
        if constexpr (kTabT) copy_to_lds<kTabVecs, WAVES * kWave>(a.exp_table + 256, sh_raw);
    };
    SampleJob job;
    if constexpr (FUSED) {
        // Small batches: a head launch of its own costs more (launch, hand-over of the job record through
        // memory) than taking the accept decisions again in each of the sequence's workgroups.  All of them run
        // the same code on the same inputs and reach the same job; one of them writes the sequence's outputs.
        job = verify_head(a, b, writer, (HeadStaged *)sh_raw, sh_lanes, shT, request_table, (a.nsl * SPLIT + WAVES - 1) / WAVES);
    } else {
        const double tv = a.exp_table[threadIdx.x & 255];
        job = a.final_jobs ? a.final_jobs[b] : a.jobs[b].job;      // vocabulary shards: the caller's copy
        request_table();
        if (!kTotals || threadIdx.x < 256) shT[threadIdx.x] = tv;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // before the rows are requested: nothing younger to wait for
    }
    WG_STAMP(g_stamps_slices, 8, wg, 1);                         // job known
    if (job.kind == 0) {
        if constexpr (kTotals)
            if (threadIdx.x < kSliceVals) a.part2[(int64_t)b * kSliceVals + threadIdx.x] = 0.0;
        return;
    }
    const Rows r = job_rows<TD, DD>(a, b, job);
    const bool live = s < a.nsl;
    const bool resid = job.kind == 1;
    const int first = s * kSampleSlice + part * (kSliceChunks * kWave * kPer), base = first + lane * kPer;
    // The wavefront's requests run kAhead chunks ahead of its arithmetic.  With one chunk ahead the kernel was bound by
    // memory latency, not by arithmetic: 2 KB in flight per wavefront, 8 MB over the chip, is 2.5 TB/s at 3 us.
    // bfloat16 pairs request the whole slice at once (32 registers), others two chunks ahead.
    constexpr int kAhead = (TD == TAPOUT_BF16 && DD == TAPOUT_BF16) || kSliceChunks < 2 ? kSliceChunks : 2;
    // whole workgroup, uniform: which rows take their exponentials from the table
    const bool tab_ok = (kTabT || kTabD) && !(a.vflags & kVerifyNoExpTable) && tab_job_ok(job);
    const bool tab_t = kTabT && tab_ok, tab_d = kTabD && tab_ok && resid;
    const double *shE = (const double *)sh_raw;
    Raw8<TD> qt[kSliceChunks];
    Raw8<DD> qd[kSliceChunks];
    // A slice that lies wholly inside the rows (all but a row's last one) is requested in straight-line code:
    // the per-request checks of the general path are branches, and across branches the compiler waits for every
    // outstanding request where the first chunk's would do.
    const bool whole = live && first + kSliceChunks * kWave * kPer <= a.V;       // wavefront-uniform
    if (__builtin_expect(whole, 1)) {
        const char *tp = r.trow + (int64_t)base * Elem<TD>::size;
        const char *dp = r.drow + (int64_t)base * Elem<DD>::size;
#pragma unroll
        for (int c = 0; c < kSliceChunks; ++c) {
            qt[c] = Raw8<TD>{}; qd[c] = Raw8<DD>{};
            if (c < kAhead) {
#pragma unroll
                for (int h = 0; h < (TD == TAPOUT_F32 ? 2 : 1); ++h)
                    qt[c].w[h] = load16<TD>(tp + (int64_t)c * kWave * kPer * Elem<TD>::size + 16 * h);
            }
        }
        if (resid) {
#pragma unroll
            for (int c = 0; c < kAhead; ++c)
#pragma unroll
                for (int h = 0; h < (DD == TAPOUT_F32 ? 2 : 1); ++h)
                    qd[c].w[h] = load16<DD>(dp + (int64_t)c * kWave * kPer * Elem<DD>::size + 16 * h);
        }
    } else {
#pragma unroll
        for (int c = 0; c < kSliceChunks; ++c) {
            qt[c] = Raw8<TD>{}; qd[c] = Raw8<DD>{};
            if (c < kAhead && live) {
                qt[c] = load_raw8<TD>(r.trow, base + c * kWave * kPer, a.V);
                if (resid) qd[c] = load_raw8<DD>(r.drow, base + c * kWave * kPer, a.V);
            }
        }
    }
    if constexpr (!FUSED) __syncthreads();                       // (FUSED: the decisions' last barrier has published the tables)
    WG_STAMP(g_stamps_slices, 8, wg, 2);                         // tables in LDS, rows requested
    // A wavefront without a slice has nothing to add; where wavefronts' sums meet (SPLIT, kTotals) it comes to the barrier with the others.
    constexpr bool kMeet = SPLIT > 1 || kTotals;
    if (!kMeet && !live) return;
    ExpRef rp, rq;
    rp.set((double)job.ref_p); rq.set((double)job.ref_q);
    const TabScale sc = tab_scale(job, tab_t, tab_d, shT);
    const double lam = sc.Lp, band = kEta * sc.Lp;
    double c2 = kExpC2;
    float top = INFINITY;
    asm volatile("" : "+v"(c2), "+v"(top));               // stay in vector registers through the loop
    // Ds = sum of b carrying the sign of a - L~ b, so that D = (B + Ds) / 2 without a select per element (an
    // element with a == L~ b lands in D; it is in the band, so U covers it).  Elements inside the band are a
    // handful per row at most: their sum and their list are kept under a branch a wavefront almost never enters.
    double A = 0.0, Bs = 0.0, R = 0.0, Ds = 0.0, U = 0.0;
    // one pass over the slice with the rows' exponentials from the table (TT, TD_) or computed; inside: the slice lies wholly
    // inside the rows, the requests need no checks
    auto pass = [&](auto tt, auto td, auto inside) {
        constexpr bool TT = decltype(tt)::value, TD_ = decltype(td)::value;
#pragma unroll
        for (int c = 0; c < kSliceChunks; ++c) {
            if (c + kAhead < kSliceChunks) {
                const int jn = base + (c + kAhead) * kWave * kPer;
                if constexpr (decltype(inside)::value) {
#pragma unroll
                    for (int h = 0; h < (TD == TAPOUT_F32 ? 2 : 1); ++h) qt[c + kAhead].w[h] = load16<TD>(r.trow + (int64_t)jn * Elem<TD>::size + 16 * h);
                    if (resid) {
#pragma unroll
                        for (int h = 0; h < (DD == TAPOUT_F32 ? 2 : 1); ++h) qd[c + kAhead].w[h] = load16<DD>(r.drow + (int64_t)jn * Elem<DD>::size + 16 * h);
                    }
                } else {
                    qt[c + kAhead] = load_raw8<TD>(r.trow, jn, a.V);
                    if (resid) qd[c + kAhead] = load_raw8<DD>(r.drow, jn, a.V);
                }
            }
            float ct[kPer], cd[kPer];
            widen8<TD>(qt[c], ct);
            widen8<DD>(qd[c], cd);
            if (resid) {
                uint64_t any_band = 0;
                if constexpr (TT && TD_) {
                    double cA = 0.0, cB = 0.0, cR = 0.0, cDs = 0.0;
                    chunk_pair_tab(qt[c].w[0], qd[c].w[0], shE, lam, band, cA, cB, cR, cDs, any_band);
                    // a chunk that holds a magnitude below the table's range is formed again, the slow way
                    if (__builtin_expect(__builtin_amdgcn_ballot_w64(cA != cA || cB != cB) != 0, 0)) {
                        asm volatile("" ::: "memory");
                        any_band = 0;
                        cA = 0.0; cB = 0.0; cR = 0.0; cDs = 0.0;
                        chunk_pair<true, true>(ct, cd, rp, rq, shT, shE, c2, top, lam, band, cA, cB, cR, cDs, any_band);
                    }
                    A += cA; Bs += cB; R += cR; Ds += cDs;
                } else {
                    static_assert(!TT && !TD_, "the table serves both rows or neither");
                    chunk_pair<false, false>(ct, cd, rp, rq, shT, shE, c2, top, lam, band, A, Bs, R, Ds, any_band);
                }
                if (__builtin_expect(any_band != 0, 0)) {
                    asm volatile("" ::: "memory");                  // keep this a branch: a select would cost every element
                    // almost never taken: form the chunk's exponentials again and treat its band elements one by one
#pragma unroll 1
                    for (int i = 0; i < kPer; ++i) {
                        const double av = TT ? tab_exp_any(ct[i], shE) : exp_fast(ct[i], rp.neg_ref_c, rp.lo, shT, c2, top);
                        const double bv = TD_ ? tab_exp_any(cd[i], shE) : exp_fast(cd[i], rq.neg_ref_c, rq.lo, shT, c2, top);
                        const double diff = fma(-lam, bv, av);
                        if (fabs(diff) < band * bv) {
                            U += bv;
                            if (!FUSED && a.final_jobs) continue;             // (vocabulary shards keep no band list)
                            const int pos = atomicAdd(&a.jobs[b].band_cnt, 1);
                            if (pos < kBandCap) a.jobs[b].band_idx[pos] = base + c * kWave * kPer + i;
                        }
                    }
                }
            } else {
                double cA = 0.0;
                if constexpr (TT) {
                    cA = chunk_one_tab(qt[c].w[0], shE);
                    if (__builtin_expect(__builtin_amdgcn_ballot_w64(cA != cA) != 0, 0)) {
                        asm volatile("" ::: "memory");
                        cA = 0.0;
#pragma unroll
                        for (int i = 0; i < kPer; ++i) cA += tab_exp_any(ct[i], shE);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < kPer; ++i) cA += exp_fast(ct[i], rp.neg_ref_c, rp.lo, shT, c2, top);
                }
                A += cA;
            }
        }
    };
    using std::false_type; using std::true_type;
    static_assert(kTabT == kTabD, "the table serves both rows or neither");
    if (kMeet && !live) {}
    else if constexpr (kTabT) {
        // (a job on one row, the bonus position, has no draft row: the pass then sums the target row alone)
        // (the whole slice was requested ahead: no request is left for the loop)
        if (__builtin_expect(tab_t, 1)) pass(true_type{}, true_type{}, true_type{}); else pass(false_type{}, false_type{}, true_type{});
    } else {
        if (__builtin_expect(whole, 1)) pass(false_type{}, false_type{}, true_type{}); else pass(false_type{}, false_type{}, false_type{});
    }
    WG_STAMP_LANE0(g_stamps_slices, 8, wg, 3 + wave);            // this wavefront's loop done (slots 3..6)
    double D = 0.5 * (Bs + Ds);
    A = wave_sum_d(A) * sc.ct;
    if (resid) { Bs = wave_sum_d(Bs) * sc.cd; R = wave_sum_d(R) * sc.ct; D = wave_sum_d(D) * sc.cd; U = wave_sum_d(U) * sc.cd; }
    double *o = a.part1 + ((int64_t)b * a.nsl + s) * kSliceVals;
    if constexpr (!kMeet) {
        if (lane == 0) { o[0] = A; o[1] = Bs; o[2] = R; o[3] = D; o[4] = U; }
    } else {
        if (lane == 0) { double *m = sh_sums[wave]; m[0] = A; m[1] = Bs; m[2] = R; m[3] = D; m[4] = U; }
        __syncthreads();
        if (live && part == 0 && lane < kSliceVals) {
            // the slice's other wavefronts: the next ones, or in the writer's workgroup the ones before
            double sum = sh_sums[wave][lane];
#pragma unroll
            for (int q = 1; q < SPLIT; ++q) sum += sh_sums[writer ? wave - q : wave + q][lane];
            o[lane] = sum;
        }
        if constexpr (kTotals)
            if (wave == 0 && lane < kSliceVals) {                // (what the job has no sum of is 0)
                double sum = 0.0;
#pragma unroll
                for (int q = 0; q < WAVES; ++q) sum += sh_sums[q][lane];
                a.part2[(int64_t)b * kSliceVals + lane] = sum;
            }
    }
    WG_STAMP(g_stamps_slices, 8, wg, 7);                         // first wavefront's sums stored
}

// ---- locate kernel: one workgroup per sequence --------------------------------------------
constexpr int kThreadPer = kSampleSlice / kVBlock;     // 8 consecutive elements per thread inside a slice

struct Weights {
    int kind;          // 1 residual max(0, a - L b), 2 target row only (a)
    double lam;        // exact S_p / S_q
    ExpRef rp, rq;
};

// Exclusive scan of one double per thread over the workgroup (thread order); *total = sum.  One barrier;
// sh4 must not be in use by a previous call that other wavefronts may still be reading.
__device__ inline double block_excl_scan_d(double v, double *sh4, double *total)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    double wtot;
    const double inc = wave_incl_scan_d(v, &wtot);
    if (lane == 0) sh4[wave] = wtot;
    __syncthreads();
    double base = 0.0;
#pragma unroll
    for (int w2 = 0; w2 < kVBlock / kWave; ++w2) base += (w2 < wave) ? sh4[w2] : 0.0;
    *total = ((sh4[0] + sh4[1]) + sh4[2]) + sh4[3];
    return base + (inc - v);
}

// Weights of the kThreadPer consecutive elements from j0 on.
template <int TD, int DD>
__device__ inline void thread_weights(const Weights &w, const Rows &r, int j0, int V, const double *T, double (&wv)[kThreadPer])
{
#pragma unroll
    for (int g = 0; g < kThreadPer / kPer; ++g) {
        // both rows' requests side by side where the run lies inside the rows (the usual case): the checks of the
        // general path are branches, and the compiler waits for the target row's data before it requests the draft row's
        const int j = j0 + g * kPer;
        const bool pair = w.kind == 1;
        Raw8<TD> qt;
        Raw8<DD> qd = Raw8<DD>{};
        if (j + kPer <= V) {
#pragma unroll
            for (int h = 0; h < (TD == TAPOUT_F32 ? 2 : 1); ++h) qt.w[h] = load16<TD>(r.trow + (int64_t)j * Elem<TD>::size + 16 * h);
            if (pair) {
#pragma unroll
                for (int h = 0; h < (DD == TAPOUT_F32 ? 2 : 1); ++h) qd.w[h] = load16<DD>(r.drow + (int64_t)j * Elem<DD>::size + 16 * h);
            }
        } else {
            qt = load_raw8<TD>(r.trow, j, V);
            if (pair) qd = load_raw8<DD>(r.drow, j, V);
        }
        float xt[kPer], xd[kPer];
        widen8<TD>(qt, xt);
        widen8<DD>(qd, xd);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            double v = exp_fast(xt[i], w.rp.neg_ref_c, w.rp.lo, T);
            if (w.kind == 1) {
                v = fma(-w.lam, exp_fast(xd[i], w.rq.neg_ref_c, w.rq.lo, T), v);
                v = v > 0.0 ? v : 0.0;
            }
            // masked (-inf) logits carry a stand-in weight of ~1e-304: exactly zero for the scan
            wv[g * kPer + i] = (j0 + g * kPer + i < V && v > 1.0e-290) ? v : 0.0;
        }
    }
}

struct LocateShared {
    double scan[2][4];      // alternating buffers of block_excl_scan_d
    int hits[2][4];         // alternating per-wavefront results of locate_in_slice
    int last;
    int band_key[kBandCap];     // band elements of the sequence, sorted by index ...
    double band_val[kBandCap];  // ... and their residual weights with the exact L
};

__device__ inline int wave_min_i32(int v)
{
    v = min(v, __builtin_amdgcn_update_dpp(0x7fffffff, v, 0xB1, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(0x7fffffff, v, 0x4E, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(0x7fffffff, v, 0x141, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(0x7fffffff, v, 0x140, 0xf, 0xf, false));
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// First of the kSampleSlice elements from `from` on (a slice, most often) whose running sum (starting at cum) exceeds target, or -1.
// With track_last, sh->last collects the largest index with positive weight seen (fallback only).
// *slice_total: their weight as scanned.  `phase` alternates between calls so that consecutive
// scans use different LDS buffers.
template <int TD, int DD>
__device__ inline int locate_in_slice(const Weights &w, const Rows &r, int from, int V, const double *T,
                                      double cum, double target, LocateShared *sh, int phase, double *slice_total,
                                      bool track_last = false)
{
    double wv[kThreadPer];
    thread_weights<TD, DD>(w, r, from + (int)threadIdx.x * kThreadPer, V, T, wv);
    double sum = 0.0;
#pragma unroll
    for (int i = 0; i < kThreadPer; ++i) sum += wv[i];
    const double excl = block_excl_scan_d(sum, sh->scan[phase & 1], slice_total);
    const int j0 = from + threadIdx.x * kThreadPer;
    double c = cum + excl;
    int hit = 0x7fffffff, lp = -1;
#pragma unroll
    for (int i = 0; i < kThreadPer; ++i) {
        c += wv[i];
        if (wv[i] > 0.0) lp = j0 + i;
        if (hit == 0x7fffffff && j0 + i < V && c > target) hit = j0 + i;
    }
    // one LDS word per wavefront instead of one atomic per thread
    hit = wave_min_i32(hit);
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) sh->hits[phase & 1][wave] = hit;
    if (track_last) {
        const int neg = wave_min_i32(-lp);                         // max of lp
        if ((threadIdx.x & (kWave - 1)) == 0 && -neg >= 0) atomicMax(&sh->last, -neg);
    }
    __syncthreads();
    const int *hh = sh->hits[phase & 1];
    const int h = min(min(hh[0], hh[1]), min(hh[2], hh[3]));
    return h == 0x7fffffff ? -1 : h;
}

// A row's slices over the lanes of a wavefront: lane l has slices [l n, (l + 1) n), n = slices_per_lane.  Every wavefront of a
// workgroup does this for itself, on the same numbers: no LDS and no barrier before the slice is known.
__device__ inline int slices_per_lane(int nsl) { return (nsl + kWave - 1) / kWave; }

// The first slice whose inclusive prefix of weights exceeds `target`, and the prefix ahead of it; -1: none.
// weight(s, q): of slice s, the q-th of the lane's.
template <class Weight>
__device__ __forceinline__ int find_slice(int nsl, double target, Weight weight, double *ahead)
{
    const int n = slices_per_lane(nsl), first = (int)(threadIdx.x & (kWave - 1)) * n;
    double z = 0.0;
    for (int q = 0; q < n; ++q)
        if (first + q < nsl) z += weight(first + q, q);
    double total;
    const double incl = wave_incl_scan_d(z, &total);
    const uint64_t past = __builtin_amdgcn_ballot_w64(incl > target);
    if (!past) { *ahead = 0.0; return -1; }
    const int l = __builtin_ctzll(past);
    // that lane's slices one by one (added in another order than the scan's: if none crosses, the next lane's first one)
    double c = incl - z;
    int found = first + n;
    for (int q = 0; q < n; ++q)
        if (found == first + n && first + q < nsl) {
            const double w = weight(first + q, q);
            if (c + w > target) found = first + q; else c += w;
        }
    found = __builtin_amdgcn_readlane(found, l);
    *ahead = lane_d(c, l);
    return found < nsl ? found : -1;
}

// Token of a draw: the first element whose running sum over the row exceeds `target`; whole workgroup (weight as find_slice;
// start(s): the element at which slice s starts).
template <int TD, int DD, class Weight, class Start>
__device__ __forceinline__ int find_token(const Weights &w, const Rows &r, int V, int nsl, const double *T, double target, Weight weight, Start start, LocateShared *sh, int &phase)
{
    double cum;
    const int s_found = find_slice(nsl, target, weight, &cum);
    LOCATE_STAMP(3);                                             // slice found
    // slice sums and the in-slice scan round differently: if the crossing is not inside the chosen
    // slice, continue into the elements behind it
    int token = -1;
    if (s_found >= 0)
        for (int j = start(s_found); j < V && token < 0; j += kSampleSlice) {
            double slice_total;
            token = locate_in_slice<TD, DD>(w, r, j, V, T, cum, target, sh, phase++, &slice_total);
            cum += slice_total;
        }
    if (__builtin_expect(token < 0, 0)) {
        // rounding left no crossing: the largest index with positive weight
        for (int j = 0; j < V; j += kSampleSlice) {
            double slice_total;
            locate_in_slice<TD, DD>(w, r, j, V, T, 0.0, INFINITY, sh, phase++, &slice_total, true);
        }
        __syncthreads();
        token = sh->last;
    }
    return token;
}
__device__ inline int whole_slice_start(int s) { return s * kSampleSlice; }

// Exact weights of all slices of a row, zs[s], and their total; whole workgroup.  A wavefront per slice, no barrier until all
// are done.  (By the whole workgroup, slice after slice with a scan each, every slice waited for its loads
// and two barriers.  Rounds with a few such sequences: V = 256000, 512 sequences 1426.9 us, this 1417.6; V = 32000, 32 sequences
// 35.6 / 34.0.)
template <int TD, int DD>
__device__ inline double slice_weights(const Weights &w, const Rows &r, int V, int nsl, const double *T, double *zs)
{
    constexpr int kWaves = kVBlock / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    for (int s = threadIdx.x / kWave; s < nsl; s += kWaves) {
        double sum = 0.0;
#pragma unroll 2
        for (int c = 0; c < kWaves; ++c) {
            double wv[kThreadPer];
            thread_weights<TD, DD>(w, r, s * kSampleSlice + (c * kWave + lane) * kThreadPer, V, T, wv);
#pragma unroll
            for (int i = 0; i < kThreadPer; ++i) sum += wv[i];
        }
        sum = wave_sum_d(sum);
        if (lane == 0) zs[s] = sum;
    }
    __threadfence_block();
    __syncthreads();
    const int n = slices_per_lane(nsl);
    double z = 0.0;
    for (int q = 0; q < n; ++q)
        if (lane * n + q < nsl) z += zs[lane * n + q];
    return lanes_sum(z, 0, 6);
}

// Band elements of a sequence (see the slice kernel).  Each listed element is evaluated with the exact L; what it
// contributed to the slice sums under L~ (recomputed here with the slice kernel's own arithmetic, hence the same
// number) is taken back: correction = max(0, a - L b) - (max(0, a - L~ b) - delta [a > L~ b] b).  The list is
// sorted by index, so that sums over it do not depend on the order in which the slice kernel's workgroups
// appended.  Leaves the sorted (index, correction) pairs in sh and returns their total.  Whole workgroup.
// E: the table of bfloat16 exponentials (memory), sc / tab_t / tab_d: the job's scales as the slice kernel formed them
// (tab_scale): the side of L~ an element was counted on is decided here on the very numbers the slice kernel compared.
// Inlined: a call that is not gives the kernel a stack, and a kernel with scratch memory starts later, whether it touches it or not (a chain of
// small kernels without / with: 1.56 / 2.03 us each, of 256 workgroups 1.70 / 2.17).  Rounds with the call / without: V = 128256, 64
// sequences 67.3 / 67.0 us, up to the stop position 58.5 / 57.9, V = 50257, 48 sequences 56.85 / 56.64.
template <int TD, int DD>
__device__ inline double settle_band(const Weights &w, const Rows &r, int V, const double *T, const double *E,
                                           const TabScale &sc, bool tab_t, bool tab_d,
                                           double delta, int n_band, int band_i, LocateShared *sh)
{
    const int tid = threadIdx.x;
    double wv = 0.0;
    if (tid < n_band && band_i < V) {
        const float xt = load_elem<TD>(r.trow, band_i), xd = load_elem<DD>(r.drow, band_i);
        const double avp = tab_t ? tab_exp_any(xt, E) : exp_fast(xt, w.rp.neg_ref_c, w.rp.lo, T);
        const double bvp = tab_d ? tab_exp_any(xd, E) : exp_fast(xd, w.rq.neg_ref_c, w.rq.lo, T);
        const double av = avp * sc.ct, bv = bvp * sc.cd;       // (scales of 1 where the row's exponentials are computed)
        const double v = fma(-w.lam, bv, av);
        const double exact = v > 1.0e-290 ? v : 0.0;           // same rule as thread_weights (masked logits weigh nothing)
        const double dt = fma(-sc.Lp, bvp, avp);
        wv = exact - (sc.ct * fmax(dt, 0.0) - delta * (dt >= 0.0 ? bv : 0.0));
    }
    if (tid < kBandCap) { sh->band_key[tid] = tid < n_band ? band_i : 0x7fffffff; sh->band_val[tid] = wv; }
    __syncthreads();
    int rank = 0;
    if (tid < n_band)
        for (int q = 0; q < n_band; ++q) rank += sh->band_key[q] < band_i ? 1 : 0;     // indices are distinct
    __syncthreads();
    if (tid < n_band) { sh->band_key[rank] = band_i; sh->band_val[rank] = wv; }
    __syncthreads();
    double total = 0.0;
    for (int q = 0; q < n_band; ++q) total += sh->band_val[q];
    return total;
}

// FIN (whole-round calls whose accept decisions did not wait for the draft epilogue): the launch carries
// that epilogue's workgroups too, one per sequence, ahead of the locate workgroups: two latency-bound kernels of a
// few dozen workgroups each run side by side instead of one after the other.
template <int TD, int DD, bool FIN>
__global__ __launch_bounds__(kVBlock) void verify_locate(VerifyArgs a, DraftFinalArgs fin)
{
    if constexpr (FIN) warm_args(a, fin); else warm_args(a);
    static_assert(kVBlock == kFinalBlock, "the draft epilogue runs in this kernel's workgroups");
    LOCATE_STAMP(0);                                             // entry
    // tapout_round: the end of the round needs nothing of this launch, only the accepted lengths of an earlier one, so it
    // rides along as workgroups of its own behind the others instead of taking a launch after this one: a few lanes per
    // sequence (UCB: one per arm, Thompson Sampling: two).  (UCB at the end of the locate workgroups themselves, behind
    // the token, made them 2 us longer: V = 128256, 64 sequences, up to the stop position 8.0 us, this 6.0.)
    if (a.bandit_tail) {
        const int wg = (int)blockIdx.x - (FIN ? 2 : 1) * a.B;
        if (wg >= 0) {
            if (a.bandit_tail == 2)
                update_select_ts_lanes(a.bandit, wg * (kVBlock / 16) + (int)(threadIdx.x >> 4), threadIdx.x & 15,
                                       a.b_arm_in, a.accept_len, a.n_draft, a.b_gamma, a.b_active, a.b_u_ts, a.b_arm_out, a.b_flags);
            else
                update_select_ucb_lanes(a.bandit, wg * (kVBlock / TAPOUT_MAX_ARMS) + (int)(threadIdx.x / TAPOUT_MAX_ARMS), threadIdx.x % TAPOUT_MAX_ARMS,
                                        a.b_arm_in, a.accept_len, a.n_draft, a.b_gamma, a.b_active, a.b_arm_out, a.b_flags);
            return;
        }
    }
    if constexpr (FIN)
        if ((int)blockIdx.x < a.B) {
            draft_finalize_on_lanes<false>(fin, blockIdx.x, DD);
#ifdef TAPOUT_WG_STAMPS
            __syncthreads();
#endif
            LOCATE_STAMP(7);                                     // the epilogue's workgroup: done
            return;
        }
    __shared__ double shT[256];
    __shared__ LocateShared shl;
    const int b = FIN ? blockIdx.x - a.B : blockIdx.x;
    const int tid = threadIdx.x;
    // the slice sums, the table and the uniform are requested before the job is looked at (one round trip)
    const double *ps = a.part1 + (int64_t)b * a.nsl * kSliceVals;
    double *zs = a.part2 + (int64_t)b * a.nsl;                       // exact slice weights (slow path only)
    // First all loads that do not depend on each other, then their uses: written so that no wait separates the
    // requests (the first two slices of each lane without a loop; 256 threads fetch the 256 table entries).
    static_assert(kVBlock == 256, "one table entry per thread");
    const int lane = tid & (kWave - 1), npl = slices_per_lane(a.nsl), s0 = lane * npl;
    const double *p0 = ps + (int64_t)min(s0, a.nsl - 1) * kSliceVals, *p1 = ps + (int64_t)min(s0 + 1, a.nsl - 1) * kSliceVals;
    double f[2][kSliceVals];
#pragma unroll
    for (int q = 0; q < kSliceVals; ++q) f[0][q] = p0[q];
    const double tv = a.exp_table[tid];
    const float u32v = a.u_sample[b];
    const int band_n = a.jobs[b].band_cnt;
    const int band_i = a.jobs[b].band_idx[tid & (kBandCap - 1)];                                  // stale beyond band_n: unused
    const SampleJob job = a.jobs[b].job;
#pragma unroll
    for (int q = 0; q < kSliceVals; ++q) f[1][q] = npl > 1 ? p1[q] : 0.0;
    // the compiler would otherwise sink these loads below the early exit and pay a second round trip for them
    asm volatile("" :: "v"(f[0][0]), "v"(f[0][1]), "v"(f[0][2]), "v"(f[0][3]), "v"(f[0][4]), "v"(tv), "v"(u32v), "v"(band_n), "v"(band_i));
    shT[tid] = tv;
    if (tid == 0) shl.last = -1;
    if (__builtin_expect(job.kind == 0, 0)) return;                  // the slice sums of such a sequence are stale: unused
    __syncthreads();                                                   // publishes the table and the inits
    LOCATE_STAMP(1);                                             // first requests answered
    // totals of the five slice quantities, every wavefront for itself, fixed order
    double tot[kSliceVals];
#pragma unroll
    for (int q = 0; q < kSliceVals; ++q) {
        double acc = s0 < a.nsl ? f[0][q] : 0.0;
        if (npl > 1) acc += s0 + 1 < a.nsl ? f[1][q] : 0.0;
        for (int k = 2; k < npl; ++k) acc += s0 + k < a.nsl ? ps[(int64_t)(s0 + k) * kSliceVals + q] : 0.0;      // vocabularies beyond 128 slices
        tot[q] = lanes_sum(acc, 0, 6);
    }
    const double Sp = tot[0], Sq = tot[1];
    Weights w;
    w.kind = job.kind;
    w.rp.set((double)job.ref_p); w.rq.set((double)job.ref_q);
    bool draft_bad = false;
    if (job.kind == 1 && (!(Sq > 0.0) || !(Sq < INFINITY))) {          // NaN / empty draft row: draw from the target row alone
        w.kind = 2;
        draft_bad = true;
    }
    w.lam = w.kind == 1 ? Sp / Sq : 0.0;
    const double delta = w.lam - job.lam;
    const Rows r = job_rows<TD, DD>(a, b, job);
    const double u = (double)u32v;
    int phase = 0;

    // slice weights: target row alone -> A_s; residual -> R~_s - delta D_s if the bound on the sign flips allows,
    // else with the listed band elements corrected one by one
    double Z = w.kind == 2 ? Sp : tot[2] - delta * tot[3];
    bool exact_sums = false;
    int n_band = 0;
    if (w.kind == 1) {
        const bool close = fabs(delta) <= kEta * job.lam;
        bool certified = close && Z > 0.0 && fabs(delta) * tot[4] <= 2.0e-10 * Z;
        if (__builtin_expect(!certified && close && band_n <= kBandCap, 0)) {
            n_band = band_n;
            const bool tab_ok = TD == TAPOUT_BF16 && DD == TAPOUT_BF16 && !(a.vflags & kVerifyNoExpTable) && tab_job_ok(job);    // as in the slice kernel
            const bool tab_t = tab_ok, tab_d = tab_ok;
            Z += settle_band<TD, DD>(w, r, a.V, shT, a.exp_table + 256, tab_scale(job, tab_t, tab_d, shT), tab_t, tab_d,
                                     delta, band_n, band_i, &shl);
            certified = Z > 0.0;
        }
        if (__builtin_expect(!certified, 0)) {
            n_band = 0;
            // slow path: exact slice weights with the exact L (also the p == q case: then Z may vanish)
            Z = slice_weights<TD, DD>(w, r, a.V, a.nsl, shT, zs);
            if (!(Z > 0.0)) {
                // the residual vanished (p == q up to rounding): draw from the target row itself
                w.kind = 2;
                __syncthreads();                                       // zs has been read
                Z = slice_weights<TD, DD>(w, r, a.V, a.nsl, shT, zs);
            }
            exact_sums = true;
            if (tid == 0) shl.last = -1;
            __threadfence_block();
            __syncthreads();
        }
    }
    const double z0 = w.kind == 2 ? f[0][0] : f[0][2] - delta * f[0][3], z1 = w.kind == 2 ? f[1][0] : f[1][2] - delta * f[1][3];
    auto slice_weight = [&](int s, int q) -> double {
        if (exact_sums) return zs[s];
        const double *at = ps + (int64_t)s * kSliceVals;
        double v = q == 0 ? z0 : (q == 1 ? z1 : (w.kind == 2 ? at[0] : at[2] - delta * at[3]));
        if (w.kind == 2) return v;
        v = v > 0.0 ? v : 0.0;
        for (int k = 0; k < n_band; ++k)
            if (shl.band_key[k] / kSampleSlice == s) v += shl.band_val[k];
        return v;
    };

    LOCATE_STAMP(2);                                             // total weight known (certified, settled or recomputed)
    int token = -1;
    if (Z > 0.0) token = find_token<TD, DD>(w, r, a.V, a.nsl, shT, u * Z, slice_weight, whole_slice_start, &shl, phase);
    LOCATE_STAMP(4);                                             // token found
    if (tid == 0) {
        if (token < 0) token = 0;
        a.out_tok[(int64_t)b * (a.K + 1) + job.row] = token;
        if (__builtin_expect(draft_bad, 0)) {
            uint32_t f = a.flags_ws[b] | TAPOUT_FLAG_BAD_ROW;
            a.flags_ws[b] = f;
            if (a.flags) a.flags[b] = f;
        }
    }
    LOCATE_STAMP(5);                                             // outputs written
}

// ---- draft-token sampling: the inverse CDF of every live draft row ---------------------------
__device__ inline float wave_max_f(float v)
{
    auto mv = [](float x, auto ctrl) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true)); };
    v = fmaxf(v, mv(v, std::integral_constant<int, 0xB1>{})); v = fmaxf(v, mv(v, std::integral_constant<int, 0x4E>{}));
    v = fmaxf(v, mv(v, std::integral_constant<int, 0x141>{})); v = fmaxf(v, mv(v, std::integral_constant<int, 0x140>{}));
    auto at = [&](int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); };
    return fmaxf(fmaxf(at(0), at(16)), fmaxf(at(32), at(48)));
}

// A row's maximum, the exponent reference of its draw, and the epilogue's bad-row rule, from the row's partials, by one
// wavefront: a NaN anywhere poisons a slice's sum (also from inside the batch the draft pass leaves out of it), a row
// without a finite maximum has no softmax.  In two steps, request and use.
struct RowRefRegs { float v1, S; };
__device__ inline RowRefRegs row_ref_issue(const Partial *p, int nsplit)
{
    const int sl = min((int)(threadIdx.x & (kWave - 1)), nsplit - 1);       // surplus lanes ask for the last partial again
    return RowRefRegs{p[sl].v1, p[sl].S};
}
__device__ inline float row_ref_finish(RowRefRegs r, const Partial *p, int nsplit, bool *bad)
{
    bool mine = !(r.S >= 0.0f) || r.S == INFINITY;
    for (int sl = (int)(threadIdx.x & (kWave - 1)) + kWave; sl < nsplit; sl += kWave) {
        const float S = p[sl].S;
        r.v1 = fmaxf(r.v1, p[sl].v1);
        mine |= !(S >= 0.0f) || S == INFINITY;
    }
    const float M = wave_max_f(r.v1);
    *bad = __builtin_amdgcn_ballot_w64(mine) != 0 || M == -INFINITY || M == INFINITY;
    return M;
}

// The row's lse in double, the same bits in every lane as the draft epilogue leaves in its outputs: its lane path's arithmetic on
// the same lanes (see draft_finalize_lanes), every group of a row's lanes with the same row.
template <int USH>
__device__ __forceinline__ double row_lse_lanes(const DraftFinalArgs &a, const int dtype, const BatchGeom &g, const u32x4 &w0, const u32x4 &w1, const int msh)
{
    const int sl = (int)(threadIdx.x >> USH) & ((1 << msh) - 1);
    const Piece t = row_on_lanes<false, USH>(a, dtype, g, w0, w1, sl < a.nsplit, threadIdx.x & ((1 << USH) - 1), msh + USH, []() { return NAN; });
    return row_signals(row_total<true>(t), a.V > 1).lse;
}

// The same of the epilogue's staged path (see draft_finalize_staged): every piece completed and rounded by a lane, then merged one
// by one; at most a wavefront of pieces.
__device__ inline double row_lse_staged(const DraftFinalArgs &a, const BatchGeom &g, const u32x4 &w0, const u32x4 &w1)
{
    const int sl = threadIdx.x & (kWave - 1);
    Piece e = piece_from_words(w0, w1);
    batch_fix(e, batch_issue(g, a.dtype, a.V, sl < a.nsplit ? e.idx : -1, a.part), a.dtype);
    Piece acc = empty_piece();
    for (int s = 0; s < a.nsplit; ++s) {
        auto at = [&](int v) { return (uint32_t)__builtin_amdgcn_readlane(v, s); };
        acc = merge_pair<true>(acc, piece_from_words(u32x4{at(__float_as_int(e.M)), at(__float_as_int((float)e.S)), at(__float_as_int((float)e.T)), at(__float_as_int(e.v2))},
                                                     u32x4{at(e.idx), at(__float_as_int(e.xt)), 0u, 0u}));
    }
    return row_signals(row_total<true>(acc), a.V > 1).lse;
}

// Tokens: one workgroup per draft row finds the draw slice (see DrawSums) and the element that hold u * Z, and forms log q(tok).
// OWN, kOwnLanes or kOwnStaged: the draft epilogue's workgroups ride in this launch, ahead of the others, and every row forms its lse itself,
// from the partials, while the elements travel, both on that path of the epilogue; 0: the epilogue has run and left it.
constexpr int kOwnLanes = 1, kOwnStaged = 2;
template <int DT, int OWN>
__global__ __launch_bounds__(kVBlock) void sample_locate_kernel(SampleArgs a, DraftFinalArgs fin)
{
    if constexpr (OWN != 0) {
        warm_args(a, fin);
        if ((int)blockIdx.x < a.B) {
            if constexpr (OWN == kOwnLanes) draft_finalize_on_lanes<false>(fin, blockIdx.x, DT);
            else {
                __shared__ __align__(16) unsigned char lds[kStagedLds];
                draft_finalize_staged<false>(fin, blockIdx.x, lds);
            }
            return;
        }
    } else warm_args(a);
    __shared__ double shT[256];
    __shared__ LocateShared shl;
    constexpr int kParts = kBlock / kWave, kVec = Elem<DT>::vec;
    const int row = (int)blockIdx.x - (OWN != 0 ? a.B : 0), b = row / a.K, k = row - b * a.K, tid = threadIdx.x;
    const int per_split = a.nb * kStreamU, n_slices = a.nsplit * per_split;
    const int nsl = (a.V + kSampleSlice - 1) / kSampleSlice;
    double *ps = a.sums + (int64_t)row * (n_slices > 0 ? n_slices * kParts : nsl);
    // everything is requested before anything is looked at: one round trip
    const int npl = slices_per_lane(n_slices), s0 = (tid & (kWave - 1)) * npl;
    typedef double d2 __attribute__((ext_vector_type(2)));
    static_assert(kParts == 4, "two loads a slice");
    const double *first = n_slices > 0 ? ps : a.sums;
    auto request = [&](int s, d2 &lo, d2 &hi) { const d2 *p = (const d2 *)(first + (int64_t)max(min(s, n_slices - 1), 0) * kParts); lo = p[0]; hi = p[1]; };
    d2 x0, y0, x1, y1;
    request(s0, x0, y0);
    request(s0 + 1, x1, y1);
    const double tv = a.exp_table[tid];
    const float u32v = a.u[row];
    const RowRefRegs rr = row_ref_issue(a.part + (int64_t)row * a.nsplit, a.nsplit);
    const int kl = a.k_len ? a.k_len[b] : a.K;
    const char *rowp = (const char *)row_address(a.base, DT, a.stride_b, a.stride_k, b, k);
    double lse = 0.0;
    [[maybe_unused]] BatchGeom g{};
    [[maybe_unused]] u32x4 w0{}, w1{};
    [[maybe_unused]] int msh = 0, ush = 0;
    if constexpr (OWN != 0) {
        if constexpr (OWN == kOwnLanes) { msh = lane_merge_shift(a.K, a.nsplit); ush = draft_lanes_shift(a.K << msh); }
        const int sl = OWN == kOwnStaged ? tid & (kWave - 1) : (tid >> ush) & ((1 << msh) - 1);
        const u32x4 *pp = (const u32x4 *)(a.part + (int64_t)row * a.nsplit + min(sl, a.nsplit - 1));
        w0 = pp[0]; w1 = pp[1];
        g = batch_geom(rowp, DT, a.V, sl, a.per);
    } else lse = a.lse[row];
    asm volatile("" :: "v"(x0), "v"(y0), "v"(x1), "v"(y1), "v"(tv), "v"(u32v), "v"(rr.v1), "v"(rr.S), "v"(lse), "v"(w0), "v"(w1));
    shT[tid] = tv;
    if (tid == 0) shl.last = -1;
    if (k >= kl) return;
    bool bad;
    const float M = row_ref_finish(rr, a.part + (int64_t)row * a.nsplit, a.nsplit, &bad);
    if (__builtin_expect(bad, 0)) {                                      // nothing to draw from
        if (tid == 0) { a.tok[row] = -1; if (a.logq_tok) a.logq_tok[row] = NAN; }
        return;
    }
    __syncthreads();                                                     // publishes the table
    Weights w;
    w.kind = 2; w.lam = 0.0;
    w.rp.set((double)M); w.rq.set(0.0);
    Rows r;
    r.trow = r.drow = rowp;
    int phase = 0, token = -1;
    if (__builtin_expect(n_slices > 0 && M >= kDrawLow + 100.0f && M < kDrawHigh, 1)) {
        // the sums in the reference of the row's maximum
        const double scale = exp_fast_d(-(double)M, shT);
        auto sum4 = [&](const d2 &lo, const d2 &hi) { return ((lo.x + lo.y) + (hi.x + hi.y)) * scale; };
        const double f0 = sum4(x0, y0), f1 = sum4(x1, y1);
        auto weight = [&](int s, int q) -> double {
            if (q == 0) return f0;
            if (q == 1) return f1;
            d2 lo, hi;
            request(s, lo, hi);
            return sum4(lo, hi);
        };
        double z = s0 < n_slices ? f0 : 0.0;
        if (npl > 1) z += s0 + 1 < n_slices ? f1 : 0.0;
        for (int q = 2; q < npl; ++q) z += s0 + q < n_slices ? weight(s0 + q, q) : 0.0;
        const double Z = lanes_sum(z, 0, 6);
        int head, nvec, tail;
        row_geometry<DT>(rowp, a.V, head, nvec, tail);
        auto start = [&](int s) {
            const int split = s / per_split;
            return s == 0 ? 0 : head + min(split * a.per + min((s - split * per_split) * kBlock, a.per), nvec) * kVec;
        };
        if (Z > 0.0) token = find_token<DT, DT>(w, r, a.V, n_slices, shT, (double)u32v * Z, weight, start, &shl, phase);
    } else {
        // logits beyond the range of the sums, or no sums: all over again in the reference of the row's maximum (the sums' place holds them)
        __syncthreads();                                                 // every wavefront has its sums
        const double Z = slice_weights<DT, DT>(w, r, a.V, nsl, shT, ps);
        if (Z > 0.0) token = find_token<DT, DT>(w, r, a.V, nsl, shT, (double)u32v * Z, [&](int s, int) { return ps[s]; }, whole_slice_start, &shl, phase);
    }
    if constexpr (OWN == kOwnStaged) lse = row_lse_staged(fin, g, w0, w1);
    else if constexpr (OWN == kOwnLanes) {
        if (__builtin_expect(a.K << msh > kFinalBlock, 0)) lse = row_lse_lanes<0>(fin, DT, g, w0, w1, msh);
        else on_lanes<-1>(msh, ush, [&](auto m, auto u) __attribute__((always_inline)) { lse = row_lse_lanes<decltype(u)::value>(fin, DT, g, w0, w1, decltype(m)::value); });
    }
    if (tid == 0) {
        if (token < 0) token = 0;
        a.tok[row] = token;
        if (a.logq_tok) a.logq_tok[row] = (float)((double)load_elem<DT>(r.trow, token) - lse);
    }
}

// ---- final token over vocabulary shards ---------------------------------------------------------
// This shard's five sums per sequence, one wavefront per sequence (fixed order).
__global__ __launch_bounds__(kVBlock) void shard_sums_kernel(ShardFinalArgs a)
{
    const int b = blockIdx.x * kWavesPerWG + (int)(threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    if (b >= a.v.B) return;
    const int kind = a.v.final_jobs[b].kind;
    const double *ps = a.v.part1 + (int64_t)b * a.v.nsl * kSliceVals;
    double s[kSliceVals] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int sl = lane; sl < a.v.nsl; sl += kWave)
#pragma unroll
        for (int q = 0; q < kSliceVals; ++q) s[q] += ps[sl * kSliceVals + q];       // stale where the job has no such sum: dropped below
#pragma unroll
    for (int q = 0; q < kSliceVals; ++q) {
        const double t = wave_sum_d(s[q]);
        if (lane == 0) a.sums_out[(int64_t)b * kSliceVals + q] = (kind != 0 && (q == 0 || kind == 1)) ? t : 0.0;
    }
}

// One workgroup per sequence.  Every shard runs this on the same sums_all, so all of them derive the same
// normaliser ratio, the same masses and the same owner; only the owner scans its slices for the token.
template <int TD, int DD>
__global__ __launch_bounds__(kVBlock) void shard_locate(ShardFinalArgs a)
{
    __shared__ double shT[256];
    __shared__ LocateShared shl;
    warm_args(a);
    const VerifyArgs &v = a.v;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1);
    // everything that does not depend on the job is requested first (one round trip): the sums of the shards (lane h of
    // every wavefront takes shards h, h + 64, ...), the slice sums of the lane's first slice, the table
    double mine[kSliceVals], tot[kSliceVals];
    const double *sa = a.sums_all + ((int64_t)min(lane, a.G - 1) * v.B + b) * kSliceVals;
#pragma unroll
    for (int q = 0; q < kSliceVals; ++q) mine[q] = sa[q];
    const double *ps = v.part1 + (int64_t)b * v.nsl * kSliceVals;
    const double *pf = ps + (int64_t)min(lane * slices_per_lane(v.nsl), v.nsl - 1) * kSliceVals;
    const double f0 = pf[0], f2 = pf[2], f3 = pf[3];
    const double tv = v.exp_table[tid];
    const float u32v = v.u_sample[b];
    const SampleJob job = v.final_jobs[b];
    asm volatile("" :: "v"(mine[0]), "v"(mine[1]), "v"(mine[2]), "v"(mine[3]), "v"(mine[4]), "v"(f0), "v"(f2), "v"(f3), "v"(tv), "v"(u32v));
    if (tid == 0) { a.tok_out[b] = -1; a.need_exact[b] = 0; a.exact_mass[b] = NAN; }
    if (job.kind == 0) return;
    shT[tid] = tv;
    if (tid == 0) shl.last = -1;
    __syncthreads();
    // totals over all shards, in one fixed order on every shard
#pragma unroll
    for (int q = 0; q < kSliceVals; ++q) {
        double t = lane < a.G ? mine[q] : 0.0;
        for (int h = lane + kWave; h < a.G; h += kWave) t += a.sums_all[((int64_t)h * v.B + b) * kSliceVals + q];
        tot[q] = wave_sum_d(t);
    }
    const double Sp = tot[0], Sq = tot[1];
    Weights w;
    w.kind = job.kind;
    w.rp.set((double)job.ref_p); w.rq.set((double)job.ref_q);
    if (job.kind == 1 && (!(Sq > 0.0) || !(Sq < INFINITY))) w.kind = 2;       // unusable draft row: draw from the target row alone
    w.lam = w.kind == 1 ? Sp / Sq : 0.0;
    const double delta = w.lam - job.lam;
    const Rows r = job_rows<TD, DD>(v, b, job);
    double *zs = v.part2 + (int64_t)b * v.nsl;
    int phase = 0;
    bool exact = false;                       // masses and own slice weights are exact recomputations
    double Z = w.kind == 2 ? Sp : tot[2] - delta * tot[3];
    if (w.kind == 1) {
        const bool certified = fabs(delta) <= kEta * job.lam && Z > 0.0 && fabs(delta) * tot[4] <= 2.0e-10 * Z;
        if (!certified) {
            // exact weights of this shard's slices with the exact ratio (every shard does this for its own slices)
            double ztot = 0.0;
            for (int s = 0; s < v.nsl; ++s) {
                double st;
                locate_in_slice<TD, DD>(w, r, s * kSampleSlice, v.V, shT, 0.0, INFINITY, &shl, phase++, &st);
                if (tid == 0) zs[s] = st;
                ztot += st;
            }
            __threadfence_block();
            __syncthreads();
            if (!a.exact_all) {                                                // first call: hand the exact mass to the caller
                if (tid == 0) { a.exact_mass[b] = ztot; a.need_exact[b] = 1; }
                return;
            }
            exact = true;
            double t = 0.0;
            for (int h = lane; h < a.G; h += kWave) t += a.exact_all[(int64_t)h * v.B + b];
            Z = wave_sum_d(t);
            if (!(Z > 0.0)) {                                                   // p == q up to rounding: draw from the target row itself
                w.kind = 2; exact = false; Z = Sp;
            }
        }
    }
    if (!(Z > 0.0)) {                                                           // nothing to draw from anywhere: the first shard answers token 0
        if (tid == 0 && a.g == 0) a.tok_out[b] = a.vocab_offset;
        return;
    }
    // owner: the first shard whose inclusive prefix of masses exceeds u * Z; the last one with mass if rounding leaves none.
    // Every wavefront walks the shards 64 at a time, lane h the mass of the h-th of them under the current weights.
    const double target = (double)u32v * Z;
    double prefix = 0.0, mine_prefix = 0.0;
    int owner = -1, last_pos = -1;
    for (int h0 = 0; h0 < a.G; h0 += kWave) {
        const int h = h0 + lane;
        double m = 0.0;
        if (h < a.G) {
            const double *sh = a.sums_all + ((int64_t)h * v.B + b) * kSliceVals;
            const double m0 = h0 == 0 ? mine[0] : sh[0], m2 = h0 == 0 ? mine[2] : sh[2], m3 = h0 == 0 ? mine[3] : sh[3];
            m = w.kind == 2 ? m0 : (exact ? a.exact_all[(int64_t)h * v.B + b] : fmax(m2 - delta * m3, 0.0));
        }
        double total;
        const double incl = wave_incl_scan_d(m, &total);
        const uint64_t past = __builtin_amdgcn_ballot_w64(h < a.G && prefix + incl > target), pos = __builtin_amdgcn_ballot_w64(m > 0.0);
        if (a.g >= h0 && a.g < h0 + kWave) mine_prefix = prefix + lane_d(incl - m, a.g - h0);
        if (owner < 0 && past) owner = h0 + __builtin_ctzll(past);
        if (pos) last_pos = h0 + 63 - __builtin_clzll(pos);
        prefix += total;
    }
    const bool fallback = owner < 0;
    if (fallback) owner = last_pos;
    if (owner != a.g) return;
    auto slice_weight = [&](int s, int q) -> double {
        const double *at = ps + (int64_t)s * kSliceVals;
        if (w.kind == 2) return q == 0 ? f0 : at[0];
        if (exact) return zs[s];
        return q == 0 ? fmax(f2 - delta * f3, 0.0) : fmax(at[2] - delta * at[3], 0.0);
    };
    // (a fallback's target lies beyond every slice: find_token then takes the last positive weight here)
    const int token = find_token<TD, DD>(w, r, v.V, v.nsl, shT, fallback ? INFINITY : target - mine_prefix, slice_weight, whole_slice_start, &shl, phase);
    if (tid == 0) a.tok_out[b] = a.vocab_offset + (token < 0 ? 0 : token);
}

// Wavefronts that share a slice, and so workgroups of the slice launch.  Few slices leave the chip idle while single wavefronts
// walk four chunks each: one chunk per wavefront, or two, then shorten the launch until its workgroups, each of which takes the
// accept decisions again, get in each other's way.  One chunk up to two workgroups per compute unit, or where it adds none; two
// up to two and a half.  Rows of more than 32 slices don't share two ways: they gain nothing there, and the rounds of binary32 rows lose.
// Measured, us per round with one / two / four wavefronts per slice: V = 32000, one sequence, binary32, up to the stop position
// 21.0 / 20.3 / 18.9; 32 sequences, bfloat16 26.1 / 24.8 / 24.1;
// V = 8000, 128 sequences, binary32 24.2 / 22.9 / 21.6; V = 128256, 8 sequences, bfloat16 22.9 / 21.2 / 20.9.  Beyond 512
// workgroups: V = 32000, 64 sequences, binary32 31.7 / 29.1 / 31.2; V = 50257, 48 sequences 34.9 / 34.0 / -; V = 128256, 16
// sequences 28.7 / 29.8 / 30.7.  Beyond 640: V = 32000, bfloat16, 96 sequences 29.7 / 29.7 / 33.6, 128 sequences 33.4 / 34.5 / 39.9.
inline int slice_split(int B, int nsl)
{
    auto wgs = [&](int split) { return (int64_t)B * ((nsl * split + kWavesPerWG - 1) / kWavesPerWG); };
    if (wgs(4) <= 512 || wgs(4) == wgs(1)) return 4;
    if ((wgs(2) <= 640 && nsl <= 32) || wgs(2) == wgs(1)) return 2;
    return 1;
}

template <int TD, int DD, bool FUSED>
void launch_slices(const VerifyArgs &a, hipStream_t st, Timing tm)
{
    const int split = slice_split(a.B, a.nsl);
    const dim3 grid((a.nsl * split + kWavesPerWG - 1) / kWavesPerWG, a.B), block(kVBlock);         // (a context holds at most 65535 sequences)
    if (split == 4) launch_kernel(verify_slices<TD, DD, FUSED, 4>, grid, block, st, tm, a);
    else if (split == 2) launch_kernel(verify_slices<TD, DD, FUSED, 2>, grid, block, st, tm, a);
    else launch_kernel(verify_slices<TD, DD, FUSED, 1>, grid, block, st, tm, a);
}

// A shard's sums: all slices of a sequence in one workgroup of sixteen wavefronts, which adds them up itself, where that workgroup has
// but one slice or the sequences alone fill the chip; else the slices spread over the chip and a launch behind them adds up (us per call apart
// / together, bfloat16: V = 2000, 64 sequences 7.2 / 5.3; V = 8016, 64 and 256 sequences 7.2 / 7.5, 10.0 / 8.1; V = 16032 8.1 / 9.7, 12.8 / 10.6;
// V = 32064 9.7 / 14.6, 19.5 / 16.5).
constexpr int kShardWaves = 16;
inline bool shard_totals(int B, int nsl) { return nsl == 1 || (B >= 192 && nsl <= kShardWaves); }
template <int TD, int DD>
hipError_t launch_shard_typed(const ShardFinalArgs &a, int pass, hipStream_t st)
{
    if (pass == 0 && shard_totals(a.v.B, a.v.nsl)) {
        VerifyArgs v = a.v;
        v.part2 = a.sums_out;
        const dim3 grid(1, v.B), block(kShardWaves * kWave);
        if (v.nsl <= kShardWaves / 4) launch_kernel(verify_slices<TD, DD, false, 4, kShardWaves>, grid, block, st, Timing{}, v);
        else if (v.nsl <= kShardWaves / 2) launch_kernel(verify_slices<TD, DD, false, 2, kShardWaves>, grid, block, st, Timing{}, v);
        else launch_kernel(verify_slices<TD, DD, false, 1, kShardWaves>, grid, block, st, Timing{}, v);
    } else if (pass == 0) {
        launch_slices<TD, DD, false>(a.v, st, Timing{});
        hipLaunchKernelGGL(shard_sums_kernel, dim3((a.v.B + kWavesPerWG - 1) / kWavesPerWG), dim3(kVBlock), 0, st, a);
    } else {
        hipLaunchKernelGGL((shard_locate<TD, DD>), dim3(a.v.B), dim3(kVBlock), 0, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_shard_dispatch(const ShardFinalArgs &a, int pass, hipStream_t st)
{
    if (!a.v.exp_table) return hipErrorInvalidValue;
    if (a.v.t_dtype == TAPOUT_F32)
        return a.v.d_dtype == TAPOUT_F32 ? launch_shard_typed<TAPOUT_F32, TAPOUT_F32>(a, pass, st) : launch_shard_typed<TAPOUT_F32, TAPOUT_BF16>(a, pass, st);
    return a.v.d_dtype == TAPOUT_F32 ? launch_shard_typed<TAPOUT_BF16, TAPOUT_F32>(a, pass, st) : launch_shard_typed<TAPOUT_BF16, TAPOUT_BF16>(a, pass, st);
}

template <int TD, int DD>
hipError_t launch_typed(const VerifyArgs &a, const DraftFinalArgs &fin, bool with_fin, int pass, hipStream_t st, Timing tm)
{
    const dim3 block(kVBlock);
    if (pass == 1) {
        if (a.fused_head) launch_slices<TD, DD, true>(a, st, tm);
        else launch_slices<TD, DD, false>(a, st, tm);
    }
    else {
        // workgroups that end the round: 32 sequences each (UCB, bandit_tail 1) or sixteen (Thompson Sampling, 2)
        const int per_wg = kVBlock / (a.bandit_tail == 2 ? 16 : TAPOUT_MAX_ARMS);
        const unsigned extra = a.bandit_tail ? (unsigned)((a.B + per_wg - 1) / per_wg) : 0u;
        if (with_fin) launch_kernel(verify_locate<TD, DD, true>, dim3(2 * a.B + extra), block, st, tm, a, fin);
        else launch_kernel(verify_locate<TD, DD, false>, dim3(a.B + extra), block, st, tm, a, fin);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_shard_final_sums(const ShardFinalArgs &a, hipStream_t st) { return launch_shard_dispatch(a, 0, st); }
hipError_t launch_shard_final_token(const ShardFinalArgs &a, hipStream_t st) { return launch_shard_dispatch(a, 1, st); }

hipError_t launch_sample(const SampleArgs &a, const DraftFinalArgs *fin, hipStream_t st, Timing tm)
{
    static const DraftFinalArgs no_fin{};
    if (!a.exp_table || (fin != nullptr) != (a.lse == nullptr)) return hipErrorInvalidValue;
    if (fin && (fin->B != a.B || fin->shards > 0 || !sample_own_lse(a.B, a.K, a.nsplit))) return hipErrorInvalidValue;
    const dim3 grid(a.B * a.K + (fin ? a.B : 0)), block(kVBlock);
    const int own = !fin ? 0 : (lane_merge_fits(a.K, a.nsplit) ? kOwnLanes : kOwnStaged);
    void (*kernel)(SampleArgs, DraftFinalArgs);
    if (a.dtype == TAPOUT_F32) kernel = own == 0 ? sample_locate_kernel<TAPOUT_F32, 0> : (own == kOwnLanes ? sample_locate_kernel<TAPOUT_F32, kOwnLanes> : sample_locate_kernel<TAPOUT_F32, kOwnStaged>);
    else kernel = own == 0 ? sample_locate_kernel<TAPOUT_BF16, 0> : (own == kOwnLanes ? sample_locate_kernel<TAPOUT_BF16, kOwnLanes> : sample_locate_kernel<TAPOUT_BF16, kOwnStaged>);
    launch_kernel(kernel, grid, block, st, tm, a, fin ? *fin : no_fin);
    return hipGetLastError();
}

hipError_t launch_verify(const VerifyArgs &a, int pass, hipStream_t st, Timing tm, const DraftFinalArgs *fin)
{
    static const DraftFinalArgs no_fin{};
    const bool with_fin = fin != nullptr;
    if (!a.exp_table) return hipErrorInvalidValue;           // every pass reads it
    if (((a.vflags & kVerifyOwnQ) != 0) != with_fin || (fin && (a.shards > 0 || fin->shards > 0 || fin->B != a.B || !own_q_shape(a.K, a.nsplit, fin->nsplit))))
        return hipErrorInvalidValue;
    if (!fin) fin = &no_fin;
    if (pass == 0) {
        if (a.fused_head) return hipErrorInvalidValue;       // the slice kernel is the head then
        const bool staged = !lane_merge_fits(a.K + 1, a.nsplit);
        if (a.shards > 0) launch_kernel(staged ? verify_head_kernel<true, true> : verify_head_kernel<true, false>, dim3(a.B), dim3(kVBlock), st, tm, a);
        else launch_kernel(staged ? verify_head_kernel<false, true> : verify_head_kernel<false, false>, dim3(a.B), dim3(kVBlock), st, tm, a);
        return hipGetLastError();
    }
    if (a.t_dtype == TAPOUT_F32)
        return a.d_dtype == TAPOUT_F32 ? launch_typed<TAPOUT_F32, TAPOUT_F32>(a, *fin, with_fin, pass, st, tm) : launch_typed<TAPOUT_F32, TAPOUT_BF16>(a, *fin, with_fin, pass, st, tm);
    return a.d_dtype == TAPOUT_F32 ? launch_typed<TAPOUT_BF16, TAPOUT_F32>(a, *fin, with_fin, pass, st, tm) : launch_typed<TAPOUT_BF16, TAPOUT_BF16>(a, *fin, with_fin, pass, st, tm);
}

}  // namespace tapout

#ifdef TAPOUT_WG_STAMPS
// Copies one stamp table to the host (synchronises the device).  table 0: slice kernel, 8 slots per workgroup
// (0 entry, 1 job known, 2 tables in LDS and rows requested, 3..6 each wavefront's loop done, 7 sums stored);
// table 1: accept decisions inside the slice kernel, 4 slots (0 first requests answered, 1 rows merged, 2 decisions
// taken, 3 first rejection published); table 2: locate kernel, 8 slots by blockIdx.x (0 entry, 1 first requests
// answered, 2 total weight known, 3 slice found, 4 token found, 5 written; 7: a draft epilogue workgroup is done).
// Units: 10 ns.  Not part of the library's interface.
extern "C" __attribute__((visibility("default"))) int tapout_debug_wg_stamps(int table, unsigned long long *host, int n_wg)
{
    if (!host || n_wg < 0) return -1;
    if (hipDeviceSynchronize() != hipSuccess) return -2;
    if (table == 0 && n_wg <= tapout::kStampWgs)
        return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(tapout::g_stamps_slices), (size_t)n_wg * 8 * sizeof(unsigned long long));
    if (table == 1 && n_wg <= tapout::kStampWgs)
        return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(tapout::g_stamps_head), (size_t)n_wg * 4 * sizeof(unsigned long long));
    if (table == 2 && n_wg <= 4096)
        return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(tapout::g_stamps_locate), (size_t)n_wg * 8 * sizeof(unsigned long long));
    return -1;
}
#endif
