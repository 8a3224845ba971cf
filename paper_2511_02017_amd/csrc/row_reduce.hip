// Streaming pass over logits rows: the one read of the vocabulary that feeds
// every signal of Table 1 / Appendix A.1 (entropy, top-1 probability,
// top-1/top-2 margin) and the normalisers the verification step needs.
//
// One launch covers all rows of a [B, KK, V] tensor.  A row is cut into
// `nsplit` slices of whole 16-byte vectors; one 256-thread workgroup reduces
// one slice to a 32-byte Partial.  Every element is loaded exactly once, with
// 16-byte non-temporal loads that are contiguous across the wavefront, four
// vectors per thread in flight; six (draft) or eight (target) wavefronts per
// SIMD hide the latency (explicit double buffering was measured: slower).
// Batches that lie wholly inside the slice are loaded without bounds checks.
//
// Per thread the softmax sums are kept online in the base-2 domain against an
// integer reference R >= max * log2 e: y = fma(x, log2e, -R) has a single
// rounding, 2^y comes from the hardware exp2, and moving to a larger reference
// is an exact ldexp.  The maximum, and for draft rows the largest value outside
// the batch of vectors in which it appeared, are kept once per batch; with the
// second largest value inside that batch, which the epilogue reads again (below),
// the latter gives the row's second maximum.  Only the 16-byte window in which
// the thread's maximum first appeared is remembered; the exact argmax index is
// recovered later from that window.
//
// Draft rows: the entropy of a peaked row is a small number made of small
// terms, and a binary32 sum that also holds the row's dominant term rounds
// them away.  So the batch of vectors in which a thread met its maximum is
// summed apart from the rest, and the workgroup leaves the batch that holds the
// slice's first maximum out of its partial altogether: the sums of a partial
// then hold "small" terms only, and the epilogue that merges the partials adds
// the few elements of that one batch back from the logits themselves, with the
// row's first maximum as an exact term of its own.
//
// Wavefront reductions use DPP row operations (no LDS traffic).  The partials
// are merged per sequence by a second, small launch (finalize.hip for draft
// rows, the head kernel in verify.hip for target rows): a
// "last workgroup finishes the sequence" scheme was measured and lost, because
// on this chip every cross-workgroup hand-over costs a memory round trip of
// about 3 us under streaming load and four of them chain up.
#include "common.h"
#include "exp_device.h"
#include "finalize_device.h"

namespace tapout {

namespace {

// max3 / med3 / max as the bare instructions.  fmaxf() and the med3 builtin first quiet every operand the compiler
// cannot prove to be a canonical number (one v_max_f32 x, x per logit, a tenth of the draft pass's vector
// instructions); the instructions themselves already return the other operand when one is a NaN, which is what the
// running maxima want (NaN logits are ignored here and poison the sums instead).
__device__ inline float max3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ inline float med3(float a, float b, float c)
{
    float r;
    asm("v_med3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ inline float max2(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Headroom (in powers of two) added to a thread's reference when it has to be
// raised, so that a slowly growing running maximum raises it only a few times.
constexpr float kHeadroom = 8.0f;

template <int N>
__device__ inline void widen(const u32x4 &w, float (&x)[N])
{
    if constexpr (N == 8) unpack<TAPOUT_BF16>(w, x);
    else if constexpr (N == 4) unpack<TAPOUT_F32>(w, x);
    else x[0] = __uint_as_float(w.x);
}

template <bool FULL>
struct ThreadState {
    float v1 = -INFINITY;   // running maximum
    float v2 = -INFINITY;   // FULL: the largest value outside the batch in which the running maximum appeared
    float R = -1.0e30f;     // integer reference: every x seen so far has x*log2e <= R (+ rounding); -1e30: none yet
    float s = 0.0f;         // sum 2^(x*log2e - R); FULL: without the batch in which the running maximum appeared
    float t = 0.0f;         // sum 2^y * y (FULL only), likewise
    float s_hi = 0.0f;      // FULL: the two sums over the batch in which the running maximum appeared
    float t_hi = 0.0f;
    int32_t cand = 0x7fffffff;

    // Raise the reference so that it covers a vector's maximum m (rare after the first few vectors).
    // sb, tb: the sums of the batch in progress.
    __device__ inline void cover(float m, float &sb, float &tb)
    {
        if (__builtin_fmaf(m, kLog2e, -R) > 0.0f) {           // also the first finite value (nothing is summed yet then)
            float Rn = ceilf(m * kLog2e) + kHeadroom;
            float d = Rn - R;
            int di = (int)fminf(fmaxf(d, -1.0e9f), 1.0e9f);
            if constexpr (FULL) {
                t = ldexpf(t - d * s, -di);
                t_hi = ldexpf(t_hi - d * s_hi, -di);
                tb = ldexpf(tb - d * sb, -di);
                s_hi = ldexpf(s_hi, -di);
            }
            s = ldexpf(s, -di);
            sb = ldexpf(sb, -di);
            R = Rn;
        }
    }

    // A batch of U vectors of N values each (vector u starts at element index first + u * stride of the row), vector by vector:
    // maximum, reference check, sums.  n: the vectors behind the n-th hold nothing in the whole wavefront and are passed over.
    //
    // What can wait is done once per batch: the running maximum, the largest value outside its batch (the row's second
    // maximum is one of those or lies in the set-apart batch, which the epilogue reads again anyway) and which vector holds
    // the maximum, the first of several (remembered as the argmax candidate).  With the second maximum and the candidate kept vector
    // by vector the maxima took 1.5 instructions an element instead of 0.5.  The tokens' draw, which this arithmetic bounds: 46.4
    // -> 44.8 us for 512 rows of 128256 bf16 logits, 33.2 -> 32.1 for 256 rows of 151936; the draft pass waits for memory: 28.6 ->
    // 28.4 at the first size.
    //
    // The entropy sum of a vector is formed without looking at the terms; a masked (-inf) logit gives 0 * -inf = NaN there, and only
    // then the vector is summed again with the exponent clamped (one comparison per vector instead of one clamp per element).
    // each(u): called when vector u has been folded.
    template <int U, int N, class Each>
    __device__ inline void fold_batch(const u32x4 (&w)[U], int n, int32_t first, int32_t stride, Each each)
    {
        float vm[U], sb = 0.0f, tb = 0.0f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            vm[u] = -INFINITY;
            if (U > 1 && u >= n) continue;
            float x[N], y[N], e[N];
            widen<N>(w[u], x);
            vm[u] = vector_max(x);
            cover(vm[u], sb, tb);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                y[i] = __builtin_fmaf(x[i], kLog2e, -R);
                e[i] = __builtin_amdgcn_exp2f(y[i]);
            }
            float sv = e[0];
            float tv = FULL ? e[0] * y[0] : 0.0f;
#pragma unroll
            for (int i = 1; i < N; ++i) {
                sv += e[i];
                if constexpr (FULL) tv = __builtin_fmaf(e[i], y[i], tv);
            }
            if constexpr (FULL) {
                if (tv != tv) {
                    tv = 0.0f;
#pragma unroll
                    for (int i = 0; i < N; ++i) tv = __builtin_fmaf(e[i], fmaxf(y[i], -200.0f), tv);
                }
                tb = u == 0 ? tv : tb + tv;
            }
            sb = u == 0 ? sv : sb + sv;                        // (a sum started from 0.0f would cost an addition: -0 + 0)
            each(u);
        }
        float bm = vm[0];
        if constexpr (U == 4) bm = max2(max3(vm[0], vm[1], vm[2]), vm[3]);
        static_assert(U == 1 || U == 4, "the maximum of a batch's vectors");
        const bool grew = bm > v1;                             // a lane mask in scalar registers
        if constexpr (FULL) v2 = med3(v1, v2, bm);
        v1 = max2(v1, bm);
        int32_t at = U - 1;
#pragma unroll
        for (int u = U - 2; u >= 0; --u) at = vm[u] == bm ? u : at;
        asm("" : "+v"(at));                                    // (a number below four is in the instruction, its product with the stride in a register)
        cand = grew ? first + at * stride : cand;
        if constexpr (FULL) {
            // If the running maximum grew inside the batch, its sums become the set-apart ones and the batch that held
            // the previous maximum joins the rest; else it joins the rest itself.
            s += grew ? s_hi : sb;
            t += grew ? t_hi : tb;
            s_hi = grew ? sb : s_hi;
            t_hi = grew ? tb : t_hi;
        } else {
            s += sb;
        }
    }

    // One element on its own (unaligned head or tail of a row): a batch of one.
    __device__ inline void fold_single(float x0, int32_t j)
    {
        u32x4 w[1];
        w[0] = u32x4{__float_as_uint(x0), 0u, 0u, 0u};
        fold_batch<1, 1>(w, 1, j, 0, [](int) {});
    }
};

// ---- wavefront reductions with DPP -------------------------------------------
// quad_perm [1,0,3,2] = 0xB1, quad_perm [2,3,0,1] = 0x4E, row_half_mirror = 0x141, row_mirror = 0x140: after the four steps every
// lane of a 16-lane row holds the row's result; row_bcast15 and row_bcast31 carry it on from row to row.
template <int CTRL, int ROWS>
__device__ inline float dpp_rows(float v) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, true)); }
// Maximum over the 64 lanes, in a scalar register (bare instructions: see max3; a DPP operand is read two wait states after it was written).
__device__ inline float wave_max(float v)
{
    asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf"
        : "+v"(v));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}
// Sum over the 64 lanes; valid in the last lane.
__device__ inline float wave_sum_last(float v)
{
    v += dpp_rows<0xB1, 0xf>(v); v += dpp_rows<0x4E, 0xf>(v); v += dpp_rows<0x141, 0xf>(v); v += dpp_rows<0x140, 0xf>(v);
    v += dpp_rows<0x142, 0xa>(v);
    v += dpp_rows<0x143, 0xc>(v);
    return v;
}
__device__ inline double wave_sum_last(double v) { return wave_sum_d(v); }
// The value of one lane, in a scalar register.
__device__ inline float of_lane(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }
__device__ inline float scaled(float v, int e) { return ldexpf(v, e); }
__device__ inline double scaled(double v, int e) { return ldexp(v, e); }
__device__ inline u32x4 two_doubles(double a, double b)
{
    return u32x4{(uint32_t)__double2loint(a), (uint32_t)__double2hiint(a), (uint32_t)__double2loint(b), (uint32_t)__double2hiint(b)};
}
__device__ inline double double_of(uint32_t lo, uint32_t hi) { return __hiloint2double((int)hi, (int)lo); }
__device__ inline int wave_min_i(int v)
{
    v = min(v, dpp_mov<0xB1>(v)); v = min(v, dpp_mov<0x4E>(v)); v = min(v, dpp_mov<0x141>(v)); v = min(v, dpp_mov<0x140>(v));
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

template <int DT> struct NegInfVec;
template <> struct NegInfVec<TAPOUT_F32>  { static constexpr uint32_t word = 0xff800000u; };
template <> struct NegInfVec<TAPOUT_BF16> { static constexpr uint32_t word = 0xff80ff80u; };

__device__ inline float quad_sum(float v) { v += dpp_mov<0xB1>(v); return v + dpp_mov<0x4E>(v); }

template <int DT, int U, bool CHECKED>
__device__ inline void load_batch(u32x4 (&w)[U], const u32x4 *vp, int i, int end)
{
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int idx = i + u * kBlock;
        if (!CHECKED || idx < end) w[u] = __builtin_nontemporal_load(vp + idx);
        else { const uint32_t ni = NegInfVec<DT>::word; w[u] = u32x4{ni, ni, ni, ni}; }   // -inf padding folds to nothing
    }
}

struct NoMore { __device__ void operator()(int) const {} };
template <int DT, bool FULL, int U, class Each = NoMore>
__device__ inline void fold_batch(ThreadState<FULL> &st, const u32x4 (&w)[U], int n, int i, int head, Each each = Each())
{
    constexpr int VEC = Elem<DT>::vec;
    st.template fold_batch<U, VEC>(w, n, head + i * VEC, kBlock * VEC, each);
}

// How many of its vectors of a batch a wavefront has to fold (first: the batch's first vector, end: behind the slice's last one), where
// the vector ALU is what bounds the pass: the draw's.  (Its launch, 1024 rows of V = 50257, bfloat16 48.5 us with the whole batch
// folded at the end of a row, 41.7 so, and 0.3 of 41 us the other way where batches are whole; the passes without a draw wait for memory,
// 0.3 % longer with it.)
template <int U>
__device__ inline int wave_vectors(int first, int end)
{
    const int left = end - __builtin_amdgcn_readfirstlane(first + ((int)threadIdx.x & (kBlock - 1) & -kWave));
    return max(min((left + kBlock - 1) / kBlock, U), 0);
}

// ---- slice sums of the draft-token draw, on the way ------------------------------------------------
// The inverse CDF of a draft row runs over sums of exponentials in double.  They need no row maximum if they are kept in the
// logits' own scale: exp(x) as it is, from the table for bfloat16 values, computed for binary32 ones, is in range for rows whose maximum
// lies in [-600, 700); others are summed again where their token is drawn.  So the pass that reads the rows for
// their statistics forms these sums too.  A draw slice is one vector per thread, kBlock vectors: a batch holds kStreamU of them,
// each wavefront leaves its own sums, [draw slice][wavefront].
// Slices a workgroup works on side by side, and workgroups of a compute unit.  bfloat16: two slices share a copy of the table, so that
// four copies in LDS serve eight wavefronts per SIMD (64 registers); binary32: no table, six wavefronts (72 registers).  The kernel
// is bound by vector instructions (rocprofv3 at V = 128256, 512 rows, bfloat16: vector ALU busy 66 %, LDS in use 34 %): us per call with four / six / eight wavefronts per
// SIMD 53.5 / 53.9 / 49.5, 64 rows 14.9 / 14.8 / 15.4; a batch asked for ahead of the one at hand changed nothing there.
template <int DT> struct DrawShape;
template <> struct DrawShape<TAPOUT_BF16> { static constexpr int parts = 2, per_cu = 4, few_per_cu = 3; };
template <> struct DrawShape<TAPOUT_F32>  { static constexpr int parts = 1, per_cu = 6, few_per_cu = 6; };
template <int DT>
struct DrawSums {
    const double *T, *E;             // tables in LDS: 2^(k/256) and, for bfloat16, exp(x)
    bool table;                      // bfloat16: look exponentials up
    double *out;                     // of the slice the workgroup is at

    __device__ inline double computed(float x) const { return exp_fast(x, 0.0, kDrawLow, T, kExpC2, kDrawHigh); }
    __device__ inline double computed(const u32x4 &w) const
    {
        constexpr int VEC = Elem<DT>::vec;
        float x[VEC];
        unpack<DT>(w, x);
        double e = 0.0;
#pragma unroll
        for (int i = 0; i < VEC; i += 2) {                   // two at a time: all of them side by side want sixty registers more
            e += computed(x[i]) + computed(x[i + 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        return e;
    }
    __device__ inline double looked_up(const u32x4 &w) const
    {
        const char *at = (const char *)E;
        double e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const TabOffsets o = tab_offsets2(w[i]);
            e[i] = *(const double *)(at + o.lo) + *(const double *)(at + o.hi);
        }
        return (e[0] + e[1]) + (e[2] + e[3]);
    }
    // The four sums of a batch over the wavefront: the first two steps halve the number of values, so that each sixteen
    // lanes end with one of them.
    __device__ inline void store(const double (&v)[kStreamU], int bi) const
    {
        static_assert(kStreamU == 4, "one value for each sixteen lanes");
        auto both = [](double a, double b, auto swap) {
            const auto h = swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b)), l = swap((unsigned)__double2loint(a), (unsigned)__double2loint(b));
            return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
        };
        auto swap32 = [](unsigned a, unsigned b) { return __builtin_amdgcn_permlane32_swap(a, b, false, false); };
        auto swap16 = [](unsigned a, unsigned b) { return __builtin_amdgcn_permlane16_swap(a, b, false, false); };
        double x = both(both(v[0], v[1], swap32), both(v[2], v[3], swap32), swap16);       // rows of sixteen lanes: v[0], v[2], v[1], v[3]
        x += dpp_d<0xB1>(x); x += dpp_d<0x4E>(x); x += dpp_d<0x141>(x); x += dpp_d<0x140>(x);
        const int lane = threadIdx.x & (kWave - 1), row = lane >> 4, wave = (threadIdx.x & (kBlock - 1)) / kWave;
        const int q = ((row & 1) << 1) | (row >> 1);
        if ((lane & 15) == 0) out[(bi * kStreamU + q) * (kBlock / kWave) + wave] = x;
    }
    // One vector's sum.
    __device__ inline double vector(const u32x4 &w) const
    {
        double e = DT == TAPOUT_BF16 ? looked_up(w) : computed(w);
        asm volatile("" : "+v"(e));                          // summed here and now: else the terms, two registers each, wait for the end of the batch
        return e;
    }
    // Which of a batch's sums v have to be formed again (again()), a bit each: those of vectors that hold a value which is not in
    // the table.
    __device__ inline uint32_t missing(const double (&v)[kStreamU]) const
    {
        if constexpr (DT != TAPOUT_BF16) return 0u;
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < kStreamU; ++u) m |= __builtin_amdgcn_ballot_w64(v[u] != v[u]) != 0 ? 1u << u : 0u;
        return m;
    }
    // Whether the slice is not for the table, which counts everything beyond it as 0: a thread of the wavefront has met a value above it, or
    // none has met one beside which what lies below doesn't matter (see kDrawLowTab).  Not where all is masked so far.  v1: the thread's
    // maximum so far.  From the batch on that shows it nothing is looked up any more, and the slice's sums are computed from its logits
    // once more when its statistics are done and their registers free.  (us per call, bfloat16 logits around -40, all of it left to the
    // one workgroup that draws a row's token / this: V = 128256, 64 sequences of 8 rows 110 / 79, of one 51 / 19, V = 50257, 48 sequences of 7
    // 54 / 37; one row of V = 128256 46.1 / 13.5, where logits in the table's range take 11.7.)
    __device__ inline bool off_table(float v1) const
    {
        return __builtin_amdgcn_ballot_w64(v1 >= kTabEnd) != 0 || (__builtin_amdgcn_ballot_w64(v1 >= kDrawLowTab) == 0 && __builtin_amdgcn_ballot_w64(v1 >= kDrawLow) != 0);
    }
    // The sum of vector u of batch bi once more, computed, with a thread's lone element (its exponential) beside it.  The lane that
    // stored the first one stores it.
    __device__ inline void again(const u32x4 &w, double lone, int bi, int u, int tid) const
    {
        asm volatile("" : "+v"(tid));                        // (else what is formed of it here waits in registers from the kernel's start on)
        const double x = wave_sum_d(computed(w) + lone);
        const int lane = tid & (kWave - 1), row = ((u & 1) << 1) | (u >> 1), wave = tid / kWave;
        if (lane == row * 16) out[(bi * kStreamU + u) * (kBlock / kWave) + wave] = x;
    }
};

// What a workgroup leaves of slice `split` of a row: the threads' sums reduced, its Partial written.  tok_bits: the logit of the row's
// token, if the slice holds it.  set: which of kSets copies of the records in LDS; on: there is a slice (all threads come to the barrier).
// RECORD > 0: the slice is the whole row, rowp, read by so many wavefronts, and what is left is the row's shard record: everything but the first maximum, whose index
// is exact and global.  From the threads on its sums are added in double, and each wavefront's first maximum as a term of its own, as the
// merge of several slices does: a row of two to four batches brings its longer sums of a thread, and a binary32 reduction would come
// on top (root mean square of the relative error of S, two batches of bfloat16, logits of spread 0.5: slices merged 4.4e-8, in binary32
// 5.8e-8, this 3.1e-8; spread 5 2.33e-7, 2.40e-7, 2.28e-7; us per call, 64 sequences of 8 rows, in binary32 / this 7.0 / 7.2).
template <int DT, bool FULL, int kSets = 1, int PARTS = 1, int RECORD = 0>
__device__ inline void finish_slice(const RowReduceArgs &a, const ThreadState<FULL> &st, const int split, const int row, const uint32_t tok_bits,
                                    const bool holds_tok, const int set = 0, const bool on = true, const char *rowp = nullptr, const int vocab_offset = 0)
{
    static_assert(RECORD == 0 || FULL, "a record holds all statistics");
    using Sum = std::conditional_t<RECORD != 0, double, float>;
    constexpr int kWaves = RECORD != 0 ? RECORD : kBlock / kWave;
    __shared__ u32x4 sh_rec[kSets][kWaves][2];
    const int tid = PARTS > 1 ? threadIdx.x & (kBlock - 1) : threadIdx.x;
    // Every wavefront brings its sums to its own maximum and leaves one record; the first wavefront merges the four, a lane each.
    // What a slice costs besides its loads is this chain of instructions (a wavefront issues one in about nine cycles here), in
    // every workgroup of a launch and, in small ones, in the open: us per pass, with the reduction
    // it replaces (every thread to the workgroup maximum first, three barriers, one thread merging) and with this: V = 128256, 64 sequences,
    // K = 8 up to the stop position 61.7 / 60.4, V = 50257, 48 sequences 57.9 / 56.5, V = 32000, one sequence 19.7 / 19.4.
    const int wave = tid / kWave, lane = tid % kWave;
    const float Mw = wave_max(st.v1), Rw = ref_of_max(Mw);
    const float d = Rw - st.R;
    const int di = (int)fminf(fmaxf(d, -1.0e9f), 1.0e9f);
    Sum s = scaled((Sum)st.s, -di);                             // exact scaling
    Sum t = 0.0f, s_hi = 0.0f, t_hi = 0.0f;
    if constexpr (FULL) {
        t = scaled((Sum)st.t - (Sum)d * (Sum)st.s, -di);
        s_hi = scaled((Sum)st.s_hi, -di);
        t_hi = scaled((Sum)st.t_hi - (Sum)d * (Sum)st.s_hi, -di);
    }
    if (st.v1 == -INFINITY && !(st.s != st.s)) { s = 0.0f; t = 0.0f; s_hi = 0.0f; t_hi = 0.0f; }   // thread saw nothing finite
    // the wavefront's vector with its first maximum: one thread's, unless several met that value
    const uint64_t met = __builtin_amdgcn_ballot_w64(st.v1 == Mw);
    int owner = __builtin_ctzll(met), cw = __builtin_amdgcn_readlane(st.cand, owner);
    if (met & (met - 1)) {
        cw = wave_min_i(st.v1 == Mw ? st.cand : 0x7fffffff);
        owner = __builtin_ctzll(__builtin_amdgcn_ballot_w64(st.v1 == Mw && st.cand == cw));
    }
    // FULL: that thread's set-apart batch stays out of the wavefront's sums and goes into the record on its own (every other
    // thread's is ordinary data).  Largest value outside that batch: of that thread the one it kept (st.v2), of the others the maximum
    float v2w = -INFINITY;
    if constexpr (FULL) {
        s += lane == owner ? (Sum)0.0f : s_hi;
        t += lane == owner ? (Sum)0.0f : t_hi;
        v2w = wave_max(lane == owner ? st.v2 : st.v1);
        t = wave_sum_last(t);
    }
    s = wave_sum_last(s);
    if constexpr (RECORD != 0) {
        if (lane == kWave - 1) {
            sh_rec[set][wave][0] = u32x4{__float_as_uint(Mw), 0u, (uint32_t)cw, __float_as_uint(v2w)};
            sh_rec[set][wave][1] = two_doubles(s, t);
        }
        __syncthreads();
        if (wave > 0) return;
        // Four lanes for each wavefront's record, one for each vector of its set-apart batch, which comes back from the logits (and poisons the
        // sums where it holds a NaN or an infinity): all but the wavefront's first maximum, which is a term of its own unless it is the row's.
        constexpr int kVecBits = 2, kBits = kWaves == 4 ? 4 : (kWaves == 8 ? 5 : 6);
        static_assert(kStreamU == 1 << kVecBits && kWaves == 1 << (kBits - kVecBits), "a wavefront's lanes");
        const int u = lane & (kStreamU - 1), from = (lane >> kVecBits) & (kWaves - 1);
        const u32x4 r0 = sh_rec[set][from][0], r1 = sh_rec[set][from][1];
        const float Ml = __uint_as_float(r0.x);
        const int cl = (int)r0.z;
        const BatchVecs<1> bt = batch_issue_vecs<1>(batch_geom(rowp, DT, a.V, 0, a.per), DT, a.V, cl, u, a.out);
        const float M = lanes_max(Ml, kVecBits, kBits), R = ref_of_max(M), dl = R - ref_of_max(Ml);
        const int dil = (int)fminf(fmaxf(dl, -1.0e9f), 1.0e9f), cand = lanes_min(Ml == M ? cl : 0x7fffffff, kVecBits, kBits);
        const bool holds = Ml == M && cl == cand;
        const double s0 = double_of(r1.x, r1.y);
        double S = ldexp(s0, -dil), T = Ml == -INFINITY ? 0.0 : ldexp(fma(-(double)dl, s0, double_of(r1.z, r1.w)), -dil);
        if (!holds && Ml > -INFINITY) {
            const float y = __builtin_fmaf(Ml, kLog2e, -R), e = __builtin_amdgcn_exp2f(y);
            S += (double)e;
            T += (double)e * (double)fmaxf(y, -200.0f);
        }
        const BatchExtra x = batch_sum<DT>(R, Ml, true, bt, u);
        const float v2 = lanes_max(fmaxf(holds ? __uint_as_float(r0.w) : Ml, x.m2), 0, kBits);
        const int idx = lanes_min(holds ? x.idx : 0x7fffffff, 0, kBits);
        S = lanes_sum(S, kVecBits, kBits) + lanes_sum((double)x.sa, 0, kBits);
        T = lanes_sum(T, kVecBits, kBits) + lanes_sum((double)x.ta, 0, kBits);
        if (tid == 0) {
            u32x4 *o = (u32x4 *)(a.out + row);
            o[0] = u32x4{__float_as_uint(M), __float_as_uint((float)S), __float_as_uint((float)T), __float_as_uint(v2)};
            o[1] = u32x4{(uint32_t)(vocab_offset + (idx >= 0 && idx < a.V ? idx : 0)), holds_tok ? (DT == TAPOUT_F32 ? tok_bits : tok_bits << 16) : 0x7fc00000u, 0u, 0u};
        }
    } else {
        const float hs = FULL ? of_lane(s_hi, owner) : 0.0f, ht = FULL ? of_lane(t_hi, owner) : 0.0f;
        if (lane == kWave - 1) {
            sh_rec[set][wave][0] = u32x4{__float_as_uint(Mw), __float_as_uint(s), (uint32_t)cw, __float_as_uint(v2w)};
            if constexpr (FULL) sh_rec[set][wave][1] = u32x4{__float_as_uint(t), __float_as_uint(hs), __float_as_uint(ht), 0u};
        }
        __syncthreads();
        if (wave > 0) return;
        constexpr int kBits = 2;                                // four records, one on each lane of a quad
        static_assert(kBlock / kWave == 1 << kBits, "a record per wavefront");
        const u32x4 r0 = sh_rec[set][lane & 3][0];
        const float Ml = __uint_as_float(r0.x), M = lanes_max(Ml, 0, kBits);
        const bool met_it = Ml == M;
        const float dl = ref_of_max(M) - ref_of_max(Ml);
        const int dil = (int)fminf(fmaxf(dl, -1.0e9f), 1.0e9f);
        Partial p;
        p.v1 = M;
        p.cand = lanes_min(met_it ? (int)r0.z : 0x7fffffff, 0, kBits);
        const float s0 = __uint_as_float(r0.y);
        p.T = 0.0f; p.v2 = -INFINITY; p.pad[1] = 0;
        if constexpr (FULL) {
            const u32x4 r1 = sh_rec[set][lane & 3][1];
            const float hs0 = __uint_as_float(r1.y);
            const bool holds = met_it && (int)r0.z == p.cand;
            // The batch with the slice's first maximum stays out (the epilogue adds its elements back from the
            // logits); the set-apart batches of the other wavefronts are ordinary data.  A NaN or an infinity
            // inside the left-out batch must still poison the sums: x - x is 0 for finite x only.
            // In double from here on: going over to the slice's reference adds up to three times the sum's own rounding to T, which four
            // records do not average out (errors, root mean square: entropy, V = 8000, logits of spread 2, 3.5e-8 in binary32, 3.1e-8 so; margin,
            // V = 32000, 32 sequences of 8 rows 8.0e-8 and 7.5e-8; us per round, V = 128256, 64 sequences 67.9 / 67.9, up to the stop position 58.7 / 59.0).
            const double s1 = (double)s0 + (double)(holds ? hs0 - hs0 : hs0), t1 = (double)__uint_as_float(r1.x) + (double)(holds ? 0.0f : __uint_as_float(r1.z));
            const double T = Ml == -INFINITY ? 0.0 : ldexp(fma(-(double)dl, s1, t1), -dil);       // (a record without a finite maximum: dl is no distance)
            p.v2 = lanes_max(holds ? __uint_as_float(r0.w) : Ml, 0, kBits);
            p.S = (float)lanes_sum(ldexp(s1, -dil), 0, kBits);
            p.T = (float)lanes_sum(T, 0, kBits);
            // the left-out batch's own sum (same reference): S + this is the slice's sum over every element, to
            // binary32 precision, for a reader that wants the row's lse before the epilogue has run
            p.pad[1] = __float_as_int(quad_sum(holds ? ldexpf(hs0, -dil) : 0.0f));
        } else {
            p.S = quad_sum(ldexpf(s0, -dil));
        }
        p.pad[0] = holds_tok ? (int)(DT == TAPOUT_F32 ? tok_bits : tok_bits << 16) : 0x7fc00000;
        if (tid == 0 && on) {
            u32x4 *o = (u32x4 *)(a.out + (int64_t)row * a.nsplit + split);
            o[0] = u32x4{__float_as_uint(p.v1), __float_as_uint(p.S), __float_as_uint(p.T), __float_as_uint(p.v2)};
            o[1] = u32x4{(uint32_t)p.cand, (uint32_t)p.pad[0], (uint32_t)p.pad[1], 0u};
        }
    }
}

// The work of one workgroup: slice `split` of row k of sequence b.  RECORD (see finish_slice): kBlock threads for every fourth
// of it, which take the row's batches in turn.
template <int DT, bool FULL, int RECORD = 0>
__device__ inline void stream_pass_body(const RowReduceArgs &a, const int split, const int k, const int b, const int vocab_offset = 0)
{
    constexpr int VEC = Elem<DT>::vec;
    // vectors in flight per thread.  Four is best for both passes: for the draft pass that means 77 registers
    // and six wavefronts per SIMD instead of eight, which still beats two vectors at full occupancy
    // (measured; three, six and eight vectors and an explicit prefetch of the next batch are all slower).
    constexpr int U = kStreamU;
    constexpr int kParts = RECORD > kBlock / kWave ? RECORD * kWave / kBlock : 1;

    const int tid = kParts > 1 ? threadIdx.x & (kBlock - 1) : threadIdx.x, part = kParts > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kBlock) : 0;
    int n_active;                                   // rows of sequence b this pass reads
    if (a.len_mode == 0) {                          // draft rows: k < k_len[b]
        n_active = a.len ? a.len[b] : a.KK;
        n_active = n_active > a.KK ? a.KK : (n_active < 0 ? 0 : n_active);
    } else {                                        // target rows: k <= n_draft[b]
        int n = a.len[b];
        n_active = (n < 1 ? 1 : (n > a.KK - 1 ? a.KK - 1 : n)) + 1;
    }
    if (a.clear_jobs && split == 0 && k == 0 && tid == 0) a.clear_jobs[b].band_cnt = 0;
    if (a.arm_dst && split == 0 && k == 0 && tid == 0) a.arm_dst[b] = a.arm_src[b];
    if (k >= n_active) return;
    // The row's token, if it has one.  Requested as a vector load (the index carries a zero the compiler cannot
    // see through): a scalar load from memory would hold up the first wait for the kernel arguments and with it
    // the first logits; this one returns with the first batch.
    int tk = -1;
    if (a.tok && k < a.tok_rows) {                          // target rows, and draft rows when the caller wants log q(tok) early
        int zero;
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
        tk = a.tok[(int64_t)b * a.tok_rows + k + zero];
        if constexpr (RECORD != 0) tk -= vocab_offset;
    }
    const char *rowp = (const char *)a.base + ((int64_t)b * a.stride_b + (int64_t)k * a.stride_k) * Elem<DT>::size;
    int head, nvec, tail;
    row_geometry<DT>(rowp, a.V, head, nvec, tail);
    const u32x4 *vp = (const u32x4 *)(rowp + (int64_t)head * Elem<DT>::size);
    // a.per: vectors per slice, chosen on the host as a multiple of 64 (whole 1 KB wavefront loads, so
    // slices of aligned rows start on cache-line boundaries) with nsplit * per >= the vectors of any row
    const int v0 = min(split * a.per, nvec), v1e = min(v0 + a.per, nvec);

    ThreadState<FULL> st;
    // unaligned head (first slice) and tail (last slice): one element per thread
    if (split == 0 && part == 0 && tid < head) st.fold_single(load_elem<DT>(rowp, tid), tid);
    {
        const int nbatch = (v1e - v0 + U * kBlock - 1) / (U * kBlock), nfull = (v1e - v0) / (U * kBlock);
        int i = v0 + part * (U * kBlock) + tid;
        // A compute unit issues the loads of its oldest wavefront first, so of the eight workgroups that share
        // it the ones dispatched first run ahead and the rest trail by up to a third of the launch; the chip
        // then drains with few loads in flight.  Lowering a wavefront's priority as it gets through its slice
        // keeps the workgroups of a compute unit level (measured: launch 0.6 us shorter for the draft pass).
        const int q1 = nbatch / 4, q2 = nbatch / 2, q3 = (3 * nbatch) / 4;
        __builtin_amdgcn_s_setprio(3);
        for (int bi = part; bi < nbatch; bi += kParts, i += kParts * U * kBlock) {
            if (bi == q1) __builtin_amdgcn_s_setprio(2);
            if (bi == q2) __builtin_amdgcn_s_setprio(1);
            if (bi == q3) __builtin_amdgcn_s_setprio(0);
            u32x4 w[U];
            if (bi < nfull) load_batch<DT, U, false>(w, vp, i, v1e);      // every vector of the batch lies inside the slice
            else load_batch<DT, U, true>(w, vp, i, v1e);
            fold_batch<DT, FULL, U>(st, w, U, i, head);
        }
        __builtin_amdgcn_s_setprio(3);      // finish the reduction promptly: the slot is wanted by the next workgroup
    }
    // The token's logit, if this slice holds it (elements [e0, e1); every index of the row lies in exactly one slice): the first
    // wavefront asks for it now and looks at it last (as the bits they are: widened in this branch, they would be waited for here).
    uint32_t tok_bits = 0;
    bool holds_tok = false;
    {
        const int t = __builtin_amdgcn_readfirstlane(tid < kWave && part == 0 ? tk : -1);
        const int e0 = split == 0 ? 0 : head + v0 * VEC, e1 = split == a.nsplit - 1 ? a.V : head + v1e * VEC;
        if (t >= e0 && t < e1) {
            // the row's address once more, from scalar registers (the zero is opaque to the compiler): holding the
            // one from the top of the kernel in vector registers through the loop costs the draft pass a wavefront per SIMD
            int zero;
            asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
            const char *rp = (const char *)a.base + ((int64_t)(b + zero) * a.stride_b + (int64_t)k * a.stride_k) * Elem<DT>::size;
            if constexpr (DT == TAPOUT_F32) tok_bits = ((const uint32_t *)rp)[t]; else tok_bits = ((const uint16_t *)rp)[t];
            holds_tok = true;
        }
    }
    if (split == a.nsplit - 1 && part == 0 && tid < tail) {
        int32_t j = head + nvec * VEC + tid;
        st.fold_single(load_elem<DT>(rowp, j), j);
    }

    finish_slice<DT, FULL, 1, 1, RECORD>(a, st, split, b * a.KK + k, tok_bits, holds_tok, 0, true, rowp, vocab_offset);
}

// grid = (slice, row of the sequence, sequence): no index arithmetic ahead of the first load.
// At least six wavefronts per SIMD (80 vector registers): the draft pass on bfloat16 sits right at that limit.
template <int DT, bool FULL>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void stream_pass_kernel(RowReduceArgs a)
{
    warm_args(a);
    stream_pass_body<DT, FULL>(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// The draft epilogue's workgroups and, behind them, target rows 0 and 1 of every sequence: up to the stop position those two are read
// whatever it turns out to be, and the epilogue alone leaves the chip idle.
template <int DD, int TD>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void epilogue_stream_kernel(DraftFinalArgs f, RowReduceArgs t, int n_seq)
{
    static_assert(kBlock == kFinalBlock, "the epilogue runs in this kernel's workgroups");
    warm_args(f, t);
    if ((int)blockIdx.x < n_seq) { draft_finalize_few(f, blockIdx.x, DD); return; }
    const int i = (int)blockIdx.x - n_seq, row = i / t.nsplit, b = row / kFirstRows;
    stream_pass_body<TD, false>(t, i - row * t.nsplit, row - b * kFirstRows, b);
}
// The target rows behind them.
template <int TD>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void stream_rest_kernel(RowReduceArgs a)
{
    warm_args(a);
    stream_pass_body<TD, false>(a, blockIdx.x, blockIdx.y + kFirstRows, blockIdx.z);
}

// A workgroup per row of a vocabulary shard: the row's record, with no launch behind this one to merge slices.  WAVES: four, or eight or sixteen
// that share the row's batches (shard_record_waves).
template <int DT, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) __attribute__((amdgpu_waves_per_eu(6))) void stream_record_kernel(RowReduceArgs a, int vocab_offset)
{
    warm_args(a);
    stream_pass_body<DT, true, WAVES>(a, 0, blockIdx.x, blockIdx.y, vocab_offset);
}

// Draft rows and target rows of a round in ONE launch: grid = (slice, row, 2 * sequences), the first half of the
// z range takes the draft tensor, the second half the target tensor (one more row per sequence).  A launch over a
// few hundred rows spends a fifth of its time filling and draining the chip; one launch over both tensors pays
// that once.  The grid has the larger of the two slice counts.
template <int DD, int TD>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void stream_pair_kernel(RowReduceArgs d, RowReduceArgs t, int n_seq)
{
    warm_args(d, t);
    const int z = blockIdx.z;
    if (z < n_seq) {
        if ((int)blockIdx.y < d.KK && (int)blockIdx.x < d.nsplit) stream_pass_body<DD, true>(d, blockIdx.x, blockIdx.y, z);
    } else {
        if ((int)blockIdx.x < t.nsplit) stream_pass_body<TD, false>(t, blockIdx.x, blockIdx.y, z - n_seq);
    }
}

// The draft pass with the slice sums of the draft-token draw (see DrawSums).  As many workgroups as are resident at once, so that the
// 36 KB table of bfloat16 exponentials is copied to LDS once per workgroup.  Every slice is as long as the next, and they are dealt out with
// a fixed stride, which keeps full drafts level.  Draft positions come first in their order: drafts that stop early leave late
// positions empty, and every workgroup has early and late ones.  (Sequences first, a stride that K times the slices of a row divides
// gave each workgroup its own positions.  us per call, V = 128256, 64 sequences of 8 rows, sequences first / this: two of the rows live
// bfloat16 44.4 / 23.2, binary32 34.3 / 29.1, four 45.3 / 32.2, 53.2 / 43.6, 2 to 8 at random 46.7 / 47.2, 62.9 / 66.6, all 52 / 52, 81 / 78;
// V = 32000, 512 sequences of 16 rows, bfloat16 173 / 67, 170 / 117, 170 / 167, 179 / 183.  Random lengths gain little: a workgroup whose
// slices are all live is as slow as in a full draft.  The sequences turned against each other from position to position as well
// 48.0 and 73.0 there, and 0.4 us in a call of one row.)
// FEW: every workgroup takes one slice (of bfloat16 rows: two side by side), and its first batch travels with the table instead of behind it: with
// few rows a slice is hardly more than that.  The batch takes registers: 80, so that three workgroups of bfloat16 rows fit a compute unit; calls of more
// (four are resident then, all with one slice as well) and of several slices to a workgroup keep 64.  us per call, one row a sequence, behind the
// table / with it: bfloat16, V = 32000, 1, 16, 64 sequences 11.2 / 10.9, 12.9 / 12.3, 13.7 / 13.0, V = 128256 12.1 / 11.6, 13.0 / 12.5, 16.2 / 15.7; binary32, which has no
// table, 9.45 / 9.2, 10.2 / 9.9, 11.2 / 11.05 and 11.4 / 11.2, 12.4 / 12.3, 18.2 / 18.0 (0.15 of each by the epilogue's straight path in the second launch).
template <int DT, bool FEW>
__global__ __launch_bounds__(kBlock * DrawShape<DT>::parts) __attribute__((amdgpu_waves_per_eu(DrawShape<DT>::parts * (FEW ? DrawShape<DT>::few_per_cu : DrawShape<DT>::per_cu)))) void stream_draw_kernel(RowReduceArgs a, DrawArgs d)
{
    constexpr bool kTab = DT == TAPOUT_BF16;
    constexpr int VEC = Elem<DT>::vec, U = kStreamU, kParts = DrawShape<DT>::parts;
    __shared__ double shT[256];
    __shared__ __align__(16) double shE[kTab ? kTabDoubles : 2];
    warm_args(a, d);
    const int tid = threadIdx.x & (kBlock - 1), part = __builtin_amdgcn_readfirstlane(threadIdx.x / kBlock);
    const double tv = d.exp_table[tid];
    if constexpr (kTab) copy_to_lds<kTabVecs, kBlock * kParts>(d.exp_table + 256, shE);
    struct Slice { int b, k, s; const char *row; int head, nvec, tail, v0, v1e, nbatch, on; } at;
    const int n_seq = a.n_rows / a.KK;
    {
        const int first = (int)blockIdx.x * kParts + part, row = first / a.nsplit;
        at.s = first - row * a.nsplit;
        at.k = row / n_seq;
        at.b = row - at.k * n_seq;
    }
    DrawSums<DT> draw;
    draw.T = shT; draw.E = shE;
    draw.table = kTab && !(d.vflags & kVerifyNoExpTable);
    // The slice at hand: its place and, once it is known, its row.
    auto take = [&]() {
        at.on = at.k < a.KK;
        at.on = at.on && (!a.len || at.k < a.len[at.b]);
        at.row = (const char *)a.base + ((int64_t)at.b * a.stride_b + (int64_t)(at.on ? at.k : 0) * a.stride_k) * Elem<DT>::size;
        row_geometry<DT>(at.row, a.V, at.head, at.nvec, at.tail);
        at.v0 = min(at.s * a.per, at.nvec);
        at.v1e = min(at.v0 + a.per, at.nvec);
        at.nbatch = (at.v1e - at.v0 + U * kBlock - 1) / (U * kBlock);
    };
    [[maybe_unused]] u32x4 first[U];
    [[maybe_unused]] int n_first = 0;
    if constexpr (FEW) {
        take();
        const u32x4 *vp = (const u32x4 *)(at.row + (int64_t)at.head * Elem<DT>::size);
        if (at.on && at.v0 + U * kBlock <= at.v1e) { load_batch<DT, U, false>(first, vp, at.v0 + tid, at.v1e); n_first = U; }
        else if (at.on) { load_batch<DT, U, true>(first, vp, at.v0 + tid, at.v1e); n_first = wave_vectors<U>(at.v0, at.v1e); }
    }
    if (part == 0) shT[tid] = tv;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // the copy to LDS
    __syncthreads();
    for (int turn = 0; turn < (FEW ? 1 : d.turns); ++turn) {
        if constexpr (!FEW) take();
        const u32x4 *vp = (const u32x4 *)(at.row + (int64_t)at.head * Elem<DT>::size);
        draw.out = d.sums + ((int64_t)(at.b * a.KK + at.k) * a.nsplit + at.s) * ((int64_t)d.nb * U * (kBlock / kWave));
        ThreadState<true> st;
        bool off = kTab && !draw.table;                                      // the slice's sums are computed, behind everything else
        if (at.on && at.s == 0 && tid < at.head) st.fold_single(load_elem<DT>(at.row, tid), tid);
        const bool heads = at.on && at.s == 0 && at.head > 0, tails = at.on && at.s == a.nsplit - 1 && at.tail > 0;
        for (int b0 = 0; at.on && b0 < d.nb; b0 += 16) {                     // sixteen batches, then what is missing of their sums
            const int b1 = min(b0 + 16, d.nb), b1d = min(b1, at.nbatch);
            uint64_t missing = 0;
            int bi = b0;
#pragma unroll 1
            for (; bi < b1d && !off; ++bi) {
                const int i = at.v0 + bi * (U * kBlock) + tid;
                u32x4 w[U];
                int n = U;
                if (FEW && bi == 0) {
                    n = n_first;
#pragma unroll
                    for (int u = 0; u < U; ++u) w[u] = first[u];
                } else if (at.v0 + (bi + 1) * (U * kBlock) <= at.v1e) load_batch<DT, U, false>(w, vp, i, at.v1e);
                else { load_batch<DT, U, true>(w, vp, i, at.v1e); n = wave_vectors<U>(at.v0 + bi * (U * kBlock), at.v1e); }
                double v[U] = {0.0, 0.0, 0.0, 0.0};
                fold_batch<DT, true, U>(st, w, n, i, at.head, [&](int u) { v[u] = draw.vector(w[u]); });
                missing |= (uint64_t)draw.missing(v) << ((bi - b0) * U);
                draw.store(v, bi);
                if constexpr (kTab) off = draw.off_table(st.v1);
            }
            if constexpr (kTab) {
#pragma unroll 1
                for (; bi < b1d; ++bi) {                                     // the statistics alone
                    const int i = at.v0 + bi * (U * kBlock) + tid;
                    u32x4 w[U];
                    load_batch<DT, U, true>(w, vp, i, at.v1e);
                    fold_batch<DT, true, U>(st, w, U, i, at.head);
                }
                if (off) continue;
            }
            for (bi = max(b0, at.nbatch); bi < b1; ++bi) {                   // a slice shorter than the others
                const double v[U] = {0.0, 0.0, 0.0, 0.0};
                draw.store(v, bi);
            }
            // (the elements ahead of the row's vectors and behind them go with its first and its last draw slice)
            if (heads && b0 == 0) missing |= 1u;
            if (tails && b1 == d.nb) missing |= 1ull << ((b1 - b0) * U - 1);
            while (__builtin_expect(missing != 0, 0)) {
                const int at_bit = __builtin_ctzll(missing), bi = b0 + at_bit / U, u = at_bit % U;
                missing &= missing - 1;
                const int i = at.v0 + bi * (U * kBlock) + u * kBlock + tid;
                constexpr uint32_t ni = NegInfVec<DT>::word;
                u32x4 w = u32x4{ni, ni, ni, ni};
                if (i < at.v1e) w = vp[i];
                int32_t j = -1;
                if (heads && bi == 0 && u == 0 && tid < at.head) j = tid;
                if (tails && bi == d.nb - 1 && u == U - 1 && tid < at.tail) j = at.head + at.nvec * VEC + tid;
                draw.again(w, j >= 0 ? draw.computed(load_elem<DT>(at.row, j)) : 0.0, bi, u, tid);
            }
        }
        if (at.on && at.s == a.nsplit - 1 && tid < at.tail) {
            const int32_t j = at.head + at.nvec * VEC + tid;
            st.fold_single(load_elem<DT>(at.row, j), j);
        }
        finish_slice<DT, true, 2 * kParts, kParts>(a, st, at.s, at.b * a.KK + at.k, 0u, false, (turn & 1) * kParts + part, at.on);
        if constexpr (kTab) {
            for (int bi = 0; __builtin_expect(off && at.on, 0) && bi < d.nb; ++bi) {
                u32x4 w[U];
                load_batch<DT, U, true>(w, vp, at.v0 + bi * (U * kBlock) + tid, at.v1e);
                double v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    v[u] = draw.computed(w[u]);
                    asm volatile("" : "+v"(v[u]));
                }
                if (heads && bi == 0 && tid < at.head) v[0] += draw.computed(load_elem<DT>(at.row, tid));
                if (tails && bi == d.nb - 1 && tid < at.tail) v[U - 1] += draw.computed(load_elem<DT>(at.row, at.head + at.nvec * VEC + tid));
                draw.store(v, bi);
            }
        }
        at.s += d.step_s; at.b += d.step_b; at.k += d.step_k;
        if (at.s >= a.nsplit) { at.s -= a.nsplit; ++at.b; }
        if (at.b >= n_seq) { at.b -= n_seq; ++at.k; }
    }
}

template <int DT, bool FULL>
hipError_t launch(const RowReduceArgs &a, hipStream_t st, Timing tm)
{
    dim3 grid((unsigned)a.nsplit, (unsigned)a.KK, (unsigned)(a.n_rows / a.KK)), block(kBlock);
    launch_kernel(stream_pass_kernel<DT, FULL>, grid, block, st, tm, a);
    return hipGetLastError();
}

template <int DT>
hipError_t launch_record(const RowReduceArgs &a, int vocab_offset, hipStream_t st, Timing tm)
{
    const int waves = shard_record_waves(a.n_rows, a.V, Elem<DT>::vec);
    void (*kernel)(RowReduceArgs, int) = waves == 4 ? stream_record_kernel<DT, 4> : (waves == 8 ? stream_record_kernel<DT, 8> : stream_record_kernel<DT, 16>);
    launch_kernel(kernel, dim3((unsigned)a.KK, (unsigned)(a.n_rows / a.KK)), dim3(waves * kWave), st, tm, a, vocab_offset);
    return hipGetLastError();
}

template <int DD, int TD>
hipError_t launch_pair(const RowReduceArgs &d, const RowReduceArgs &t, hipStream_t st, Timing tm)
{
    const int n_seq = t.n_rows / t.KK;
    dim3 grid((unsigned)(d.nsplit > t.nsplit ? d.nsplit : t.nsplit), (unsigned)t.KK, (unsigned)(2 * n_seq)), block(kBlock);
    launch_kernel(stream_pair_kernel<DD, TD>, grid, block, st, tm, d, t, n_seq);
    return hipGetLastError();
}

}  // namespace

// d: the draft tensor ([B, K, V], all statistics), t: the target tensor of the same sequences ([B, K + 1, V]).
hipError_t launch_row_reduce_pair(const RowReduceArgs &d, int d_dtype, const RowReduceArgs &t, int t_dtype, hipStream_t st, Timing tm)
{
    if (d.n_rows / d.KK != t.n_rows / t.KK || d.KK + 1 != t.KK || 2 * (t.n_rows / t.KK) > 65535) return hipErrorInvalidValue;
    if (d_dtype == TAPOUT_F32)
        return t_dtype == TAPOUT_F32 ? launch_pair<TAPOUT_F32, TAPOUT_F32>(d, t, st, tm) : launch_pair<TAPOUT_F32, TAPOUT_BF16>(d, t, st, tm);
    return t_dtype == TAPOUT_F32 ? launch_pair<TAPOUT_BF16, TAPOUT_F32>(d, t, st, tm) : launch_pair<TAPOUT_BF16, TAPOUT_BF16>(d, t, st, tm);
}

template <int DT>
static hipError_t launch_draw(const RowReduceArgs &a, DrawArgs d, hipStream_t st, Timing tm)
{
    // every part of every workgroup the same number of slices, and no more workgroups than are resident
    constexpr int kParts = DrawShape<DT>::parts;
    const int64_t units = (int64_t)a.n_rows * a.nsplit, slots = 256 * DrawShape<DT>::per_cu * kParts;
    d.turns = (int)((units + slots - 1) / slots);
    const int wgs = (int)((units + (int64_t)d.turns * kParts - 1) / ((int64_t)d.turns * kParts)), step = wgs * kParts;
    const int n_seq = a.n_rows / a.KK;
    d.step_s = step % a.nsplit; d.step_b = step / a.nsplit % n_seq; d.step_k = step / a.nsplit / n_seq;
    const bool few = wgs <= 256 * DrawShape<DT>::few_per_cu && d.turns == 1;      // all resident at once (see the kernel)
    launch_kernel(few ? stream_draw_kernel<DT, true> : stream_draw_kernel<DT, false>, dim3(wgs), dim3(kBlock * kParts), st, tm, a, d);
    return hipGetLastError();
}

hipError_t launch_stream_draw(const RowReduceArgs &a, int dtype, DrawArgs d, hipStream_t st, Timing tm)
{
    if (!d.exp_table || !d.sums || a.tok || a.clear_jobs || a.arm_dst || a.len_mode != 0) return hipErrorInvalidValue;
    return dtype == TAPOUT_F32 ? launch_draw<TAPOUT_F32>(a, d, st, tm) : launch_draw<TAPOUT_BF16>(a, d, st, tm);
}

hipError_t launch_row_reduce(const RowReduceArgs &a, int dtype, bool full, hipStream_t st, Timing tm)
{
    if (dtype == TAPOUT_F32) return full ? launch<TAPOUT_F32, true>(a, st, tm) : launch<TAPOUT_F32, false>(a, st, tm);
    return full ? launch<TAPOUT_BF16, true>(a, st, tm) : launch<TAPOUT_BF16, false>(a, st, tm);
}

hipError_t launch_epilogue_stream(const DraftFinalArgs &f, RowReduceArgs t, int t_dtype, hipStream_t st, Timing tm)
{
    const int n_seq = t.n_rows / t.KK;
    if (!epilogue_streams(f.B, f.K, f.nsplit, t.nsplit) || f.shards > 0 || f.B != n_seq || f.K + 1 != t.KK || t.arm_dst) return hipErrorInvalidValue;
    t.len = nullptr; t.len_mode = 0;                          // rows 0 and 1 whatever the stop position
    const dim3 grid((unsigned)(n_seq + n_seq * kFirstRows * t.nsplit)), block(kBlock);
    void (*kernel)(DraftFinalArgs, RowReduceArgs, int);
    if (t_dtype == TAPOUT_F32) kernel = f.dtype == TAPOUT_F32 ? epilogue_stream_kernel<TAPOUT_F32, TAPOUT_F32> : epilogue_stream_kernel<TAPOUT_BF16, TAPOUT_F32>;
    else kernel = f.dtype == TAPOUT_F32 ? epilogue_stream_kernel<TAPOUT_F32, TAPOUT_BF16> : epilogue_stream_kernel<TAPOUT_BF16, TAPOUT_BF16>;
    launch_kernel(kernel, grid, block, st, tm, f, t, n_seq);
    return hipGetLastError();
}
hipError_t launch_stream_rest(RowReduceArgs t, int t_dtype, hipStream_t st, Timing tm)
{
    if (t.KK <= kFirstRows || t.len_mode != 1 || t.arm_dst) return hipErrorInvalidValue;
    t.clear_jobs = nullptr;                                   // (done with row 0)
    const dim3 grid((unsigned)t.nsplit, (unsigned)(t.KK - kFirstRows), (unsigned)(t.n_rows / t.KK)), block(kBlock);
    if (t_dtype == TAPOUT_F32) launch_kernel(stream_rest_kernel<TAPOUT_F32>, grid, block, st, tm, t);
    else launch_kernel(stream_rest_kernel<TAPOUT_BF16>, grid, block, st, tm, t);
    return hipGetLastError();
}

hipError_t launch_shard_records(const RowReduceArgs &a, int vocab_offset, int dtype, hipStream_t st, Timing tm)
{
    if (a.nsplit != 1) return hipErrorInvalidValue;
    return dtype == TAPOUT_F32 ? launch_record<TAPOUT_F32>(a, vocab_offset, st, tm) : launch_record<TAPOUT_BF16>(a, vocab_offset, st, tm);
}

}  // namespace tapout
