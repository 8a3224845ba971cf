// Device code of the double-precision exponentials that the final token and the draft-token draw are made of: computed ones
// (exp_fast), those of bfloat16 logits from a table in LDS, and the wavefront sums over them.
#pragma once
#include "common.h"

namespace tapout {

// ---- double-precision helpers ---------------------------------------------------
constexpr double kExpC = 369.3299304675746;            // 256 / ln 2
constexpr double kExpC1 = 0.0027076061740622863;       // ln2/256
constexpr double kExpC2 = kExpC1 * kExpC1 / 2.0;
constexpr double kExpC3 = kExpC1 * kExpC1 * kExpC1 / 6.0;
constexpr double kMagic = 6755399441055744.0;          // 1.5 * 2^52: adding it rounds to an integer held in the low mantissa bits

// exp(x - ref) for x <= ref + small.  neg_ref_c = -ref * 256/ln2; lo = ref - 700 as binary32: inputs
// below it (masked -inf logits, NaN) are treated as ref - 700, i.e. as weight 1e-304.
// c2 is kExpC2 and top is +inf: a caller with many exponentials in a row keeps them in vector registers (an
// instruction takes one scalar constant only, and the compiler would otherwise move c2 into a register before
// every use; with a top it cannot see through, the clamp stays a med3, which unlike fmaxf needs no quieting of
// its input first).
__device__ inline double exp_fast(float x, double neg_ref_c, float lo, const double *T, double c2 = kExpC2, float top = INFINITY)
{
    const double xd = (double)__builtin_amdgcn_fmed3f(x, lo, top);      // max(x, lo) for numbers, lo for NaN
    const double t = fma(xd, kExpC, neg_ref_c);          // (x - ref) * 256/ln2
    const double tm = t + kMagic;
    const int ni = __double2loint(tm);                   // round(t) in two's complement
    const double rs = t - (tm - kMagic);                 // remainder in units of ln2/256, |rs| <= 1/2
    const double q = rs * fma(rs, fma(rs, kExpC3, c2), kExpC1);
    const double tk = T[ni & 255];
    const double e = fma(tk, q, tk);                     // in [1, 2): scale by 2^(ni >> 8) through the exponent field
    int hi;                                              // high word + ((ni >> 8) << 20), as mask and one shift-add
    asm("v_lshl_add_u32 %0, %1, 12, %2" : "=v"(hi) : "v"(ni & (int)0xffffff00), "v"(__double2hiint(e)));
    return __hiloint2double(hi, __double2loint(e));
}

// exp(x) for a double argument, same table and polynomial: relative error < 2e-13, underflowing like exp: to denormal numbers and,
// below log(2^-1075) = -745.13, to 0 (arguments are clamped to [-746, 700], NaN to -746): a token of probability 0 has the
// ratio 0, which a uniform of 0 is not below.  ([-700, ..] made that ratio 1e-304, and u = 0 accepted the token.)
__device__ inline double exp_fast_d(double x, const double *T)
{
    const double t = fmin(fmax(x, -746.0), 700.0) * kExpC;
    const double tm = t + kMagic;
    const int ni = __double2loint(tm);
    const double rs = t - (tm - kMagic);
    const double q = rs * fma(rs, fma(rs, kExpC3, kExpC2), kExpC1);
    const double tk = T[ni & 255];
    return ldexp(fma(tk, q, tk), ni >> 8);
}

struct ExpRef {
    double neg_ref_c; float lo;
    __device__ inline void set(double ref) { neg_ref_c = -ref * kExpC; lo = (float)(ref - 700.0); }
};

// ---- wavefront reductions and scans of doubles with DPP (no LDS round trips) ---------------
// quad_perm [1,0,3,2] = 0xB1, quad_perm [2,3,0,1] = 0x4E, row_half_mirror = 0x141, row_mirror = 0x140,
// row_shr:n = 0x110 + n (lanes without a source inside their 16-lane row read 0).
template <int CTRL>
__device__ inline double dpp_d(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ inline double lane_d(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// Sum over the 64 lanes, same value in every lane, fixed order.
__device__ inline double wave_sum_d(double v)
{
    v += dpp_d<0xB1>(v); v += dpp_d<0x4E>(v); v += dpp_d<0x141>(v); v += dpp_d<0x140>(v);
    return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}
// Inclusive prefix sum over the 64 lanes (lane order); *total = sum of all lanes.
__device__ inline double wave_incl_scan_d(double v, double *total)
{
    v += dpp_d<0x111>(v); v += dpp_d<0x112>(v); v += dpp_d<0x114>(v); v += dpp_d<0x118>(v);   // inside each 16-lane row
    const double t0 = lane_d(v, 15), t1 = lane_d(v, 31), t2 = lane_d(v, 47), t3 = lane_d(v, 63);
    const int rowid = (threadIdx.x & (kWave - 1)) >> 4;
    const double t01 = t0 + t1, t012 = t01 + t2;
    v += rowid == 0 ? 0.0 : (rowid == 1 ? t0 : (rowid == 2 ? t01 : t012));
    *total = t012 + t3;
    return v;
}

// ---- exponentials of bfloat16 logits from a table -----------------------------------------
// A bfloat16 logit has 2^16 possible values, and those between 2^-12 and 2^6 in magnitude (all a softmax row holds
// besides masked entries and the odd tiny one) are 2 * 2302 of them: exp(x) itself, correctly rounded on the host,
// comes from a table of 36 KB in LDS with three integer instructions and one LDS read instead of the thirteen
// instructions of exp_fast.  The row's exponent reference is applied once per slice, to the sums:
//   a_j = exp(t_j - ref_p) = E[t_j] c_t,  b_j = exp(d_j - ref_q) = E[d_j] c_d,   c_t = exp(-ref_p), c_d = exp(-ref_q)
//   a_j - L~ b_j = c_t (E[t_j] - L' E[d_j]),  L' = L~ c_d / c_t
// so the slice kernel sums E[t], E[d], max(0, E[t] - L' E[d]), ... and scales A, R~ by c_t and B, D, U by c_d at the
// end.  A row of another element type keeps exp_fast and c = 1.
// Layout: T[2 idx] for positive values, T[2 idx + 1] for negative ones.  Entry pair idx = 1 .. kTabTop - 1 is the magnitude with
// bfloat16 bits kTabLo15 + idx - 1.
// Pair kTabTop stands for every magnitude from kTabEnd = 63.5 up (and NaN): 0 for either sign.  That is exact for -inf (a
// masked entry) and an error below e^-49 of the row's largest term for any other logit <= -63.5 given the condition
// on the references that tab_job_ok checks (row maxima in [-14, 63)); a job outside it takes the computed
// exponentials, as does a slice of a draft-token draw whose maximum is not in the table's range (see DrawSums).  Pair 0 stands for
// the magnitudes below 2^-12 (and zeros), which are not in the table, and holds NaN: a vector's or chunk's sums show that it met one.
// The draft pass of a draw then forms the sum again, computed; the slice kernel forms the chunk again with tab_exp_any, which
// evaluates 1 + x + x^2/2 + x^3/6 for them (error < 2e-16).
constexpr int kTabTop = 18 * 128 - 1;
constexpr uint32_t kTabLo15 = (uint32_t)(127 - 12) << 7;            // bfloat16 magnitude bits of 2^-12
constexpr int kTabDoubles = 2 * (kTabTop + 1);                       // 4608 doubles = 36,864 bytes
constexpr int kTabVecs = kTabDoubles / 2;                            // 16-byte vectors
static_assert(kTabVecs % kBlock == 0, "the table is copied to LDS in whole rounds of the workgroup");
static_assert(kTabDoubles == kExpBf16Doubles, "the host builds the table");
static_assert(2 * kTabTop + 1 < 65536, "an entry's number fits sixteen bits");

// Two bfloat16 values as they lie in one word -> the byte offsets of their entries.  Both halves are worked on at once with the packed
// 16-bit integer instructions, and the shift to bytes takes the word apart: six instructions for two look-ups (with the signs in
// separate halves of the table, masked off and added back, nine; one value at a time nine each).  us per pass, nine / six: V = 151936, 256
// sequences, K = 16 437.6 / 434.7; V = 128256, 64 sequences 69.7 / 69.2, draft rows with sampled tokens 49.3 / 47.9.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
struct TabOffsets { uint32_t lo, hi; };
__device__ inline TabOffsets tab_offsets2(uint32_t w)
{
    const u16x2 v = __builtin_bit_cast(u16x2, w), sign = v >> (u16x2)(unsigned short)15;
    u16x2 d;                                                                       // 2 magnitude + sign
    asm("v_pk_mad_u16 %0, %1, 2, %2 op_sel_hi:[1,0,1]" : "=v"(d) : "v"(v), "v"(sign));
    d = __builtin_elementwise_sub_sat(d, (u16x2)(unsigned short)(2 * (kTabLo15 - 1)));        // 0, 1: below the table
    d = __builtin_elementwise_min(d, (u16x2)(unsigned short)(2 * kTabTop + 1));
    const uint32_t three = 3;
    TabOffsets o;
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(o.lo) : "s"(three), "v"(d));
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(o.hi) : "s"(three), "v"(d));
    return o;
}
// x: a bfloat16 value widened to binary32 (low 16 bits zero); same entry as tab_offsets2 finds.
__device__ inline double tab_lookup(float x, const double *T)
{
    const uint32_t u = __float_as_uint(x);
    const uint32_t m = (u >> 16) & 0x7fffu;
    const uint32_t d = min(max(m, kTabLo15 - 1) - (kTabLo15 - 1), (uint32_t)kTabTop);
    return T[2 * d + (u >> 31)];
}
// Any binary32-widened bfloat16 value, with the same bits as the table wherever it applies.
__device__ inline double tab_exp_any(float x, const double *T)
{
    const uint32_t u = __float_as_uint(x);
    if (((u >> 16) & 0x7fffu) < kTabLo15) {
        const double t = (double)x;
        return fma(t, fma(t, fma(t, 1.0 / 6.0, 0.5), 1.0), 1.0);
    }
    return tab_lookup(x, T);
}
// One row alone: the sum of its exponentials over a chunk.
__device__ inline double chunk_one_tab(const u32x4 &wt, const double *shE)
{
    const char *E = (const char *)shE;
    double cA = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const TabOffsets ot = tab_offsets2(wt[k]);
        cA += *(const double *)(E + ot.lo);
        cA += *(const double *)(E + ot.hi);
    }
    return cA;
}

// N 16-byte vectors (a multiple of 64) from memory to LDS, without passing through registers, by a workgroup of kThreads.
// The copy is complete when every wavefront has waited for its loads (vmcnt) and a barrier has been passed.
template <int N, int kThreads>
__device__ inline void copy_to_lds(const void *src, void *dst)
{
    typedef const __attribute__((address_space(1))) void *Global;
    typedef __attribute__((address_space(3))) void *Lds;
    constexpr int kWaves = kThreads / kWave, kTurns = N / kWave;
    static_assert(N % kWave == 0, "whole wavefronts");
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int q = 0; q < (kTurns + kWaves - 1) / kWaves; ++q) {
        const int turn = q * kWaves + wave, first = turn * kWave;              // the wavefront's 64 vectors: lane l's goes to first + l
        if ((q + 1) * kWaves <= kTurns || turn < kTurns)
            __builtin_amdgcn_global_load_lds((Global)((const char *)src + (int64_t)(first + lane) * 16), (Lds)((char *)dst + first * 16), 16, 0, 0);
    }
}

}  // namespace tapout
