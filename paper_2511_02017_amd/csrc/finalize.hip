// Per-sequence epilogue of the draft pass: merges the slice partials of every
// draft row into the signals of Table 1 / Appendix A.1 (entropy, top-1
// probability, top-1/top-2 margin, lse, log q(tok)) and runs the stop scan of
// Algorithm 1's draft loop: the token drafted at the step where the selected
// rule fires is kept, so n_stop = first firing k + 1.
//
// The partials of the draft pass leave out the batch of vectors in which each
// slice met its first maximum (row_reduce.hip): every (row, slice) piece first
// gets the elements of that batch back from the logits, except the first
// maximum itself, which enters the row's sums at the end as an exact double
// term.  That is what keeps the entropy of a peaked row (a small number made
// of small terms) accurate to binary32 relative precision.
//
// One workgroup per sequence.  The kernel is latency bound (O(K * nsplit)
// work), so it is written to keep dependent memory round trips few: the partials
// are requested by all threads at once, the token gather and the left-out batches
// travel together in a second round trip, and every row decides "fires / does not
// fire" for itself.  Few rows and slices: lanes of their own for every (row,
// slice) piece, a row's first lane emits it, and ballots over the rows give the
// stop position.  Long drafts and many pieces: partials staged in LDS, one thread
// per row, a scan over decision bytes.  The two rules that look at more than the
// current row's signals (SVIP-Difference: previous row's entropy; AdaEDL: the
// sequence's adaptive threshold) decide once all entropies of the sequence are
// in LDS.
#include "finalize_device.h"

namespace tapout {

namespace {

// A kernel for each path (and element type): compiled together they kept 124 scalars in vector registers' lanes, to be written and read back
// one by one on the way.
template <bool SHARDED, int DT, bool ONCE>
__global__ __launch_bounds__(kFinalBlock) void draft_finalize_lanes_kernel(DraftFinalArgs a)
{
    __shared__ __align__(16) unsigned char lds[kLanesLds];
    warm_args(a);
    draft_finalize_lanes<SHARDED, ONCE>(a, blockIdx.x, lds, DT, lane_merge_shift(a.K, a.nsplit));
}
template <bool SHARDED>
__global__ __launch_bounds__(kFinalBlock) void draft_finalize_staged_kernel(DraftFinalArgs a)
{
    __shared__ __align__(16) unsigned char lds[kStagedLds];
    warm_args(a);
    draft_finalize_staged<SHARDED>(a, blockIdx.x, lds);
}

// ---- vocabulary shards -----------------------------------------------------------------------
// One record per row of the shard from its slice partials, with the exact global argmax and, if this shard owns it, the logit
// of the drafted token.  Every slice partial gets its left-out batch back (all but the first maximum), then the slices are
// merged; the record leaves the row slice's first maximum out of its two sums.  2^sh lanes per row, one slice each (rows of
// more than sixteen slices: one lane that walks them; sh = 0).
__global__ __launch_bounds__(kFinalBlock) void shard_merge_kernel(ShardMergeArgs a, int sh)
{
    warm_args(a);
    const int64_t t = (int64_t)blockIdx.x * kFinalBlock + threadIdx.x;
    const int row_i = (int)(t >> sh), sl0 = (int)threadIdx.x & ((1 << sh) - 1);
    const bool in = row_i < a.B * a.KK;
    const int i = in ? row_i : 0;
    const int b = i / a.KK, k = i - b * a.KK;
    const void *row = row_address(a.base, a.dtype, a.stride_b, a.stride_k, b, k);
    const int KT = a.KK - a.rows_mode;                       // tokens per sequence (the last target row has none)
    // first round trip: the row count, the token, the partial; second: the token's logit and the partial's left-out batch
    const int n = a.len ? a.len[b] : a.KK;
    int tok = -1;
    if (a.tok && k < KT && sl0 == 0) tok = a.tok[(int64_t)b * KT + k] - a.vocab_offset;
    const int n_live = a.rows_mode == 0 ? min(n, a.KK) : (n < 1 ? 1 : min(n, a.KK - 1)) + 1;
    const bool live = in && k < n_live;
    const int64_t at = (int64_t)i * a.nsplit;
    Piece acc = empty_piece();
    if (live && sl0 < a.nsplit) acc = piece_from_partial(a.part[at + sl0]);
    float xt = NAN;
    if (live && tok >= 0 && tok < a.Vs) xt = load_elem_rt(row, a.dtype, tok);
    BatchRegs bt = batch_issue(row, a.dtype, a.Vs, live && sl0 < a.nsplit ? acc.idx : -1, sl0, a.per, a.part);
    batch_fix(acc, bt, a.dtype);
    if (sh == 0)
        for (int sl = 1; live && sl < a.nsplit; ++sl) {
            Piece e = piece_from_partial(a.part[at + sl]);
            bt = batch_issue(row, a.dtype, a.Vs, e.idx, sl, a.per, a.part);
            batch_fix(e, bt, a.dtype);
            acc = merge_pair<true>(acc, e);
        }
    acc = lane_group_merge<true>(acc, sh);
    if (!live || sl0 != 0) return;
    Partial o;
    o.v1 = acc.M; o.S = (float)acc.S; o.T = (float)acc.T; o.v2 = acc.v2;
    o.cand = a.vocab_offset + ((acc.idx >= 0 && acc.idx < a.Vs) ? acc.idx : 0);
    o.pad[0] = __float_as_int(xt); o.pad[1] = o.pad[2] = 0;
    a.out[i] = o;
}

}  // namespace

hipError_t launch_draft_finalize(const DraftFinalArgs &a, hipStream_t st, Timing tm)
{
    void (*kernel)(DraftFinalArgs);
    auto lanes = [&](auto sharded, auto dtype) -> void (*)(DraftFinalArgs) {
        return lanes_in_one_pass(a.K, a.nsplit) ? draft_finalize_lanes_kernel<decltype(sharded)::value, decltype(dtype)::value, true>
                                                : draft_finalize_lanes_kernel<decltype(sharded)::value, decltype(dtype)::value, false>;
    };
    using F32 = std::integral_constant<int, TAPOUT_F32>; using BF16 = std::integral_constant<int, TAPOUT_BF16>;
    if (!lane_merge_fits(a.K, a.nsplit)) kernel = a.shards > 0 ? draft_finalize_staged_kernel<true> : draft_finalize_staged_kernel<false>;
    else if (a.shards > 0) kernel = lanes(std::true_type{}, F32{});      // (records have no element type)
    else kernel = a.dtype == TAPOUT_F32 ? lanes(std::false_type{}, F32{}) : lanes(std::false_type{}, BF16{});
    launch_kernel(kernel, dim3(a.B), dim3(kFinalBlock), st, tm, a);
    return hipGetLastError();
}

hipError_t launch_shard_merge(const ShardMergeArgs &a, hipStream_t st, Timing tm)
{
    int sh = 0;
    while ((1 << sh) < a.nsplit) ++sh;
    if (sh > 4) sh = 0;
    const int64_t n = ((int64_t)a.B * a.KK) << sh;
    launch_kernel(shard_merge_kernel, dim3((unsigned)((n + kFinalBlock - 1) / kFinalBlock)), dim3(kFinalBlock), st, tm, a, sh);
    return hipGetLastError();
}

}  // namespace tapout
