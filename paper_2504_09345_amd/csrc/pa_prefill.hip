// Causal chunked-prefill rows on MFMA (gfx950), sharing a varlen call with the
// decode rows.
//
// A sequence with context C issuing a chunk of L > 1 query rows has the
// chunk's own K/V already in its pages (the library's reading of the
// paper's GPU prefill, MoE-Lens Sec. 6.4); row j sits at position C - L + j
// and attends to keys 0 .. C - L + j (Sec. 2 GQA groups, Sec. 5.5 paged KV).
// Unlike a decode row, a chunk reuses every K/V page across many query rows,
// so the contraction is dense enough for the matrix cores.
//
// Work item: (sequence, KV head g, block of PB chunk positions).  The block's
// M = PB * s query rows (position-major, the s heads of group g) are split
// over 8 waves of two 16-row MFMA blocks each (256 rows), so every operand
// read from LDS feeds two matrix products (or of one block each, 128 rows, in
// calls too small to fill the CUs: prefill_blocks).  Per step of two 16-key pages:
//   S^T[key][row] = K . Q^T   (v_mfma_f32_16x16x32_bf16 per page, K as the A
//                  operand)
//   online softmax per row (each lane owns one row and 8 of its keys)
//   O^T[dim][row] += V^T . P^T (one v_mfma_f32_16x16x32_f16 over the step's
//                  keys: P rounded to fp16, V staged in LDS as fp16)
// fp16 keeps 11 significant bits against bf16's 8, so P's rounding error is
// 2^-11 relative (bf16 P alone missed the relative tolerance; fp16 P adds a
// tenth of what the bf16 rounding of the output costs), and bf16 V converts
// to fp16 exactly for magnitudes in [2^-17, 2^16).  An item whose V holds a
// value of 2^16 or more (or inf / NaN; in fp16 each makes every row of the
// item non-finite), or whose output rows have an RMS below 2^-14 (where
// fp16's subnormal V could matter), is computed again in a bf16 pass: V as
// loaded, P as its bf16 high and low parts in two v_mfma_f32_16x16x32_bf16
// (fp32-level accuracy).  Both conditions are read off the first pass's
// output rows.
// head_dim 64 takes the bf16 form only, with P in three parts (its chunks ran
// with fp32 weights on the split-K kernel before, and fp16 P or two parts would
// hold fewer bits), four pages per step, so that a step stages the same bytes
// and keeps as many products between barriers; an item with a row that is not
// finite is computed again row by row, so that a V that is infinite or NaN
// reaches only the rows that see its key.  Bound by the matrix products and the
// softmax's vector instructions like head_dim 128: 4 chunks of 200-400 rows on
// 0-1,024 tokens 205 -> 58 us (130 TFLOP/s), 8 of 512 rows on 768 813 -> 86 us
// (399 TFLOP/s), 8 of 2,048 rows on 890 10.7 ms -> 0.59 ms (433 TFLOP/s); with
// P in two parts 49, 74 and 493 us.
// Computing the transposed products keeps "lane l % 16 = query row" in every
// accumulator, so the softmax statistics, the P operand and the O rescale all
// stay in the lane that owns the row: no register transposes.
// The pages' K and V tiles are staged in LDS once per workgroup, two pages
// per synchronised step, and read by all 8 waves, both with 16-byte chunks
// XOR-swizzled by key (conflict-free operand reads); each lane's PV operand
// (4 keys of one dim) is one ds_read_b64_tr_b16 from the [key][dim] V tile.
// The step loop is software-pipelined: the QK products of step t + 1 are
// issued before the softmax and PV of step t, so the matrix cores and the
// VALU work side by side.  Global loads run up to four steps ahead through two
// register sets and a three-step LDS ring, and the item's block-table
// entries are read from an LDS window.
// A persistent grid walks the items in a snake order (item x and 2G-1-x per
// workgroup) so early and late causal blocks pair up.
#include "pa_prefill_body.h"

namespace pa {

template <int D, int S, bool TR, int NB>
__global__ __launch_bounds__(kPfThreads) void prefill_kernel(PrefillArgs a) {
  __shared__ PrefillSmem sm;
  extern __shared__ int32_t s_cum[];  // [B + 1] prefix of items per sequence
  prefill_body<D, S, TR, NB>(a, sm, s_cum, blockIdx.x, gridDim.x);
}

template <int D, bool TR, int NB>
static const void* prefill_pick(int s) {
  switch (s) {
    case 1: return reinterpret_cast<const void*>(&prefill_kernel<D, 1, TR, NB>);
    case 2: return reinterpret_cast<const void*>(&prefill_kernel<D, 2, TR, NB>);
    case 4: return reinterpret_cast<const void*>(&prefill_kernel<D, 4, TR, NB>);
    case 6: return reinterpret_cast<const void*>(&prefill_kernel<D, 6, TR, NB>);
    case 8: return reinterpret_cast<const void*>(&prefill_kernel<D, 8, TR, NB>);
  }
  return nullptr;
}

// trace: the gather-trace instantiation (also records the rows it loads)
template <int NB>
static const void* prefill_fn_blocks(int D, int s, bool trace) {
  if (D == 128) return trace ? prefill_pick<128, true, NB>(s) : prefill_pick<128, false, NB>(s);
  if (D == 64) return trace ? prefill_pick<64, true, NB>(s) : prefill_pick<64, false, NB>(s);
  return nullptr;
}
static const void* prefill_fn(int D, int s, int blocks, bool trace = false) {
  return blocks == 1 ? prefill_fn_blocks<1>(D, s, trace) : prefill_fn_blocks<kPfBlocksMax>(D, s, trace);
}

bool prefill_supported(int dtype, int D, int s) { return dtype == 0 && prefill_fn(D, s, kPfBlocksMax) != nullptr; }

int prefill_occupancy(int D, int s, int blocks, int B) {
  const void* fn = prefill_fn(D, s, blocks);
  if (fn == nullptr) return 0;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, kPfThreads, (size_t)(B + 1) * sizeof(int32_t)) != hipSuccess)
    return 0;
  return n;
}

hipError_t launch_prefill(int D, int s, int blocks, const PrefillArgs& a, int G, hipStream_t st, KernelEvents ev) {
  const void* fn = prefill_fn(D, s, blocks, a.trace != nullptr);
  if (fn == nullptr || G <= 0) return hipErrorInvalidValue;
  void* args[] = {const_cast<PrefillArgs*>(&a)};
  hipError_t e = hipExtLaunchKernel(fn, dim3(G), dim3(kPfThreads), args, (size_t)(a.B + 1) * sizeof(int32_t), st,
                                    ev.start, ev.stop, 0);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace pa
