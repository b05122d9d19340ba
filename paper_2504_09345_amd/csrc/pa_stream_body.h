// Body of the persistent stream-K decode workgroup, shared by the stream-K
// kernel and the mixed prefill + decode kernel (see pa_stream.hip for the
// design).
#pragma once

#include <type_traits>

#include "pa_counter.h"
#include "pa_device.h"
#include "pa_kernels.h"
#include "pa_tile.h"

namespace pa {

// info word of a unit: valid tokens (5 bits) | item start | item end | head
// block (6 bits) | q/out row (19 bits)
__device__ __forceinline__ int info_valid(int i) { return i & 31; }
__device__ __forceinline__ bool info_start(int i) { return (i >> 5) & 1; }
__device__ __forceinline__ bool info_end(int i) { return (i >> 6) & 1; }
__device__ __forceinline__ int info_hb(int i) { return (i >> 7) & 63; }
__device__ __forceinline__ int info_row(int i) { return (int)((unsigned)i >> 13); }

// Merge n <= 64 partial records of an item, those of ranges xs, xs + step, ...
// (record slot 1 of the item's first range x0, slot 0 of the others), in range
// order, by one wave; lane l takes the records' 16-byte chunks l, l + 64, ...
// (Rec: a chunk's head and dims).  final: normalise and write the output row;
// otherwise write the merged record over the first one's.  Every record is
// stored before its part counts its arrival, and whichever part arrives last
// merges all of them, so the result does not depend on which one it is.
//
// The merge is a chain of memory round trips (1 to 2 us each: the records
// bypass the L2, which is not coherent between XCDs), so the (m, l) of all
// records, record i by lane i, are loaded with the first kBatch records'
// outputs, and the outputs kBatch records at a time.  One sequence of 200 tokens
// (13 parts) takes 12 us per call, of 2,000 tokens 17 us and of 32,000 tokens
// 36 us; with every record waited for in turn, every range between the parts
// looked at with 64-bit divisions, and one merging wave per head for any number
// of parts, they took 147, 615 and 1,274 us.
template <typename T, int D, int S, int W, typename Rec>
__device__ __forceinline__ void merge_records(const StreamArgs& a, int x0, int xs, int step, int n, bool final, int w,
                                              int lane, T* out) {
  constexpr int kChunks = S * D / 4;
  constexpr int C = (kChunks + 63) / 64;  // chunks per lane
  constexpr int kBatch = 8;
  asm volatile("" ::: "memory");  // (the record loads stay below the arrival)
  auto slot = [&](int i) {
    const int x = xs + i * step;
    return ((int64_t)x * 2 + (x == x0 ? 1 : 0)) * W + w;
  };
  f32x4_dev_t v[kBatch][C];
  auto load = [&](int i0) {
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {  // (past the last record: that one again, unused)
      const __amdgpu_buffer_rsrc_t r = record_rsrc(a.ws_o + slot(min(i0 + b, n - 1)) * S * D, S * D);
#pragma unroll
      for (int u = 0; u < C; ++u) v[b][u] = load_dev4(r, (u * 64 + lane) * 4);
    }
  };
  // lane i: record i's maxima and sums, then its weight for each head
  float c[S], l[S], M[S];
  {
    const float* ml = a.ws_ml + slot(min(lane, n - 1)) * S * 2;
#pragma unroll
    for (int j = 0; j < S; ++j) load_dev2(ml + j * 2, c[j], l[j]);
  }
  load(0);
#pragma unroll
  for (int j = 0; j < S; ++j) {
    M[j] = across_groups_max<1>(fmaxf(kMInit, c[j]));
    c[j] = fast_exp2(c[j] - M[j]);
  }
  auto bcast = [](float v, int i) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), i));
  };
  // Value of head h among the S wave-uniform ones.  (Chosen between as values:
  // an array indexed at run time moves to LDS, and addressing it there reads
  // the dispatch packet from host memory, 10 us for the grid's workgroups.)
  auto pick = [&](const float (&v)[S], int h) {
    float x = v[0];
#pragma unroll
    for (int j = 1; j < S; ++j) {
      const float vj = v[j];
      x = h == j ? vj : x;
    }
    return x;
  };
  float L[S];
  f32x4_dev_t acc[C];
#pragma unroll
  for (int j = 0; j < S; ++j) L[j] = 0.0f;
#pragma unroll
  for (int u = 0; u < C; ++u) acc[u] = f32x4_dev_t{0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < n; i0 += kBatch) {
    if (i0 > 0) load(i0);
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      if (i0 + b < n) {  // wave-uniform
        float ci[S];
#pragma unroll
        for (int j = 0; j < S; ++j) {
          ci[j] = bcast(c[j], i0 + b);
          L[j] = fmaf(bcast(l[j], i0 + b), ci[j], L[j]);
        }
#pragma unroll
        for (int u = 0; u < C; ++u) {
          const float ch = pick(ci, Rec::head(u * 64 + lane));
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[u][e] = fmaf(v[b][u][e], ch, acc[u][e]);
        }
      }
    }
  }
  const __amdgpu_buffer_rsrc_t r = record_rsrc(a.ws_o + slot(0) * S * D, S * D);
#pragma unroll
  for (int u = 0; u < C; ++u) {
    const int ch = u * 64 + lane;
    if (final) {
      const float Lh = pick(L, Rec::head(ch));
      if (kChunks % 64 == 0 || ch < kChunks) {
#pragma unroll
        for (int e = 0; e < 4; ++e) store_out<T>(out + Rec::head(ch) * D + Rec::dim(ch) + e, acc[u][e] / Lh);
      }
    } else {
      store_dev4(r, ch * 4, acc[u]);  // (a chunk past the record is out of the descriptor's range)
    }
  }
  if (!final && lane == 0) {
#pragma unroll
    for (int j = 0; j < S; ++j) store_dev(a.ws_ml + slot(0) * S * 2 + j * 2, M[j], L[j]);
  }
}

// The record of an item's other part, loaded ahead of merge_held: (M, L) and
// the unnormalised O of this lane's head column in the matrix-core layout
// (lanes of heads >= S load nothing).
template <int D, int S>
struct HeldRecord {
  float m = 0.0f, l = 0.0f;
  f32x4_dev_t o[D / 16] = {};
};
template <int D, int S>
__device__ __forceinline__ void load_held(HeldRecord<D, S>& r, const float* o, const float* ml, int lane) {
  asm volatile("" ::: "memory");  // (the loads stay below the look at the counter)
  const __amdgpu_buffer_rsrc_t rec = record_rsrc(o, S * D);
  const int n = lane & 15, G = lane >> 4;
  if (n < S) {
    load_dev2(ml + n * 2, r.m, r.l);
#pragma unroll
    for (int mb = 0; mb < D / 16; ++mb) r.o[mb] = load_dev4(rec, mfma::Record<D, S>::chunk(n, mb, G) * 4);
  }
}

// merge_records for an item of two parts whose first part is this wave's
// matrix-core state (its record never stored) and whose second part is the
// record r: the same operations in the same order as merge_records over the two
// records, so the output bits do not depend on which of the two parts merged.
template <typename T, int D, int S>
__device__ __forceinline__ void merge_held(const mfma::State<D, S>& st, const HeldRecord<D, S>& r, int lane, T* out) {
  const float l0 = mfma::total_l(st);  // (every lane: a cross-lane sum)
  const int n = lane & 15, G = lane >> 4;
  if (n < S) {
    const float M = fmaxf(fmaxf(kMInit, st.m), r.m);
    const float c0 = fast_exp2(st.m - M), c1 = fast_exp2(r.m - M);
    const float L = fmaf(r.l, c1, fmaf(l0, c0, 0.0f));
#pragma unroll
    for (int mb = 0; mb < D / 16; ++mb) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        store_out<T>(out + n * D + mb * 16 + 4 * G + i,
                     fmaf(r.o[mb][i], c1, fmaf(st.acc[mb][i], c0, 0.0f)) / L);
    }
  }
}

// Arrival counters of cut items (pa_counter.h), one per range, counted once per
// workgroup.  Device-scope atomics on one line complete about 30 ns apart, so
// they are kept few, one fetch-and-add per part: with every wave counting by
// itself, in a compare-and-swap loop that retries once per other part, 8
// sequences cut into 26 parts each took 60 us.
struct DeviceCounter {
  unsigned long long* p;
  __device__ __forceinline__ uint64_t fetch_add(uint64_t x) {
    return __hip_atomic_fetch_add(p, (unsigned long long)x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ bool swap(uint64_t& expected, uint64_t x) {
    unsigned long long e = expected;
    const bool done = __hip_atomic_compare_exchange_strong(p, &e, (unsigned long long)x, __ATOMIC_RELAXED,
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    expected = e;
    return done;
  }
  __device__ __forceinline__ void store(uint64_t x) {
    __hip_atomic_store(p, (unsigned long long)x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

// An item cut over ranges x0 .. x1 merges its n = x1 - x0 + 1 records at once
// when n <= 16, and otherwise in two levels: the last part of each group of
// ranges leaves the group's record in the place of its first, then counts the
// group, so that no workgroup reads more than a group of records, or one per
// group, alone.  Groups of 8 up to 64 parts, 16 up to 256, then 32: the two
// levels then take about as many batches of records, and a level has at most
// 64 records, one per lane.  The counters: x0's for the item; for a group, that
// of its first range, or x0 + 1 for the first group.  Those ranges lie wholly
// inside the item, so no other item uses their counters (a group of one range
// needs none).
struct CutItem {
  int x0, x1;
  __device__ bool grouped() const { return x1 - x0 >= 16; }
  __device__ int shift() const { return x1 - x0 < 64 ? 3 : x1 - x0 < 256 ? 4 : 5; }
  __device__ int group_first(int x) const { return x0 + ((x - x0) >> shift() << shift()); }
  __device__ bool group_of_one(int x) const { return group_first(x) == x1; }
  // level 0: range x's group; level 1: the item.  Its first record's range,
  // the distance between records, their number, and the counter's range.
  __device__ int first(int level, int x) const { return level == 0 ? group_first(x) : x0; }
  __device__ int step(int level) const { return level == 1 && grouped() ? 1 << shift() : 1; }
  __device__ int parts(int level, int x) const {
    return level == 0 ? min(1 << shift(), x1 - group_first(x) + 1)
                      : grouped() ? ((x1 - x0) >> shift()) + 1 : x1 - x0 + 1;
  }
  __device__ int counter(int level, int x) const { return first(level, x) + (level == 0 && group_first(x) == x0 ? 1 : 0); }
};
static_assert(kStreamMaxGrid <= 32 * 64, "one record per lane at either level");

// First unit of range x, and the range that holds unit e (the largest x with
// U x / G <= e), of G equal ranges over U units.  U <= kStreamMaxUnits *
// kStreamMaxGrid = 2^21 (the host plans the grid for that) and x <= G <= 2^10,
// so the products fit 32 bits.
__device__ __forceinline__ int range_begin(int x, int U, int G) { return (int)((uint32_t)U * (uint32_t)x / (uint32_t)G); }
__device__ __forceinline__ int range_of(int e, int U, int G) {
  return (int)(((uint32_t)(e + 1) * (uint32_t)G - 1u) / (uint32_t)U);
}
static_assert((int64_t)kStreamMaxUnits * kStreamMaxGrid * kStreamMaxGrid <= 0xffffffffll, "32-bit range products");

// Sequence of unit u: the largest r with nb * cum[r] <= u (a non-empty one).
__device__ __forceinline__ int info_row_seq(const int32_t* cum, int R, int nb, int u) {
  int lo = 0, hi = R - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (nb * cum[mid] <= u) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// LDS of one stream-K workgroup of SUB teams of W waves.
template <int W, int SUB, int D, bool MF>
struct StreamSmem {
  static constexpr int kTeamUnits = kStreamMaxUnits / SUB;
  int32_t cum[kStreamMaxRows + 1];  // page prefix sums over rows
  uint8_t tail[kStreamMaxRows];     // valid tokens of each row's last page
  int32_t scan[64 * W * SUB];
  struct Team {
    int32_t page[kTeamUnits];  // unit table of the range: page id
    int32_t info[kTeamUnits];  //   and info word
    CutItem cut[2];            // the items cut by the range's start and by its end (x0 = -1: none)
    int32_t last[2];           // whether this team's part of each completed its counter
    int32_t held;              // whether the last item's other part has counted
  } team[SUB];
  __attribute__((aligned(16))) uint8_t kv[MF ? W * SUB : 1][MF ? 2 * mfma::kTileBytes<D> : 16];  // per-wave tile staging
};

// Codes in s_tail for rows without units (a row with units holds 1 .. 16,
// the tokens in its last page).
constexpr uint8_t kRowZeros = 0x20, kRowNaN = 0x40;

// The stream-K decode workgroup `wg` of a grid of n_wg (see pa_stream.hip): SUB
// teams of W waves (a wave per KV head of a head block), each streaming a range
// of its own in step with the others; range x is team x / n_wg of workgroup
// x mod n_wg, so a small batch spreads over the workgroups first.  Teams only
// share the workgroup's barriers and its prefix sums.
// TR: gather-trace instantiation (records every loaded token's pool row in
// a.trace besides computing the attention).  SPLIT: with the matrix-core
// fold, load K and V half a unit apart (the decode-only kernel); without it,
// through the ring of NBUF whole tiles (the mixed kernel, whose decode
// workgroups share HBM with prefill workgroups and need the longer lead).
template <typename T, int D, int S, int W, int SUB, int NBUF, bool MF, bool TR = false, bool SPLIT = kStreamSplitKV>
__device__ __forceinline__ void stream_body(const StreamArgs& a, StreamSmem<W, SUB, D, MF>& sm, int wg, int n_wg) {
  using Sh = DecodeShape<T, D, S>;
  constexpr int NT = 64 * W * SUB;
  int32_t* s_cum = sm.cum;
  uint8_t* s_tail = sm.tail;
  int32_t* s_scan = sm.scan;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int team = SUB == 1 ? 0 : wave / W;
  const int w = SUB == 1 ? wave : wave % W;  // the wave's KV head in a head block
  const int bid = team * n_wg + wg;          // the team's range
  auto& tm = sm.team[team];
  int32_t* s_page = tm.page;
  int32_t* s_info = tm.info;
  const int R = a.B;  // items are sequences
  // bf16, head_dim 128: what the chunk kernel took before decode-only calls ran
  // without it
  constexpr bool kChunkRows = MF && D == 128 && SPLIT;

  // 1. pages per sequence and their prefix sums (every workgroup, redundantly)
  {
    const int per = (R + NT - 1) / NT;
    const int r0 = min(R, tid * per), r1 = min(R, r0 + per);
    int local = 0;
    bool chunks = false;
    for (int r = r0; r < r1; ++r) {
      int row, nv;
      const int status = seq_decode_row(a.query_start_loc, a.context_lens, a.max_context_len, r, row, nv);
      if constexpr (kChunkRows) chunks |= status == 0 && a.chunk_rows > 0 && a.query_start_loc[r + 1] > row + 1;
      int np = status == 1 ? (nv + kPage - 1) / kPage : 0;
      const bool bad = status < 0 || np > (int)a.bt_stride;  // contract violation: a NaN row (below)
      if (bad) np = 0;
      // tokens in the last page, or for a row without units what its output
      // gets: kRowZeros (empty decode context), kRowNaN (violation), 0 (none)
      s_tail[r] = (uint8_t)(np ? nv - (np - 1) * kPage : bad ? kRowNaN : status == 1 ? kRowZeros : 0);
      s_cum[r] = local;
      local += np;
    }
    const int off = block_exclusive_scan<NT>(local, s_scan);
    for (int r = r0; r < r1; ++r) s_cum[r] += off;
    if (tid == NT - 1) s_cum[R] = off + local;
    if constexpr (kChunkRows) {
      // Chunks that the call's max_q_len does not allow, and for which no chunk
      // kernel was launched: the wave that met one takes this workgroup's share
      // of its rows, one (row, query head) after the other.
      for (uint64_t met = __builtin_amdgcn_ballot_w64(chunks); met != 0; met &= met - 1) {
        const int c0 = __builtin_amdgcn_readlane(r0, __builtin_ctzll(met));
        const int c1 = __builtin_amdgcn_readlane(r1, __builtin_ctzll(met));
        for (int r = c0; r < c1; ++r) {
          const int q0 = a.query_start_loc[r], L = a.query_start_loc[r + 1] - q0, C = a.context_lens[r];
          if (L < 2) continue;
          const bool bad = C > a.max_context_len || L > C || (C + kPage - 1) / kPage > (int)a.bt_stride;
          for (int i = wg; i < L * a.H_q; i += n_wg) {
            const int j = i / a.H_q, h = i - j * a.H_q;
            if (q0 + j < 0 || q0 + j >= a.chunk_rows) continue;
            const int64_t at = ((int64_t)(q0 + j) * a.H_q + h) * D;
            T* o = reinterpret_cast<T*>(a.out) + at;
            if (bad)
              for (int e = lane; e < D; e += 64) store_out<T>(o + e, NAN);
            else
              attend_row<T, D, 1>(reinterpret_cast<const T*>(a.q) + at, reinterpret_cast<const T*>(a.k_pages),
                                  reinterpret_cast<const T*>(a.v_pages), BlockTable{a.block_table, a.bt_stride}, r,
                                  h / S, a.H_kv, C - L + j + 1, a.scale_log2, lane, o,
                                  TR ? a.trace + ((int64_t)(h / S) * R + r) * (a.bt_stride * kPage) : nullptr);
          }
        }
      }
    }
    __syncthreads();
  }
  const int U = a.nb * s_cum[R];
  // A batch of fewer units than workgroups runs on the first U of them, one
  // unit each (no range is ever empty).  Ranges of at least two or three units
  // would save parts to merge but stream alone for longer: within 3 % on most
  // small batches, 35 % slower on 8 sequences of 20 to 60 tokens.  Nor does it
  // pay to use the fewest ranges that keep the longest one's length: 8 to 12
  // sequences -13 to +25 %.
  // Teams beyond the first of each workgroup join once a range has kJoinUnits
  // units (more parts to merge otherwise).  Batches of 4,096 to 8,192 units on one
  // KV head are 1, 3 and 11 % behind the best grid with bounds of 2, 4 and 8 units,
  // larger ones (those that teams are used for unless the declared contexts are
  // far above the real ones) the same with each.
  constexpr int kJoinUnits = 4;
  const int G = max(1, SUB == 1 ? min(n_wg, U) : min(n_wg * SUB, max(min(n_wg, U), U / kJoinUnits)));
  // Rows without units: zeros for an empty decode context, NaN for a contract
  // violation (flagged in s_tail above); rows r = wg (mod n_wg) are this
  // workgroup's to write.
  for (int r = wg; r < R; r += n_wg) {
    if (s_cum[r + 1] != s_cum[r]) continue;  // the row has units
    const int code = s_tail[r];
    if (code != kRowZeros && code != kRowNaN) continue;
    const int qrow = a.query_start_loc != nullptr ? a.query_start_loc[r] : r;
    const float fill = code == kRowNaN ? NAN : 0.0f;
    T* o = reinterpret_cast<T*>(a.out) + (int64_t)qrow * a.H_q * D;
    for (int i = tid; i < a.H_q * D; i += NT) store_out<T>(o + i, fill);
  }
  if (wg >= G || U == 0) return;
  auto units_of = [&](int x) { return x < G ? range_begin(x + 1, U, G) - range_begin(x, U, G) : 0; };
  const int u0 = range_begin(min(bid, G), U, G);
  const int n_units = units_of(bid);
  int n_steps = n_units;  // the longest range of the workgroup's teams
  if constexpr (SUB > 1) {
#pragma unroll
    for (int t = 0; t < SUB; ++t) n_steps = max(n_steps, units_of(t * n_wg + wg));
  }

  // 2. unit table of this range, and the items cut by its start and its end
  const BlockTable bt{a.block_table, a.bt_stride};
  for (int i = w * 64 + lane; i < n_units; i += 64 * W) {
    const int u = u0 + i;
    const int r = info_row_seq(s_cum, R, a.nb, u);
    const int np = s_cum[r + 1] - s_cum[r];
    const int rem = u - a.nb * s_cum[r];
    const int hb = rem / np, p = rem - hb * np;
    const int qrow = a.query_start_loc != nullptr ? a.query_start_loc[r] : r;
    s_page[i] = bt.page(r, p);
    const int valid = p == np - 1 ? (int)s_tail[r] : kPage;
    s_info[i] = valid | (p == 0) << 5 | (p == np - 1) << 6 | hb << 7 | qrow << 13;
    if (i == 0 || i == n_units - 1) {
      const CutItem cut{range_of(u - p, U, G), range_of(u - p + np - 1, U, G)};
      if (i == 0) tm.cut[0] = p == 0 ? CutItem{-1, -1} : cut;
      if (i == n_units - 1) tm.cut[1] = p == np - 1 ? CutItem{-1, -1} : cut;
    }
  }
  __syncthreads();

  // 3. stream the units: wave w handles KV head hb * W + w of every unit
  const int dl = lane % Sh::LPT, row = lane / Sh::LPT;
  const int lane_off = lane * 16;
  const T* kp = reinterpret_cast<const T*>(a.k_pages);
  const T* vp = reinterpret_cast<const T*>(a.v_pages);
  const T* qbase = reinterpret_cast<const T*>(a.q);

  DecodeState<T, D, S> st;
  mfma::State<D, S> ms;  // matrix-core variant (bf16)
  auto& s_kv = sm.kv;
  bool head_partial = false;
  int first_unit = 0;   // of the present item, in this range
  bool redone = false;  // its state was made again (below)

  // Element offset and live tokens of unit k's tile for this wave (a null
  // tile past the range); the trace instantiation records the tile's rows.
  auto unit_tile = [&](int k, int64_t& off, int& valid, bool record) {
    valid = 0;
    off = 0;
    if (k < n_units) {
      const int page = __builtin_amdgcn_readfirstlane(s_page[k]);
      const int info = __builtin_amdgcn_readfirstlane(s_info[k]);
      off = tile_offset(page, info_hb(info) * W + w, a.H_kv, D);
      valid = info_valid(info);
      if constexpr (TR) {
        if (record) {
          // (sequence, head block, page) of the unit, from the unit's index
          const int r = info_row_seq(s_cum, R, a.nb, u0 + k);
          const int np = s_cum[r + 1] - s_cum[r];
          const int rem = u0 + k - a.nb * s_cum[r];
          const int hb = rem / np, p = rem - hb * np;
          if (lane < valid)
            trace_put(a.trace, ((int64_t)(hb * W + w) * R + r) * (a.bt_stride * kPage) + p * kPage + lane,
                      off / D + lane);
        }
      }
    }
  };
  auto issue = [&](u32x4 (&kr)[Sh::NI], u32x4 (&vr)[Sh::NI], int k) {
    int64_t off;
    int valid;
    unit_tile(k, off, valid, true);
    issue_tile<Sh::NI>(tile_rsrc<T, D>(kp + off, valid), tile_rsrc<T, D>(vp + off, valid), lane_off, kr, vr);
  };

  // Items cut by range boundaries.  Every part (the item's first part ends
  // its range; a later part starts one) stores its partial records, one per
  // wave, and then counts its arrival; the workgroup whose part arrives last
  // merges the records in range order and writes the output.  Nothing waits on
  // another workgroup, so the result and the kernel's completion do not depend
  // on how many workgroups are resident or in which order they run.  Records
  // travel through device-coherent stores and loads.
  //
  // A range leaves at most two records per wave: job 0, the item cut by its
  // start, and job 1, that cut by its end (a range inside one item has only
  // job 0).  A job moves one phase at a time, at the barriers that the units
  // have anyway: record stores issued (1), completed in every wave (2), counted
  // by wave 0 (3).  A part that was the last merges when the range has
  // streamed, where no tile is held in registers and a merge can keep many
  // records in flight (4).
  int phase[2] = {0, 0}, level[2] = {1, 1}, job_row[2] = {0, 0}, job_g[2] = {0, 0};
  auto of_job = [](int j, int v0, int v1) { return j == 0 ? v0 : v1; };
  auto job_begin = [&](auto j_, int qrow, int g) {
    constexpr int j = decltype(j_)::value;
    const CutItem cut = tm.cut[j];
    phase[j] = 1;
    level[j] = cut.grouped() && !cut.group_of_one(bid) ? 0 : 1;
    job_row[j] = qrow;
    job_g[j] = g;
  };
  // (wait: the s_waitcnt encoding that leaves only the loads just issued
  // outstanding, as a std::integral_constant: waiting for the record stores
  // then does not drain them, since the vector-memory counter retires in
  // issue order)
  auto jobs_stored = [&](auto wait) {
    if (phase[0] == 1 || phase[1] == 1) {  // wave-uniform
      asm volatile("" ::: "memory");  // (the record stores stay above)
      __builtin_amdgcn_s_waitcnt(decltype(wait)::value);
#pragma unroll
      for (int j = 0; j < 2; ++j) phase[j] = phase[j] == 1 ? 2 : phase[j];
    }
  };
  auto jobs_step = [&]() {  // after a barrier
    if ((phase[0] | phase[1]) < 2) return;
#pragma unroll
    for (int j = 0; j < 2; ++j) phase[j] = phase[j] == 3 ? tm.last[j] ? 4 : 0 : phase[j];
    if (w == 0 && lane < 2) {
      const int ph = of_job(lane, phase[0], phase[1]), lv = of_job(lane, level[0], level[1]);
      if (ph == 2) {
        const CutItem cut = tm.cut[lane];
        DeviceCounter ctr{a.ws_flag + (int64_t)cut.counter(lv, bid) * W};
        tm.last[lane] = counter_arrive(ctr, a.key, cut.parts(lv, bid));
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) phase[j] = phase[j] == 2 ? 3 : phase[j];
  };
  // Range-end merge from registers (the matrix-core split loop sets these):
  // the item ending the range has one other part, which has counted, and
  // its record is in held_rec.
  bool held_now = false;
  HeldRecord<D, S> held_rec;

  // Start of unit k, every wave in step (without the barrier the older wave
  // of each SIMD runs ahead, waves 0..3 finish ~30% before waves 4..7, and
  // those then stream the rest alone with half the loads in flight; in step,
  // the W waves also issue the W adjacent head tiles of a page together).
  // A new (row, head) item loads its queries.  Returns the unit's info word.
  auto begin_unit = [&](int k) {
    __syncthreads();
    jobs_step();
    int info = 0;
    if (k < n_units) {
      info = __builtin_amdgcn_readfirstlane(s_info[k]);
      if (info_start(info) || k == 0) {
        head_partial = !info_start(info);
        first_unit = k;
        redone = false;
        const int g = info_hb(info) * W + w;
        const T* qg = qbase + ((int64_t)info_row(info) * a.H_q + (int64_t)g * S) * D;
        if constexpr (MF) {
          mfma::begin_item<D, S>(ms, reinterpret_cast<const uint16_t*>(qg), lane);
        } else {
          const T* qp = qg + dl * Sh::VEC;
#pragma unroll
          for (int j = 0; j < S; ++j) {
            st.q[j] = *reinterpret_cast<const u32x4*>(qp + j * D);
            st.m[j] = kMInit;
            st.l[j] = 0.0f;
#pragma unroll
            for (int e = 0; e < Sh::VEC; ++e) st.o[j][e] = 0.0f;
          }
        }
      }
    }
    return info;
  };
  // At head_dim 64, the matrix-core state of an item's part that is not finite
  // is made again from the part's units (first_unit .. k) with the VALU fold, as
  // every part was before: V . (p1 + p2 + p3) is NaN for an infinite V whose
  // weight needs fewer parts, and weights up to 2^kRescaleSlack overflow sooner.
  // One head at a time, so that this rare path holds few registers.
  constexpr bool kRedo = MF && D == 64;
  auto not_finite = [&]() {
    float t[4] = {ms.l, ms.l, ms.l, ms.l};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      t[i] *= 0.0f;  // (0, or NaN where a value is infinite or NaN)
#pragma unroll
      for (int mb = 0; mb < D / 16; ++mb) t[i] = fmaf(ms.acc[mb][i], 0.0f, t[i]);
    }
    return __builtin_amdgcn_ballot_w64((t[0] + t[1]) + (t[2] + t[3]) != 0.0f && (lane & 15) < S) != 0;
  };
  auto redo = [&](int k) {
    redone = true;  // (until the next item starts)
    const int info = __builtin_amdgcn_readfirstlane(s_info[k]);
    const T* qg = qbase + ((int64_t)info_row(info) * a.H_q + (int64_t)(info_hb(info) * W + w) * S) * D;
    const int n = lane & 15, Gl = lane >> 4;
#pragma unroll 1
    for (int j = 0; j < S; ++j) {
      using Sh1 = DecodeShape<T, D, 1>;
      DecodeState<T, D, 1> s1;
      s1.q[0] = *reinterpret_cast<const u32x4*>(qg + j * D + dl * Sh1::VEC);
      s1.m[0] = kMInit;
      s1.l[0] = 0.0f;
#pragma unroll
      for (int e = 0; e < Sh1::VEC; ++e) s1.o[0][e] = 0.0f;
#pragma unroll 1
      for (int u = first_unit; u <= k; ++u) {
        int64_t off;
        int valid;
        unit_tile(u, off, valid, false);
        u32x4 kr[Sh1::NI], vr[Sh1::NI];
        issue_tile<Sh1::NI>(tile_rsrc<T, D>(kp + off, valid), tile_rsrc<T, D>(vp + off, valid), lane_off, kr, vr);
        fold_tile<T, D, 1>(s1, kr, vr, row, valid, a.scale_log2);
      }
      float M[1], L[1], O[1][Sh1::VEC];
      merge_rows<T, D, 1>(s1, M, L, O);
      // lane (n = j, Gl) takes dims 16 mb + 4 Gl + i, from the lane of those dims
#pragma unroll
      for (int mb = 0; mb < D / 16; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int from = (16 * mb + 4 * Gl) / Sh1::VEC;
          const float even = __shfl(O[0][i], from), odd = __shfl(O[0][(4 + i) % Sh1::VEC], from);
          if (n == j) ms.acc[mb][i] = Gl & 1 ? odd : even;
        }
      if (n == j) {
        ms.m = M[0];
        ms.l = Gl == 0 ? L[0] : 0.0f;
      }
    }
  };
  // End of unit k (k < n_units): an item that ends here is finished in place
  // when it lies wholly in the range; a part cut by the range stores its
  // record and begins its job.
  auto end_unit = [&](int k, int info) {
    const bool tail_partial = k == n_units - 1 && !info_end(info);
    if (info_end(info) || k == n_units - 1) {
      const int r = info_row(info);
      const int g = info_hb(info) * W + w;
      T* outp = reinterpret_cast<T*>(a.out) + ((int64_t)r * a.H_q + (int64_t)g * S) * D;
      if (!head_partial && !tail_partial) {  // the whole item in this range
        if constexpr (MF)
          mfma::finish<D, S, T>(ms, lane, outp, redone);
        else
          finish_rows<T, D, S>(st, row, dl, outp);
      } else {  // (uniform over the team)
        if constexpr (MF) {
          if (held_now && k == n_units - 1) {
            merge_held<T, D, S>(ms, held_rec, lane, outp);
            if (w == 0 && lane == 0) DeviceCounter{a.ws_flag + (int64_t)bid * W}.store(0);
            return;
          }
        }
        const int64_t slot = ((int64_t)bid * 2 + (head_partial ? 0 : 1)) * W + w;
        if constexpr (MF)
          mfma::partial<D, S>(ms, lane, a.ws_o + slot * S * D, a.ws_ml + slot * S * 2);
        else
          partial_rows<T, D, S>(st, row, dl, lane, a.ws_o + slot * S * D, a.ws_ml + slot * S * 2);
        if (head_partial) job_begin(std::integral_constant<int, 0>{}, r, g);
        else job_begin(std::integral_constant<int, 1>{}, r, g);
      }
    }
  };
  // The jobs left when the range has streamed.
  auto jobs_finish = [&]() {
    // (every team runs every step of a two-level merge: stored and counted,
    // merged and stored, counted, merged)
    for (int step = 0; SUB > 1 ? step < 4 : (phase[0] | phase[1]) != 0; ++step) {
      jobs_stored(std::integral_constant<int, 0>{});
      __syncthreads();
      jobs_step();
#pragma unroll 1
      for (int j = 0; j < 2; ++j) {
        if (of_job(j, phase[0], phase[1]) != 4) continue;
        const int lv = of_job(j, level[0], level[1]);
        const CutItem cut = tm.cut[j];
        T* outp = reinterpret_cast<T*>(a.out) + ((int64_t)of_job(j, job_row[0], job_row[1]) * a.H_q +
                                                 (int64_t)of_job(j, job_g[0], job_g[1]) * S) * D;
        using Rec = std::conditional_t<MF, mfma::Record<D, S>, RowsRecord<D, S>>;
        merge_records<T, D, S, W, Rec>(a, cut.x0, cut.first(lv, bid), cut.step(lv), cut.parts(lv, bid), lv == 1, w,
                                       lane, outp);
        // (a group's record counts in the item next)
        phase[0] = j == 0 ? 1 - lv : phase[0];
        phase[1] = j == 1 ? 1 - lv : phase[1];
        level[0] = j == 0 ? 1 : level[0];
        level[1] = j == 1 ? 1 : level[1];
      }
    }
  };

  if constexpr (MF && SPLIT) {
    // Matrix-core fold: a unit's K and V loads go out half a unit apart.  The
    // K loads of unit k + 1 (after the queries of the item it starts, if it
    // starts one) follow unit k's QK half, and its V loads follow unit k's PV
    // half, before the unit's end (an output, or a record and maybe a merge);
    // each is waited for about a unit after it was issued, so about one K and
    // one V tile (8 KiB) are in flight per wave instead of two whole tiles,
    // and one register set of each suffices.  These loads are issued as
    // inline assembly, which the compiler's wait counting does not see (its
    // own counting, across the merge paths, waited for every load at each
    // unit), and are waited for explicitly: when unit k + 1's QK half starts,
    // its V loads (NI instructions) went out after its K loads and queries,
    // and when unit k's PV half starts, unit k + 1's K loads went out after
    // unit k's V loads, so vmcnt(NI) suffices at both points whatever else
    // (records, merges, outputs) went out in between.
    static_assert(Sh::NI < 16, "vmcnt range");
    const int n_q = lane & 15, g_q = lane >> 4;
    auto load_queries = [&](int info) {
      const int g = info_hb(info) * W + w;
      const T* qg = qbase + ((int64_t)info_row(info) * a.H_q + (int64_t)g * S) * D;
      // lane (n, G): row n of the group (zeros past the S rows), dims
      // 32 s + 8 G .. +8 of Q^T operand s
      asm_issue<D / 32, 64>(scalar_rsrc(qg, S * D * 2), (n_q * D + g_q * 8) * 2, ms.qt);
    };
    auto tile_k = [&](int k, u32x4 (&x)[Sh::NI]) {
      int64_t off;
      int valid;
      unit_tile(k, off, valid, true);
      asm_issue<Sh::NI>(scalar_rsrc(kp + off, valid * D * (int)sizeof(T)), lane_off, x);
    };
    auto tile_v = [&](int k, u32x4 (&x)[Sh::NI]) {
      int64_t off;
      int valid;
      unit_tile(k, off, valid, false);
      asm_issue<Sh::NI>(scalar_rsrc(vp + off, valid * D * (int)sizeof(T)), lane_off, x);
    };
    //
    // The range's last item, when cut by the range's end, usually finishes
    // last: its other part started the next range and counted long before.
    // If that item has two parts (it ends in the next range), wave 0 loads its
    // counter (inline assembly too) in the next-to-last unit's QK half, older
    // than the K loads of the last unit, so the waits above cover it
    // unchanged, and looks at it at that unit's end; if the other part has
    // counted, every wave loads its record when the last unit starts, and the
    // last unit ends by merging from registers (merge_held): no record stored,
    // no arrival counted (every other part has counted, so no part reads the
    // counter again in this call), the record's latency hidden behind the
    // unit's fold.  With a single unit the counter is loaded between its K and
    // V loads and looked at before it starts.
    const bool held = n_units > 0 && tm.cut[1].x0 == bid && tm.cut[1].x1 == bid + 1;
    const uint64_t counted = a.key.step;  // one part counted
    u32x2_t ctr = u32x2_t{0u, 0u};

    // (one block for a team with units, left only past the last wait: no path
    // leads from a load around its wait)
    if (SUB == 1 || n_units > 0) {
      u32x4 kc[Sh::NI], vc[Sh::NI];
      load_queries(__builtin_amdgcn_readfirstlane(s_info[0]));
      tile_k(0, kc);
      if (held && w == 0 && n_units == 1) asm_load_dev(a.ws_flag + (int64_t)bid * W, ctr);
      tile_v(0, vc);
      auto look = [&](auto newer) {  // newer: the tile loads issued after the counter's
        vm_wait<decltype(newer)::value>(ctr);
        if (lane == 0) tm.held = ((uint64_t)ctr.y << 32 | ctr.x) == counted;
      };
      if (held && w == 0 && n_units == 1) look(std::integral_constant<int, Sh::NI>{});
      int k = 0;
      do {
        __syncthreads();  // lockstep, as in begin_unit
        jobs_step();
        const int info = __builtin_amdgcn_readfirstlane(s_info[k]);
        if (info_start(info) || k == 0) {
          head_partial = !info_start(info);
          first_unit = k;
          redone = false;
          mfma::reset<D, S>(ms);
        }
        vm_wait<Sh::NI>(kc);  // K of unit k and the queries (issued before it)
        vm_wait<Sh::NI>(ms.qt);
        if (held && w == 0 && k + 2 == n_units) asm_load_dev(a.ws_flag + (int64_t)bid * W, ctr);
        if (held && k == n_units - 1) {
          held_now = tm.held;
          if (held_now) {
            const int64_t slot = ((int64_t)(bid + 1) * 2 + 0) * W + w;
            load_held<D, S>(held_rec, a.ws_o + slot * S * D, a.ws_ml + slot * S * 2, lane);
          }
        }
        mfma::Weights<mfma::kParts<D>> pt;
        mfma::fold_qk<D, S>(ms, kc, s_kv[wave], lane, info_valid(info), a.scale_log2, pt);
        if (k + 1 < n_units) {  // the queries are free once the QK half is done
          const int next = __builtin_amdgcn_readfirstlane(s_info[k + 1]);
          if (info_start(next)) load_queries(next);
        }
        tile_k(k + 1, kc);
        jobs_stored(std::integral_constant<int, (Sh::NI & 15) | (7 << 4) | (15 << 8)>{});
        vm_wait<Sh::NI>(vc);  // V of unit k
        mfma::fold_pv<D, S>(ms, vc, s_kv[wave], lane, pt);
        tile_v(k + 1, vc);
        if constexpr (kRedo) {
          if ((info_end(info) || k == n_units - 1) && not_finite()) {
            vm_wait<0>(kc);  // (all loads, before their registers may move)
            vm_wait<0>(vc);
            vm_wait<0>(ms.qt);
            vm_wait<0>(ctr);
            redo(k);
          }
        }
        end_unit(k, info);
        if (held && w == 0 && k + 2 == n_units) look(std::integral_constant<int, 2 * Sh::NI>{});
      } while (++k < n_units);
      vm_wait<0>(kc);  // the last (null) tiles' loads, before their registers serve anything else
      vm_wait<0>(vc);
    }
    for (int k = n_units; k < n_steps; ++k) {  // another team has a unit more
      __syncthreads();
      jobs_step();
      jobs_stored(std::integral_constant<int, 0>{});
    }
    jobs_finish();
  } else {
    // A ring of NBUF register tiles: the tile of unit k + NBUF - 1 is issued
    // at the start of unit k.
    constexpr int kRingLoads = 2 * Sh::NI;  // load instructions of one issue()
    constexpr int kWaitRing = (kRingLoads & 15) | (7 << 4) | (15 << 8) | ((kRingLoads >> 4) << 14);
    static_assert(kRingLoads < 64, "vmcnt range");
    u32x4 kr[NBUF][Sh::NI], vr[NBUF][Sh::NI];
#pragma unroll
    for (int u = 0; u + 1 < NBUF; ++u) issue(kr[u], vr[u], u);
    for (int base = 0; base < n_steps; base += NBUF) {
#pragma unroll
      for (int u = 0; u < NBUF; ++u) {
        const int k = base + u;
        const int info = begin_unit(k);
        issue(kr[(u + NBUF - 1) % NBUF], vr[(u + NBUF - 1) % NBUF], k + NBUF - 1);
        jobs_stored(std::integral_constant<int, kWaitRing>{});
        if (k < n_units) {
          if constexpr (MF)
            mfma::fold<D, S>(ms, kr[u], vr[u], s_kv[wave], lane, info_valid(info), a.scale_log2);
          else
            fold_tile<T, D, S>(st, kr[u], vr[u], row, info_valid(info), a.scale_log2);
          if constexpr (kRedo) {
            if ((info_end(info) || k == n_units - 1) && not_finite()) redo(k);
          }
          end_unit(k, info);
        }
      }
    }
    jobs_finish();
  }
}

}  // namespace pa
