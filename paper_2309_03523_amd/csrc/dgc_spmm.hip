// Normalised neighbour aggregation of the GCN convolution (the structure encoder Section 6
// names) over the fused batch, and the stale-cache gather (Section 5.2).
//
//   M[row of (t,i)] = d_i^-1/2 * sum_j d_j^-1/2 * src(t,j)
//   src(t,j) = fresh[t,j] if j lies in the row's chunk vertex range, else the cache row.
// (With generated chunks the stored columns come pre-marked instead: j = fresh, ~j = cache row.)
//
// HBM/L2-bound work: one wavefront owns one work item (a group of consecutive rows, or one
// part of a split row).  The 64 lanes span the feature dimension (1, 2 or 4 floats each), so
// every neighbour row is one fully coalesced load; column indices and their degree scalings
// are fetched 64 at a time, one per lane, and handed out with v_readlane so that the row
// address is wave-uniform.  Eight neighbour rows are in flight per wave.  Rows of 65 to 128
// floats take the two-rows-per-load variant instead (each half of the wave one neighbour, 16
// bytes per lane, sixteen rows in flight).
#include <algorithm>

#include "dgc_internal.h"

namespace dgc {
namespace {

constexpr int kInflight = 8;
constexpr int kInflightPair = 8;   // pairs of rows in flight in the two-rows-per-load variant (4 and 12 measured slower)

template <int VEC> struct Vec;
template <> struct Vec<1> { using T = float; };
template <> struct Vec<2> { using T = float2; };
template <> struct Vec<4> { using T = float4; };

template <int VEC>
__device__ __forceinline__ void vload(float (&v)[VEC], const float* p) {
  if constexpr (VEC == 1) { v[0] = *p; }
  if constexpr (VEC == 2) { const float2 t = *reinterpret_cast<const float2*>(p); v[0] = t.x; v[1] = t.y; }
  if constexpr (VEC == 4) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
}

// Output rows are written once and read later by another kernel: streaming stores, so that
// they do not push the neighbour rows being re-read out of L2.
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
template <int VEC>
__device__ __forceinline__ void vstore(float* p, const float (&v)[VEC]) {
  if constexpr (VEC == 1) { __builtin_nontemporal_store(v[0], p); }
  if constexpr (VEC == 2) { floatx2 t = {v[0], v[1]}; __builtin_nontemporal_store(t, reinterpret_cast<floatx2*>(p)); }
  if constexpr (VEC == 4) {
    floatx4 t = {v[0], v[1], v[2], v[3]};
    __builtin_nontemporal_store(t, reinterpret_cast<floatx4*>(p));
  }
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int lane) {
  const int lo = __builtin_amdgcn_readlane((int)(v & 0xffffffff), lane);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
  return ((int64_t)hi << 32) | (uint32_t)lo;
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Per-work-item constants, all wave-uniform.
struct RowCtx {
  const int32_t* cj;        // colidx of the snapshot
  const int32_t* cl;        // col_local of the segment, indexed by (e - e0)   (STAGED)
  const float* dinv_t;
  const float* fresh_t; int64_t ld_fresh;
  const float* stale_t; int64_t ld_stale;   // IN_PLACE: cache snapshot; STAGED: segment's halo rows
  int64_t v_lo, v_hi, e0;
  bool skip_stale;          // neighbours outside the range contribute nothing (input-gradient pass)
};

// MODE of the neighbour lookup
constexpr int kInPlace = 0;   // by the segment's vertex range, rows read where they are
constexpr int kStaged = 1;    // local slots: fresh rows, then the segment's gathered halo rows
constexpr int kSigned = 2;    // pre-marked columns (j fresh, ~j cache), rows read where they are

// acc += sum over stored non-zeros e in [ea, eb) of dinv[col] * src row, features fi..fi+VEC-1.
template <int VEC, int MODE>
__device__ __forceinline__ void accumulate_edges(const RowCtx& c, int64_t ea, int64_t eb, int lane, int fi,
                                                 bool active, float (&acc)[VEC]) {
  for (int64_t eb0 = ea; eb0 < eb; eb0 += kWave) {
    const int m = (int)((eb - eb0) < kWave ? (eb - eb0) : kWave);
    int j = 0, loc = 0;
    float wj = 0.f;
    if (lane < m) {
      j = __builtin_nontemporal_load(c.cj + eb0 + lane);  // streamed once
      wj = c.dinv_t[(MODE == kSigned && j < 0) ? ~j : j];
      if constexpr (MODE == kStaged) loc = __builtin_nontemporal_load(c.cl + (eb0 - c.e0) + lane);
    }
    for (int k = 0; k < m; k += kInflight) {
      float v[kInflight][VEC];
      float w[kInflight];
#pragma unroll
      for (int u = 0; u < kInflight; ++u) {
        w[u] = 0.f;
#pragma unroll
        for (int q = 0; q < VEC; ++q) v[u][q] = 0.f;
        if (k + u < m) {  // wave-uniform
          const int jj = __builtin_amdgcn_readlane(j, k + u);
          w[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wj), k + u));
          const float* src;
          if constexpr (MODE == kStaged) {
            const int ll = __builtin_amdgcn_readlane(loc, k + u);
            const int64_t nv = c.v_hi - c.v_lo;
            src = ll < nv ? c.fresh_t + (c.v_lo + ll) * c.ld_fresh : c.stale_t + (ll - nv) * c.ld_stale;
          } else {
            const bool in = MODE == kSigned ? jj >= 0 : (jj >= c.v_lo && jj < c.v_hi);   // wave-uniform
            const int64_t col = (MODE == kSigned && !in) ? ~jj : jj;
            src = in ? c.fresh_t + col * c.ld_fresh : c.stale_t + col * c.ld_stale;
            if (!in && c.skip_stale) { w[u] = 0.f; continue; }
          }
          if (active) vload<VEC>(v[u], src + fi);
        }
      }
#pragma unroll
      for (int u = 0; u < kInflight; ++u)
#pragma unroll
        for (int q = 0; q < VEC; ++q) acc[q] = fmaf(w[u], v[u][q], acc[q]);
    }
  }
}

template <int VEC>
__device__ __forceinline__ void store_row(float* out, int fi, int F, int64_t ldm, const float (&acc)[VEC], float scale);

// The same sum for rows of at most 128 floats, two neighbours per load instruction: lanes 0-31 take
// the even non-zeros of the batch and lanes 32-63 the odd ones, four floats per lane, so that one
// 16-byte load per lane fetches two whole rows (twice the bytes per instruction of a 64-lane
// 8-byte load; the aggregation is bound by the rate of load instructions, not by bytes).  Each
// half ends with the sum over its own neighbours; the caller adds the two halves.
template <int MODE>
__device__ __forceinline__ void accumulate_edges_pair(const RowCtx& c, int64_t ea, int64_t eb, int lane, int fi,
                                                      bool active, float (&acc)[4]) {
  const bool odd = lane >= 32;
  for (int64_t eb0 = ea; eb0 < eb; eb0 += kWave) {
    const int m = (int)((eb - eb0) < kWave ? (eb - eb0) : kWave);
    int j = 0, loc = 0;
    float wj = 0.f;
    if (lane < m) {
      j = __builtin_nontemporal_load(c.cj + eb0 + lane);  // streamed once
      wj = c.dinv_t[(MODE == kSigned && j < 0) ? ~j : j];
      if constexpr (MODE == kStaged) loc = __builtin_nontemporal_load(c.cl + (eb0 - c.e0) + lane);
    }
    for (int k = 0; k < m; k += 2 * kInflightPair) {
      float v[kInflightPair][4];
      float w[kInflightPair];
#pragma unroll
      for (int u = 0; u < kInflightPair; ++u) {
        w[u] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[u][q] = 0.f;
        const int e = k + 2 * u;                      // e + 1 <= 63
        if (e < m) {                                  // wave-uniform
          const int j0 = __builtin_amdgcn_readlane(j, e), j1 = __builtin_amdgcn_readlane(j, e + 1);
          const int w0 = __builtin_amdgcn_readlane(__float_as_int(wj), e);
          const int w1 = __builtin_amdgcn_readlane(__float_as_int(wj), e + 1);
          const int jj = odd ? j1 : j0;
          bool take = !odd || e + 1 < m;              // the last non-zero of an odd batch has no partner
          w[u] = take ? __int_as_float(odd ? w1 : w0) : 0.f;
          const float* src;
          if constexpr (MODE == kStaged) {
            const int l0 = __builtin_amdgcn_readlane(loc, e), l1 = __builtin_amdgcn_readlane(loc, e + 1);
            const int ll = odd ? l1 : l0;
            const int64_t nv = c.v_hi - c.v_lo;
            src = ll < nv ? c.fresh_t + (c.v_lo + ll) * c.ld_fresh : c.stale_t + (ll - nv) * c.ld_stale;
          } else {
            const bool in = MODE == kSigned ? jj >= 0 : (jj >= c.v_lo && jj < c.v_hi);
            const int64_t col = (MODE == kSigned && !in) ? ~jj : jj;
            src = in ? c.fresh_t + col * c.ld_fresh : c.stale_t + col * c.ld_stale;
            if (!in && c.skip_stale) { w[u] = 0.f; take = false; }
          }
          if (active && take) vload<4>(v[u], src + fi);
        }
      }
#pragma unroll
      for (int u = 0; u < kInflightPair; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = fmaf(w[u], v[u][q], acc[q]);
    }
  }
}

// One output row from the paired sum: halves added, lanes 0-31 store columns 0-127, lanes 32-63
// zero-fill the pad columns from 128 to the pitch.
template <int MODE>
__device__ __forceinline__ void pair_row(const RowCtx& c, int64_t ea, int64_t eb, int lane, int F, int64_t ldm,
                                         float* out, float scale) {
  const int fi = (lane & 31) * 4;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  accumulate_edges_pair<MODE>(c, ea, eb, lane, fi, fi < F, acc);
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] += __shfl_xor(acc[q], 32);
  if (lane < 32) {
    store_row<4>(out, fi, F, ldm, acc, scale);
  } else if (128 + fi < ldm) {
    const float z[4] = {0.f, 0.f, 0.f, 0.f};
    vstore<4>(out + 128 + fi, z);
  }
}

template <int MODE>
__device__ __forceinline__ RowCtx make_ctx(const SpmmArgs& a, const Segment& sg) {
  constexpr bool STAGED = MODE == kStaged;
  RowCtx c;
  // (the marked columns are stored segment after segment; e counts from the snapshot's start)
  c.cj = MODE == kSigned ? a.col_signed + (sg.nnz_off - sg.e0) : a.g.colidx[sg.t];
  c.cl = STAGED ? a.col_local + sg.nnz_off : nullptr;
  c.dinv_t = a.dinv + (int64_t)sg.t * a.g.N;
  c.fresh_t = a.fresh + (int64_t)sg.t * a.g.N * a.ld_fresh;
  c.ld_fresh = a.ld_fresh;
  if (STAGED) {
    c.stale_t = a.halo + sg.halo_off * a.ld_halo;
    c.ld_stale = a.ld_halo;
  } else {
    c.stale_t = a.stale + (int64_t)sg.t * a.g.N * a.ld_stale;
    c.ld_stale = a.ld_stale;
  }
  c.v_lo = sg.v_lo; c.v_hi = sg.v_hi; c.e0 = sg.e0;
  c.skip_stale = a.skip_stale;
  return c;
}

template <int VEC>
__device__ __forceinline__ void store_row(float* out, int fi, int F, int64_t ldm, const float (&acc)[VEC], float scale) {
  if (fi >= ldm) return;
  float o[VEC];
#pragma unroll
  for (int q = 0; q < VEC; ++q) o[q] = (fi + q < F) ? acc[q] * scale : 0.f;
  vstore<VEC>(out + fi, o);
}

// One wave per group of consecutive rows of a segment.  Rows longer than long_nnz are left to
// the split-row kernels.
template <int VEC, int MODE, bool PAIR>
__global__ __launch_bounds__(256) void k_spmm_short(SpmmArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t item = (int64_t)blockIdx.x * (256 / kWave) + (threadIdx.x / kWave);
  if (item >= a.n_short) return;
  const int seg = uniform(a.work_short[3 * item + 0]);
  const int r0 = uniform(a.work_short[3 * item + 1]);
  const int n = uniform(a.work_short[3 * item + 2]);
  const Segment sg = a.segs[seg];
  const RowCtx c = make_ctx<MODE>(a, sg);
  const int64_t* rp = a.g.rowptr[sg.t] + sg.v_lo + r0;
  const int64_t my_rp = lane <= n ? rp[lane] : 0;
  // optional output permutation: row_map[packed row] = row of M to write, < 0 = row not wanted
  const int64_t my_map = a.row_map ? (lane < n ? a.row_map[sg.row_off + r0 + lane] : -1) : sg.row_off + r0 + lane;
  for (int r = 0; r < n; ++r) {
    const int64_t ea = readlane64(my_rp, r), eb = readlane64(my_rp, r + 1);
    if (eb - ea > a.long_nnz) continue;
    const int64_t orow = readlane64(my_map, r);
    if (orow < 0) continue;
    const float di = c.dinv_t[sg.v_lo + r0 + r];
    float* out = a.M + orow * (a.ld_out ? a.ld_out : a.ldm);
    if constexpr (PAIR) {
      pair_row<MODE>(c, ea, eb, lane, a.F, a.ldm, out, di);
    } else {
      for (int f0 = 0; f0 < a.ldm; f0 += kWave * VEC) {
        const int fi = f0 + lane * VEC;
        float acc[VEC];
#pragma unroll
        for (int q = 0; q < VEC; ++q) acc[q] = 0.f;
        accumulate_edges<VEC, MODE>(c, ea, eb, lane, fi, fi < a.F, acc);
        store_row<VEC>(out, fi, a.F, a.ldm, acc, di);
      }
    }
  }
}

// One wave per part of a split row: unscaled partial sums.
template <int VEC, int MODE, bool PAIR>
__global__ __launch_bounds__(256) void k_spmm_long(SpmmArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t item = (int64_t)blockIdx.x * (256 / kWave) + (threadIdx.x / kWave);
  if (item >= a.n_long) return;
  const int seg = uniform(a.work_long[4 * item + 0]);
  const int row = uniform(a.work_long[4 * item + 1]);
  const int part = uniform(a.work_long[4 * item + 2]);
  const Segment sg = a.segs[seg];
  const RowCtx c = make_ctx<MODE>(a, sg);
  const int64_t* rp = a.g.rowptr[sg.t] + sg.v_lo + row;
  const int64_t ra = rp[0], rb = rp[1];
  const int64_t ea = ra + (int64_t)part * a.part_nnz;
  const int64_t eb = (ea + a.part_nnz < rb) ? ea + a.part_nnz : rb;
  float* out = a.partial + item * a.ldm;
  if constexpr (PAIR) {
    pair_row<MODE>(c, ea, eb, lane, a.F, a.ldm, out, 1.0f);
  } else {
    for (int f0 = 0; f0 < a.ldm; f0 += kWave * VEC) {
      const int fi = f0 + lane * VEC;
      float acc[VEC];
#pragma unroll
      for (int q = 0; q < VEC; ++q) acc[q] = 0.f;
      accumulate_edges<VEC, MODE>(c, ea, eb, lane, fi, fi < a.F, acc);
      store_row<VEC>(out, fi, a.F, a.ldm, acc, 1.0f);
    }
  }
}

// Sum the parts of each split row in part order (fixed order: results are reproducible), in
// double: a hub row's sum runs over tens of thousands of terms, and the merge of its parts is the
// one place where a wider accumulator costs nothing (a few thousand rows per launch).
template <int VEC>
__global__ __launch_bounds__(256) void k_spmm_long_reduce(SpmmArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t item = (int64_t)blockIdx.x * (256 / kWave) + (threadIdx.x / kWave);
  if (item >= a.n_long) return;
  if (uniform(a.work_long[4 * item + 2]) != 0) return;
  const int seg = uniform(a.work_long[4 * item + 0]);
  const int row = uniform(a.work_long[4 * item + 1]);
  const int parts = uniform(a.work_long[4 * item + 3]);
  const Segment sg = a.segs[seg];
  const float di = a.dinv[(int64_t)sg.t * a.g.N + sg.v_lo + row];
  const int64_t orow = a.row_map ? a.row_map[sg.row_off + row] : sg.row_off + row;
  if (orow < 0) return;
  float* out = a.M + orow * (a.ld_out ? a.ld_out : a.ldm);
  for (int f0 = 0; f0 < a.ldm; f0 += kWave * VEC) {
    const int fi = f0 + lane * VEC;
    if (fi >= a.ldm) continue;
    double sum[VEC];
#pragma unroll
    for (int q = 0; q < VEC; ++q) sum[q] = 0.0;
    // parts requested together (past the last: the last one, not added): two of a row that has no more, else eight
    auto add = [&](int p0, auto ahead) {
      constexpr int kAhead = decltype(ahead)::value;
      float v[kAhead][VEC];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) vload<VEC>(v[k], a.partial + (item + min(p0 + k, parts - 1)) * a.ldm + fi);
#pragma unroll
      for (int k = 0; k < kAhead; ++k)
#pragma unroll
        for (int q = 0; q < VEC; ++q) sum[q] += p0 + k < parts ? (double)v[k][q] : 0.0;
    };
    if (parts <= 2) add(0, std::integral_constant<int, 2>());
    else
      for (int p0 = 0; p0 < parts; p0 += 8) add(p0, std::integral_constant<int, 8>());
    float acc[VEC];
#pragma unroll
    for (int q = 0; q < VEC; ++q) acc[q] = (float)(sum[q] * (double)di);
    store_row<VEC>(out, fi, a.F, a.ldm, acc, 1.0f);
  }
}


// ---------------------------------------------------------------------------------------------
// Second generation of the aggregation kernels (IN_PLACE and generated chunks, equal pitches of the
// fresh and the cache tensor).  The first generation above spends some
// thirty vector instructions per gathered row on broadcasting column ids, range tests and 64-bit
// address arithmetic, and is bound by instruction issue, not by memory.  Here the per-non-zero
// work is prepared once, at packing time, in an edge table (SpmmArgs::etab): the marked column and the neighbour's scaling.
//
// What bounds them on large graphs is what passes the L2s: random rows of a table that does not fit them come at 7.2 to 8 TB/s
// whatever a kernel does (100 000 x 32 rows of 128 floats: 64 % of 211 M lines of 128 bytes miss; with the stores 6.5 TB/s pass); on small
// ones the latency of the few gathers that are under way.  Both want many rows at once, of few columns each:
//   A wave takes one slice of 4 LPR columns of up to kAggRows rows, LPR lanes of 16 bytes a row, so G = 64 / LPR rows at a time; where
// one ends, its lanes take the next of the list.  Entries come eight to a load, one a lane and a batch ahead, and go to the LPR lanes by
// swizzles.  Past a row's end a batch loads zeros, so nothing but the row's neighbours gets into its sum.  Rows of more than kAggLong non-zeros, and parts of
// split rows, are shared by the G groups.  A row's sum runs in two chains.
//   One row for the whole width of a wave and, where it is narrower, two or four of at most 16 non-zeros at a time took 2853 us where 64
// columns a wave take 2660 (100 000 x 32 rows of 128 floats), 7151 and 6630 (62 500 x 64 of 256), 694 and 613 (30 001 x 24 of 128), 1200
// and 1129 (40 000 x 32 of 172), 458 and 366 (20 000 x 8 of 300), 65 and 50 (12 345 x 10 of 50), 10.7 and 9.5 (1000 x 8 of 32).  32 columns
// a wave are 2 to 4 % slower from 128 floats on (of a pitch of 704 bytes, where a line of 128 then lies across two, 11 %), 128 columns 2 to 12 %
// (but see wide_slices).
//   A slice of all rows after the other, so that an XCD's L2 holds more of it: 104 M lines pass the L2s instead of 134 M, but the
// launches take 2974 and 9238 us, since a slice of a power-of-two pitch lies in a quarter or an eighth of an L2's channels.  Two batches
// under way: 3.5 % slower.  Items of 8, 16, 24, 32 rows: 2770, 2660, 2657, 2670 and 372, 374, 399, 404 us.
constexpr int kAggLong = 64;

struct AggRow {
  int64_t orow;      // row of M
  int start, end;    // entries, from the item's first
  float scale;
};

__device__ const float4 agg_zero = {0.f, 0.f, 0.f, 0.f};

template <int LPR, int U>
__device__ __forceinline__ int of_lane(int v) {      // lane U of each LPR
  return __builtin_amdgcn_ds_swizzle(v, (U << 5) | (0x20 - LPR));
}

// SKIP: neighbours that are marked stale add nothing.
template <int LPR, bool SKIP>
struct AggGather {
  gbyte *fresh, *stale;      // this lane's 16 bytes of row 0
  uint32_t ld_bytes;
  template <int U>
  __device__ __forceinline__ void one(int2 e, int n, float4& v, float& w) const {
    const int col = of_lane<LPR, U>(e.x), b = of_lane<LPR, U>(e.y);
    gbyte* const base = SKIP || col >= 0 ? fresh : stale;
    gbyte* const at = base + (uint64_t)(uint32_t)(col ^ (col >> 31)) * ld_bytes;
    v = __builtin_bit_cast(float4, load16(U < n && (!SKIP || col >= 0) ? at : in_global(&agg_zero)));
    w = __int_as_float(b);
  }
  // the n (of at most eight) non-zeros whose entries the lanes hold
  __device__ __forceinline__ void batch(int2 e, int n, float4 (&v)[8], float (&w)[8]) const {
    one<0>(e, n, v[0], w[0]); one<1>(e, n, v[1], w[1]); one<2>(e, n, v[2], w[2]); one<3>(e, n, v[3], w[3]);
    one<4>(e, n, v[4], w[4]); one<5>(e, n, v[5], w[5]); one<6>(e, n, v[6], w[6]); one<7>(e, n, v[7], w[7]);
  }
};
__device__ __forceinline__ void agg_add(const float4 (&v)[8], const float (&w)[8], float (&acc)[2][4]) {
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    acc[u & 1][0] = fmaf(w[u], v[u].x, acc[u & 1][0]);
    acc[u & 1][1] = fmaf(w[u], v[u].y, acc[u & 1][1]);
    acc[u & 1][2] = fmaf(w[u], v[u].z, acc[u & 1][2]);
    acc[u & 1][3] = fmaf(w[u], v[u].w, acc[u & 1][3]);
  }
}
// this lane's entry of the eight from pos on (past the row's end its last; kEtabPad spare ones end the table)
__device__ __forceinline__ int2 agg_entry(const int2* tab, int start, int pos, int end) {
  return tab[max(start, min(pos + (int)(threadIdx.x & 7), end - 1))];    // (read again by the other slices: not as a stream, 95 -> 90 us of 10 x 12 345 rows)
}
// this slice's columns of an output row, and zeros up to the pitch behind the last slice
template <int LPR>
__device__ __forceinline__ void agg_store(const SpmmArgs& a, float* out, int fi, int c1, const float (&acc)[4], float scale) {
  if (fi < c1) {
    float o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = fi + q < a.F ? acc[q] * scale : 0.f;
    if (a.keep_out) *reinterpret_cast<float4*>(out + fi) = make_float4(o[0], o[1], o[2], o[3]);
    else vstore<4>(out + fi, o);
  }
  const float z[4] = {0.f, 0.f, 0.f, 0.f};
  for (int c = fi + 4 * LPR; c < c1; c += 4 * LPR) vstore<4>(out + c, z);
}

// The sum over [from, end), a share for every lane group; every group ends with all of it.
template <int LPR, bool SKIP>
__device__ __forceinline__ void agg_shared(const AggGather<LPR, SKIP>& rows, const int2* tab, int from, int end, float (&sum)[4]) {
  constexpr int kBatch = 8 * (64 / LPR);
  const int g8 = from + 8 * ((threadIdx.x & 63) / LPR);
  float acc[2][4] = {};
  int2 e = agg_entry(tab, from, g8, end);
  for (int i = 0; from + i < end; i += kBatch) {
    float4 v[8];
    float w[8];
    const int n = end - (i + g8);
    const int2 now = e;
    e = agg_entry(tab, from, i + kBatch + g8, end);
    rows.batch(now, n, v, w);
    agg_add(v, w, acc);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) sum[q] = acc[0][q] + acc[1][q];
#pragma unroll
  for (int m = LPR; m < 64; m <<= 1)
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[q] += __shfl_xor(sum[q], m);
}

// A wave's slice: columns fi .. +3 of this lane; stored up to column c1.
template <int LPR, bool SKIP>
struct AggSlice {
  int fi, c1, c0;
  __device__ __forceinline__ AggSlice(const SpmmArgs& a, int slice) {
    c0 = 4 * LPR * slice;
    fi = c0 + 4 * ((threadIdx.x & 63) % LPR);
    c1 = c0 + 4 * LPR < a.F ? c0 + 4 * LPR : (int)a.ldm;
  }
  __device__ __forceinline__ AggGather<LPR, SKIP> of(const SpmmArgs& a, int t) const {
    const int64_t col = (int64_t)t * a.g.N * a.ld_fresh + (fi < a.F ? fi : c0);     // lanes past the row's end re-read its first columns (never stored)
    return AggGather<LPR, SKIP>{in_global(a.fresh + col), in_global(a.stale + col), (uint32_t)(a.ld_fresh * sizeof(float))};
  }
};

// A part of a split row, or a row that a workgroup's waves share.
struct TeamRow {
  int64_t e;        // table entry of the first non-zero
  int64_t orow;     // row of M (a part: of the partial sums)
  int nnz, t;
  float scale;
};
constexpr int kTeam = 4;
template <int LPR> constexpr int kShared = 4 * 8 * (64 / LPR);    // four batches of a wave

// The part of a split row that `item` is; false if nobody wants the row (the merge skips it too).
__device__ __forceinline__ bool agg_part(const SpmmArgs& a, int64_t item, TeamRow* to) {
  const int32_t* w = a.work_long + 4 * item;
  const Segment sg = a.segs[uniform(w[0])];
  const int row = uniform(w[1]), p = uniform(w[2]), n_parts = uniform(w[3]);
  if (a.row_map && a.row_map[sg.row_off + row] < 0) return false;
  to->orow = item;
  to->t = sg.t;
  to->scale = 1.0f;
  if (a.eptr) {          // equal shares of what the row has in this table
    const int64_t ra = a.eptr[sg.row_off + row], n = a.eptr[sg.row_off + row + 1] - ra;
    to->e = ra + n * p / n_parts;
    to->nnz = (int)(ra + n * (p + 1) / n_parts - to->e);
  } else {
    const int64_t* rp = a.g.rowptr[sg.t] + sg.v_lo + row;
    const int64_t ea = rp[0] + (int64_t)p * a.part_nnz, eb = rp[1];
    to->e = sg.nnz_off + (ea - sg.e0);
    to->nnz = (int)(min(ea + a.part_nnz, eb) - ea);
  }
  return true;
}

// The rows of an item.  TEAM: those of more than kShared<LPR> non-zeros are left in `queue`.
template <int LPR, bool SKIP, bool TEAM>
__device__ __forceinline__ void agg_rows(const SpmmArgs& a, const AggSlice<LPR, SKIP>& slice, int64_t item, AggRow* list, TeamRow* queue, int* queued) {
  constexpr int G = 64 / LPR;
  const int lane = threadIdx.x & (kWave - 1), g = lane / LPR, l = lane % LPR;
  if (item >= a.n_items) {
    if (TEAM && lane == 0) *queued = 0;
    return;
  }
  const AggItem it = a.items[item];
  const int n = uniform(it.n), t = uniform(it.t), v0 = uniform(it.v0);
  const int64_t* rp = a.g.rowptr[t] + v0;
  const int64_t stored = lane <= n ? rp[lane] : 0;
  const int64_t ptr = lane <= n ? (a.eptr ? a.eptr[it.row + lane] : stored + it.base) : 0;
  const int64_t first = readlane64(ptr, 0);
  const int after = lane + 1 < kWave ? lane + 1 : lane;
  const int start = (int)(ptr - first), end = __shfl(start, after);
  const int64_t full = __shfl((long long)stored, after) - stored;
  const int2* const tab = a.etab + first;
  const AggGather<LPR, SKIP> from = slice.of(a, t);
  const int64_t ldo = a.ld_out ? a.ld_out : a.ldm;
  int64_t orow = -1;
  float scale = 0.f;
  if (lane < n) {
    orow = a.row_map ? a.row_map[it.row + lane] : it.row + lane;
    scale = a.dinv[(int64_t)t * a.g.N + v0 + lane];
  }
  // (rows whose output nobody wants, row_map < 0, and those that the parts make, are not taken)
  const bool wanted = lane < n && orow >= 0 && full <= a.long_nnz;
  const uint64_t below = (1ull << lane) - 1;
  const uint64_t teams = TEAM ? __ballot(wanted && end - start > kShared<LPR>) : 0;
  uint64_t shared = __ballot(wanted && end - start > kAggLong) & ~teams;
  const uint64_t own = __ballot(wanted) & ~shared & ~teams;
  if (own >> lane & 1) list[__popcll(own & below)] = AggRow{orow, start, end, scale};
  if constexpr (TEAM) {
    if (teams >> lane & 1) queue[__popcll(teams & below)] = TeamRow{ptr, orow, end - start, t, scale};
    if (lane == 0) *queued = __popcll(teams);
  }
  const int listed = __popcll(own);
  __builtin_amdgcn_wave_barrier();
  while (shared) {
    const int r = __builtin_ctzll(shared);
    shared &= shared - 1;
    float sum[4];
    agg_shared<LPR, SKIP>(from, tab, __builtin_amdgcn_readlane(start, r), __builtin_amdgcn_readlane(end, r), sum);
    if (g == 0)
      agg_store<LPR>(a, a.M + readlane64(orow, r) * ldo, slice.fi, slice.c1, sum, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(scale), r)));
  }
  if (!listed) return;
  int row = min(g, listed - 1), next = G;
  bool busy = g < listed;
  int pos = list[row].start, from_e = pos, to_e = list[row].end;
  int2 e = agg_entry(tab, from_e, pos, to_e);
  float acc[2][4] = {};
  for (;;) {
    float4 v[8];
    float w[8];
    const int left = busy ? to_e - pos : 0;
    from.batch(e, left, v, w);
    // where the next batch is: further in the row, or in the next row that no group has
    const bool done = busy && left <= 8;
    const uint64_t ends = __ballot(done && l == 0);
    const int mine = row;
    pos += 8;
    if (done) {
      const int r = next + __popcll(ends & ((1ull << (lane & ~(LPR - 1))) - 1));
      busy = r < listed;
      row = min(r, listed - 1);
      pos = from_e = list[row].start;
      to_e = list[row].end;
    }
    next += __popcll(ends);
    e = agg_entry(tab, from_e, pos, to_e);
    agg_add(v, w, acc);
    if (done) {
      const AggRow out = list[mine];
      float sum[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        sum[q] = acc[0][q] + acc[1][q];
        acc[0][q] = acc[1][q] = 0.f;
      }
      agg_store<LPR>(a, a.M + out.orow * ldo, slice.fi, slice.c1, sum, out.scale);
    }
    if (!__ballot(busy)) break;
  }
}

// One launch for parts and rows, the parts first: one of them is the longest work there is, and on a small graph
// a launch of its own waits for one.  A wave a part, a wave an item; ns slices of each.  first: the launch's first block of all.
template <int LPR, bool SKIP>
__global__ __launch_bounds__(256) void k_agg(SpmmArgs a, int ns, int64_t part_blocks, int64_t first) {
  __shared__ AggRow list[kTeam][kAggRows];
  const int wave = uniform(threadIdx.x / kWave);
  const int64_t block = first + blockIdx.x;
  const bool part = block < part_blocks;
  const int64_t place = (block - (part ? 0 : part_blocks)) * kTeam + wave, item = place / ns;
  const AggSlice<LPR, SKIP> slice(a, (int)(place - item * ns));
  if (!part) {
    agg_rows<LPR, SKIP, false>(a, slice, item, list[wave], nullptr, nullptr);
  } else if (item < a.n_long) {
    TeamRow p;
    if (!agg_part(a, item, &p)) return;
    float sum[4];
    agg_shared<LPR, SKIP>(slice.of(a, p.t), a.etab + p.e, 0, p.nnz, sum);
    if ((threadIdx.x & (kWave - 1)) < LPR) agg_store<LPR>(a, a.partial + item * a.ldm, slice.fi, slice.c1, sum, 1.0f);
  }
}

// The same where there are rows long enough to be shared: on a graph that does not fill the chip for long the longest row is
// what the launch waits for (1024 non-zeros are 32 batches of gathers, each waited for), so the four waves of a workgroup share a
// part, and the longer rows of their four items once they have done the shorter ones.  A row's quarters are added in wave order.
template <int LPR, bool SKIP>
__global__ __launch_bounds__(256) void k_agg_team(SpmmArgs a, int ns, int64_t part_blocks) {
  __shared__ AggRow list[kTeam][kAggRows];
  __shared__ TeamRow queue[kTeam][kAggRows];
  __shared__ int queued[kTeam];
  __shared__ float4 sums[2][kTeam][LPR];
  const int lane = threadIdx.x & (kWave - 1), wave = uniform(threadIdx.x / kWave);
  const int g = lane / LPR, l = lane % LPR;
  const bool part = blockIdx.x < part_blocks;
  const int64_t block = blockIdx.x - (part ? 0 : part_blocks), four = block / ns;
  const AggSlice<LPR, SKIP> slice(a, (int)(block - four * ns));
  if (part) {
    TeamRow p;
    const bool there = wave == 0 && agg_part(a, four, &p);
    if (lane == 0) {
      queued[wave] = there;
      if (there) queue[0][0] = p;
    }
  } else {
    agg_rows<LPR, SKIP, true>(a, slice, four * kTeam + wave, list[wave], queue[wave], queued + wave);
  }
  __syncthreads();
  float* const out = part ? a.partial : a.M;
  const int64_t ldo = part || !a.ld_out ? a.ldm : a.ld_out;
  int turn = 0;
  for (int from = 0; from < kTeam; ++from)
    for (int i = 0; i < queued[from]; ++i, ++turn) {
      const TeamRow row = queue[from][i];
      const int nnz = uniform(row.nnz), quarter = (nnz + kTeam - 1) / kTeam, e0 = min(wave * quarter, nnz);
      float part_sum[4];
      agg_shared<LPR, SKIP>(slice.of(a, uniform(row.t)), a.etab + row.e, e0, min(e0 + quarter, nnz), part_sum);
      if (g == 0) sums[turn & 1][wave][l] = make_float4(part_sum[0], part_sum[1], part_sum[2], part_sum[3]);
      __syncthreads();       // (the next row's sums go to the other buffer)
      if (wave == (turn & (kTeam - 1)) && g == 0) {
        const float4 s0 = sums[turn & 1][0][l], s1 = sums[turn & 1][1][l], s2 = sums[turn & 1][2][l], s3 = sums[turn & 1][3][l];
        const float sum[4] = {((s0.x + s1.x) + s2.x) + s3.x, ((s0.y + s1.y) + s2.y) + s3.y, ((s0.z + s1.z) + s2.z) + s3.z,
                              ((s0.w + s1.w) + s2.w) + s3.w};
        agg_store<LPR>(a, out + row.orow * ldo, slice.fi, slice.c1, sum, row.scale);
      }
    }
}

// The team is for launches that the chip holds a few times over at most (it holds some 6000 waves): there the longest row is what they
// wait for (12 345 x 10 rows of 50 floats 59 -> 51 us, 3000 x 16 of 64 40 -> 33); where there is more to do, waves of one item's slices side by side
// are the faster ones (62 500 x 64 rows of 256 6.74 ms, 7.33 with the team; 20 000 x 8 of 300 374 us and 404).  And parts shorter than a
// shared row are a workgroup's only while the chip holds all of them at once.
template <int LPR, bool SKIP>
void launch_agg(SpmmArgs a, hipStream_t st) {
  // Outputs of the size of the L2s are still there when the next kernel reads them; larger ones are streamed past the rows that are
  // read again (8 x 1000 rows of 32 floats: a forward of 19.1 us takes 18.3, 10 x 12 345 of 50 95 and 92; 64 x 62 500 of 256, kept: 22.26 ms
  // becomes 22.48).
  a.keep_out = a.n_items * kAggRows * a.ldm * (int64_t)sizeof(float) <= 64 << 20;
  const int64_t ns = (a.F + 4 * LPR - 1) / (4 * LPR), few = 14 * 1024;
  const bool team = LPR < 32 && a.longest_row > kShared<LPR> && a.n_items * ns <= few && a.n_long * ns <= (a.part_nnz > kShared<LPR> ? few : kTeamsAtOnce);
  const int64_t parts = team ? a.n_long * ns : (a.n_long * ns + kTeam - 1) / kTeam;
  const int64_t rows = team ? (a.n_items + kTeam - 1) / kTeam * ns : (a.n_items * ns + kTeam - 1) / kTeam;
  if constexpr (LPR < 32) if (team) {
    if (parts + rows > 0) hipLaunchKernelGGL((k_agg_team<LPR, SKIP>), (unsigned)(parts + rows), 256, 0, st, a, (int)ns, parts);
    return;
  }
  for (int64_t first = 0; first < parts + rows; first += kMostBlocks)
    hipLaunchKernelGGL((k_agg<LPR, SKIP>), (unsigned)std::min(kMostBlocks, parts + rows - first), 256, 0, st, a, (int)ns, parts, first);
}

// Two slices of 128 columns instead of three or four of 64, the last of which may hold few: on large graphs (from where no team is
// wanted), where a row's own cost counts (few neighbours, a narrow fourth slice) or the table's lines do (many neighbours, a narrow third).
// One wave for all columns -> slices of 64 -> of 128, us.  4 x 400 000 rows of 200 floats, Chung-Lu degrees: 4.5 neighbours a row 1191 -> 1323 ->
// 1178, 14 2393 -> 2524 -> 2361; of 256: 1253 -> 1360 -> 1226; 16 x 30 000 of 200, 5 neighbours: 367 -> 395 -> 361, of 256, 9: 634 -> 545 -> 591;
// 16 x 8000 of 200: 98 -> 89 -> 98.  4 x 400 000 of 132, equal degrees: 33 neighbours 4618 -> 4925 -> 4608, 17 2444 -> 2558 -> 2361; of 176: 33
// 5519 -> 5814 -> 5603; 32 x 40 000 of 160, 17 neighbours: 1462 -> 1316 -> 1351.
bool wide_slices(const SpmmArgs& a) {
  if (a.F <= 128 || a.F > 256 || a.n_rows < 1 << 18 || a.skip_stale) return false;
  const bool hubs = a.longest_row > 1024;
  if (a.F > 224) return hubs && a.nnz < 8 * a.n_rows;
  if (a.F > 192) return a.nnz < (hubs ? 16 : 9) * a.n_rows;
  return a.n_rows >= 1 << 20 && a.nnz >= (a.F <= 160 ? 16 : 24) * a.n_rows;
}

void launch_agg_all(const SpmmArgs& a, hipStream_t st) {
  const bool skip = a.skip_stale && !a.eptr;       // (a table of a row's own chunk has none to leave out)
  if (a.F <= 32) skip ? launch_agg<8, true>(a, st) : launch_agg<8, false>(a, st);
  else if (wide_slices(a)) launch_agg<32, false>(a, st);
  else skip ? launch_agg<16, true>(a, st) : launch_agg<16, false>(a, st);
  const unsigned gl = (unsigned)((a.n_long + 3) / 4);
  if (!gl) return;
  if (a.ldm <= 64) hipLaunchKernelGGL((k_spmm_long_reduce<1>), gl, 256, 0, st, a);
  else if (a.ldm <= 128) hipLaunchKernelGGL((k_spmm_long_reduce<2>), gl, 256, 0, st, a);
  else hipLaunchKernelGGL((k_spmm_long_reduce<4>), gl, 256, 0, st, a);
}

// The first entry of every row in a table of the neighbours of its own chunk alone, counted (FILL: their entries, in order).  A wave an item,
// whose rows' entries lie one behind the other and do so in the other table: lane r counts what lies before row r, and the fill does not
// look at rows at all.  Bound by the reads, of which eight are under way (16 x 3000 vertices, 0.8 M non-zeros, 6 us, 64 x 62 500,
// 68 M, 0.23 ms; a wave a row that waited for each of its reads took 25 us and 1.69 ms).
template <bool FILL>
__global__ __launch_bounds__(256) void k_inside(SpmmArgs a, int64_t* eptr, int2* inside, int64_t first) {
  constexpr int kAhead = 8;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t item = (first + blockIdx.x) * kTeam + uniform(threadIdx.x / kWave);
  // (what a last row without neighbours reads: its weight is multiplied with zero)
  if (FILL && item == 0 && lane == 0) inside[eptr[a.n_rows]] = make_int2(0, 0);
  if (item >= a.n_items) return;
  const AggItem it = a.items[item];
  const int64_t ptr = (a.g.rowptr[it.t] + it.v0)[min(lane, it.n)], begin = readlane64(ptr, 0);
  const int at = (int)(ptr - begin), end = __builtin_amdgcn_readlane(at, kWave - 1);      // (an item has at most kAggRows rows)
  const int2* const tab = a.etab + begin + it.base;
  int64_t out = FILL ? eptr[it.row] : 0;
  int before = 0, mine = 0;
  for (int e = 0; e < end; e += kAhead * kWave) {
    int2 entry[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) entry[u] = tab[min(e + u * kWave + lane, end - 1)];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int p = e + u * kWave;
      const bool is = p + lane < end && entry[u].x >= 0;
      const uint64_t in = __ballot(is);
      if constexpr (FILL) {
        if (is) inside[out + __popcll(in & ((1ull << lane) - 1))] = entry[u];
        out += __popcll(in);
      } else {
        if (at >= p && at < p + kWave) mine = before + __popcll(in & ((1ull << (at - p)) - 1));
        before += __popcll(in);
      }
    }
  }
  if constexpr (!FILL) {
    if (at == end) mine = before;
    const int next = __shfl_down(mine, 1);
    if (lane < it.n) eptr[it.row + lane] = next - mine;
  }
}

// etab[p] = (marked column, scaling of the neighbour) for packed non-zero p
__global__ __launch_bounds__(256) void k_edge_table(GraphDev g, const Segment* segs, int64_t nseg, int64_t total_nnz,
                                                    const float* dinv, const int32_t* col_signed, int2* etab) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= total_nnz + kEtabPad) return;
  if (p >= total_nnz) { etab[p] = make_int2(0, 0); return; }
  int64_t lo = 0, hi = nseg - 1;     // the segment of p: largest s with nnz_off[s] <= p
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) >> 1;
    if (segs[mid].nnz_off <= p) lo = mid; else hi = mid - 1;
  }
  const Segment sg = segs[lo];
  const int32_t j = g.colidx[sg.t][sg.e0 + (p - sg.nnz_off)];
  const int32_t marked = col_signed ? col_signed[p] : ((j >= sg.v_lo && j < sg.v_hi) ? j : ~j);
  const bool valid = j >= 0 && j < g.N;
  const float w = valid ? dinv[(int64_t)sg.t * g.N + j] : 0.f;
  etab[p] = make_int2(valid ? marked : 0, __float_as_int(w));
}

template <int VEC, bool PAIR = false>
void launch_spmm_v(const SpmmArgs& a, hipStream_t st) {
  constexpr int RV = PAIR ? 2 : VEC;   // the merge of split rows walks the pitch 64 x RV floats at a time
  const int mode = a.halo != nullptr ? kStaged : a.col_signed != nullptr ? kSigned : kInPlace;
  const unsigned gs = (unsigned)((a.n_short + 3) / 4), gl = (unsigned)((a.n_long + 3) / 4);
  if (gs) {
    if (mode == kStaged) hipLaunchKernelGGL((k_spmm_short<VEC, kStaged, PAIR>), gs, 256, 0, st, a);
    else if (mode == kSigned) hipLaunchKernelGGL((k_spmm_short<VEC, kSigned, PAIR>), gs, 256, 0, st, a);
    else hipLaunchKernelGGL((k_spmm_short<VEC, kInPlace, PAIR>), gs, 256, 0, st, a);
  }
  if (gl) {
    if (mode == kStaged) hipLaunchKernelGGL((k_spmm_long<VEC, kStaged, PAIR>), gl, 256, 0, st, a);
    else if (mode == kSigned) hipLaunchKernelGGL((k_spmm_long<VEC, kSigned, PAIR>), gl, 256, 0, st, a);
    else hipLaunchKernelGGL((k_spmm_long<VEC, kInPlace, PAIR>), gl, 256, 0, st, a);
    hipLaunchKernelGGL((k_spmm_long_reduce<RV>), gl, 256, 0, st, a);
  }
}

// halo[p] = C[t(p), halo_idx[p], :] for every packed halo slot p.  One thread per float4.
__global__ __launch_bounds__(256) void k_gather(const Segment* segs, int64_t nseg, const int32_t* halo_idx,
                                                const int64_t* halo_ptr, int64_t total_halo, int64_t N,
                                                const float* C, int64_t ldc, int32_t f4, float* halo,
                                                int64_t ldh) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t p = idx / f4;
  if (p >= total_halo) return;
  const int c = (int)(idx - p * f4);
  int64_t lo = 0, hi = nseg - 1;  // largest s with halo_ptr[s] <= p
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) >> 1;
    if (halo_ptr[mid] <= p) lo = mid; else hi = mid - 1;
  }
  const int64_t t = segs[lo].t;
  const float4 v = *reinterpret_cast<const float4*>(C + (t * N + halo_idx[p]) * ldc + 4 * c);
  *reinterpret_cast<float4*>(halo + p * ldh + 4 * c) = v;
}

}  // namespace

void launch_edge_table(const GraphDev& g, const Segment* segs, int64_t nseg, int64_t total_nnz, const float* dinv,
                       const int32_t* col_signed, int2* etab, hipStream_t st) {
  const int64_t n = total_nnz + kEtabPad;
  hipLaunchKernelGGL(k_edge_table, (unsigned)((n + 255) / 256), 256, 0, st, g, segs, nseg, total_nnz, dinv, col_signed, etab);
}


void launch_spmm(const SpmmArgs& a, hipStream_t st) {
  // the edge-table kernels: rows read in place, one pitch for both sources
  if (a.etab && !a.halo && a.ld_fresh == a.ld_stale && a.ld_fresh * 4 < (int64_t(1) << 31)) {
    launch_agg_all(a, st);
    return;
  }
  if (a.F <= 64) launch_spmm_v<1>(a, st);
  else if (a.F <= 128) launch_spmm_v<4, true>(a, st);
  else launch_spmm_v<4>(a, st);
}

void launch_inside(const SpmmArgs& a, int64_t* eptr, int2* inside, hipStream_t st) {
  const int64_t all = (a.n_items + kTeam - 1) / kTeam;
  for (int64_t first = 0; first < all; first += kMostBlocks) {
    const unsigned blocks = (unsigned)std::min(kMostBlocks, all - first);
    if (inside) hipLaunchKernelGGL(k_inside<true>, blocks, 256, 0, st, a, eptr, inside, first);
    else hipLaunchKernelGGL(k_inside<false>, blocks, 256, 0, st, a, eptr, inside, first);
  }
}

void launch_gather(const Segment* segs, int64_t nseg, const int32_t* halo_idx, const int64_t* halo_ptr,
                   int64_t total_halo, int64_t N, const float* C, int64_t ldc, int32_t F, float* halo,
                   int64_t ldh, hipStream_t st) {
  const int32_t f4 = (F + 3) / 4;
  const int64_t n = total_halo * f4;
  if (n > 0)
    hipLaunchKernelGGL(k_gather, (unsigned)((n + 255) / 256), 256, 0, st, segs, nseg, halo_idx, halo_ptr,
                       total_halo, N, C, ldc, f4, halo, ldh);
}

}  // namespace dgc
