// Graph-attention structure encoder + causal temporal self-attention time encoder (the
// DySAT-style DGNN of the paper's Sections 2.1 and 6) over a fused batch of chunks, bf16 storage
// with fp32 accumulation: forward pass.  S = F = 128, 8 heads of 16 dims, windows of up to 32
// snapshots.
//
//   z = W x (own rows) / W c (cache rows, Section 5.2);  e_ij^h = LeakyReLU_0.2(a_dst^h.z_i^h + a_src^h.z_j^h)
//   alpha = softmax over the stored row;  u_i = sum_j alpha_ij z_j;  g = ELU(u)
//   p_s = g_s + pos[s];  q, k, v = W_q p, W_k p, W_v p;  y_s^h = sum_{r<=s} softmax_r(q_s^h.k_r^h / 4) v_r^h
#include "dgc_dysat_dev.h"

namespace dgc {
using namespace dysat;
namespace {

// ---------------------------------------------------------------------------------------------
// Weights [n_out = 128][n_in = 128] fp32 -> bf16 operand fragments, 16 bytes per lane.
//  mode 0: fragment (jb, kb) of W as the 32-row operand: lane l holds W[32 jb + l%32][16 kb + 8 (l/32) + 0..7].
//  mode 1: fragment (ib, ks) of W^T, for products whose contraction index is W's row index:
//          lane l holds W[16 ks + 8 (l/32) + 0..7][32 ib + l%32].
//  mode 2: as mode 1, of what W loses when it is rounded to bf16 (the low part).
__global__ void k_pack_w_bf16(const float* W, uint4* packed, int mode) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;   // (blk * 8 + k) * 64 + lane
  if (idx >= 4 * 8 * 64) return;
  const int lane = idx & 63, k = (idx >> 6) & 7, blk = idx >> 9;
  const int r32 = lane & 31, hh = lane >> 5;
  float x[8];
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    if (mode == 0) x[p] = W[(blk * 32 + r32) * kS + k * 16 + 8 * hh + p];
    else x[p] = W[(k * 16 + 8 * hh + p) * kS + blk * 32 + r32];
  }
  if (mode == 2) {
    bf16x8 hi, lo;
    split8(x, hi, lo);
    packed[idx] = __builtin_bit_cast(uint4, lo);
  } else {
    packed[idx] = __builtin_bit_cast(uint4, pack8(x));
  }
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// owner[t*N + v] = chunk that covers (t, v); one block per segment
__global__ void k_owner(const Segment* segs, int64_t N, int32_t* owner) {
  const Segment s = segs[blockIdx.x];
  for (int64_t v = s.v_lo + threadIdx.x; v < s.v_hi; v += blockDim.x) owner[(int64_t)s.t * N + v] = s.chunk;
}

// x of this lane where the lane's row of 16 (half of 32) has the even number, else y, each plus its partner's
__device__ __forceinline__ float add_rows16(float x, float y) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_rows32(float x, float y) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// ---------------------------------------------------------------------------------------------
// Projection z = W x for every vertex of every snapshot in use: zC from the cache rows (any
// vertex can be somebody's out-of-chunk neighbour), zX from the input rows of covered vertices,
// plus the attention scalars s_src[h] = a_src^h . z^h, s_dst[h] = a_dst^h . z^h (from the fp32
// accumulators).  A wave takes 32 vertices at a time; the workgroup keeps W (32 KB) in LDS.  Bound by memory: 4.4 GB in 1.27 ms
// for 4 000 000 vertices (1.70 ms with W from the caches and 8-byte stores).
struct ProjArgs {
  const uint16_t* X; int64_t ldx;
  const uint16_t* C; int64_t ldc;
  const uint4* Wp;
  const float* a_src; const float* a_dst;
  const int32_t* owner; const int32_t* used_t; int32_t n_used; int64_t N;
  uint16_t* zX; uint16_t* zC;   // half precision
  float* sX;   // [T*N][16]: s_src[8], s_dst[8]
  float* sC;   // [T*N][8]:  s_src
};

__global__ __launch_bounds__(512, 4) void k_gat_project(ProjArgs a) {
  __shared__ uint4 w[4 * 8 * 64];
  __shared__ float4 att[2][kS / 4];     // a_src, a_dst
  for (int i = threadIdx.x; i < 4 * 8 * 64; i += 512) w[i] = a.Wp[i];
  if (threadIdx.x < kS / 4) att[0][threadIdx.x] = reinterpret_cast<const float4*>(a.a_src)[threadIdx.x];
  else if (threadIdx.x < kS / 2) att[1][threadIdx.x - kS / 4] = reinterpret_cast<const float4*>(a.a_dst)[threadIdx.x - kS / 4];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 31, hh = lane >> 5;
  const int64_t tiles_per_t = (a.N + 31) / 32, n_tiles = tiles_per_t * a.n_used;
  for (int64_t tile = (int64_t)blockIdx.x * 8 + wave; tile < n_tiles; tile += (int64_t)gridDim.x * 8) {
    const int32_t t = a.used_t[tile / tiles_per_t];
    const int64_t v = (tile % tiles_per_t) * 32 + n;
    const bool valid = v < a.N;
    const int64_t row = (int64_t)t * a.N + (valid ? v : a.N - 1);
    const bool covered = valid && a.owner[row] >= 0;
    const bool any_cov = __ballot(covered) != 0ull;
#pragma unroll 1
    for (int side = 0; side < 2; ++side) {          // 0: cache rows, 1: input rows
      if (side == 1 && !any_cov) break;
      const uint16_t* src = side ? a.X + row * a.ldx : a.C + row * a.ldc;
      const bool wr = side ? covered : valid;
      bf16x8 xf[8];
#pragma unroll
      for (int kb = 0; kb < 8; ++kb) xf[kb] = as_frag(*reinterpret_cast<const uint4*>(src + kb * 16 + 8 * hh));
      uint16_t* z = (side ? a.zX : a.zC) + row * kS;
#pragma unroll 1
      for (int jb = 0; jb < 4; ++jb) {
        floatx16 acc = {};
        float ssrc[2], sdst[2];
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) acc = mfma(as_frag(w[(jb * 8 + kb) * 64 + lane]), xf[kb], acc);
#pragma unroll
        for (int hd = 0; hd < 2; ++hd) {
          const int h = 2 * jb + hd;
          const uint2 z0 = packh4(acc[8 * hd], acc[8 * hd + 1], acc[8 * hd + 2], acc[8 * hd + 3]);
          const uint2 z1 = packh4(acc[8 * hd + 4], acc[8 * hd + 5], acc[8 * hd + 6], acc[8 * hd + 7]);
          const uint4 o = head_order(make_uint4(z0.x, z0.y, z1.x, z1.y));
          if (wr) *reinterpret_cast<uint4*>(z + h * kD + 8 * hh) = o;
          float ps = 0.f, pd = 0.f;
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const float4 as = att[0][h * 4 + 2 * c + hh], ad = att[1][h * 4 + 2 * c + hh];
            const int r = 8 * hd + 4 * c;
            ps += as.x * acc[r] + as.y * acc[r + 1] + as.z * acc[r + 2] + as.w * acc[r + 3];
            pd += ad.x * acc[r] + ad.y * acc[r + 1] + ad.z * acc[r + 2] + ad.w * acc[r + 3];
          }
          ssrc[hd] = add_rows32(ps, ps);
          sdst[hd] = add_rows32(pd, pd);
        }
        if (wr && side == 0 && hh == 0) *reinterpret_cast<float2*>(a.sC + row * 8 + 2 * jb) = make_float2(ssrc[0], ssrc[1]);
        if (wr && side == 1)
          *reinterpret_cast<float2*>(a.sX + row * 16 + 8 * hh + 2 * jb) =
              hh ? make_float2(sdst[0], sdst[1]) : make_float2(ssrc[0], ssrc[1]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Edge softmax + aggregation.  One wavefront per group of rows of one segment.  Lane = 16 * slot + sub: the four
// slots take four neighbours at a time, the 16 sub-lanes of a slot span a neighbour's 128 features (8 per lane, one
// 16-byte load; head = sub / 2), so that a logit's exponential is computed by two lanes and not by eight.  A batch
// is kBatch neighbours per slot, and the next batch is requested before the current one is used; the next row's
// column ids before the current row.  The softmax is accumulated online with one running maximum per head for all
// slots; the slots' sums are added at the row's end.
// Bound by the latency of the gathers where rows are few: 51 us for 12 snapshots of 5001 vertices and about 60 000
// non-zeros (83 us without the team); by their bytes where they are many: 2.9 ms for 16 of 250 000 and 3 million, 5.8 TB/s
// with U.
// Rows longer than long_nnz (hubs of the power-law graphs) are cut into parts of part_nnz non-zeros, one wavefront
// each, in the same launch and begun first; a part leaves its (maximum, sum, weighted sum) in a scratch record and a
// second kernel merges the records of a row in part order.
struct GatArgs {
  GraphDev g;
  const Segment* segs;
  const int32_t* work; int64_t n_work;     // [n][3]: segment, first local row, rows
  const int32_t* work_long; int64_t n_long;   // [n][4]: segment, local row, part, parts
  int32_t long_nnz, part_nnz;
  float* long_partial;                     // [n_long][kLongRec]
  const uint16_t* zX; const uint16_t* zC;
  const float* sX; const float* sC;
  float* U;        // [T*N][128] pre-ELU output (fp32: every later stage is sensitive to it)
  float* lse;      // [T*N][8] log-sum-exp of the logits of every (row, head)
};

struct SoftAcc { float m, l, a0, a1; };
constexpr float kLowest = -3.4028234663852886e38f;

constexpr int kBatch = 4;    // neighbours per slot and batch
struct GatBatch { uint4 z[kBatch]; float e[kBatch]; };

__device__ __forceinline__ float slots_max(float x) {    // over lanes l, l^16, l^32, l^48
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
// first of the two features whose sums a lane holds after gat_row_range
__device__ __forceinline__ int own_feature(int lane) { return 8 * (lane & 15) + 4 * ((lane >> 4) & 1) + 2 * (lane >> 5); }

// online softmax-weighted sum over n stored non-zeros, first, of a row of segment s.  ids: column id of non-zero
// `lane` of them, loaded by the caller.  m and l are those of the lane's head (lane % 16 / 2), a0 and a1 those of
// features own_feature(lane) and the next.
__device__ __forceinline__ SoftAcc gat_row_range(const GatArgs& a, const Segment& s, const int32_t* first, int64_t base,
                                                 float sd, int n, int32_t ids, int lane) {
  const int slot = lane >> 4, sub = lane & 15, head = sub >> 1;
  // The maximum starts at the lowest float, so that neighbours of weight zero (logit -inf) leave zeros where they come first in
  // a part or a quarter, as they do behind others.
  float m = kLowest, l = 0.f, acc[8];
#pragma unroll
  for (int d = 0; d < 8; ++d) acc[d] = 0.f;
  int32_t ahead = 64 + lane < n ? first[64 + lane] : 0;
  auto request = [&](int k, GatBatch& b) {
    if (k > 0 && (k & 63) == 0) {
      ids = ahead;
      ahead = k + 64 + lane < n ? first[k + 64 + lane] : 0;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = k + 4 * u + slot;
      const int32_t j = __shfl(ids, i & 63);
      b.z[u] = make_uint4(0, 0, 0, 0);
      b.e[u] = -INFINITY;
      if (i < n) {
        const bool in = j >= s.v_lo && j < s.v_hi;
        b.z[u] = *reinterpret_cast<const uint4*>((in ? a.zX : a.zC) + (base + j) * kS + 8 * sub);
        b.e[u] = *(in ? a.sX + (base + j) * 16 + head : a.sC + (base + j) * 8 + head);
      }
    }
  };
  auto use = [&](const GatBatch& b) {
    float e[kBatch], bm = -INFINITY;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      e[u] = lrelu(sd + b.e[u]);       // -inf stays -inf (no neighbour)
      bm = fmaxf(bm, e[u]);
    }
    const float mn = fmaxf(m, slots_max(bm));
    const float sc = __expf(m - mn);
    m = mn;
    l *= sc;
#pragma unroll
    for (int d = 0; d < 8; ++d) acc[d] *= sc;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float p = __expf(e[u] - mn);
      float z[8];
      unpackh8(b.z[u], z);
      l += p;
#pragma unroll
      for (int d = 0; d < 8; ++d) acc[d] += p * z[d];
    }
  };
  GatBatch x, y;
  if (n > 0) {
    request(0, x);
    for (int k = 0;; k += 8 * kBatch) {
      const bool more = k + 4 * kBatch < n;
      if (more) request(k + 4 * kBatch, y);
      use(x);
      if (!more) break;
      const bool again = k + 8 * kBatch < n;
      if (again) request(k + 8 * kBatch, x);
      use(y);
      if (!again) break;
    }
  }
  float h[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) h[d] = add_rows16(acc[d], acc[4 + d]);
  const float l2 = add_rows16(l, l);
  return {m, add_rows32(l2, l2), add_rows32(h[0], h[2]), add_rows32(h[1], h[3])};
}

// stored: the row has neighbours; then a sum of zero means that no logit is above -inf, and the softmax is NaN
__device__ __forceinline__ void gat_row_store(const GatArgs& a, int64_t row, const SoftAcc& r, int feature, bool lse_lane, int head,
                                              bool stored = true) {
  const float l = stored && r.l == 0.f ? NAN : r.l;
  const float inv = l > 0.f ? 1.f / l : l;
  *reinterpret_cast<float2*>(a.U + row * kS + feature) = make_float2(r.a0 * inv, r.a1 * inv);
  if (lse_lane) a.lse[row * 8 + head] = r.m + __logf(l);
}

// TEAM: rows of more than kShared non-zeros are left in `queue` for the four waves of the workgroup.
constexpr int kTeam = 4, kShared = 8 * 4 * kBatch;     // eight batches of a wave (four: the same on small graphs, 0.5 % more on large ones)
struct TeamRow { int64_t e0; int32_t seg, i, n; };     // first non-zero, segment, vertex, non-zeros


// Rows of at most kSlotRow non-zeros: one to each of a wave's four slots of 16 lanes, eight neighbours at a time; where one ends, its
// slot takes the next of the item's.  What a row costs beside its neighbours is paid once for four, and nothing is summed across
// slots: the kernel was bound by the vector units (323 instructions of a wave a row, where a wave took one row after the other).
// 16 x 250 000 vertices 2826 -> 2212 us, 12 x 5001 51.6 -> 47.  (16, 24, 48, 64 non-zeros a slot: 98.8, 99.4, 101.9, 105 us of the whole
// forward of the smaller, the same of the larger within 0.3 %; four waves a SIMD: 2313 us.)
constexpr int kSlotRow = 24, kSlots = 4;
struct SlotRow { int start, end, r; };        // non-zeros from the item's first; row of the item
__device__ const uint4 kNoRow = {0, 0, 0, 0};      // what a slot loads past its row's end

template <int U>
__device__ __forceinline__ int of_slot(int v) {      // lane U of each 16
  return __builtin_amdgcn_ds_swizzle(v, (U << 5) | 0x10);
}

struct SlotBatch { uint4 z[8]; float s[8]; };
struct SlotRows {
  gbyte *zx, *zc, *sx, *sc;       // vertex 0 of the snapshot: this lane's 16 bytes of a projection, its head's scalar
  uint32_t lo, span;
  template <int U>
  __device__ __forceinline__ void one(int32_t ids, int n, SlotBatch& b) const {
    const uint32_t j = (uint32_t)of_slot<U>(ids);
    const bool in = j - lo < span;
    gbyte* const z = (in ? zx : zc) + (uint64_t)j * (kS * 2);
    b.z[U] = __builtin_bit_cast(uint4, load16(U < n ? z : in_global(&kNoRow)));
    b.s[U] = *(const __attribute__((address_space(1))) float*)((in ? sx : sc) + (uint64_t)j * (in ? 64u : 32u));
  }
  __device__ __forceinline__ void batch(int32_t ids, int n, SlotBatch& b) const {
    one<0>(ids, n, b); one<1>(ids, n, b); one<2>(ids, n, b); one<3>(ids, n, b);
    one<4>(ids, n, b); one<5>(ids, n, b); one<6>(ids, n, b); one<7>(ids, n, b);
  }
};

__device__ __forceinline__ void gat_slots(const GatArgs& a, const Segment& s, const int32_t* col, int64_t base, int64_t i0, const SlotRow* list,
                                          int listed, int lane) {
  const int slot = lane >> 4, sub = lane & 15, head = sub >> 1;
  const SlotRows from{in_global(a.zX + base * kS + 8 * sub), in_global(a.zC + base * kS + 8 * sub), in_global(a.sX + base * 16 + head),
                      in_global(a.sC + base * 8 + head), (uint32_t)s.v_lo, (uint32_t)(s.v_hi - s.v_lo)};
  const float* const sd_of = a.sX + (base + i0) * 16 + 8 + head;
  auto ids_at = [&](int pos, int end) { return end > pos ? col[min(pos + (sub & 7), end - 1)] : 0; };
  int k = min(slot, listed - 1), next = kSlots;
  bool busy = slot < listed;
  SlotRow row = list[k];
  int pos = row.start;
  int32_t ids = ids_at(pos, row.end);
  float sd = sd_of[row.r * 16], m = kLowest, l = 0.f, acc[8] = {};
  for (;;) {
    SlotBatch b;
    const int left = busy ? row.end - pos : 0;
    from.batch(ids, left, b);
    const bool done = busy && left <= 8;
    const uint64_t ends = __ballot(done && sub == 0);
    const int r = row.r;
    const bool stored = row.end > row.start;
    const float sd_now = sd;
    pos += 8;
    if (done) {
      k = next + __popcll(ends & ((1ull << (lane & ~15)) - 1));
      busy = k < listed;
      row = list[min(k, listed - 1)];
      pos = row.start;
      sd = sd_of[row.r * 16];
    }
    next += __popcll(ends);
    ids = ids_at(pos, row.end);
    float e[8], mn = m;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      e[u] = u < left ? lrelu(sd_now + b.s[u]) : -INFINITY;
      mn = fmaxf(mn, e[u]);
    }
    const float sc = __expf(m - mn);
    m = mn;
    l *= sc;
#pragma unroll
    for (int d = 0; d < 8; ++d) acc[d] *= sc;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float p = __expf(e[u] - mn);
      float z[8];
      unpackh8(b.z[u], z);
      l += p;
#pragma unroll
      for (int d = 0; d < 8; ++d) acc[d] += p * z[d];
    }
    if (done) {
      const int64_t at = base + i0 + r;
      const float sum = stored && l == 0.f ? NAN : l;      // (no logit above -inf: the softmax is NaN)
      const float inv = sum > 0.f ? 1.f / sum : sum;
      float4* const u = reinterpret_cast<float4*>(a.U + at * kS + 8 * sub);
      u[0] = make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
      u[1] = make_float4(acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv);
      if (!(sub & 1)) a.lse[at * 8 + head] = m + __logf(sum);
      m = kLowest;
      l = 0.f;
#pragma unroll
      for (int d = 0; d < 8; ++d) acc[d] = 0.f;
    }
    if (!__ballot(busy)) break;
  }
}

template <bool TEAM>
__device__ __forceinline__ void gat_short(const GatArgs& a, int64_t item, int lane, SlotRow* list, TeamRow* queue, int* n_queued) {
  if constexpr (TEAM) {
    if (lane == 0) *n_queued = 0;
  }
  if (item >= a.n_work) return;
  const int32_t si = a.work[3 * item], r0 = a.work[3 * item + 1], nr = a.work[3 * item + 2];      // (at most 32 rows)
  const Segment s = a.segs[si];
  const int64_t base = (int64_t)s.t * a.g.N, i0 = s.v_lo + r0;
  const int64_t rp = a.g.rowptr[s.t][i0 + min(lane, nr)];
  const int64_t first = ((int64_t)__builtin_amdgcn_readfirstlane((int)(rp >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)rp);
  const int64_t len64 = __shfl_down((long long)rp, 1) - rp;
  const int start = (int)(rp - first), len = (int)len64;
  const int32_t* col = a.g.colidx[s.t] + first;
  const bool here = lane < nr && len64 <= a.long_nnz;      // (split rows: gat_long)
  const uint64_t below = (1ull << lane) - 1;
  const uint64_t teams = TEAM ? __ballot(here && len > kShared) : 0;
  uint64_t waves = __ballot(here && (len > kSlotRow || nr < kSlots)) & ~teams;
  const uint64_t own = __ballot(here) & ~waves & ~teams;
  if (own >> lane & 1) list[__popcll(own & below)] = SlotRow{start, start + len, lane};
  if constexpr (TEAM) {
    if (teams >> lane & 1) queue[__popcll(teams & below)] = TeamRow{rp, si, (int32_t)(i0 + lane), len};
    if (lane == 0) *n_queued = __popcll(teams);
  }
  __builtin_amdgcn_wave_barrier();
  const int head = (lane & 15) >> 1, listed = __popcll(own);
  while (waves) {
    const int r = __builtin_ctzll(waves);
    waves &= waves - 1;
    const int n = __builtin_amdgcn_readlane(len, r);
    const int32_t* at = col + __builtin_amdgcn_readlane(start, r);
    const SoftAcc sum = gat_row_range(a, s, at, base, a.sX[(base + i0 + r) * 16 + 8 + head], n, lane < n ? at[lane] : 0, lane);
    gat_row_store(a, base + i0 + r, sum, own_feature(lane), lane < 16 && !(lane & 1), head, n > 0);
  }
  if (listed) gat_slots(a, s, col, base, i0, list, listed, lane);
}

// record of one part of a split row: weighted sum [128], maximum [8], sum [8]
constexpr int kLongRec = 144;
__device__ __forceinline__ void put_record(float* rec, const SoftAcc& r, int lane) {
  *reinterpret_cast<float2*>(rec + own_feature(lane)) = make_float2(r.a0, r.a1);
  if (lane < 16 && !(lane & 1)) {
    rec[128 + (lane >> 1)] = r.m;
    rec[136 + (lane >> 1)] = r.l;
  }
}
// n records in their order; the lane's features are 2 lane and the next, its head lane / 8
__device__ __forceinline__ SoftAcc merge_records(const float* recs, int n, int lane) {
  const int head = lane >> 3;
  float mx = -INFINITY;
  for (int p = 0; p < n; ++p) mx = fmaxf(mx, recs[p * kLongRec + 128 + head]);
  SoftAcc r{mx, 0.f, 0.f, 0.f};
  for (int p = 0; p < n; ++p) {
    const float* rec = recs + p * kLongRec;
    const float sc = __expf(rec[128 + head] - mx);
    const float2 v = *reinterpret_cast<const float2*>(rec + 2 * lane);
    r.l += sc * rec[136 + head];
    r.a0 += sc * v.x;
    r.a1 += sc * v.y;
  }
  return r;
}

__device__ __forceinline__ void gat_long(const GatArgs& a, int64_t item, int lane) {
  if (item >= a.n_long) return;
  const int32_t* w = a.work_long + 4 * item;
  const Segment s = a.segs[w[0]];
  const int64_t i = s.v_lo + w[1];
  const int64_t* rowptr = a.g.rowptr[s.t];
  const int64_t base = (int64_t)s.t * a.g.N;
  const int head = (lane & 15) >> 1;
  const int64_t e0 = rowptr[i] + (int64_t)w[2] * a.part_nnz, e1 = min(rowptr[i + 1], e0 + a.part_nnz);
  const float sd = a.sX[(base + i) * 16 + 8 + head];
  const int32_t* first = a.g.colidx[s.t] + e0;
  const int n = (int)(e1 - e0);
  const SoftAcc r = gat_row_range(a, s, first, base, sd, n, lane < n ? first[lane] : 0, lane);
  put_record(a.long_partial + item * kLongRec, r, lane);
}

__global__ __launch_bounds__(256, 5) void k_gat_aggregate(GatArgs a, int64_t long_blocks) {
  const int lane = threadIdx.x & 63;
  __shared__ SlotRow list[kTeam][32];
  const int64_t block = blockIdx.x, wave = threadIdx.x >> 6;
  if (block < long_blocks) gat_long(a, block * kTeam + wave, lane);
  else gat_short<false>(a, (block - long_blocks) * kTeam + wave, lane, list[wave], nullptr, nullptr);
}

// The same where a row is longer than kShared: the launch on a small graph waits for its longest row (1024 non-zeros are 64
// batches in turn), so the four waves of a workgroup share a part, and the longer rows of their groups
// once the others are done.  The quarters' records meet in LDS and are merged in wave order.
__global__ __launch_bounds__(256, 5) void k_gat_aggregate_team(GatArgs a, int64_t long_blocks) {
  __shared__ SlotRow list[kTeam][32];
  __shared__ TeamRow queue[kTeam][32];          // a group has at most 32 rows
  __shared__ int queued[kTeam];
  __shared__ __align__(16) float recs[2][kTeam][kLongRec];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t block = blockIdx.x;
  const bool part = block < long_blocks;
  if (part) {
    if (lane == 0) {
      queued[wave] = wave == 0;
      if (wave == 0) {
        const int32_t* w = a.work_long + 4 * block;
        const Segment s = a.segs[w[0]];
        const int64_t i = s.v_lo + w[1];
        const int64_t* rowptr = a.g.rowptr[s.t];
        const int64_t e0 = rowptr[i] + (int64_t)w[2] * a.part_nnz;
        queue[0][0] = TeamRow{e0, w[0], (int32_t)i, (int32_t)(min(rowptr[i + 1], e0 + a.part_nnz) - e0)};
      }
    }
  } else {
    gat_short<true>(a, (block - long_blocks) * kTeam + wave, lane, list[wave], queue[wave], queued + wave);
  }
  __syncthreads();
  int turn = 0;
  for (int from = 0; from < kTeam; ++from)
    for (int k = 0; k < queued[from]; ++k, ++turn) {
      const TeamRow row = queue[from][k];
      const Segment s = a.segs[__builtin_amdgcn_readfirstlane(row.seg)];
      const int64_t base = (int64_t)s.t * a.g.N;
      const int n = __builtin_amdgcn_readfirstlane(row.n), quarter = (n + kTeam - 1) / kTeam;
      const int b = min(n, wave * quarter), m = min(n, b + quarter) - b;
      const float sd = a.sX[(base + row.i) * 16 + 8 + ((lane & 15) >> 1)];
      const int32_t* first = a.g.colidx[s.t] + row.e0 + b;
      put_record(recs[turn & 1][wave], gat_row_range(a, s, first, base, sd, m, lane < m ? first[lane] : 0, lane), lane);
      __syncthreads();        // (the next row's records go to the other buffer)
      if (wave == (turn & (kTeam - 1))) {
        const SoftAcc r = merge_records(recs[turn & 1][0], kTeam, lane);
        const int head = lane >> 3;
        if (part) {
          float* rec = a.long_partial + block * kLongRec;
          *reinterpret_cast<float2*>(rec + 2 * lane) = make_float2(r.a0, r.a1);
          if ((lane & 7) == 0) {
            rec[128 + head] = r.m;
            rec[136 + head] = r.l;
          }
        } else {
          gat_row_store(a, base + row.i, r, 2 * lane, (lane & 7) == 0, head);
        }
      }
    }
}

// one wavefront per split row (the item of its part 0) merges the parts in order
__global__ __launch_bounds__(256) void k_gat_aggregate_merge(GatArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= a.n_long) return;
  const int32_t* w = a.work_long + 4 * item;
  if (w[2] != 0) return;
  const Segment s = a.segs[w[0]];
  const SoftAcc r = merge_records(a.long_partial + item * kLongRec, w[3], lane);
  gat_row_store(a, (int64_t)s.t * a.g.N + s.v_lo + w[1], r, 2 * lane, (lane & 7) == 0, lane >> 3);
}

// ---------------------------------------------------------------------------------------------
// Temporal self-attention, forward.  One wavefront per two vertices of a chunk: 32 rows
// n = 16 a + s (a = vertex 0/1, s = step in the window).  Per block jb of 32 output features
// (two heads): Q and K in row layout, V in column layout; per head one product K Q^T gives the
// transposed score block of both vertices (lane (n_s, hh) holds the scores of its own query row
// against key rows 8g + 4hh + e; those of its own vertex are registers 8a .. 8a+7), the softmax
// is lane-local plus one exchange with lane l^32, and the probabilities are directly the B
// operand of the product with V (A operand = V in column layout; B masked
// to the vertex), which lands in row layout, ready to be stored.
// Every in-register operand (P, Q, K, V, the probabilities) is carried as a hi + lo pair of bf16
// values, so that the only roundings to bf16 are those of the stored tensors (z, U, Y).
struct TemporalArgs {
  const ChunkInfo* chunks; int32_t n_chunks;
  const int64_t* tile_ptr;   // [n_chunks+1] first tile of every chunk (2 vertices per tile; WIDE: 1)
  int64_t n_tiles;
  int64_t N; int32_t T;
  const float* U;
  const float* pos;          // [T][128]
  const uint4* Wq; const uint4* Wk; const uint4* Wv;   // mode-0 fragments
  uint16_t* Y; int64_t ldy;
};

// softmax over the key steps r <= s of the lane's own vertex; x[p] is the raw score against key
// step r = 8 (p/4) + 4 hh + p%4 (NP = 8: windows up to 16; NP = 16: up to 32); returns
// probabilities (0 for masked positions)
template <int NP>
__device__ __forceinline__ void causal_softmax(float* x, int s, int hh) {
  float mx = -INFINITY;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = 8 * (p >> 2) + 4 * hh + (p & 3);
    x[p] = keep_or_ninf(r <= s, 0.25f * x[p]);
    mx = fmaxf(mx, x[p]);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  float sum = 0.f;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    x[p] = __expf(x[p] - mx);
    sum += x[p];
  }
  sum += __shfl_xor(sum, 32);
  const float inv = 1.f / sum;
#pragma unroll
  for (int p = 0; p < NP; ++p) x[p] *= inv;
}

// The three weight matrices (96 KB of fragments) are staged in LDS once per workgroup; the
// workgroup's waves then walk the tiles with a grid stride and never synchronise again.
constexpr int kFragsPerW = 4 * 8 * 64;   // uint4 fragments of one 128 x 128 weight

__device__ __forceinline__ void stage_weights(uint4* lds, const uint4* w0, const uint4* w1, const uint4* w2) {
  for (int i = threadIdx.x; i < kFragsPerW; i += blockDim.x) {
    lds[i] = w0[i];
    lds[kFragsPerW + i] = w1[i];
    lds[2 * kFragsPerW + i] = w2[i];
  }
  __syncthreads();
}

// Twelve waves, three a SIMD, are what 155 registers allow: 12 x 5001 vertices, 2508 tiles, are one round of them on 256
// CUs, 35 us, and were two of eight, 44; an inference of 16 x 250 000 vertices takes 5.32 ms, with eight 5.43.  A wave's tiles lie gridDim apart, so
// that few tiles spread over all CUs.
constexpr int kTemporalWaves = 12;

// WIDE: one vertex per tile, windows of up to 32 snapshots: the score block of a head is the whole
// 32 x 32 product (all 16 registers of a lane are keys of its own vertex), and the product with V
// contracts over the two halves of the keys (registers 0..7 and 8..15) instead of over two vertices.
template <bool WIDE>
__global__ __launch_bounds__(64 * kTemporalWaves) void k_temporal_fwd(TemporalArgs a) {
  extern __shared__ uint4 wlds[];
  stage_weights(wlds, a.Wq, a.Wk, a.Wv);
  const int lane = threadIdx.x & 63;
  const int hh = lane >> 5;
  for (int64_t tile = (int64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x; tile < a.n_tiles; tile += (int64_t)gridDim.x * kTemporalWaves) {
  const TileRow r = tile_row<WIDE>(a.chunks, a.n_chunks, a.tile_ptr, tile, a.N, lane);
  const uint32_t m_vert[2] = {r.a == 0 ? 0xffffffffu : 0u, r.a == 1 ? 0xffffffffu : 0u};
  bf16x8 pf[8], pl[8];
  load_p_frags<true>(a.U, a.pos, r, hh, pf, pl);
#pragma unroll 1
  for (int jb = 0; jb < 4; ++jb) {
    floatx16 q = {}, k = {}, vt = {};
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
      const int fi = (jb * 8 + kb) * 64 + lane;
      const bf16x8 wq = as_frag(wlds[fi]), wk = as_frag(wlds[kFragsPerW + fi]), wv = as_frag(wlds[2 * kFragsPerW + fi]);
      q = mfma(wq, pf[kb], q);
      q = mfma(wq, pl[kb], q);
      k = mfma(wk, pf[kb], k);
      k = mfma(wk, pl[kb], k);
      vt = mfma(pf[kb], wv, vt);
      vt = mfma(pl[kb], wv, vt);
    }
    bf16x8 vh[2], vl[2];        // steps of the two vertices, or (WIDE) of the two halves of the window
#pragma unroll
    for (int av = 0; av < 2; ++av) split8v(vt, 8 * av, vh[av], vl[av]);
#pragma unroll
    for (int hd = 0; hd < 2; ++hd) {
      bf16x8 kh, kl, qh, ql;
      split8v(k, 8 * hd, kh, kl);
      split8v(q, 8 * hd, qh, ql);
      floatx16 st = {};
      st = mfma3(kh, kl, qh, ql, st);                 // st[i = key row][j = query row]
      constexpr int NP = WIDE ? 16 : 8;
      float pr[NP];
#pragma unroll
      for (int p = 0; p < NP; ++p) pr[p] = WIDE ? st[p] : pick_half(st, p, m_vert[0], m_vert[1]);
      causal_softmax<NP>(pr, r.s, hh);
      bf16x8 ph[NP / 8], plo[NP / 8];
#pragma unroll
      for (int c = 0; c < NP / 8; ++c) split8(pr + 8 * c, ph[c], plo[c]);
      floatx16 y = {};        // of both heads' features; this head's are registers 8 hd ..
#pragma unroll
      for (int av = 0; av < 2; ++av) {
        const bf16x8 pa = WIDE ? ph[WIDE ? av : 0] : and_mask(ph[0], m_vert[av]);
        const bf16x8 pb = WIDE ? plo[WIDE ? av : 0] : and_mask(plo[0], m_vert[av]);
        y = mfma3(vh[av], vl[av], pa, pb, y);
      }
      const uint4 o = head_order(__builtin_bit_cast(uint4, pack8v(y, 8 * hd)));
      if (r.valid) *reinterpret_cast<uint4*>(a.Y + r.row * a.ldy + jb * 32 + 16 * hd + 8 * hh) = o;
    }
  }
  }
}

}  // namespace

void dysat_build_owner(const Segment* segs, int64_t nseg, int32_t T, int64_t N, int32_t* owner, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_i32, blocks_for((int64_t)T * N, 256), 256, 0, st, owner, -1, (int64_t)T * N);
  hipLaunchKernelGGL(k_owner, (unsigned)nseg, 256, 0, st, segs, N, owner);
}

void dysat_pack_params(const DysatWs& ws, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_W], ws.Wp, 0);
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_WQ], ws.Wqp, 0);
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_WK], ws.Wkp, 0);
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_WV], ws.Wvp, 0);
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_WQ], ws.WqT, 1);
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_WK], ws.WkT, 1);
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_WV], ws.WvT, 1);
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_W], ws.WT, 1);
  hipLaunchKernelGGL(k_pack_w_bf16, 8, 256, 0, st, ws.P[DY_W], ws.WTlo, 2);
}

void dysat_forward(const DysatWs& ws, const void* X, int64_t ldx, const void* C, int64_t ldc, void* Y, int64_t ldy,
                   hipEvent_t* ev, hipStream_t st) {
  ProjArgs pa{};
  pa.X = static_cast<const uint16_t*>(X); pa.ldx = ldx;
  pa.C = static_cast<const uint16_t*>(C); pa.ldc = ldc;
  pa.Wp = ws.Wp; pa.a_src = ws.P[DY_ASRC]; pa.a_dst = ws.P[DY_ADST];
  pa.owner = ws.owner; pa.used_t = ws.used_t; pa.n_used = ws.n_used; pa.N = ws.N;
  pa.zX = ws.zX; pa.zC = ws.zC; pa.sX = ws.sX; pa.sC = ws.sC;
  const int64_t ptiles = (ws.N + 31) / 32 * ws.n_used;
  if (ev) (void)hipEventRecord(ev[0], st);
  hipLaunchKernelGGL(k_gat_project, (unsigned)std::min<int64_t>(512, (ptiles + 7) / 8), 512, 0, st, pa);
  if (ev) (void)hipEventRecord(ev[1], st);
  GatArgs ga{};
  ga.g = ws.g; ga.segs = ws.segs; ga.work = ws.work_fwd; ga.n_work = ws.n_fwd;
  ga.work_long = ws.work_long; ga.n_long = ws.n_long; ga.long_nnz = ws.long_nnz; ga.part_nnz = ws.part_nnz;
  ga.long_partial = ws.long_partial;
  ga.zX = ws.zX; ga.zC = ws.zC; ga.sX = ws.sX; ga.sC = ws.sC; ga.U = ws.U; ga.lse = ws.lse;
  // else there is nothing to share, or parts shorter than that are more than the chip holds at once (8 x 30 000 vertices of 60
  // neighbours, 0.5 M parts of 32: an inference 0.99 -> 2.03 ms)
  const bool team = ws.longest_row > kShared && ws.n_long <= (ws.part_nnz > kShared ? kMostTeams : kTeamsAtOnce);
  const int64_t long_blocks = team ? ws.n_long : (ws.n_long + kTeam - 1) / kTeam;
  hipLaunchKernelGGL(team ? k_gat_aggregate_team : k_gat_aggregate, (unsigned)(long_blocks + (ws.n_fwd + kTeam - 1) / kTeam), 256, 0, st,
                     ga, long_blocks);
  if (ws.n_long > 0) hipLaunchKernelGGL(k_gat_aggregate_merge, blocks_for(ws.n_long, 4), 256, 0, st, ga);
  if (ev) (void)hipEventRecord(ev[2], st);
  TemporalArgs ta{};
  ta.chunks = ws.chunks; ta.n_chunks = ws.n_chunks; ta.tile_ptr = ws.tile_ptr; ta.n_tiles = ws.n_tiles;
  ta.N = ws.N; ta.T = ws.T; ta.U = ws.U; ta.pos = ws.P[DY_POS];
  ta.Wq = ws.Wqp; ta.Wk = ws.Wkp; ta.Wv = ws.Wvp;
  ta.Y = static_cast<uint16_t*>(Y); ta.ldy = ldy;
  {
    static std::atomic<uint64_t> ready{0}, ready_wide{0};
    const size_t lds = sizeof(uint4) * 3 * kFragsPerW;
    (void)(ws.wide ? allow_lds(reinterpret_cast<const void*>(k_temporal_fwd<true>), lds, ready_wide)
                   : allow_lds(reinterpret_cast<const void*>(k_temporal_fwd<false>), lds, ready));   // if not, the launch is an error
    const unsigned grid = (unsigned)std::min<int64_t>(256, ws.n_tiles);
    if (ws.wide) hipLaunchKernelGGL(k_temporal_fwd<true>, grid, 64 * kTemporalWaves, lds, st, ta);
    else hipLaunchKernelGGL(k_temporal_fwd<false>, grid, 64 * kTemporalWaves, lds, st, ta);
  }
  if (ev) (void)hipEventRecord(ev[3], st);
}

}  // namespace dgc
