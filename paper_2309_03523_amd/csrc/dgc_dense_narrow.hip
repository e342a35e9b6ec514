// Time encoder of narrow layers (S = H of 32 or 64): the transform, the input-side and hidden-side products and the gates of
// dgc_dense_split.hip, its products (fp32 numbers as sums of three bf16 parts, six MFMAs) and its operands' order, on tiles of
// 16 vertices and 16 columns a wave.
//
// What bounds a narrow layer is the chain of one step: a wave's products, its gates and two barriers, on a few vertices.  In
// 32 x 32 blocks a layer of 32 is one wave a tile, and 8 snapshots of 1000 vertices occupy 34 of 1024 SIMDs for 34 us.
// v_mfma_f32_16x16x32_bf16 makes twice as many tiles, twice as many waves a tile and a quarter of the vector work a wave.  Half
// of a workgroup's waves follow the state, the others the input, which does not wait for it: they are a step ahead, so a
// step's chain is the hidden-side products and the gates (the 34 us become 12; with all of it in one wave, 14).
// The gates' weights (72 registers a product for 64 wide GRU gates) stay in registers for all tiles that a workgroup takes,
// the transform's in LDS.  The small part products of every sum go apart from the large one (in one sum the registers
// would do for twice the waves of a 64 wide GRU, which is 5 % on 200 000 vertices and nothing on few).
//   Weights are the A operand: lane l holds of row l % 16 of a 16-row block the columns
//   32 kb + 16 (e / 4) + 4 (l / 16) + e % 4, e = 0..7.  Activations are the B operand, column l % 16 (a vertex) in the same order,
//   and the lane receives of that vertex columns 4 (l / 16) .. +3 of the block: the lower or upper half of its next operand.
#include <algorithm>

#include "dgc_internal.h"
#include "dgc_split_dev.h"

namespace dgc {
namespace {

using namespace split;

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float sigmoid_fast(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }
__device__ __forceinline__ float tanh_fast(float x) { return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + __expf(2.0f * x)); }

__device__ __forceinline__ floatx4 mfma(const uint4& w, const uint4& x, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(w), as_frag(x), c, 0, 0, 0);
}
// large(g) += w[g] x (its large part product), small(g) += the five others, smallest first; one sum's after another's, so
// that none waits for the one before it
template <int NG, class Large, class Small>
__device__ __forceinline__ void six_each(Large&& large, Small&& small, const uint4 (&w)[NG][3], const uint4 (&x)[3]) {
  constexpr int kw[5] = {0, 2, 1, 0, 1}, kx[5] = {2, 0, 1, 1, 0};
#pragma unroll
  for (int k = 0; k < 5; ++k)
#pragma unroll
    for (int g = 0; g < NG; ++g) small(g) = mfma(w[g][kw[k]], x[kx[k]], small(g));
#pragma unroll
  for (int g = 0; g < NG; ++g) large(g) = mfma(w[g][0], x[0], large(g));
}

__device__ __forceinline__ floatx4 load4(const float* p) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  return floatx4{v.x, v.y, v.z, v.w};
}
__device__ __forceinline__ void store4(float* p, const floatx4& v) { *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]); }

// Where a workgroup is in the steps of its half tiles (the same for all lanes); the next one's tables are there before
// it is needed.
struct HalfTile {
  ChunkInfo ch;
  int64_t at;
  int v0, first, nrows;      // nrows = 0: there is none
};
__device__ __forceinline__ HalfTile half_tile_from(const DenseArgs& a, int64_t at) {
  HalfTile t{};
  for (; at < 2 * a.n_tiles32; at += gridDim.x) {
    const DenseTile tile = table_entry(a.tiles32, at >> 1);
    const int first = 16 * (int)(at & 1);
    if (tile.nrows > first) {
      t.ch = table_entry(a.chunks, tile.chunk);
      t.at = at;
      t.v0 = tile.v0;
      t.first = first;
      t.nrows = min(16, tile.nrows - first);
      break;
    }
  }
  return t;
}
struct Place {
  HalfTile cur, next;
  int s;
  __device__ __forceinline__ void start(const DenseArgs& a) {
    cur = half_tile_from(a, blockIdx.x);
    next = cur.nrows ? half_tile_from(a, cur.at + gridDim.x) : cur;
    s = 0;
  }
  __device__ __forceinline__ void advance(const DenseArgs& a) {
    if (++s < cur.ch.w) return;
    s = 0;
    cur = next;
    if (cur.nrows) next = half_tile_from(a, cur.at + gridDim.x);
  }
};

template <int KIND, int NW>
struct Narrow {
  static constexpr bool kLstm = KIND == DGC_TIME_LSTM;
  static constexpr int NG = kLstm ? 4 : 3, KBH = NW / 2, H = 16 * NW;
};
struct Lds {
  uint4 *wz, *xs, *hs, *zs;   // [NW][nkb0][3][64] transform weights, then this lane's places: input row, state, transformed row
  float4* pre;                // [NW][NG][64] input-side sums of the gates
};

__device__ __forceinline__ void put_cols(uint4* frag, int w, const floatx4& v) {   // a wave's 16 columns -> their half of k-block w / 2
  const float x[4] = {v[0], v[1], v[2], v[3]};
  uint2 p[3];
  split4(x, p);
#pragma unroll
  for (int k = 0; k < 3; ++k) reinterpret_cast<uint2*>(frag + ((w >> 1) * 3 + k) * kFrag)[w & 1] = p[k];
}

template <int NG, int KBH>
__device__ __forceinline__ void load_gates(uint4 (&to)[KBH][NG][3], const float4* from, int nw, int w, int lane) {
#pragma unroll
  for (int kb = 0; kb < KBH; ++kb)
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int p = 0; p < 3; ++p) to[kb][g][p] = reinterpret_cast<const uint4*>(from)[(((g * nw + w) * KBH + kb) * 3 + p) * kFrag + lane];
}

// The waves of the state: hidden-side products, gates, outputs.
template <int KIND, bool SEQ, int NW>
__device__ __forceinline__ void narrow_state(const DenseArgs& a, const Lds& l, int w, int lane) {
  using C = Narrow<KIND, NW>;
  constexpr int NG = C::NG, KBH = C::KBH, H = C::H;
  constexpr bool kLstm = C::kLstm;
  const int n16 = lane & 15, col0 = 16 * w + 4 * (lane >> 4);     // this lane's columns: col0 .. +3
  uint4 wh[KBH][NG][3];
  load_gates(wh, a.Whh, NW, w, lane);
  const floatx4 nbias = kLstm ? (floatx4)(0.f) : load4(a.bhh + 2 * H + col0);
  const int64_t V = a.total_state_rows;
  const bool mapped = SEQ && a.y_map != nullptr;
  Place at;
  at.start(a);
  floatx4 h = (floatx4)(0.f), c = (floatx4)(0.f), hin = (floatx4)(0.f), cin = (floatx4)(0.f);
  // Row of the tile that this lane stands for (past the end: the last one, never stored), and the state that enters step s:
  // with sequences that of state row sr where one starts, else the chunk's at its first snapshot, zero where the mask says so.
  auto row_of = [&](const HalfTile& t) { return t.v0 + t.first + min(n16, t.nrows - 1); };
  auto slot_of = [&](const HalfTile& t, int s) { return (int64_t)(t.ch.t_lo + s) * a.N + t.ch.v_lo + row_of(t); };
  int64_t sr = -1;
  bool taken = false;
  auto request_state = [&](const HalfTile& t, int s) {
    if constexpr (SEQ) sr = a.seq_in[slot_of(t, s)];
    else sr = s == 0 ? t.ch.state_off + row_of(t) : -1;
    taken = sr >= 0;
    if (a.H0) {
      const int64_t r = max(sr, (int64_t)0);
      if (SEQ || s == 0) {
        hin = load4(a.H0 + r * H + col0);
        if constexpr (kLstm) cin = load4(a.H0 + (V + r) * H + col0);
      }
    }
  };
  auto enter = [&](const HalfTile& t, int s) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      h[v] = taken ? hin[v] : h[v];
      if constexpr (kLstm) c[v] = taken ? cin[v] : c[v];
    }
    if constexpr (!SEQ) {
      if (a.reset_mask && a.reset_mask[slot_of(t, s)]) {
        h = (floatx4)(0.f);
        c = (floatx4)(0.f);
      }
    }
  };
  if (at.cur.nrows) {
    request_state(at.cur, 0);
    enter(at.cur, 0);
    put_cols(l.hs, w, h);
  }
  __syncthreads();
  __syncthreads();
  while (at.cur.nrows) {
    const HalfTile& t = at.cur;
    const int64_t slot = slot_of(t, at.s);
    int64_t so = -1, yr = slot;                 // state row that leaves after this step; row of Y
    if constexpr (SEQ) {
      so = a.seq_out[slot];
      if (mapped) yr = a.y_map[slot];
    } else if (at.s + 1 == t.ch.w) {
      so = t.ch.state_off + row_of(t);
    }
    const bool valid = n16 < t.nrows, last = at.s + 1 == t.ch.w;
    const HalfTile& nt = last ? at.next : t;
    const bool more = nt.nrows > 0;
    if (more) request_state(nt, last ? 0 : at.s + 1);
    __syncthreads();
    floatx4 acc[4], small[4];                   // LSTM: i, f, g, o; GRU: r, z, input part of n, hidden part of n
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      acc[g] = small[g] = (floatx4)(0.f);
      if (g < NG) {
        const float4 v = l.pre[(w * NG + g) * 64];
        acc[g] = floatx4{v.x, v.y, v.z, v.w};
      } else {
        acc[g] = nbias;
      }
    }
#pragma unroll
    for (int kb = 0; kb < KBH; ++kb) {
      uint4 x[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) x[p] = l.hs[(kb * 3 + p) * kFrag];
      six_each<NG>([&](int g) -> floatx4& { return acc[!kLstm && g == 2 ? 3 : g]; },
                   [&](int g) -> floatx4& { return small[!kLstm && g == 2 ? 3 : g]; }, wh[kb], x);
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] += small[g];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if constexpr (kLstm) {
        const float ig = sigmoid_fast(acc[0][v]), fg = sigmoid_fast(acc[1][v]);
        const float gg = tanh_fast(acc[2][v]), og = sigmoid_fast(acc[3][v]);
        c[v] = fg * c[v] + ig * gg;
        h[v] = og * tanh_fast(c[v]);
      } else {
        const float r = sigmoid_fast(acc[0][v]), zg = sigmoid_fast(acc[1][v]);
        const float n = tanh_fast(acc[2][v] + r * acc[3][v]);
        h[v] = (1.0f - zg) * n + zg * h[v];
      }
    }
    if (valid) {
      if (yr >= 0) store4(a.Y + yr * a.ldy + col0, h);
      if (a.HN && so >= 0) {
        store4(a.HN + so * H + col0, h);
        if constexpr (kLstm) store4(a.HN + (V + so) * H + col0, c);
      }
    }
    if (more) {
      enter(nt, last ? 0 : at.s + 1);
      put_cols(l.hs, w, h);
    }
    at.advance(a);
  }
}

// The waves of the input, a step ahead of the state's: input rows, the transform, input-side products.
template <int KIND, int NW>
__device__ __forceinline__ void narrow_input(const DenseArgs& a, const Lds& l, int w, int lane) {
  using C = Narrow<KIND, NW>;
  constexpr int NG = C::NG, KBH = C::KBH, H = C::H;
  constexpr int XP = NW == 2 ? 4 : 2;          // k-blocks of the input row that a wave requests ahead
  const int n16 = lane & 15, q4 = 4 * (lane >> 4), col0 = 16 * w + q4;
  const int nkb0 = (a.K0 + 31) / 32, kpad = (a.K0 + 15) / 16 * 16;
  uint4 wi[KBH][NG][3];
  load_gates(wi, a.Wih, NW, w, lane);
  const floatx4 zbias = a.bg ? load4(a.bg + col0) : (floatx4)(0.f);
  floatx4 gbias[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    gbias[g] = load4(a.bih + g * H + col0);
    if (C::kLstm || g < 2) gbias[g] += load4(a.bhh + g * H + col0);
  }
  // the input row in fragments: wave w takes k-blocks w, w + NW, ..; columns past the row's whole 16 are zero
  Place at;                                    // of the rows requested last
  at.start(a);
  float4 xq[XP][2];
  auto x_row = [&]() {
    const HalfTile& t = at.cur;
    return a.M + (t.ch.row_off0 + (int64_t)at.s * t.ch.nv + t.v0 + t.first + min(n16, t.nrows - 1)) * a.ldm + q4;
  };
  auto load_x = [&](const float* p, int kb, float4 (&x)[2]) {
    x[0] = *reinterpret_cast<const float4*>(p + 32 * kb);
    x[1] = 32 * kb + 16 < kpad ? *reinterpret_cast<const float4*>(p + 32 * kb + 16) : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  auto request_x = [&]() {
    if (!at.cur.nrows) return;
    const float* p = x_row();
#pragma unroll
    for (int k = 0; k < XP; ++k) load_x(p, min(w + k * NW, nkb0 - 1), xq[k]);
  };
  auto put_x = [&](int kb, const float4 (&x)[2]) {
    const float v[8] = {x[0].x, x[0].y, x[0].z, x[0].w, x[1].x, x[1].y, x[1].z, x[1].w};
    put(l.xs + kb * 3 * kFrag, v);
  };
  int staged = 0;
  auto stage_x = [&]() {                       // the rows requested last, and the request of the next
    if (!at.cur.nrows) return;
    ++staged;
#pragma unroll
    for (int k = 0; k < XP; ++k)
      if (w + k * NW < nkb0) put_x(w + k * NW, xq[k]);
    for (int kb = w + XP * NW; kb < nkb0; kb += NW) {
      float4 x[2];
      load_x(x_row(), kb, x);
      put_x(kb, x);
    }
    at.advance(a);
    request_x();
  };
  auto transform = [&]() {
    floatx4 z = zbias, small = (floatx4)(0.f);
    for (int kb = 0; kb < nkb0; ++kb) {
      uint4 x[3], wk[1][3];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        x[p] = l.xs[(kb * 3 + p) * kFrag];
        wk[0][p] = l.wz[((w * nkb0 + kb) * 3 + p) * kFrag + lane];
      }
      six_each<1>([&](int) -> floatx4& { return z; }, [&](int) -> floatx4& { return small; }, wk, x);
    }
    z += small;
    if (a.act == DGC_ACT_RELU)
#pragma unroll
      for (int v = 0; v < 4; ++v) z[v] = fmaxf(z[v], 0.f);
    put_cols(l.zs, w, z);
  };
  auto gates = [&]() {
    floatx4 acc[NG], small[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      acc[g] = gbias[g];
      small[g] = (floatx4)(0.f);
    }
#pragma unroll
    for (int kb = 0; kb < KBH; ++kb) {
      uint4 x[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) x[p] = l.zs[(kb * 3 + p) * kFrag];
      six_each<NG>([&](int g) -> floatx4& { return acc[g]; }, [&](int g) -> floatx4& { return small[g]; }, wi[kb], x);
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const floatx4 v = acc[g] + small[g];
      l.pre[(w * NG + g) * 64] = make_float4(v[0], v[1], v[2], v[3]);
    }
  };
  request_x();
  stage_x();
  __syncthreads();
  if (staged) transform();
  __syncthreads();
  if (staged) gates();
  stage_x();
  for (int done = 0; done < staged; ++done) {  // `staged` grows with the rows staged here
    const bool ahead = done + 1 < staged;      // the next step's rows are there
    __syncthreads();
    if (ahead) transform();
    __syncthreads();
    if (ahead) {
      gates();
      stage_x();
    }
  }
}

// 2 * NW waves (H = 16 NW): NW for the state and NW for the input, which keep a step's distance.  Two barriers a step.  Between the
// first and the second the state's waves read hs and pre and the input's read xs and write zs; after the second
// hs is written, zs read, pre and xs written.  SEQ: as the fields of DenseArgs say.
template <int KIND, bool SEQ, int NW, int PER_SIMD>
__global__ __launch_bounds__(128 * NW, PER_SIMD) void k_dense_narrow(DenseArgs a) {
  using C = Narrow<KIND, NW>;
  extern __shared__ __align__(16) uint4 lds[];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nkb0 = (a.K0 + 31) / 32;
  Lds l;
  l.wz = lds;
  l.xs = l.wz + NW * nkb0 * 3 * kFrag + lane;
  l.hs = l.xs + nkb0 * 3 * kFrag;
  l.zs = l.hs + C::KBH * 3 * kFrag;
  l.pre = reinterpret_cast<float4*>(l.zs + C::KBH * 3 * kFrag);
  const uint4* const Wg = reinterpret_cast<const uint4*>(a.Wg);
  for (int i = threadIdx.x; i < NW * nkb0 * 3 * kFrag; i += 128 * NW) l.wz[i] = Wg[i];
  if (w < NW) narrow_state<KIND, SEQ, NW>(a, l, w, lane);
  else narrow_input<KIND, NW>(a, l, w - NW, lane);
}

// W [n_out][n_in] -> packed[((block*nkb + kb)*3 + part)*64 + lane], zero beyond n_in
__global__ void k_pack_narrow(const float* W, int32_t n_out, int32_t n_in, uint4* packed) {
  const int nkb = (n_in + 31) / 32;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)(n_out / 16) * nkb * 64) return;
  const int lane = (int)(idx & 63);
  const int64_t f = idx >> 6;
  const int kb = (int)(f % nkb);
  const float* w = W + ((f / nkb) * 16 + (lane & 15)) * n_in;
  float x[8];
  for (int e = 0; e < 8; ++e) {
    const int col = 32 * kb + 16 * (e / 4) + 4 * (lane >> 4) + e % 4;
    x[e] = col < n_in ? w[col] : 0.f;
  }
  uint4 part[3];
  split8(x, part);
  for (int p = 0; p < 3; ++p) packed[f * 3 * 64 + p * 64 + lane] = part[p];
}

constexpr size_t kFragBytes = 3 * kFrag * sizeof(uint4);
size_t narrow_lds(int32_t H, int32_t K0, int32_t time_kind) {
  const int nw = H / 16, nkb0 = (K0 + 31) / 32, ng = time_kind == DGC_TIME_LSTM ? 4 : 3;
  return kFragBytes * (nw * nkb0 + nkb0 + nw) + sizeof(float4) * 64 * nw * ng;
}

template <int KIND, bool SEQ, int NW, int PER_SIMD>
bool launch(const DenseArgs& a, hipStream_t st, std::string* why) {
  const size_t lds = narrow_lds(16 * NW, a.K0, KIND);
  static std::atomic<uint64_t> ready{0};
  auto* kernel = &k_dense_narrow<KIND, SEQ, NW, PER_SIMD>;
  if (!allow_lds(reinterpret_cast<const void*>(kernel), 160 * 1024, ready, why)) return false;
  const int64_t per_cu = std::min<int64_t>(PER_SIMD * 4 / (2 * NW), 160 * 1024 / lds);
  const int64_t grid = std::min<int64_t>(2 * a.n_tiles32, 256 * per_cu);
  if (grid > 0) hipLaunchKernelGGL(kernel, (unsigned)grid, 128 * NW, lds, st, a);
  return true;
}

}  // namespace

bool dense_narrow_supported(int32_t S, int32_t H, int32_t K0, int32_t time_kind) {
  return S == H && (H == 32 || H == 64) && (time_kind == DGC_TIME_GRU || time_kind == DGC_TIME_LSTM) && narrow_lds(H, K0, time_kind) <= 160 * 1024;
}

// Against k_dense_split, which takes the folded transform where there is one, and half the matrix instructions.  What this kernel
// has the less of is the chain of a step and the transform's time; what it pays is that a workgroup loads all weights first (with
// windows of one step for nothing) and, where tiles are many, that fewer of them are on the chip at once.  So it is for few tiles,
// the more the longer the windows are, for more where the other kernel's transform is not folded, and for many where the input is
// so wide that few of the other kernel's workgroups fit a CU's LDS.
// How many times as long the other kernel takes for a forward, GRU (LSTM: up to a tenth more); w: the windows' snapshots.
//   64 wide, folded, 64 columns:  128 tiles w 1 1.04 to 1.12, w 2 1.08 to 1.2, w 4 1.36, w 8 1.43; 256 tiles w 2 and 4 0.98, w 8 1.06; 384 tiles
//                                 w 4 0.99, w 8 1.03, w 16 1.05; 512 tiles w 8 0.89 (GRU over 64: 76 us and 86), 1024 0.72, 2048 0.82
//            folded, 80 columns:  256 tiles w 4 1.07, 384 1.04, 512 0.91
//            96 columns:          384 tiles w 2 1.05, 512 0.98, w 4 1.02, w 8 1.02, 768 0.89 to 0.95
//            128 columns:         128 tiles w 1 1.0, 256 0.95; 384 w 2 1.01, w 4 1.10; 512 w 2 0.94, w 4 1.0, w 8 1.02; 768 w 8 0.91
//            132 to 176 columns:  512 tiles w 2 0.95, w 4 1.0, w 8 1.05; 640 w 2 1.12, w 8 1.33; 768 w 2 1.08, w 8 1.2; 1024 w 2 1.0, w 8 1.06; 2048 w 2
//                                 and w 8 1.07, w 1 1.0
//   32 wide, folded, 32 columns:  256 tiles w 1 1.01, w 2 1.1, 512 w 2 0.87, 768 w 4 1.01, w 8 1.07, 1024 w 4 0.94, w 16 0.99; 2048 w 8 0.77
//            48 columns:          512 tiles w 1 0.98, w 2 1.04, 1024 w 2 0.94, w 4 1.07, w 8 1.1; 2048 w 8 0.91
//            64 columns:          1024 tiles w 1 0.9, w 2 0.95, w 8 1.1; 2048 w 1 1.01, w 2 1.04, w 8 1.17
//            80 columns, 128:     1024 tiles w 1 0.94, 1.17, w 8 1.14, 1.53; 2048 w 1 1.03, 1.18, w 8 1.14, 1.33
bool dense_narrow_wanted(int32_t H, int32_t K0, bool folds, int64_t n_tiles32, int32_t window) {
  const int64_t w = std::min(window, 4);
  if (H == 32) {
    if (K0 > 64) return true;
    if (K0 > 48) return window > 1 || n_tiles32 >= 2048;
    return n_tiles32 <= (folds ? 256 * (w - 1) : std::min<int64_t>(512 * (w - 1), 1024));
  }
  if (window == 1) return n_tiles32 <= 128;
  if (folds) return n_tiles32 <= (window >= (K0 > 64 ? 4 : 6) ? 384 : 128);
  return n_tiles32 <= (K0 > 128 ? 2048 : window == 2 ? 384 : 512);
}

bool launch_dense_narrow(const DenseArgs& a, hipStream_t st, std::string* why) {
  const bool seq = a.seq_in != nullptr;
  if (a.time_kind == DGC_TIME_GRU) {
    if (a.H == 32) return seq ? launch<DGC_TIME_GRU, true, 2, 3>(a, st, why) : launch<DGC_TIME_GRU, false, 2, 3>(a, st, why);
    return seq ? launch<DGC_TIME_GRU, true, 4, 2>(a, st, why) : launch<DGC_TIME_GRU, false, 4, 2>(a, st, why);
  }
  if (a.H == 32) return seq ? launch<DGC_TIME_LSTM, true, 2, 3>(a, st, why) : launch<DGC_TIME_LSTM, false, 2, 3>(a, st, why);
  return seq ? launch<DGC_TIME_LSTM, true, 4, 2>(a, st, why) : launch<DGC_TIME_LSTM, false, 4, 2>(a, st, why);
}

int64_t narrow_weight_bytes(int32_t n_out, int32_t n_in) { return (int64_t)(n_out / 16) * ((n_in + 31) / 32) * kFragBytes; }

void launch_pack_narrow(const float* W, int32_t n_out, int32_t n_in, void* packed, hipStream_t st) {
  const int64_t total = (int64_t)(n_out / 16) * ((n_in + 31) / 32) * 64;
  hipLaunchKernelGGL(k_pack_narrow, (unsigned)((total + 255) / 256), 256, 0, st, W, n_out, n_in, static_cast<uint4*>(packed));
}

}  // namespace dgc
