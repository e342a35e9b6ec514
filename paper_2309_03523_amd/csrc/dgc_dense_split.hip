// Dense part of the layer on the matrix cores of 16-bit numbers at fp32 accuracy.
//
// Transforms alone: an fp32 number is the exact sum of three bf16 numbers, each the nearest to what is left (split8), so a
// product of fp32 operands is six bf16 MFMAs: hi*hi, hi*mid, mid*hi, mid*mid, hi*lo, lo*hi, all accumulated in fp32.  What is
// left out (mid*lo, lo*mid, lo*lo) is within 2^-24 of the product and of either sign: over random operands 2^-28 in the mean,
// without a bias.  (Parts cut off instead of rounded leave out up to 2^-21, always of the product's own sign: EvolveGCN-O's
// gradients are then twice to three times as far off.)  v_mfma_f32_32x32x16_bf16 does 16 times the work of
// v_mfma_f32_32x32x2f32 per cycle, so the six cost 2.7 times less than the fp32 instruction and add up in fewer roundings.  No
// scaling is needed, but at the ends of the range fp32 has a little more: a product within 1 % of the largest float may
// overflow (its rounded high parts do), and of a number below 2^-110 the parts below the smallest bf16 number are lost (a
// transform of nothing but such rows is 3e-7 off at 2^-112 and 3e-3 at 2^-126).
//
// Time encoders: their sums go into sigmoid and tanh, which are at most 1 and off by a rounding of 1, so an error that is small
// beside 1 does.  There a number is two half-precision numbers (halve8), and a product three MFMAs: hi*lo, lo*hi, hi*hi.  Two
// halves hold 22 to 24 bits of a number, and nothing below 2^-36 of an input or a state (taken 2048 times) and 2^-37 of a weight
// (4096 times); what is left out, lo*lo, is within 2^-22 of the product and of either sign.  tanh_of, whose series keeps what
// 1 - 2 / (1 + e^2x) loses below 1/2, takes back more than that, as long as the sums are of the size of 1.
// What is not: an input from 32 on, a bias above 1e30, and weights whose rows are longer than kLongestRow: there
// the tile goes on from that step, which it does again, to its window's end (for weights from the first) on three bf16 parts: a whole forward
// where all rows are 10 x 12 345, width 64, 85 -> 100 us, 32 x 100 000 of 128 5.0 -> 6.0 ms, MPNN-LSTM 5.3 -> 6.2, LSTM over labels 1.39 -> 1.73,
// GRU 256 over 300 0.88 -> 1.13, all of them no slower than on six products with the plain formula; where one row in a thousand of the last
// step is, nothing.
// Distance from 64 bits in that of six bf16 products with the plain formula: 0.58 in the mean and 1.003 at most of 206 outputs of drawn
// cases, 0.62 to 0.79 of GRUs 96 to 256 wide over 30 and 60 snapshots.  Over inputs of N(0, 1) times x and Xavier weights times w (GRU and LSTM 128 and 256 wide, one and two layers): x up to 1e-3 0.00 to 0.01
// without biases (1e-10: 0.3 to 0.9) and 0.17 to 0.5 with them, x = 1 0.3 to 0.8, 2 0.3 to 1.03, 5 0.5 to 1.23, 12 0.6 to 1.3, from 30 on 0.7 to 1.0 (three
// parts); w = 2, x = 1 0.7 to 1.14, 12 1.0 to 1.4, w = 4 0.9 to 1.03 (three parts).  Where it is above 1, by 22 bits instead of 24, lo*lo and the
// small products that are not summed apart, it is 1.5 to 4e-7 of the outputs.  All small products apart or added by link would take 0.05 to 0.1 off that
// and cost 1 to 10 %, lo*lo as well 0.1 and 5 %.  Inputs taken 64 times, up to 1023: 1.7 at x = 300, and 32 times as far at 1e-5 and below.
// GRU 128 wide, 3.2 M rows: 3.5 -> 2.35 ms; the two LSTM layers of MPNN-LSTM over 1.28 M rows 2.78 + 1.99 -> 1.9 + 1.2.
//
// With the weights as A operand (lane l: A[l%32][8*(l/32) .. +7]) and 32 activation rows as B operand
// (B[8*(l/32) .. +7][l%32]), lane (n = l%32, half = l/32) receives of row n the columns 8*g4 + 4*half + e in
// register 4*g4 + e.  Registers 0..7 (8..15) are then one k-half of a 16-wide k-block whose slots
// 8*half + 4*p + e stand for columns 8*p + 4*half + e: with the weights' columns packed in that order a
// result is the next product's operand without moving between lanes.
//
// What bounds them.  Transforms: the matrix cores' power.  Random operands through a loop of nothing but this MFMA reach
// 1.8 PFLOP/s of bf16 on this GPU (2.46 with zeros), a library product 1.33.
// Time encoders: the weights' way from the L2 to the registers, 64 bytes a cycle and CU.  With a third of the products they take
// the same time, with three waves a SIMD instead of two, too (2.35 ms of GRU 128 wide, of 3.2 M rows, at 40 % of the matrix cores' cycles);
// with every weight read from the nearest cache 2.1.
//
// k_dense_split (time encoders): a workgroup owns 32 vertices of one chunk and walks the chunk's window; wave jb
// owns columns 32*jb .. +31 of Z, of every gate and of the state.  So a weight fragment is read from L2 by one
// wave of the workgroup, and only the split activations (h, M, Z in turn) go through LDS.
// k_rows_split (transforms alone): wave jb keeps its columns of the weights in registers and a workgroup streams
// row tiles past them, so that nothing but rows is read (4 M rows, 256 -> 256: 5.16 ms on the fp32 instruction, 3.67
// with the weights from L2 for every 64 rows, 3.5 like this, of which the rows alone take 2.0 and the products alone
// 2.3; 1.28 M rows, 172 -> 128: 0.85 -> 0.39 ms).  From 13 k-blocks on (four waves; 15 with eight) 256 registers do not
// hold the weights, both sums and the requested rows: 8 to 36 of them go to scratch.
#include <algorithm>

#include "dgc_internal.h"
#include "dgc_split_dev.h"

namespace dgc {
namespace {

using namespace split;

constexpr int kUnitBytes = 3 * kFrag * 16; // a weight fragment's three parts
template <int P> constexpr int kUnit = P * kFrag * 16;    // P parts

constexpr float kActScale = 2048.f, kWeightScale = 4096.f, kSumScale = kActScale * kWeightScale;
constexpr float kMostBias = 1e30f;

// Of x scale: the gates' arguments come in the scale of their sums.
__device__ __forceinline__ float sigmoid_of(float x, float scale) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * (-1.4426950408889634f * scale)));
}
// Below 1/2 by x + x^3 P(x^2), P the polynomial of least relative error there (1.5e-8): 1 - 2 / (1 + e^2x) leaves an error of the
// size of 1's rounding however small x is.
__device__ __forceinline__ float tanh_of(float x, float scale) {
  const float y = x * scale, z = y * y;
  const float p = fmaf(fmaf(fmaf(0.01724136434495449f, z, -0.05304544046521187f), z, 0.13325878977775574f), z, -0.333331435918808f);
  const float t = fmaf(-2.0f, __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * (2.8853900817779268f * scale))), 1.0f);
  return fabsf(y) < 0.5f ? fmaf(y * z, p, y) : t;
}
// Weights come by buffer loads: resource descriptor in scalar registers, the fragment's place as scalar
// offset, the lane's 16 bytes as vector offset.  A vector offset beyond the resource reads as zero without
// touching memory: that is what a fragment past the end of a product gets, so that the loops have no branches.
struct WeightStream {
  __amdgpu_buffer_rsrc_t rsrc;
  template <int P>
  __device__ __forceinline__ void unit(uint4 (&w)[P], int lane16, int off, bool there) const {
    const int v = lane16 + (there ? 0 : 0x40000000);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const intx4 x = __builtin_amdgcn_raw_buffer_load_b128(rsrc, v, off + p * kFrag * 16, 0);
      w[p] = make_uint4(x.x, x.y, x.z, x.w);
    }
  }
};
__device__ __forceinline__ WeightStream make_stream(const void* p, int64_t bytes) {
  WeightStream w;
  w.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
  return w;
}

// A matrix of `units` fragments as k_pack_split leaves it: three bf16 parts a fragment, two halves a fragment, and a word that is not
// zero where the halves do not stand for the matrix (k_halves_word).
struct Weights {
  const uint4* parts;
  int units;
  __device__ __forceinline__ Weights(const void* p, int n) : parts(static_cast<const uint4*>(p)), units(n) {}
  __device__ __forceinline__ WeightStream stream(std::integral_constant<int, 3>) const { return make_stream(parts, (int64_t)units * kUnit<3>); }
  __device__ __forceinline__ WeightStream stream(std::integral_constant<int, 2>) const {
    return make_stream(parts + (int64_t)units * 3 * kFrag, (int64_t)units * kUnit<2>);
  }
  __device__ __forceinline__ bool halves_good() const {
    return table_entry(reinterpret_cast<const int32_t*>(parts + (int64_t)units * 5 * kFrag), 0) == 0;
  }
};

// The weight fragments of a product are read in the order (k-block, gate), D - 1 of them ahead of their use.
// fetch_ahead: the first D - 1, before the barrier that the product waits at.  nkb: k-blocks that have weights.
template <int NG, int D, int P>
__device__ __forceinline__ void fetch_ahead(uint4 (&w)[D][P], const WeightStream& ws, int off, int gstride, int nkb, int lane16) {
#pragma unroll
  for (int u = 0; u < D - 1; ++u) ws.unit(w[u], lane16, off + (u % NG) * gstride + (u / NG) * kUnit<P>, u / NG < nkb);
}

// acc(g) + small(g) += W_g x rows, over nkb k-blocks (small: the five small products; may be acc); fr: this lane's
// first operand of the staged rows.  LINKS: the small products of every k-block go to a sum of their own, which is added
// to acc by rounding additions.
template <int NG, int D, int P, bool LINKS = false, class Acc, class Small>
__device__ __forceinline__ void product(Acc&& acc, Small&& small, const uint4* fr, const WeightStream& ws, int off, int gstride, int nkb,
                                        int lane16, uint4 (&w)[D][P]) {
  constexpr int UK = D > NG ? D / NG : 1;
  static_assert((UK * NG) % D == 0, "the buffers come round within the unrolled k-blocks");
  auto add = [](floatx16& c, floatx16& s, const uint4 (&a)[P], const uint4 (&b)[P]) {
    if constexpr (P == 3) six(c, s, a, b);
    else three(c, s, a, b);
  };
  uint4 b[P];
#pragma unroll
  for (int p = 0; p < P; ++p) b[p] = fr[p * kFrag];
  __builtin_amdgcn_s_setprio(1);   // the other workgroups of the CU do their vector work beside this
#pragma unroll 1
  for (int kb = 0; kb < nkb; kb += UK) {
#pragma unroll
    for (int i = 0; i < UK; ++i) {
      const int k = kb + i;
      if (UK > 1 && k >= nkb) break;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int u = i * NG + g;
        const int kn = k + (g + D - 1) / NG, gn = (g + D - 1) % NG;
        ws.unit(w[(u + D - 1) % D], lane16, off + gn * gstride + kn * kUnit<P>, kn < nkb);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (LINKS) {
          floatx16 link = (floatx16)(0.f);
          add(acc(g), link, w[u % D], b);
          acc(g) += link;
        } else {
          add(acc(g), small(g), w[u % D], b);
        }
        if (g == NG - 1) {
          const uint4* next = fr + min(k + 1, nkb - 1) * (P * kFrag);
#pragma unroll
          for (int p = 0; p < P; ++p) b[p] = next[p * kFrag];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// columns 16*kb .. +15 of an input row (a pitch is a multiple of 16 floats); row: the lane's first column
__device__ __forceinline__ void load_x(const float* row, int kb, float4 (&x)[2]) {
  x[0] = *reinterpret_cast<const float4*>(row + 16 * kb);
  x[1] = *reinterpret_cast<const float4*>(row + 16 * kb + 8);
}
__device__ __forceinline__ void put_x(uint4* frag, const float4 (&x)[2]) {
  const float v[8] = {x[0].x, x[0].y, x[0].z, x[0].w, x[1].x, x[1].y, x[1].z, x[1].w};
  put(frag, v);
}
// x scale as two halves; whether one of them is too large
__device__ __forceinline__ bool put_halves(uint4* frag, const float (&v)[8], float scale) {
  uint4 p[2];
  const float top = halve8(v, scale, p);
#pragma unroll
  for (int q = 0; q < 2; ++q) frag[q * kFrag] = p[q];
  return top * scale > kHalfMost;
}
// a lane's 16 values of a 32-column block in global memory or LDS; p: its first column
__device__ __forceinline__ floatx16 load_block(const float* p) {
  floatx16 r;
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    const float4 b = *reinterpret_cast<const float4*>(p + 8 * g4);
    r[4 * g4] = b.x; r[4 * g4 + 1] = b.y; r[4 * g4 + 2] = b.z; r[4 * g4 + 3] = b.w;
  }
  return r;
}
__device__ __forceinline__ void store_block(float* p, const floatx16& v) {
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4)
    *reinterpret_cast<float4*>(p + 8 * g4) = make_float4(v[4 * g4], v[4 * g4 + 1], v[4 * g4 + 2], v[4 * g4 + 3]);
}
__device__ __forceinline__ void relu(floatx16& z) {
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = fmaxf(z[v], 0.f);
}

// What a row of M is to the time encoder: Z's operand; its input by way of the folded weights (no transform: where no
// activation stands between them, W_ih (W_g m + b_g) = (W_ih W_g) m + W_ih b_g); its input as it is (a second recurrent layer).
// Folding takes 8 of 56 products of 16-wide links a tile, step and wave from a GRU 128 wide over 128 columns, the pass of Z through
// LDS and a barrier: on three parts 32 x 100 000 vertices 4.05 -> 3.5 ms (2.45 on halves).  The product of
// the weights is summed in double and rounded once, where Z was rounded, so nothing gets further from 64 bits (on three parts 0.87 of
// the distance in the mean of 46 outputs of GRUs, 0.94 of 24 of LSTMs, 0.999 at most).
enum Input { kTransform, kFolded, kStack };

template <int NG, bool FEW, int P> constexpr int kHeldOf = FEW && P == 3 ? 2 : NG;     // weight fragments held of the gates

// KIND: DGC_TIME_GRU or DGC_TIME_LSTM.  SEQ, CAT: as the fields of DenseArgs say (sequences inside the window;
// the time encoder's input is [X2 row, Z]).
// HALVES: on two halves a number while these hold them, and on three bf16 parts from the step on where one does not.
template <int KIND, bool SEQ, bool CAT, Input INPUT, bool HALVES>
__device__ __forceinline__ void dense_split(const DenseArgs& a) {
  constexpr bool kLstm = KIND == DGC_TIME_LSTM, STACK = INPUT == kStack, FOLD = INPUT == kFolded;
  const float* const bih = FOLD ? a.bf : a.bih;
  constexpr int NG = kLstm ? 4 : 3;
  constexpr int DZ = SEQ ? 3 : 4;             // weight fragments held of the transform
  extern __shared__ __align__(16) uint4 lds[];
  const int njb = blockDim.x >> 6, kbh = 2 * njb, H = 32 * njb;
  const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
  const int jb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane16 = lane * 16;
  const int kbc = a.kb_chunk;                 // k-blocks that a staging buffer holds
  // Two staging buffers in turn: a buffer is written again after a barrier that every wave reached past its
  // reads of it.
  uint4* buf = lds + lane;
  uint4* other = buf + kbc * 3 * kFrag;
  float* gbias = reinterpret_cast<float*>(lds + 2 * kbc * 3 * kFrag);
  float* zbias = gbias + 4 * H;
  int* said = reinterpret_cast<int*>(zbias + H);    // the last two products with an operand out of range; [2]: a bias is
  if constexpr (HALVES) {
    if (threadIdx.x < 3) said[threadIdx.x] = 0;
    __syncthreads();
  }
  float most_bias = 0.f;
  for (int i = threadIdx.x; i < H; i += blockDim.x) {
    zbias[i] = a.bg ? a.bg[i] : 0.f;
    if constexpr (kLstm) {
#pragma unroll
      for (int g = 0; g < 4; ++g) gbias[g * H + i] = bih[g * H + i] + a.bhh[g * H + i];
    } else {
      gbias[i] = bih[i] + a.bhh[i];
      gbias[H + i] = bih[H + i] + a.bhh[H + i];
      gbias[2 * H + i] = bih[2 * H + i];
      gbias[3 * H + i] = a.bhh[2 * H + i];
    }
    most_bias = fmaxf(most_bias, fabsf(zbias[i]));
#pragma unroll
    for (int g = 0; g < 4; ++g) most_bias = fmaxf(most_bias, fabsf(gbias[g * H + i]));
  }
  if (HALVES && most_bias > kMostBias) said[2] = 1;
  const DenseTile tile = table_entry(a.tiles32, blockIdx.x);
  const ChunkInfo ch = table_entry(a.chunks, tile.chunk);
  const int nkb0 = STACK ? kbh : (a.K0 + 15) / 16, nchunk = (nkb0 + kbc - 1) / kbc;
  const int kbx = CAT ? 2 * kbh : kbh;        // k-blocks of the time encoder's input
  const int64_t V = a.total_state_rows;
  const Weights wsg(FOLD ? a.Wf : a.Wg, STACK ? 0 : (FOLD ? NG : 1) * njb * nkb0);
  const Weights wsi(a.Wih, NG * njb * kbx);
  const Weights wsh(a.Whh, NG * njb * kbh);
  const int uz = jb * nkb0;                   // first fragments of this wave, and from gate to gate
  const int ux = jb * kbx, gx = njb * kbx, uh = jb * kbh, gh = njb * kbh;
  const int uf = jb * nkb0, gf = njb * nkb0;
  const int col0 = 32 * jb + 4 * half;        // this lane's columns: col0 + 8*g4 + e
  const bool valid = l32 < tile.nrows;        // rows past the tile's end repeat its last row and are never stored
  const int row = min(l32, tile.nrows - 1);
  const int64_t v0 = ch.v_lo + tile.v0 + row, s0 = ch.state_off + tile.v0 + row;
  auto slot = [&](int64_t ts) { return ts * a.N + v0; };

  // SEQ with a row map: row of Y of this step and of the next one
  const bool mapped = SEQ && a.y_map != nullptr;
  int yrow = 0, yrow_next = 0;
  if (mapped) yrow_next = (int)a.y_map[slot(ch.t_lo)];
  auto in_row = [&](int s) -> const float* {
    int64_t r;
    if constexpr (STACK) r = mapped ? (int64_t)max(yrow_next, 0) : slot(ch.t_lo + s);
    else r = ch.row_off0 + (int64_t)s * ch.nv + tile.v0 + row;
    return a.M + r * a.ldm + 4 * half;
  };
  // Staging: wave w takes k-blocks 2w, 2w + 1 (then 2w + 2*njb ...).  The first two are requested ahead (past the
  // row's end: its last one).
  float4 xq[2][2];
  auto request_x = [&](int s, int c) {
    const float* p = in_row(s);
#pragma unroll
    for (int q = 0; q < 2; ++q) load_x(p, min(c * kbc + 2 * jb + q, nkb0 - 1), xq[q]);
  };
  // a 16-column block of numbers -> its place in a buffer of P parts a k-block; whether it is out of the halves' range
  auto put_parts = [&](auto parts, int kb, const float (&x)[8], float scale) -> bool {
    constexpr int P = decltype(parts)::value;
    uint4* const frag = buf + kb * P * kFrag;
    if constexpr (P == 2) return put_halves(frag, x, scale);
    put(frag, x);
    return false;
  };
  // An infinite input makes NaN of the gates: Z's infinities have either sign, and so the gates' sums (k_fold finds the weights
  // of which this is not true, and they are not folded).  The folded weights would hide that.
  auto put_row = [&](auto parts, int kb, const float4 (&x)[2]) -> bool {
    float v[8] = {x[0].x, x[0].y, x[0].z, x[0].w, x[1].x, x[1].y, x[1].z, x[1].w};
    if constexpr (FOLD)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = fmaf(v[e], 0.f, v[e]);
    return put_parts(parts, kb, v, kActScale);
  };
  auto stage_x = [&](auto parts, int s, int c) -> bool {
    const int k0 = c * kbc, n = min(kbc, nkb0 - k0);
    bool out = false;
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (2 * jb + q < n) out |= put_row(parts, 2 * jb + q, xq[q]);
    for (int kb = 2 * (jb + njb); kb < n; kb += 2 * njb)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (kb + q < n) {
          float4 x[2];
          load_x(in_row(s), k0 + kb + q, x);
          out |= put_row(parts, kb + q, x);
        }
    return out;
  };
  // a 32-column block in registers -> k-blocks 2*jb, 2*jb + 1
  auto turn = [&]() { uint4* x = buf; buf = other; other = x; };
  auto put_block = [&](auto parts, const floatx16& v, float scale) -> bool {
    bool out = false;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float x[8] = {v[8 * q], v[8 * q + 1], v[8 * q + 2], v[8 * q + 3], v[8 * q + 4], v[8 * q + 5], v[8 * q + 6], v[8 * q + 7]};
      out |= put_parts(parts, 2 * jb + q, x, scale);
    }
    return out;
  };

  floatx16 h = (floatx16)(0.f), c = (floatx16)(0.f);
  // The state that enters a snapshot: a masked row starts from zero; with SEQ a row where a sequence starts takes
  // the sequence's state, which is requested well before (rows where none starts request the first state row).
  int64_t sr = -1;
  floatx16 hin = (floatx16)(0.f), cin = (floatx16)(0.f);
  auto request_state = [&]() {
    if (a.H0) {
      const int64_t r = max(sr, (int64_t)0);
      hin = load_block(a.H0 + r * H + col0);
      if constexpr (kLstm) cin = load_block(a.H0 + (V + r) * H + col0);
    }
  };
  auto enter = [&](int64_t ts) {
    if constexpr (SEQ) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        h[v] = sr >= 0 ? hin[v] : h[v];
        if constexpr (kLstm) c[v] = sr >= 0 ? cin[v] : c[v];
      }
    } else if (a.reset_mask && a.reset_mask[slot(ts)]) {
      h = (floatx16)(0.f);
      c = (floatx16)(0.f);
    }
  };
  if constexpr (SEQ) {
    sr = a.seq_in[slot(ch.t_lo)];
    request_state();
  } else if (a.H0) {
    h = load_block(a.H0 + s0 * H + col0);
    if constexpr (kLstm) c = load_block(a.H0 + (V + s0) * H + col0);
  }
  enter(ch.t_lo);
  if constexpr (HALVES) __syncthreads();
  int number = 0;                             // of products so far

  // A step on P parts.  False: an operand is out of the halves' range, and nothing has changed yet.
  auto step = [&](auto parts, auto& wg, int s) -> bool {
    constexpr int P = decltype(parts)::value;
    constexpr float up = P == 2 ? kSumScale : 1.f, down = 1.f / up;     // the sums are in the scale of the products
    const int64_t ts = ch.t_lo + s;
    if constexpr (SEQ) sr = a.seq_in[slot(min(ts + 1, (int64_t)ch.t_lo + ch.w - 1))];    // of the next step
    int64_t so = -1;                          // state row that leaves after this step
    if constexpr (SEQ) so = a.seq_out[slot(ts)];
    else if (s + 1 == ch.w) so = s0;
    auto scaled = [&](floatx16 v) {
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] *= up;
      return v;
    };
    // The barrier before a product; out: this wave's share of the operand is out of range.
    auto meet = [&](bool out) -> bool {
      ++number;
      if constexpr (P == 2) {
        if (__any(out)) said[number & 1] = number;
      }
      __syncthreads();
      return P == 3 || __builtin_expect(__builtin_amdgcn_readfirstlane(said[number & 1]) != number, 1);
    };
    auto gates = [&](auto links, auto&& to, auto&& small, const Weights& ws, int u, int gstride, int n) {
      product<NG, kHeldOf<NG, SEQ && kLstm, P>, P, decltype(links)::value>(to, small, buf, ws.stream(parts), u * kUnit<P>, gstride * kUnit<P>, n, lane16, wg);
    };
    auto ahead = [&](const Weights& ws, int u, int gstride, int n) {
      fetch_ahead<NG, kHeldOf<NG, SEQ && kLstm, P>>(wg, ws.stream(parts), u * kUnit<P>, gstride * kUnit<P>, n, lane16);
    };
    constexpr std::bool_constant<STACK && P == 3> stack_links;
    // hidden side first: the state is there while the input rows are on their way
    floatx16 acc[4];
    auto hidden = [&](int g) -> floatx16& { return acc[!kLstm && g == 2 ? 3 : g]; };
    auto in = [&](int g) -> floatx16& { return acc[g]; };
    // Small part products in sums of their own (the matrix unit truncates when it adds, and a small sum is truncated by less): on halves those
    // that go into a GRU's tanh (0.92 of the distance from 64 bits; of 120 drawn outputs up to 96 to 256 wide 1.095 of six products' at most
    // without, 0.93 with them; 32 x 100 000 vertices 5.01 -> 5.06 ms, the other cases as before.  All four sums 0.917, and 4.5 % more
    // with sequences, whose registers they overflow), on three parts those of a GRU's folded weights.
    constexpr bool kTanhApart = P == 2 && !kLstm, kApart = P == 3 && FOLD && !kLstm;
    floatx16 sums[kTanhApart ? 2 : kApart ? NG : 1];
    auto small_hidden = [&](int g) -> floatx16& { return kTanhApart && g == 2 ? sums[kTanhApart ? 1 : 0] : hidden(g); };
    auto small_in = [&](int g) -> floatx16& { return kTanhApart && g == 2 ? sums[0] : in(g); };
    if constexpr (kTanhApart || kApart)
#pragma unroll
      for (floatx16& x : sums) x = (floatx16)(0.f);
    turn();
    if (!meet(put_block(parts, h, kActScale))) return false;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (kLstm || g != 2) acc[g] = scaled(load_block(gbias + g * H + col0));
    gates(stack_links, hidden, small_hidden, wsh, uh, gh, kbh);
    auto other_half = [&]() -> bool {         // the other half of the time encoder's input first
      ahead(wsi, ux, gx, kbh);
      int64_t r2 = slot(ts);
      if (a.x2_map) r2 = max(a.x2_map[r2], (int64_t)0);   // an empty slot reads row 0; its output is not used
      turn();
      if (!meet(put_block(parts, load_block(a.X2 + r2 * a.ldx2 + col0), kActScale))) return false;
      gates(std::false_type(), in, small_in, wsi, ux, gx, kbh);
      return true;
    };
    auto input_bias = [&]() {
      if constexpr (!kLstm) acc[2] = scaled(load_block(gbias + 2 * H + col0));
    };
    if constexpr (FOLD) {
      input_bias();
      if constexpr (CAT)
        if (!other_half()) return false;
      // Three parts: the small part products apart, as in the transform that this stands for: a GRU's in sums of their own, an
      // LSTM's (whose registers do not hold four more) for every k-block.
      auto small = [&](int g) -> floatx16& { return kApart ? sums[kApart ? g : 0] : small_in(g); };
      for (int k = 0; k < nchunk; ++k) {
        const int n = min(kbc, nkb0 - k * kbc);
        turn();
        const bool out = stage_x(parts, s, k);
        ahead(wsg, uf + k * kbc, gf, n);
        if (k + 1 < nchunk) request_x(s, k + 1);
        if (!meet(out)) return false;
        gates(std::bool_constant<P == 3 && kLstm>(), in, small, wsg, uf + k * kbc, gf, n);
      }
    } else if constexpr (!STACK) {
      floatx16 z = scaled(load_block(zbias + col0)), zs = (floatx16)(0.f);
      for (int k = 0; k < nchunk; ++k) {
        const int n = min(kbc, nkb0 - k * kbc);
        turn();
        uint4 wz[DZ][P];
        const bool out = stage_x(parts, s, k);
        fetch_ahead<1, DZ>(wz, wsg.stream(parts), (uz + k * kbc) * kUnit<P>, 0, n, lane16);
        if (k + 1 < nchunk) request_x(s, k + 1);
        if (!meet(out)) return false;
        product<1, DZ, P>([&](int) -> floatx16& { return z; }, [&](int) -> floatx16& { return zs; }, buf, wsg.stream(parts),
                          (uz + k * kbc) * kUnit<P>, 0, n, lane16, wz);
      }
      z += zs;
      if (a.act == DGC_ACT_RELU) relu(z);
      if constexpr (CAT)
        if (!other_half()) return false;
      ahead(wsi, ux + kbx - kbh, gx, kbh);
      turn();
      if (!meet(put_block(parts, z, kActScale * down))) return false;
      input_bias();
      gates(std::false_type(), in, small_in, wsi, ux + kbx - kbh, gx, kbh);
    } else {
      ahead(wsi, ux, gx, kbh);
      turn();
      if (!meet(stage_x(parts, s, 0))) return false;
      input_bias();
      gates(stack_links, in, small_in, wsi, ux, gx, kbh);
    }
    if constexpr (kTanhApart) {
      acc[2] += sums[0];
      acc[3] += sums[1];
    } else if constexpr (kApart) {
#pragma unroll
      for (int g = 0; g < NG; ++g) acc[g] += sums[g];
    }
    // requests of the next step go out before this step's stores: memory operations retire in order
    if (mapped) {
      yrow = yrow_next;
      if (s + 1 < ch.w) yrow_next = (int)a.y_map[slot(ts + 1)];
    }
    if (s + 1 < ch.w) {
      ahead(wsh, uh, gh, kbh);
      if constexpr (SEQ) request_state();
      request_x(s + 1, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      if constexpr (kLstm) {                  // i, f, g, o
        const float ig = sigmoid_of(acc[0][v], down), fg = sigmoid_of(acc[1][v], down);
        const float gg = tanh_of(acc[2][v], down), og = sigmoid_of(acc[3][v], down);
        c[v] = fg * c[v] + ig * gg;
        h[v] = og * tanh_of(c[v], 1.f);
      } else {                                // r, z, input part of n, hidden part of n
        const float r = sigmoid_of(acc[0][v], down), zg = sigmoid_of(acc[1][v], down);
        const float n = tanh_of(acc[2][v] + r * acc[3][v], down);
        h[v] = (1.0f - zg) * n + zg * h[v];
      }
    }
    if (valid) {
      const int64_t yr = mapped ? (int64_t)yrow : slot(ts);
      if (yr >= 0) store_block(a.Y + yr * a.ldy + col0, h);
      if (a.HN && so >= 0) {
        store_block(a.HN + so * H + col0, h);
        if constexpr (kLstm) store_block(a.HN + (V + so) * H + col0, c);
      }
    }
    if (s + 1 < ch.w) enter(ts + 1);
    return true;
  };
  int s = 0;
  if constexpr (HALVES) {
    if (wsh.halves_good() && (STACK || wsg.halves_good()) && ((FOLD && !CAT) || wsi.halves_good()) &&
        __builtin_amdgcn_readfirstlane(said[2]) == 0) {
      const std::integral_constant<int, 2> parts;
      uint4 wg[kHeldOf<NG, SEQ && kLstm, 2>][2];
      fetch_ahead<NG, kHeldOf<NG, SEQ && kLstm, 2>>(wg, wsh.stream(parts), uh * kUnit<2>, gh * kUnit<2>, kbh, lane16);
      request_x(0, 0);
      while (s < ch.w && step(parts, wg, s)) ++s;
      if (s == ch.w) return;
    }
  }
  const std::integral_constant<int, 3> parts;
  uint4 wg[kHeldOf<NG, SEQ && kLstm, 3>][3];
  fetch_ahead<NG, kHeldOf<NG, SEQ && kLstm, 3>>(wg, wsh.stream(parts), uh * kUnit<3>, gh * kUnit<3>, kbh, lane16);
  request_x(s, 0);
  for (; s < ch.w; ++s) step(parts, wg, s);
}

// Whether the weights can be folded is known on the device (k_fold), where a graph that was captured before other weights were
// set finds it, too.
template <int KIND, bool SEQ, bool CAT, Input INPUT, int MAXW>
__global__ __launch_bounds__(64 * MAXW, 2) void k_dense_split(DenseArgs a) {
  if constexpr (INPUT == kFolded) {
    if (table_entry(a.fold_bad, 0)) {
      dense_split<KIND, SEQ, CAT, kTransform, false>(a);
      return;
    }
  }
  dense_split<KIND, SEQ, CAT, INPUT, true>(a);
}

// Transforms alone, Y = act(M W^T + b): a workgroup takes a run of the row tiles (ordered by snapshot).  Its waves
// hold the weights, NKB k-blocks of them, and read them again only when the snapshot (and with it the weights)
// changes; the rows of the next tile are on their way while a tile is multiplied.
// kb0: first k-block of this launch (rows wider than the registers hold take a second launch, which goes on from Y).
template <int NKB, int MAXW, bool FIRST>
__global__ __launch_bounds__(64 * MAXW, 2) void k_rows_split(DenseArgs a, int kb0) {
  constexpr int XP = NKB > 2 * MAXW ? 4 : 2;  // k-blocks that a wave requests ahead
  extern __shared__ __align__(16) uint4 lds[];
  const int njb = blockDim.x >> 6;
  const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
  const int jb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nkb_all = (a.K0 + 15) / 16, nkb0 = min(nkb_all - kb0, NKB), col0 = 32 * jb + 4 * half;
  const bool last = kb0 + nkb0 == nkb_all;
  const bool two = a.kb_chunk == 2 * NKB;     // two staging buffers, or one
  uint4* buf = lds + lane;
  uint4* other = buf + (two ? NKB * 3 * kFrag : 0);
  const float* zbias = reinterpret_cast<float*>(lds + a.kb_chunk * 3 * kFrag);
  for (int i = threadIdx.x; i < 32 * njb; i += blockDim.x) const_cast<float*>(zbias)[i] = a.bg[i];
  for (int i = threadIdx.x; i < a.kb_chunk * 3 * kFrag; i += blockDim.x) lds[i] = make_uint4(0, 0, 0, 0);   // k-blocks past the row stay zero
  __syncthreads();
  const int64_t i0 = a.n_row_tiles * blockIdx.x / gridDim.x, i1 = a.n_row_tiles * (blockIdx.x + 1) / gridDim.x;
  float4 xq[XP][2];
  auto kb_of = [&](int q) { return 2 * jb + (q / 2) * 2 * njb + q % 2; };
  auto m_row = [&](const DenseTile& t, const ChunkInfo& ch) {
    return a.M + (ch.row_off0 + (int64_t)t.step * ch.nv + t.v0 + min(l32, t.nrows - 1)) * a.ldm + 16 * kb0 + 4 * half;
  };
  auto request_x = [&](const float* p) {
#pragma unroll
    for (int q = 0; q < XP; ++q) load_x(p, min(kb_of(q), nkb0 - 1), xq[q]);
  };
  if (i0 >= i1) return;
  DenseTile tile = table_entry(a.row_tiles, i0);
  ChunkInfo ch = table_entry(a.chunks, tile.chunk);
  request_x(m_row(tile, ch));
  uint4 w[NKB][3];
  int64_t have = -1;
  for (int64_t i = i0; i < i1; ++i) {
    const int64_t t = ch.t_lo + tile.step;
    const int64_t want = a.wg_step_bytes ? t : 0;
    if (want != have) {
      const WeightStream ws = make_stream(reinterpret_cast<const char*>(a.Wg) + t * a.wg_step_bytes, (int64_t)njb * nkb_all * kUnitBytes);
#pragma unroll
      for (int k = 0; k < NKB; ++k) ws.unit(w[k], lane * 16, (jb * nkb_all + kb0 + k) * kUnitBytes, k < nkb0);
      __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt 0, here: else every tile would wait for the weights, and so for the stores before it
      have = want;
    }
    if (two) { uint4* x = buf; buf = other; other = x; }
    else __syncthreads();
#pragma unroll
    for (int q = 0; q < XP; ++q)
      if (kb_of(q) < nkb0) put_x(buf + kb_of(q) * 3 * kFrag, xq[q]);
    for (int kb = kb_of(XP); kb < nkb0; kb += 2 * njb)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (kb + q < nkb0) {
          float4 x[2];
          load_x(m_row(tile, ch), kb + q, x);
          put_x(buf + (kb + q) * 3 * kFrag, x);
        }
    const int nrows = tile.nrows;
    float* y = a.Y + (t * a.N + ch.v_lo + tile.v0 + l32) * a.ldy + col0;
    if (i + 1 < i1) {
      tile = table_entry(a.row_tiles, i + 1);
      ch = table_entry(a.chunks, tile.chunk);
      request_x(m_row(tile, ch));
    }
    __syncthreads();
    floatx16 z = load_block(zbias + col0);
    if constexpr (!FIRST) {
      if (l32 < nrows) z = load_block(y);
    }
    floatx16 small = (floatx16)(0.f);
#pragma unroll
    for (int k = 0; k < NKB; ++k) {
      uint4 b[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) b[p] = buf[(k * 3 + p) * kFrag];
      six(z, small, w[k], b);
    }
    z += small;
    if (last && a.act == DGC_ACT_RELU) relu(z);
    if (l32 < nrows) store_block(y, z);
  }
}

// W [n_out][n_in] (strides so, si) -> three bf16 parts per fragment: packed[((jb*nkb + kb)*3 + part)*64 + lane] holds of
// row jb*32 + lane%32 the columns 16*kb + 8*p + 4*(lane/32) + e (p = 0, 1; e = 0..3), zero beyond n_in.
// half (or nullptr): behind these, the same as two half-precision parts of 4096 w.
__global__ void k_pack_split(const float* W, int64_t per_w, int64_t so, int64_t si, int32_t n_out, int32_t n_in, int64_t count,
                             uint4* packed, uint4* half) {
  const int nkb = (n_in + 15) / 16;
  const int64_t per = (int64_t)(n_out / 32) * nkb * 64;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= per * count) return;
  const int64_t m = idx / per, i = idx - m * per;
  const int lane = (int)(i & 63);
  const int64_t f = i >> 6;
  const int kb = (int)(f % nkb);
  const int64_t out = (f / nkb) * 32 + (lane & 31);
  const float* w = W + m * per_w + out * so;
  float x[8];
  for (int k = 0; k < 8; ++k) {
    const int col = 16 * kb + 8 * (k / 4) + 4 * (lane >> 5) + k % 4;
    x[k] = col < n_in ? w[col * si] : 0.f;
  }
  uint4 part[3];
  split8(x, part);
  for (int p = 0; p < 3; ++p) packed[((m * per + (f << 6)) * 3 + p * 64) + lane] = part[p];
  if (!half) return;
  uint4 two[2];
  halve8(x, kWeightScale, two);
  for (int p = 0; p < 2; ++p) half[(f << 6) * 2 + p * 64 + lane] = two[p];
}

// A wave a row: *word is set where a row of W is longer than kLongestRow, or not finite.  The error that inputs cut at 2^-36 make of a gate's
// argument is 2^-37 times the length of the row that they are multiplied with, for a transform's times that of the gate's as well; and
// where rows are so long the gates' arguments are, too (above).
constexpr float kLongestRow = 8.f;
__global__ __launch_bounds__(256) void k_halves_word(const float* W, int64_t so, int64_t si, int32_t n_out, int32_t n_in, int32_t* word) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n_out) return;
  float sum = 0.f;
  for (int k = lane; k < n_in; k += 64) {
    const float w = W[row * so + k * si];
    sum = fmaf(w, w, sum);
  }
  for (int m = 1; m < 64; m <<= 1) sum += __shfl_xor(sum, m);
  if (lane == 0 && !(sum <= kLongestRow * kLongestRow)) atomicOr(word, 1);
}

// out[r][k] = sum over s of wih[r][s] wg[s][k], bias[r] = bih[r] + sum over s of wih[r][s] bg[s], both summed in double.
// *bad where the transform would do better: a value is not finite; it is below what three bf16 parts hold (2^-110); or an
// infinity in column k need not make NaN of gate r.  It does, whatever the other columns hold, where a weight is zero or the
// products have both signs, as those of ordinary weights do; products of one sign would leave a saturated gate.
// One workgroup of 64 per (row, 64 columns); column K0 is the bias.
struct FoldArgs { const float *wih, *wg, *bg, *bih; int64_t ld_wih; int32_t S, K0; float *out, *bias; int32_t* bad; };
__global__ __launch_bounds__(64) void k_fold(FoldArgs a) {
  const int r = blockIdx.y, k = blockIdx.x * 64 + threadIdx.x;
  if (k > a.K0) return;
  const float* w = a.wih + r * a.ld_wih;
  double sum = k < a.K0 ? 0.0 : (double)a.bih[r];
  const float* x = k < a.K0 ? a.wg + k : a.bg;
  const int ldx = k < a.K0 ? a.K0 : 1;
  bool up = k == a.K0, down = up;       // some product is positive (zero), negative (zero)
#pragma unroll 8
  for (int s = 0; s < a.S; ++s) {
    const double p = (double)w[s] * (double)x[s * ldx];
    up |= p >= 0.0;
    down |= p <= 0.0;
    sum += p;
  }
  const float f = (float)sum;
  if (k < a.K0) a.out[(int64_t)r * a.K0 + k] = f;
  else a.bias[r] = f;
  const bool small = k < a.K0 && sum != 0.0 && fabs(sum) < 0x1p-110;
  if (!(fabsf(f) <= 3.4028234663852886e38f) || small || !up || !down) atomicOr(a.bad, 1);
}

constexpr size_t kMaxLds = 160 * 1024;
constexpr int kCus = 256;

template <int KIND, bool SEQ, bool CAT, Input INPUT, int MAXW>
bool launch_time(DenseArgs a, int njb, hipStream_t st, std::string* why) {
  const int nkb0 = INPUT == kStack ? 2 * njb : (a.K0 + 15) / 16;
  // a staging buffer holds the state's k-blocks, and of a wider input row what 48 KB take
  a.kb_chunk = std::max(2 * njb, std::min(nkb0, 48 * 1024 / kUnitBytes));
  const size_t lds = (size_t)2 * a.kb_chunk * kUnitBytes + sizeof(float) * 5 * 32 * njb + 4 * sizeof(int32_t);
  static std::atomic<uint64_t> ready{0};
  auto* kernel = &k_dense_split<KIND, SEQ, CAT, INPUT, MAXW>;
  if (!allow_lds(reinterpret_cast<const void*>(kernel), kMaxLds, ready, why)) return false;
  if (a.n_tiles32 > 0) hipLaunchKernelGGL(kernel, (unsigned)a.n_tiles32, 64 * njb, lds, st, a);
  return true;
}

template <int KIND, bool CAT, Input INPUT, int MAXW>
bool launch_seq(const DenseArgs& a, int njb, hipStream_t st, std::string* why) {
  return a.seq_in ? launch_time<KIND, true, CAT, INPUT, MAXW>(a, njb, st, why) : launch_time<KIND, false, CAT, INPUT, MAXW>(a, njb, st, why);
}

template <int KIND, int MAXW>
bool launch_variant(const DenseArgs& a, int njb, hipStream_t st, std::string* why) {
  if (a.input_is_z) return launch_seq<KIND, false, kStack, MAXW>(a, njb, st, why);
  if constexpr (KIND == DGC_TIME_LSTM) {
    if (a.X2) return a.Wf ? launch_seq<KIND, true, kFolded, MAXW>(a, njb, st, why) : launch_seq<KIND, true, kTransform, MAXW>(a, njb, st, why);
  }
  return a.Wf ? launch_seq<KIND, false, kFolded, MAXW>(a, njb, st, why) : launch_seq<KIND, false, kTransform, MAXW>(a, njb, st, why);
}

template <int KIND>
bool launch_kind(const DenseArgs& a, int njb, hipStream_t st, std::string* why) {
  return njb <= 4 ? launch_variant<KIND, 4>(a, njb, st, why) : launch_variant<KIND, 8>(a, njb, st, why);
}

template <int NKB, int MAXW, bool FIRST>
bool launch_rows(DenseArgs a, int kb0, hipStream_t st, std::string* why) {
  const int njb = a.S / 32;
  // eight waves per CU hold 256 registers each; two staging buffers if they then still fit
  const int per_cu = 8 / njb > 0 ? 8 / njb : 1;
  const size_t one = (size_t)NKB * kUnitBytes, bias = sizeof(float) * 32 * njb;
  const bool two = (2 * one + bias) * per_cu <= kMaxLds;
  a.kb_chunk = two ? 2 * NKB : NKB;
  const size_t lds = a.kb_chunk * kUnitBytes + bias;
  static std::atomic<uint64_t> ready{0};
  auto* kernel = &k_rows_split<NKB, MAXW, FIRST>;
  if (!allow_lds(reinterpret_cast<const void*>(kernel), kMaxLds, ready, why)) return false;
  // Runs of tiles: as many as fit the chip at once.  Beside a launch that holds some compute units, two to four times as many
  // while each keeps 16 tiles, so that the other units share what these do not take (64 x 62 500 rows, 256 -> 256, beside the
  // back-propagation through the weights: a training step of 25.04 ms takes 24.64; by itself the launch is 1.5 % slower so, and
  // 1.2 times as many runs as fit are worse than as many).
  const int64_t fit = (int64_t)kCus * per_cu;
  const int64_t runs = fit * (a.shares_chip ? std::max<int64_t>(1, std::min<int64_t>(4, a.n_row_tiles / (16 * fit))) : 1);
  const int64_t grid = std::min(a.n_row_tiles, runs);
  if (grid > 0) hipLaunchKernelGGL(kernel, (unsigned)grid, 64 * njb, lds, st, a, kb0);
  return true;
}

template <int MAXW, bool FIRST>
bool launch_rows_k(const DenseArgs& a, int kb0, hipStream_t st, std::string* why) {
  switch ((std::min((a.K0 + 15) / 16 - kb0, 16) + 1) / 2) {
    case 1: return launch_rows<2, MAXW, FIRST>(a, kb0, st, why);
    case 2: return launch_rows<4, MAXW, FIRST>(a, kb0, st, why);
    case 3: return launch_rows<6, MAXW, FIRST>(a, kb0, st, why);
    case 4: return launch_rows<8, MAXW, FIRST>(a, kb0, st, why);
    case 5: return launch_rows<10, MAXW, FIRST>(a, kb0, st, why);
    case 6: return launch_rows<12, MAXW, FIRST>(a, kb0, st, why);
    case 7: return launch_rows<14, MAXW, FIRST>(a, kb0, st, why);
    case 8: return launch_rows<16, MAXW, FIRST>(a, kb0, st, why);
  }
  return false;
}

template <int MAXW>
bool launch_transform(const DenseArgs& a, hipStream_t st, std::string* why) {
  if (!launch_rows_k<MAXW, true>(a, 0, st, why)) return false;
  return a.K0 <= 256 || launch_rows_k<MAXW, false>(a, 16, st, why);
}

}  // namespace

bool dense_split_supported(int32_t S, int32_t H, int32_t time_kind) {
  return S % 32 == 0 && S >= 32 && S <= 256 && (time_kind == DGC_TIME_NONE || H == S);
}

bool launch_dense_split(const DenseArgs& a, hipStream_t st, std::string* why) {
  const int njb = a.S / 32;
  switch (a.time_kind) {
    case DGC_TIME_NONE: return njb <= 4 ? launch_transform<4>(a, st, why) : launch_transform<8>(a, st, why);
    case DGC_TIME_GRU: return launch_kind<DGC_TIME_GRU>(a, njb, st, why);
    case DGC_TIME_LSTM: return launch_kind<DGC_TIME_LSTM>(a, njb, st, why);
  }
  return false;
}

// Products of a tile and 32 columns, in k-blocks: the gates over the input's width against the transform and the gates over its
// output's.  Any that are saved pay, and the pass of Z through LDS with them: on three parts GRU 96 to 256 wide, 2 saved of 44 to 113: 5 to 10 %;
// LSTM 160 to 256 wide, 1 of 93 and more: 2 %; on halves LSTM 96 and 128 wide, 3 of 48 (8 x 500 vertices 65.1 -> 56.4 us, 8 x 20 000 204 -> 187),
// 5 of 73 (75.7 -> 65.3, 282 -> 261), 2 of 74 (80.0 -> 71.5, 294 -> 279; 16 x 60 000 1515 -> 1464).
bool dense_fold_wanted(int32_t S, int32_t K0, int32_t time_kind) {
  const int ng = time_kind == DGC_TIME_LSTM ? 4 : 3, kbh = S / 16, nkb0 = (K0 + 15) / 16;
  const int saved = nkb0 + ng * kbh - ng * nkb0;
  return saved >= 1;
}

void launch_fold(const float* wih, int64_t ld_wih, const float* wg, const float* bg, const float* bih, int32_t gH, int32_t S, int32_t K0,
                 float* out, float* bias, int32_t* bad, hipStream_t st) {
  hipLaunchKernelGGL(k_fold, dim3((unsigned)(K0 / 64 + 1), (unsigned)gH), 64, 0, st, FoldArgs{wih, wg, bg, bih, ld_wih, S, K0, out, bias, bad});
}

void launch_pack_split(const float* W, int64_t per_w, int64_t out_stride, int64_t in_stride, int32_t n_out, int32_t n_in,
                       int64_t count, void* packed, hipStream_t st) {
  const int64_t total = count * (n_out / 32) * ((n_in + 15) / 16) * 64;
  uint4* const p = static_cast<uint4*>(packed);
  if (total > 0)
    hipLaunchKernelGGL(k_pack_split, (unsigned)((total + 255) / 256), 256, 0, st, W, per_w, out_stride, in_stride, n_out, n_in,
                       count, p, per_w == 0 ? p + 3 * total : nullptr);
  if (total > 0 && per_w == 0)
    hipLaunchKernelGGL(k_halves_word, (unsigned)((n_out + 3) / 4), 256, 0, st, W, out_stride, in_stride, n_out, n_in,
                       reinterpret_cast<int32_t*>(p + 5 * total));
}

}  // namespace dgc
