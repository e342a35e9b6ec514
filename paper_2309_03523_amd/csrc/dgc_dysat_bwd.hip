// Graph-attention + causal temporal self-attention layer, bf16: backward pass (gradients of the
// seven parameter tensors and, if asked for, of the input rows; the cache is a constant).
//
// Stages: (1) temporal attention backward per 2-vertex tile (recomputes P, Q, K, V and the
// probabilities; writes dU, dQ, dK, dV and the position-table gradient), (2) dW_q, dW_k, dW_v as
// products over all rows, (3) graph attention row pass (gradients of the destination logits),
// (4) reverse-edge pass (gradients of both projections of every vertex, of a_src and a_dst),
// (5) dW of the projection from the input and the cache rows, (6) dX.  Every reduction over rows goes
// through per-wave (per-workgroup) slots that are added in slot order: no floating-point atomics.
#include "dgc_dysat_dev.h"

namespace dgc {
using namespace dysat;
namespace {

__global__ void k_fill_f32(float* p, float v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

struct TemporalBwdArgs {
  const ChunkInfo* chunks; int32_t n_chunks;
  const int64_t* tile_ptr; int64_t n_tiles;
  int64_t N; int32_t T;
  const float* U; const float* pos;
  const uint4 *Wq, *Wk, *Wv;       // row-operand fragments
  const uint16_t* Y; int64_t ldy;          // with target: dY = scale * (Y - target)
  const uint16_t* dY; int64_t lddy;        // or the upstream gradient itself
  const uint16_t* target; int64_t ldt;
  float scale;
  uint16_t *dQ, *dK, *dV;
  float* loss_partial;   // [gridDim.x * waves per block]
};

// value of lane l^32
__device__ __forceinline__ float xor32(float x, int hh) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(hh ? r[0] : r[1]);
}

// raw 16-byte pieces of the upstream gradient (or of Y and the target) of features [off, off+8)
struct DyRaw { uint4 a, b; };

__device__ __forceinline__ DyRaw load_dy_raw(const TemporalBwdArgs& a, int64_t row, int off, bool valid) {
  DyRaw r;
  r.a = make_uint4(0, 0, 0, 0);
  r.b = r.a;
  if (valid) {
    if (a.dY) {
      r.a = *reinterpret_cast<const uint4*>(a.dY + row * a.lddy + off);
    } else {
      r.a = *reinterpret_cast<const uint4*>(a.Y + row * a.ldy + off);
      r.b = *reinterpret_cast<const uint4*>(a.target + row * a.ldt + off);
    }
  }
  return r;
}
// -> dL/dY of those 8 features; adds (Y - target)^2 to sq (rows that are not valid give zeros)
__device__ __forceinline__ void dy_from_raw(const TemporalBwdArgs& a, const DyRaw& r, float* out, float& sq) {
  unpack8(r.a, out);
  if (!a.dY) {
    float g[8];
    unpack8(r.b, g);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float d = out[i] - g[i];
      out[i] = a.scale * d;
      sq += d * d;
    }
  }
}

constexpr int kFragsPerW = 4 * 8 * 64;   // uint4 fragments of one 128 x 128 weight

__device__ __forceinline__ void stage_weights(uint4* lds, const uint4* w0, const uint4* w1, const uint4* w2) {
  for (int i = threadIdx.x; i < kFragsPerW; i += blockDim.x) {
    lds[i] = w0[i];
    lds[kFragsPerW + i] = w1[i];
    lds[2 * kFragsPerW + i] = w2[i];
  }
  __syncthreads();
}

// One head of a row-layout tensor in column layout: out[c] = rows 16 c .. of the lane's feature, zero for the
// features that sel does not take.  Exact: a product with 0 and 1.
__device__ __forceinline__ void to_columns(bf16x8 x, bf16x8 sel, bf16x8* out) {
  floatx16 t = {};
  t = mfma(x, sel, t);
  out[0] = pack8v(t, 0);
  out[1] = pack8v(t, 8);
}

// Temporal self-attention, backward, first half: dQ, dK, dV (and the loss).  The workgroup stages
// W_q, W_k, W_v in LDS; each of its waves then walks 2-vertex tiles with a grid stride.  Per tile
// it recomputes P, Q, K, V.  Per head, the "query-major" score block
// (lane = query row, registers = key steps) gives the probabilities p, delta = sum_r p dp and dS;
// dQ needs dS in that orientation, dK and dV need dS and p "key-major" (lane = key row,
// registers = query steps): those are obtained by one product each with a selection operand
// (a 16 x 16 transpose per vertex on the matrix core, exact for the hi and the lo part); so are Q, K and dY in
// column layout, which the three products take as their other operand.  A head's 16 dims go to memory (bf16) before the
// next head is begun.
// All operands are hi + lo pairs.
// Bound by the vector units (softmax, splits) and the matrix cores side by side (the memory's share is 1.5 of
// 2.9 ms at 4 000 000 rows): at most 256 registers, so that a SIMD has two waves to overlap them
// (4.2 ms with one wave of 392 registers, which held Q, K by a second set of products and the three results).
// WIDE (one vertex per tile, windows of up to 32 snapshots): a lane's 16 score registers are all
// keys of its own vertex, the transposes are 32 x 32 (two selection products, one per half of the
// keys), and the three final products contract over the two halves of the keys / queries instead
// of over two vertices.
template <bool WIDE>
__global__ __launch_bounds__(512) void k_temporal_bwd(TemporalBwdArgs a) {
  extern __shared__ uint4 wlds[];
  stage_weights(wlds, a.Wq, a.Wk, a.Wv);
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6, wave = threadIdx.x >> 6;
  const int hh = lane >> 5;
  float sq = 0.f;
  constexpr int NP = WIDE ? 16 : 8, NH = NP / 8;
  // B operands: element p of lane (j, hh) is 1 where 16 c + 8 (p/4) + 4 hh + p%4 == j
  bf16x8 sel[2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int p = 0; p < 8; ++p)
      sel[c][p] = 16 * c + 8 * (p >> 2) + 4 * hh + (p & 3) == (lane & 31) ? (__bf16)1.0f : (__bf16)0.0f;
  for (int64_t tile = (int64_t)blockIdx.x * nw + wave; tile < a.n_tiles; tile += (int64_t)gridDim.x * nw) {
    const TileRow r = tile_row<WIDE>(a.chunks, a.n_chunks, a.tile_ptr, tile, a.N, lane);
    const uint32_t m_vert[2] = {r.a == 0 ? 0xffffffffu : 0u, r.a == 1 ? 0xffffffffu : 0u};
    bf16x8 pf[8], pl[8];
    load_p_frags<true>(a.U, a.pos, r, hh, pf, pl);
#pragma unroll 1
    for (int jb = 0; jb < 4; ++jb) {
      DyRaw raw[2];
      raw[0] = load_dy_raw(a, r.row, 2 * jb * 16 + 8 * hh, r.valid);
      raw[1] = load_dy_raw(a, r.row, (2 * jb + 1) * 16 + 8 * hh, r.valid);
      bf16x8 kh[2], kl[2], qh[2], ql[2], vh[2], vl[2];
      {
        floatx16 q = {}, k = {}, v = {};
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) {
          const int fi = (jb * 8 + kb) * 64 + lane;
          q = mfma2b(as_frag(wlds[fi]), pf[kb], pl[kb], q);
          k = mfma2b(as_frag(wlds[kFragsPerW + fi]), pf[kb], pl[kb], k);
          v = mfma2b(as_frag(wlds[2 * kFragsPerW + fi]), pf[kb], pl[kb], v);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          split8v(q, 8 * c, qh[c], ql[c]);
          split8v(k, 8 * c, kh[c], kl[c]);
          split8v(v, 8 * c, vh[c], vl[c]);
        }
      }
      // dL/dY of features [32 jb, 32 jb + 32), head c in row-layout order (requested before the products above)
      bf16x8 dyh[2], dyl[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        float d8[8];
        dy_from_raw(a, raw[c], d8, sq);
        bf16x8 h, l;
        split8(d8, h, l);
        dyh[c] = as_frag(head_order(__builtin_bit_cast(uint4, h)));
        dyl[c] = as_frag(head_order(__builtin_bit_cast(uint4, l)));
      }
#pragma unroll
      for (int hd = 0; hd < 2; ++hd) {
        bf16x8 dsth[NH], dstl[NH], prh[NH], prl[NH];
        {
          floatx16 st = {}, dpt = {};
          st = mfma3(kh[hd], kl[hd], qh[hd], ql[hd], st);         // [key row][query row]
          dpt = mfma3(vh[hd], vl[hd], dyh[hd], dyl[hd], dpt);
          float pr[NP], dst[NP];
          float mx = -INFINITY;
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            const int rk = 8 * (p >> 2) + 4 * hh + (p & 3);
            pr[p] = keep_or_ninf(rk <= r.s, 0.25f * (WIDE ? st[p] : pick_half(st, p, m_vert[0], m_vert[1])));
            mx = fmaxf(mx, pr[p]);
          }
          mx = fmaxf(mx, xor32(mx, hh));
          float sum = 0.f;
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            pr[p] = __expf(pr[p] - mx);
            sum += pr[p];
          }
          sum += xor32(sum, hh);
          const float inv = 1.f / sum;
          float delta = 0.f;
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            pr[p] *= inv;
            dst[p] = WIDE ? dpt[p] : pick_half(dpt, p, m_vert[0], m_vert[1]);
            delta += pr[p] * dst[p];
          }
          delta += xor32(delta, hh);
#pragma unroll
          for (int p = 0; p < NP; ++p) dst[p] = 0.25f * pr[p] * (dst[p] - delta);
#pragma unroll
          for (int c = 0; c < NH; ++c) {
            split8(dst + 8 * c, dsth[c], dstl[c]);
            split8(pr + 8 * c, prh[c], prl[c]);
          }
        }
        // d[f][row] = sum over av (the two vertices, or, WIDE, the two halves of the window's steps) of
        // x[f][steps of av] b[steps of av][row]; dims of this head: registers 8 hd ..
        auto product = [&](bf16x8 xh, bf16x8 xl, const bf16x8* bh, const bf16x8* bl, uint16_t* out) {
          bf16x8 xth[2], xtl[2];
          to_columns(xh, sel[hd], xth);
          to_columns(xl, sel[hd], xtl);
          floatx16 d = {};
#pragma unroll
          for (int av = 0; av < 2; ++av) {
            const uint32_t mv = WIDE ? 0xffffffffu : m_vert[av];
            d = mfma3(xth[av], xtl[av], and_mask(bh[av], mv), and_mask(bl[av], mv), d);
          }
          const uint4 o = head_order(__builtin_bit_cast(uint4, pack8v(d, 8 * hd)));
          if (r.valid) *reinterpret_cast<uint4*>(out + r.row * kS + jb * 32 + 16 * hd + 8 * hh) = o;
        };
        // key-major copy of one part: T[i = query row][j = key row], the query rows of vertex (half) c in bt[c]
        auto key_major = [&](const bf16x8* b, bf16x8* bt) {
          floatx16 t = {};
          if (WIDE) {
#pragma unroll
            for (int c = 0; c < NH; ++c) t = mfma(b[c], sel[c], t);
          } else {
            const uint4 s0 = __builtin_bit_cast(uint4, sel[0]), s1 = __builtin_bit_cast(uint4, sel[1]);
            t = mfma(b[0], as_frag(make_uint4(s0.x | s1.x, s0.y | s1.y, s0.z | s1.z, s0.w | s1.w)), t);   // j % 16
          }
          bt[0] = pack8v(t, 0);
          bt[1] = pack8v(t, 8);
        };
        bf16x8 bh[2], bl[2];
        bh[0] = dsth[0]; bh[1] = dsth[NH - 1];
        bl[0] = dstl[0]; bl[1] = dstl[NH - 1];
        product(kh[hd], kl[hd], bh, bl, a.dQ);
        key_major(dsth, bh);
        key_major(dstl, bl);
        product(qh[hd], ql[hd], bh, bl, a.dK);
        key_major(prh, bh);
        key_major(prl, bl);
        product(dyh[hd], dyl[hd], bh, bl, a.dV);
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
  if (lane == 0) a.loss_partial[blockIdx.x * nw + wave] = sq;
}

// Temporal self-attention, backward, second half: dP = dQ W_q + dK W_k + dV W_v from the stored
// gradients, dU = dP * ELU'(U), c = du . u per head for the passes over the non-zeros, and the gradient of the
// position table (column sums of dP per
// snapshot).  Rows are the covered vertices of the snapshots in use, 32 per tile; the transposed
// weights are staged in LDS; dQ/dK/dV row fragments are B operands as they come from memory, a quarter of the row at a
// time with the next two quarters on their way (also those of the next tile).  They are loaded whether or not the row
// counts and masked when used: loads under a condition are waited for one by one.
// Every wave sums dP over its tiles in registers (lane = row slot) and, when the snapshot
// changes, adds the 32 row slots and writes the sums to its own slot of the scratch buffer.
// Bound by memory: 6.3 GB in 1.72 ms for 4 000 000 rows (2.13 ms with three conditional loads in flight).
struct TemporalBwd2Args {
  const int32_t* used_t; int32_t n_used; int64_t N; int32_t T;
  const int32_t* owner;
  const float* U;
  const uint4 *WqT, *WkT, *WvT;
  const uint16_t *dQ, *dK, *dV;
  uint16_t* dU;
  float* c;              // [T*N][16]: c^h = du^h . u^h of the graph attention in the first 8
  float* dpos_partial;   // [gridDim.x * waves per block][T][128], zero on entry
};

__device__ __forceinline__ void flush_dpos(float* slot, int t, int lane, floatx16* acc) {
  const int n = lane & 31, hh = lane >> 5;
#pragma unroll
  for (int ib = 0; ib < 4; ++ib) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float x = acc[ib][v];
      x += __shfl_xor(x, 1); x += __shfl_xor(x, 2); x += __shfl_xor(x, 4); x += __shfl_xor(x, 8); x += __shfl_xor(x, 16);
      acc[ib][v] = x;
    }
    if (n == 0) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4* p = reinterpret_cast<float4*>(slot + (int64_t)t * kS + ib * 32 + 8 * g + 4 * hh);
        float4 o = *p;
        o.x += acc[ib][4 * g]; o.y += acc[ib][4 * g + 1]; o.z += acc[ib][4 * g + 2]; o.w += acc[ib][4 * g + 3];
        *p = o;
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[ib][v] = 0.f;
  }
}

__global__ __launch_bounds__(512) void k_temporal_bwd2(TemporalBwd2Args a) {
  extern __shared__ uint4 wlds[];
  stage_weights(wlds, a.WqT, a.WkT, a.WvT);
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6, wave = threadIdx.x >> 6;
  const int n = lane & 31, hh = lane >> 5;
  const int64_t tiles_per_t = (a.N + 31) / 32, n_tiles = tiles_per_t * a.n_used;
  const int64_t gw = (int64_t)blockIdx.x * nw + wave, n_gw = (int64_t)gridDim.x * nw;
  const int64_t per = (n_tiles + n_gw - 1) / n_gw;
  const int64_t tile0 = gw * per, tile1 = min(n_tiles, tile0 + per);
  float* slot = a.dpos_partial + gw * a.T * kS;
  floatx16 dpos[4] = {};
  int cur_t = -1;
  struct Quarter { uint4 q[2], k[2], v[2]; };      // a quarter of the lane's rows
  auto request = [&](int64_t row, int part, Quarter& x) {
    const int64_t o = row * kS + 32 * part + 8 * hh;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      x.q[i] = *reinterpret_cast<const uint4*>(a.dQ + o + 16 * i);
      x.k[i] = *reinterpret_cast<const uint4*>(a.dK + o + 16 * i);
      x.v[i] = *reinterpret_cast<const uint4*>(a.dV + o + 16 * i);
    }
  };
  int64_t row = 0, next_row = 0;
  auto row_of = [&](int64_t tile) {      // always a row of the tensors
    return (int64_t)a.used_t[tile / tiles_per_t] * a.N + min(a.N - 1, (tile % tiles_per_t) * 32 + n);
  };
  Quarter x, y;
  if (tile0 < tile1) {
    next_row = row_of(tile0);
    request(next_row, 0, x);
    request(next_row, 1, y);
  }
  for (int64_t tile = tile0; tile < tile1; ++tile) {
    const int32_t t = a.used_t[tile / tiles_per_t];
    if (t != cur_t) {
      if (cur_t >= 0) flush_dpos(slot, cur_t, lane, dpos);
      cur_t = t;
    }
    row = next_row;
    const bool ok = (tile % tiles_per_t) * 32 + n < a.N && a.owner[row] >= 0;
    const uint32_t keep = ok ? 0xffffffffu : 0u;     // a row no chunk covers was never written
    floatx16 dP[4] = {};
    auto add = [&](const Quarter& g, int part) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const bf16x8 uq = and_mask(as_frag(g.q[i]), keep), uk = and_mask(as_frag(g.k[i]), keep), uv = and_mask(as_frag(g.v[i]), keep);
#pragma unroll
        for (int ib = 0; ib < 4; ++ib) {
          const int fi = (ib * 8 + 2 * part + i) * 64 + lane;
          dP[ib] = mfma(as_frag(wlds[fi]), uq, dP[ib]);
          dP[ib] = mfma(as_frag(wlds[kFragsPerW + fi]), uk, dP[ib]);
          dP[ib] = mfma(as_frag(wlds[2 * kFragsPerW + fi]), uv, dP[ib]);
        }
      }
    };
    add(x, 0);
    request(row, 2, x);
    add(y, 1);
    request(row, 3, y);
    const bool more = tile + 1 < tile1;
    if (more) next_row = row_of(tile + 1);
    add(x, 2);
    if (more) request(next_row, 0, x);
    add(y, 3);
    if (more) request(next_row, 1, y);
    float c[kHeads];
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) {
      dpos[ib] += dP[ib];
#pragma unroll
      for (int hd = 0; hd < 2; ++hd) {
        const int64_t o = row * kS + ib * 32 + 16 * hd;
        const float4 u0 = *reinterpret_cast<const float4*>(a.U + o + 4 * hh);
        const float4 u1 = *reinterpret_cast<const float4*>(a.U + o + 8 + 4 * hh);
        const floatx16& p = dP[ib];
        const uint2 d0 = pack4(p[8 * hd] * delu(u0.x), p[8 * hd + 1] * delu(u0.y), p[8 * hd + 2] * delu(u0.z), p[8 * hd + 3] * delu(u0.w));
        const uint2 d1 = pack4(p[8 * hd + 4] * delu(u1.x), p[8 * hd + 5] * delu(u1.y), p[8 * hd + 6] * delu(u1.z), p[8 * hd + 7] * delu(u1.w));
        const uint4 out = head_order(make_uint4(d0.x, d0.y, d1.x, d1.y));
        if (ok) *reinterpret_cast<uint4*>(a.dU + o + 8 * hh) = out;
        // of the values as stored: what the passes over the non-zeros read
        const float part = bf_lo(d0.x) * u0.x + bf_hi(d0.x) * u0.y + bf_lo(d0.y) * u0.z + bf_hi(d0.y) * u0.w +
                           bf_lo(d1.x) * u1.x + bf_hi(d1.x) * u1.y + bf_lo(d1.y) * u1.z + bf_hi(d1.y) * u1.w;
        c[2 * ib + hd] = part + xor32(part, hh);
      }
    }
    if (ok)
      *reinterpret_cast<float4*>(a.c + row * 16 + 4 * hh) =
          hh ? make_float4(c[4], c[5], c[6], c[7]) : make_float4(c[0], c[1], c[2], c[3]);
  }
  if (cur_t >= 0) flush_dpos(slot, cur_t, lane, dpos);
}

// ---------------------------------------------------------------------------------------------
// Weight gradients  dW_G[out][in] = sum over rows of G[row][out] * A[row][in]  for NG tensors G
// sharing one A (A = the rows of a bf16 tensor, or P = ELU(U) + pos recomputed from U).  Rows are
// the vertices of the snapshots in use, 32 per tile.  A workgroup walks a contiguous
// range of tiles.  Both operands need the
// row index as contraction index, i.e. column layout: obtained from natural row fragments with
// the selection products described above.  Each of the eight waves does that for a part of the tile, 32 columns of A
// (waves 0..3) or of every G (4..7), and leaves the fragments in one of two LDS buffers for all; then wave w adds
// output rows [32 (w%4), +32) x input columns [64 (w/4), +64) of every dW_G.  The next tile is on its way from memory.
// Bound by memory: for 4 000 000 rows dW_q, dW_k, dW_v 5.1 GB in 1.31 ms, and dW from the input and the cache rows (one
// launch, blockIdx.y) 4.1 GB in 0.88 ms; with every wave converting what it multiplies, 2.06 and 2 x 0.80 ms.  (Two tiles
// ahead: the registers spill.)
struct DwBf16Args {
  const int32_t* used_t; int32_t n_used; int64_t N;
  const int32_t* owner; int32_t covered_only;
  const uint16_t* A; int64_t lda;        // bf16 rows, or
  const float* Uf; const float* pos;     // A = ELU(Uf) + pos (fp32 rows of pitch 128), carried as hi + lo
  const uint16_t* G[3];
  float* partial;      // [n_groups][NG][128][128]
  int32_t n_groups;
};

struct DwRow {
  int64_t row;
  int32_t k;
  bool ok;
};

__device__ __forceinline__ DwRow dw_row(const DwBf16Args& a, bool covered_only, int64_t tile, int64_t tiles_per_t, int n) {
  DwRow r;
  r.k = (int32_t)(tile / tiles_per_t);
  const int64_t v = (tile % tiles_per_t) * 32 + n;
  const bool valid = v < a.N;
  r.row = (int64_t)a.used_t[r.k] * a.N + (valid ? v : a.N - 1);    // always a row of the tensors
  r.ok = valid && (!covered_only || a.owner[r.row] >= 0);       // rows that do not count are zeroed when used
  return r;
}

__device__ __forceinline__ uint4 keep_if(bool ok, uint4 u) {
  return make_uint4(ok ? u.x : 0u, ok ? u.y : 0u, ok ? u.z : 0u, ok ? u.w : 0u);
}

template <int NG, bool AU>
constexpr int dw_frags() { return 8 * (AU ? 2 : 1) + 8 * NG; }     // of a tile: A (hi, and lo if AU), then the G

// second: the arguments of the workgroups of blockIdx.y = 1
template <int NG, bool AU>
__global__ __launch_bounds__(512) void k_dw_bf16(DwBf16Args a, DwBf16Args second) {
  constexpr int NA = AU ? 2 : 1, kFrags = dw_frags<NG, AU>();
  const bool other = !AU && blockIdx.y;
  const uint16_t* const A = other ? second.A : a.A;
  const uint16_t* const G0 = other ? second.G[0] : a.G[0];
  const int64_t lda = other ? second.lda : a.lda;
  const bool covered_only = other ? second.covered_only : a.covered_only;
  float* const partial = other ? second.partial : a.partial;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ob = wave & 3, ih = wave >> 2;
  const int n = lane & 31, hh = lane >> 5;
  const int64_t tiles_per_t = (a.N + 31) / 32, n_tiles = tiles_per_t * a.n_used;
  const int64_t per = (n_tiles + a.n_groups - 1) / a.n_groups;
  const int64_t tile0 = (int64_t)blockIdx.x * per, tile1 = min(n_tiles, tile0 + per);
  const bf16x8 sel0 = sel_frag(0, lane), sel1 = sel_frag(1, lane);
  floatx16 acc[NG][2] = {};
  extern __shared__ uint4 dw_lds[];    // [2][kFrags][64], then (AU) the position rows of the snapshots of the range
  float* pos_lds = reinterpret_cast<float*>(dw_lds + 2 * kFrags * 64);
  const int32_t k0 = (int32_t)(tile0 / tiles_per_t);
  if (AU) {
    if (tile0 < tile1) {
      const int32_t nk = (int32_t)((tile1 - 1) / tiles_per_t) - k0 + 1;
      for (int i = threadIdx.x; i < nk * kS; i += 512) pos_lds[i] = a.pos[(int64_t)a.used_t[k0 + i / kS] * kS + (i % kS)];
    }
    __syncthreads();
  }
  struct Raw { uint4 r0, r1, r2, r3, r4, r5; int32_t k; bool ok; };     // the lane's pieces of a tile as they come from memory
  auto request = [&](int64_t tile, Raw& q) {
    const DwRow rw = dw_row(a, covered_only, tile, tiles_per_t, n);
    q.k = rw.k;
    q.ok = rw.ok;
    const int off = 32 * ob + 8 * hh;
    auto at = [&](const uint16_t* p, int64_t ld, int c) { return *reinterpret_cast<const uint4*>(p + rw.row * ld + off + 16 * c); };
    if (wave >= 4) {
      q.r0 = at(G0, kS, 0);
      q.r1 = at(G0, kS, 1);
      if constexpr (NG == 3) {
        q.r2 = at(a.G[1], kS, 0);
        q.r3 = at(a.G[1], kS, 1);
        q.r4 = at(a.G[2], kS, 0);
        q.r5 = at(a.G[2], kS, 1);
      }
    } else if constexpr (AU) {
      const uint4* u = reinterpret_cast<const uint4*>(a.Uf + rw.row * kS + off);
      q.r0 = u[0];
      q.r1 = u[1];
      q.r2 = u[4];
      q.r3 = u[5];
    } else {
      q.r0 = at(A, lda, 0);
      q.r1 = at(A, lda, 1);
    }
  };
  auto columns = [&](bf16x8 x0, bf16x8 x1, uint4* out) {     // the fragments of both halves of the rows
    floatx16 tr = {};
    tr = mfma(x0, sel0, tr);
    tr = mfma(x1, sel1, tr);
    out[0] = __builtin_bit_cast(uint4, pack8v(tr, 0));
    out[64] = __builtin_bit_cast(uint4, pack8v(tr, 8));
  };
  auto convert = [&](const Raw& q, uint4* buf) {
    buf += lane;
    auto kept = [&](uint4 u) { return as_frag(keep_if(q.ok, u)); };
    if (wave >= 4) {
      uint4* g = buf + (8 * NA + 2 * ob) * 64;
      columns(kept(q.r0), kept(q.r1), g);
      if constexpr (NG == 3) {
        columns(kept(q.r2), kept(q.r3), g + 8 * 64);
        columns(kept(q.r4), kept(q.r5), g + 16 * 64);
      }
    } else if constexpr (AU) {
      const float* pp = pos_lds + (q.k - k0) * kS + 32 * ob + 8 * hh;
      auto part = [&](uint4 ua, uint4 ub, const float* pp, bf16x8& xh, bf16x8& xl) {
        const float4 u0 = __builtin_bit_cast(float4, ua), u1 = __builtin_bit_cast(float4, ub);
        const float4 p0 = *reinterpret_cast<const float4*>(pp), p1 = *reinterpret_cast<const float4*>(pp + 4);
        float x[8];
        x[0] = elu(u0.x) + p0.x; x[1] = elu(u0.y) + p0.y; x[2] = elu(u0.z) + p0.z; x[3] = elu(u0.w) + p0.w;
        x[4] = elu(u1.x) + p1.x; x[5] = elu(u1.y) + p1.y; x[6] = elu(u1.z) + p1.z; x[7] = elu(u1.w) + p1.w;
        split8(x, xh, xl);
        xh = kept(__builtin_bit_cast(uint4, xh));
        xl = kept(__builtin_bit_cast(uint4, xl));
      };
      bf16x8 xh0, xl0, xh1, xl1;
      part(q.r0, q.r1, pp, xh0, xl0);
      part(q.r2, q.r3, pp + 16, xh1, xl1);
      columns(xh0, xh1, buf + 2 * ob * 64);
      columns(xl0, xl1, buf + (8 + 2 * ob) * 64);
    } else {
      columns(kept(q.r0), kept(q.r1), buf + 2 * ob * 64);
    }
  };
  auto multiply = [&](const uint4* buf) {
    buf += lane;
    bf16x8 at[NA][2][2];
#pragma unroll
    for (int p = 0; p < NA; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) at[p][i >> 1][i & 1] = as_frag(buf[(8 * p + 4 * ih + i) * 64]);
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      const bf16x8 g0 = as_frag(buf[(8 * NA + 8 * gi + 2 * ob) * 64]), g1 = as_frag(buf[(8 * NA + 8 * gi + 2 * ob + 1) * 64]);
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int p = 0; p < NA; ++p) {
          acc[gi][ib] = mfma(g0, at[p][ib][0], acc[gi][ib]);
          acc[gi][ib] = mfma(g1, at[p][ib][1], acc[gi][ib]);
        }
    }
  };
  Raw q;
  if (tile0 < tile1) request(tile0, q);
  uint4* buf = dw_lds;
  // a buffer is written again only after the barrier of the tile between, which every wave reaches after its products
  for (int64_t tile = tile0; tile < tile1; ++tile) {
    convert(q, buf);
    if (tile + 1 < tile1) request(tile + 1, q);
    __syncthreads();
    multiply(buf);
    buf = buf == dw_lds ? dw_lds + kFrags * 64 : dw_lds;
  }
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    float* out = partial + ((int64_t)blockIdx.x * NG + gi) * kS * kS;
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int vv = 0; vv < 16; ++vv)
        out[(ob * 32 + 8 * (vv >> 2) + 4 * hh + (vv & 3)) * kS + (2 * ih + ib) * 32 + n] = acc[gi][ib][vv];
  }
}

// out[e] = scale * sum over slots of partial[slot * stride + e].  A block of 1024 threads covers 64
// elements x 16 slot groups (group g adds slots g, g+16, ... in ascending order); the 16 group
// sums are then added in group order, so the result does not depend on the launch.
__global__ __launch_bounds__(1024) void k_reduce_slots(const float* partial, int64_t n_slots, int64_t stride,
                                                       int64_t n_elem, float scale, float* out) {
  __shared__ float sh[16][64];
  const int el = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + el;
  float s = 0.f;
  if (e < n_elem) {
    // eight of the group's slots requested together (past its last: that one, not added): 16 384 elements of 512 slots
    // took 36 us with every load waited for
    constexpr int kAhead = 8;
    for (int64_t k0 = grp; k0 < n_slots; k0 += 16 * kAhead) {
      float v[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) v[k] = partial[min(k0 + 16 * k, n_slots - 1) * stride + e];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) s += k0 + 16 * k < n_slots ? v[k] : 0.f;
    }
  }
  sh[grp][el] = s;
  __syncthreads();
  if (grp == 0 && e < n_elem) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) t += sh[g][el];
    out[e] = scale * t;
  }
}

// ---------------------------------------------------------------------------------------------
// Graph attention backward, row pass: for every covered row i, with c_i^h = du_i^h . u_i^h,
// d s_dst_i^h = sum_j dpre_ij^h,  dpre = alpha (du_i^h . z_j^h - c_i^h) LeakyReLU'(e_ij^h).
// Lane = (neighbour slot lane/8, head lane%8): eight neighbours at a time, each lane reads its
// head's 32-byte slice of the neighbour's z row and does the 16-dim dot product on its own.  Two neighbours per slot
// are a batch, and the next batch is requested before the current one is used; the next row's column ids and own
// values before the current row.
// Bound by the gathers' bytes: 2.7 ms for 16 snapshots of 250 000 vertices and 3 million non-zeros (one batch at a
// time, c computed here from rows of U, split rows in a launch of their own: 2.74 and 0.44 ms).
// Rows longer than long_nnz are cut into parts (one wavefront each, in the same launch and begun first) whose sums a
// merge kernel adds in part order.
constexpr int kLongRec = 144;    // floats per scratch record of a part of a split row (forward, row pass)

struct GatBwdRowsArgs {
  GraphDev g;
  const Segment* segs;
  const int32_t* work; int64_t n_work;
  const int32_t* work_long; int64_t n_long;
  int32_t long_nnz, part_nnz;
  float* long_partial;
  const uint16_t* zX; const uint16_t* zC;
  const float* sX; const float* sC;
  const uint16_t* dU;
  const float* c;    // [T*N][16], the first 8
  const float* lse;
  float4* st2;    // [T*N][8]: per head (s_dst, lse, c, d s_dst): what the reverse-edge pass needs of a row
};

struct RowOwn { uint4 du[2]; float c, sd, lse; };    // what a lane keeps about its own row and head

__device__ __forceinline__ RowOwn row_own(const GatBwdRowsArgs& a, int64_t row, int h) {
  RowOwn o;
  const uint4* p = reinterpret_cast<const uint4*>(a.dU + row * kS + 16 * h);
  o.du[0] = p[0];
  o.du[1] = p[1];
  o.c = a.c[row * 16 + h];
  o.sd = a.sX[row * 16 + 8 + h];
  o.lse = a.lse[row * 8 + h];
  return o;
}

constexpr int kRowBatch = 2;    // neighbours per slot and batch
struct RowBatch { uint4 z[kRowBatch][2]; float s[kRowBatch]; };

// sum_j dpre_ij^h over n stored non-zeros of row i, from `first` (the same in every slot); ids: column id of non-zero
// `lane` of them
__device__ __forceinline__ float gat_bwd_row_range(const GatBwdRowsArgs& a, const Segment& s, const int32_t* first,
                                                   int64_t base, const RowOwn& o, int n, int32_t ids, int lane) {
  const int slot = lane >> 3, h = lane & 7;
  float dsd = 0.f, du[16];
  unpack8(o.du[0], du);
  unpack8(o.du[1], du + 8);
  int32_t ahead = 64 + lane < n ? first[64 + lane] : 0;
  auto request = [&](int k, RowBatch& b) {
    if (k > 0 && (k & 63) == 0) {
      ids = ahead;
      ahead = k + 64 + lane < n ? first[k + 64 + lane] : 0;
    }
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      const int i = k + 8 * u + slot;
      const int32_t j = __shfl(ids, i & 63);
      b.z[u][0] = make_uint4(0, 0, 0, 0);
      b.z[u][1] = b.z[u][0];
      b.s[u] = -INFINITY;     // no weight
      if (i < n) {
        const bool in = j >= s.v_lo && j < s.v_hi;
        const uint4* zp = reinterpret_cast<const uint4*>((in ? a.zX : a.zC) + (base + j) * kS + 16 * h);
        b.z[u][0] = zp[0];
        b.z[u][1] = zp[1];
        b.s[u] = *(in ? a.sX + (base + j) * 16 + h : a.sC + (base + j) * 8 + h);
      }
    }
  };
  auto use = [&](const RowBatch& b) {
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      float z[16];
      unpackh8(b.z[u][0], z);      // half precision
      unpackh8(b.z[u][1], z + 8);
      const float e = o.sd + b.s[u];
      const float al = __expf(lrelu(e) - o.lse);
      float da = 0.f;
#pragma unroll
      for (int d = 0; d < 16; ++d) da += du[d] * z[d];
      dsd += al * (da - o.c) * (e > 0.f ? 1.f : kSlope);
    }
  };
  RowBatch x, y;
  constexpr int kStep = 8 * kRowBatch;
  if (n > 0) {
    request(0, x);
    for (int k = 0;; k += 2 * kStep) {
      const bool more = k + kStep < n;
      if (more) request(k + kStep, y);
      use(x);
      if (!more) break;
      const bool again = k + 2 * kStep < n;
      if (again) request(k + 2 * kStep, x);
      use(y);
      if (!again) break;
    }
  }
  dsd += __shfl_xor(dsd, 8);
  dsd += __shfl_xor(dsd, 16);
  dsd += __shfl_xor(dsd, 32);
  return dsd;
}

__device__ __forceinline__ void rows_short(const GatBwdRowsArgs& a, int64_t item, int lane) {
  if (item >= a.n_work) return;
  const int32_t si = a.work[3 * item], r0 = a.work[3 * item + 1], nr = a.work[3 * item + 2];
  const Segment s = a.segs[si];
  const int32_t* col = a.g.colidx[s.t];
  const int64_t base = (int64_t)s.t * a.g.N, i0 = s.v_lo + r0;
  const int slot = lane >> 3, h = lane & 7;
  const int64_t rp = a.g.rowptr[s.t][i0 + min(lane, nr)];      // of the whole group (at most 32 rows)
  const int32_t rlo = (int32_t)(rp & 0xffffffff), rhi = (int32_t)(rp >> 32);
  auto row_ptr = [&](int r) {
    return ((int64_t)__builtin_amdgcn_readlane(rhi, r) << 32) | (uint32_t)__builtin_amdgcn_readlane(rlo, r);
  };
  int64_t e0 = row_ptr(0), e1 = row_ptr(1);
  int32_t ids = e0 + lane < e1 ? col[e0 + lane] : 0;
  RowOwn o = row_own(a, base + i0, h);
  for (int rr = 0; rr < nr; ++rr) {
    int64_t ne1 = e1;
    int32_t nids = 0;
    RowOwn no = o;
    if (rr + 1 < nr) {
      ne1 = row_ptr(rr + 2);
      nids = e1 + lane < ne1 ? col[e1 + lane] : 0;
      no = row_own(a, base + i0 + rr + 1, h);
    }
    if (e1 - e0 <= a.long_nnz) {    // split rows: rows_long
      const float dsd = gat_bwd_row_range(a, s, col + e0, base, o, (int)(e1 - e0), ids, lane);
      if (slot == 0) a.st2[(base + i0 + rr) * 8 + h] = make_float4(o.sd, o.lse, o.c, dsd);
    }
    e0 = e1; e1 = ne1; ids = nids; o = no;
  }
}

__device__ __forceinline__ void rows_long(const GatBwdRowsArgs& a, int64_t item, int lane) {
  if (item >= a.n_long) return;
  const int32_t* w = a.work_long + 4 * item;
  const Segment s = a.segs[w[0]];
  const int64_t i = s.v_lo + w[1];
  const int64_t* rowptr = a.g.rowptr[s.t];
  const int64_t base = (int64_t)s.t * a.g.N;
  const int64_t e0 = rowptr[i] + (int64_t)w[2] * a.part_nnz, e1 = min(rowptr[i + 1], e0 + a.part_nnz);
  const int32_t* first = a.g.colidx[s.t] + e0;
  const int n = (int)(e1 - e0), h = lane & 7;
  const RowOwn o = row_own(a, base + i, h);
  const float dsd = gat_bwd_row_range(a, s, first, base, o, n, lane < n ? first[lane] : 0, lane);
  if (lane < 8) a.long_partial[item * kLongRec + h] = dsd;
}

__global__ __launch_bounds__(256) void k_gat_bwd_rows(GatBwdRowsArgs a, int64_t long_blocks) {
  const int lane = threadIdx.x & 63;
  const int64_t block = blockIdx.x, wave = threadIdx.x >> 6;
  if (block < long_blocks) rows_long(a, block * 4 + wave, lane);
  else rows_short(a, (block - long_blocks) * 4 + wave, lane);
}

__global__ void k_gat_bwd_rows_merge(GatBwdRowsArgs a) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t item = idx >> 3;
  const int h = (int)(idx & 7);
  if (item >= a.n_long) return;
  const int32_t* w = a.work_long + 4 * item;
  if (w[2] != 0) return;
  const Segment s = a.segs[w[0]];
  float dsd = 0.f;
  for (int p = 0; p < w[3]; ++p) dsd += a.long_partial[(item + p) * kLongRec + h];
  const int64_t row = (int64_t)s.t * a.g.N + s.v_lo + w[1];
  a.st2[row * 8 + h] = make_float4(a.sX[row * 16 + 8 + h], a.lse[row * 8 + h], a.c[row * 16 + h], dsd);
}

// Graph attention backward, reverse-edge pass: for every vertex j of every snapshot in use, the
// gradients of its two projections (z_j as seen from inside its own chunk: zX; as an
// out-of-chunk neighbour: zC) are gathered over the rows i that list j, i.e. over j's own stored
// row (the adjacency is symmetric):
//   dz_j += alpha_ij du_i,   d s_src_j^h += dpre_ij^h,
// then  dzX_j += d s_dst_j a_dst + d s_srcX_j a_src,  dzC_j += d s_srcC_j a_src, and the gradients
// of a_src, a_dst are accumulated per wave.  Lanes span the 128 features (two per lane).  Long
// rows are split as in the other passes (list of (snapshot, vertex, part, parts)).
struct GatBwdColsArgs {
  GraphDev g;
  const int32_t* used_t; int32_t n_used;
  const int32_t* owner;
  const uint8_t* ecode;          // per stored non-zero (j, i) of the snapshots in use: 0 = row i is not covered,
  const int64_t* ecode_off;      //   1 = i and j are rows of the same chunk, 2 = of different chunks; [T] first entry
  const int32_t* cols_long; int64_t n_cols_long;
  int32_t long_nnz, part_nnz;
  float* long_partial;
  const uint16_t* zX; const uint16_t* zC;
  const float* sX; const float* sC;
  const uint16_t* dU;
  const float4* st2;
  const float* a_src; const float* a_dst;
  uint16_t* dzX; uint16_t* dzC;
  uint16_t* dzXlo;      // nullptr, or: what dzX loses to rounding (for the input gradient)
  float* dss;           // [T*N][16]: d s_src of the row as an in-chunk neighbour [8], as a cache row [8]
};

constexpr int kSlotRow = 16;     // rows of at most this many non-zeros are taken one per slot (k_gat_bwd_cols_slot)
constexpr int kSlotU = 2;        // neighbours in flight per slot there (4 or 8, with fewer waves per SIMD, measured slower)
constexpr int kSlotWaves = 4;    // waves per SIMD of that kernel
constexpr int kColsRec = 272;    // floats per scratch record of a part of a split row: dzX[128], dzC[128], dsx[8], dsc[8]

// Lane layout of the reverse-edge pass: lane = 16 * slot + sub.  The four slots work on four
// neighbours at a time; the 16 sub-lanes of a slot span the 128 features (8 per lane, one
// 16-byte load), two sub-lanes per head.
struct ColOwn {      // what a lane keeps about the wave's own vertex j
  int32_t oj;
  float zx[8], zc[8], ssx, ssc;
};
struct ColAcc { float ax[8], ac[8], dsx, dsc; };

__device__ __forceinline__ float quad_xor1(float x) {   // value of lane l^1
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));
}
// sum over the four slots (lanes l, l^16, l^32, l^48), same result in all of them
__device__ __forceinline__ float slot_sum(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

__device__ __forceinline__ ColOwn col_own(const GatBwdColsArgs& a, int64_t row, int sub) {
  ColOwn o;
  const int head = sub >> 1;
  // zX / sX of a vertex no chunk covers hold stale values: they are never used (no neighbour
  // can be "of the same chunk"), and loading them unconditionally keeps the loads independent
  o.oj = a.owner[row];
  unpackh8(*reinterpret_cast<const uint4*>(a.zC + row * kS + 8 * sub), o.zc);
  unpackh8(*reinterpret_cast<const uint4*>(a.zX + row * kS + 8 * sub), o.zx);
  o.ssx = a.sX[row * 16 + head];
  o.ssc = a.sC[row * 8 + head];
  return o;
}

// contributions of the stored non-zeros [e0, e1) of row j; the four slots are already summed.
// il / cl: column id and code of non-zero e0 + lane (the first 64), loaded by the caller so that
// they are in flight while the previous row is being processed.
__device__ __forceinline__ ColAcc gat_bwd_col_range(const GatBwdColsArgs& a, const int32_t* col, const uint8_t* code,
                                                    int64_t base, const ColOwn& o, int64_t e0, int64_t e1,
                                                    int32_t il, int32_t cl, int lane) {
  const int slot = lane >> 4, sub = lane & 15, head = sub >> 1;
  ColAcc r;
#pragma unroll
  for (int d = 0; d < 8; ++d) { r.ax[d] = 0.f; r.ac[d] = 0.f; }
  r.dsx = 0.f; r.dsc = 0.f;
  for (int64_t eb = e0; eb < e1; eb += 64) {
    const int cnt = (int)min((int64_t)64, e1 - eb);
    if (eb != e0) {
      il = lane < cnt ? col[eb + lane] : 0;
      cl = lane < cnt ? code[eb + lane] : 0;
    }
    for (int q0 = 0; q0 < cnt; q0 += 8) {
      uint4 dv[2];
      float4 st[2];
      int32_t cc[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int idx = q0 + 4 * u + slot;
        const int32_t ii = __shfl(il, idx);
        const int32_t cs = __shfl(cl, idx);   // outside the select: every lane has to take part
        cc[u] = idx < cnt ? cs : 0;
        dv[u] = make_uint4(0, 0, 0, 0);
        st[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (cc[u] != 0) {
          dv[u] = *reinterpret_cast<const uint4*>(a.dU + (base + ii) * kS + 8 * sub);
          st[u] = a.st2[(base + ii) * 8 + head];
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float du[8];
        unpack8(dv[u], du);
        const bool sm = cc[u] == 1;
        const float e = st[u].x + (sm ? o.ssx : o.ssc);
        float al = __expf(lrelu(e) - st[u].y);
        float da = 0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) da += du[d] * (sm ? o.zx[d] : o.zc[d]);
        da += quad_xor1(da);
        al = cc[u] != 0 ? al : 0.f;
        const float dpre = al * (da - st[u].z) * (e > 0.f ? 1.f : kSlope);
        const float alx = sm ? al : 0.f, alc = sm ? 0.f : al;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          r.ax[d] += alx * du[d];
          r.ac[d] += alc * du[d];
        }
        r.dsx += sm ? dpre : 0.f;
        r.dsc += sm ? 0.f : dpre;
      }
    }
  }
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    r.ax[d] = slot_sum(r.ax[d]);
    r.ac[d] = slot_sum(r.ac[d]);
  }
  r.dsx = slot_sum(r.dsx);
  r.dsc = slot_sum(r.dsc);
  return r;
}

struct AttVec { float as[8], ad[8]; };

__device__ __forceinline__ AttVec att_init(const GatBwdColsArgs& a, int sub) {
  AttVec v;
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    v.as[d] = a.a_src[8 * sub + d];
    v.ad[d] = a.a_dst[8 * sub + d];
  }
  return v;
}

template <bool LO, bool EVERY_SLOT = false>   // LO: also keep what dzX loses to rounding (asked for with the input gradient)
__device__ __forceinline__ void gat_bwd_col_finish(const GatBwdColsArgs& a, int64_t row, const ColOwn& o,
                                                   const ColAcc& r, const AttVec& v, int lane) {
  const int slot = lane >> 4, sub = lane & 15, head = sub >> 1;
  if (!EVERY_SLOT && slot != 0) return;      // EVERY_SLOT: each slot holds a row of its own
  float out[8];
  if (o.oj >= 0) {
    const float dsd = a.st2[row * 8 + head].w;
#pragma unroll
    for (int d = 0; d < 8; ++d) out[d] = r.ax[d] + dsd * v.ad[d] + r.dsx * v.as[d];
    const bf16x8 hi = pack8(out);
    *reinterpret_cast<uint4*>(a.dzX + row * kS + 8 * sub) = __builtin_bit_cast(uint4, hi);
    if constexpr (LO) {
      float rest[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) rest[d] = out[d] - (float)hi[d];
      *reinterpret_cast<uint4*>(a.dzXlo + row * kS + 8 * sub) = __builtin_bit_cast(uint4, pack8(rest));
    }
  }
#pragma unroll
  for (int d = 0; d < 8; ++d) out[d] = r.ac[d] + r.dsc * v.as[d];
  *reinterpret_cast<uint4*>(a.dzC + row * kS + 8 * sub) = __builtin_bit_cast(uint4, pack8(out));
  if ((sub & 1) == 0) {
    a.dss[row * 16 + head] = r.dsx;
    a.dss[row * 16 + 8 + head] = r.dsc;
  }
}

// Rows of at most kSlotRow non-zeros (nine vertices in ten of a power-law graph, a third of the
// non-zeros): ONE ROW PER SLOT, four rows per wave side by side.  What a row costs apart from its
// non-zeros (its own projections and scalars, the final combination and stores) is then paid once
// per four rows, and nothing has to be summed across the slots.  The 16 lanes of a slot first
// fetch the row's column ids and codes, one neighbour per lane, and hand them round with a
// shuffle inside the slot; two neighbours per slot are in flight (eight gathered rows per wave).
template <bool LO>
__global__ __launch_bounds__(256, kSlotWaves) void k_gat_bwd_cols_slot(GatBwdColsArgs a) {
  const int lane = threadIdx.x & 63, slot = lane >> 4, sub = lane & 15, head = sub >> 1;
  const int64_t N = a.g.N;
  const int64_t quads_per_t = (N + 3) / 4, n_items = quads_per_t * a.n_used;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= n_items) return;
  const int32_t t = a.used_t[item / quads_per_t];
  const int64_t j = (item % quads_per_t) * 4 + slot;
  const bool live = j < N;
  const int64_t base = (int64_t)t * N, row = base + (live ? j : N - 1);
  const int64_t* rp = a.g.rowptr[t] + (live ? j : N - 1);
  const int64_t e0 = rp[0], len = rp[1] - e0;
  const int n = (live && len <= kSlotRow && len <= a.long_nnz) ? (int)len : 0;     // 0: not this kernel's row
  const int32_t* col = a.g.colidx[t];
  const uint8_t* code = a.ecode + a.ecode_off[t];
  const int32_t il = sub < n ? col[e0 + sub] : 0;
  const int32_t cl = sub < n ? code[e0 + sub] : 0;
  const ColOwn o = col_own(a, row, sub);
  const AttVec v = att_init(a, sub);
  int nmax = __builtin_amdgcn_readlane(n, 0);
  nmax = max(nmax, __builtin_amdgcn_readlane(n, 16));
  nmax = max(nmax, __builtin_amdgcn_readlane(n, 32));
  nmax = max(nmax, __builtin_amdgcn_readlane(n, 48));
  ColAcc r;
#pragma unroll
  for (int d = 0; d < 8; ++d) { r.ax[d] = 0.f; r.ac[d] = 0.f; }
  r.dsx = 0.f; r.dsc = 0.f;
  for (int k0 = 0; k0 < nmax; k0 += kSlotU) {
    uint4 dv[kSlotU];
    float4 st[kSlotU];
    int32_t cc[kSlotU];
#pragma unroll
    for (int u = 0; u < kSlotU; ++u) {
      const int k = k0 + u;                              // < 16 + 1: the shuffle wraps inside the slot, the code is masked
      const int32_t ii = __shfl(il, (lane & 48) | (k & 15));
      const int32_t cs = __shfl(cl, (lane & 48) | (k & 15));
      cc[u] = k < n ? cs : 0;
      dv[u] = make_uint4(0, 0, 0, 0);
      st[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (cc[u] != 0) {
        dv[u] = *reinterpret_cast<const uint4*>(a.dU + (base + ii) * kS + 8 * sub);
        st[u] = a.st2[(base + ii) * 8 + head];
      }
    }
#pragma unroll
    for (int u = 0; u < kSlotU; ++u) {
      float du[8];
      unpack8(dv[u], du);
      const bool sm = cc[u] == 1;
      const float e = st[u].x + (sm ? o.ssx : o.ssc);
      float al = __expf(lrelu(e) - st[u].y);
      float da = 0.f;
#pragma unroll
      for (int d = 0; d < 8; ++d) da += du[d] * (sm ? o.zx[d] : o.zc[d]);
      da += quad_xor1(da);
      al = cc[u] != 0 ? al : 0.f;
      const float dpre = al * (da - st[u].z) * (e > 0.f ? 1.f : kSlope);
      const float alx = sm ? al : 0.f, alc = sm ? 0.f : al;
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        r.ax[d] += alx * du[d];
        r.ac[d] += alc * du[d];
      }
      r.dsx += sm ? dpre : 0.f;
      r.dsc += sm ? 0.f : dpre;
    }
  }
  if (n > 0) gat_bwd_col_finish<LO, true>(a, row, o, r, v, lane);
}

__device__ __forceinline__ void cols_long_part(const GatBwdColsArgs& a, int64_t item, int lane) {
  if (item >= a.n_cols_long) return;
  const int32_t* w = a.cols_long + 4 * item;   // snapshot, vertex, part, parts
  const int64_t base = (int64_t)w[0] * a.g.N, j = w[1];
  const int sub = lane & 15;
  const int64_t* rowptr = a.g.rowptr[w[0]];
  const int64_t e0 = rowptr[j] + (int64_t)w[2] * a.part_nnz, e1 = min(rowptr[j + 1], e0 + a.part_nnz);
  const ColOwn o = col_own(a, base + j, sub);
  const int32_t* col = a.g.colidx[w[0]];
  const uint8_t* code = a.ecode + a.ecode_off[w[0]];
  const int32_t il = e0 + lane < e1 ? col[e0 + lane] : 0;
  const int32_t cl = e0 + lane < e1 ? code[e0 + lane] : 0;
  const ColAcc r = gat_bwd_col_range(a, col, code, base, o, e0, e1, il, cl, lane);
  if ((lane >> 4) == 0) {
    float* rec = a.long_partial + item * kColsRec;
    float4* x = reinterpret_cast<float4*>(rec + 8 * sub);
    x[0] = make_float4(r.ax[0], r.ax[1], r.ax[2], r.ax[3]);
    x[1] = make_float4(r.ax[4], r.ax[5], r.ax[6], r.ax[7]);
    float4* c = reinterpret_cast<float4*>(rec + kS + 8 * sub);
    c[0] = make_float4(r.ac[0], r.ac[1], r.ac[2], r.ac[3]);
    c[1] = make_float4(r.ac[4], r.ac[5], r.ac[6], r.ac[7]);
    if ((sub & 1) == 0) {
      rec[256 + (sub >> 1)] = r.dsx;
      rec[264 + (sub >> 1)] = r.dsc;
    }
  }
}

template <bool LO>
__global__ __launch_bounds__(256, 4) void k_gat_bwd_cols(GatBwdColsArgs a, int64_t long_blocks) {   // 4 waves per SIMD: 128 registers
  const int lane = threadIdx.x & 63;
  const int64_t block = (int64_t)blockIdx.x - long_blocks;
  if (block < 0) {       // parts of split rows go first
    cols_long_part(a, (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), lane);
    return;
  }
  const int64_t N = a.g.N;
  const int64_t groups_per_t = (N + 15) / 16, n_items = groups_per_t * a.n_used;
  const int64_t item = block * 4 + (threadIdx.x >> 6);
  if (item >= n_items) return;
  const int sub = lane & 15;
  const AttVec v = att_init(a, sub);
  const int32_t t = a.used_t[item / groups_per_t];
  const int64_t j0 = (item % groups_per_t) * 16;
  const int32_t* col = a.g.colidx[t];
  const uint8_t* code = a.ecode + a.ecode_off[t];
  const int64_t base = (int64_t)t * N;
  const int nr = (int)min((int64_t)16, N - j0);
  // row pointers of the whole group at once; the next row's column ids and codes are requested
  // before the current row is processed
  const int64_t rp = a.g.rowptr[t][j0 + min(lane, nr)];
  const int32_t rlo = (int32_t)(rp & 0xffffffff), rhi = (int32_t)(rp >> 32);
  auto row_ptr = [&](int r) {
    return ((int64_t)__builtin_amdgcn_readlane(rhi, r) << 32) | (uint32_t)__builtin_amdgcn_readlane(rlo, r);
  };
  int64_t e0 = row_ptr(0), e1 = row_ptr(1);
  int32_t il = e0 + lane < e1 ? col[e0 + lane] : 0;
  int32_t cl = e0 + lane < e1 ? code[e0 + lane] : 0;
  for (int rr = 0; rr < nr; ++rr) {
    int64_t ne0 = e1, ne1 = e1;
    int32_t nil = 0, ncl = 0;
    if (rr + 1 < nr) {
      ne1 = row_ptr(rr + 2);
      nil = ne0 + lane < ne1 ? col[ne0 + lane] : 0;
      ncl = ne0 + lane < ne1 ? code[ne0 + lane] : 0;
    }
    if (e1 - e0 <= a.long_nnz && e1 - e0 > kSlotRow) {     // shorter rows: k_gat_bwd_cols_slot
      const ColOwn o = col_own(a, base + j0 + rr, sub);
      const ColAcc r = gat_bwd_col_range(a, col, code, base, o, e0, e1, il, cl, lane);
      gat_bwd_col_finish<LO>(a, base + j0 + rr, o, r, v, lane);
    }
    e0 = ne0; e1 = ne1; il = nil; cl = ncl;
  }
}

template <bool LO>
__global__ __launch_bounds__(256) void k_gat_bwd_cols_merge(GatBwdColsArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= a.n_cols_long) return;
  const int32_t* w = a.cols_long + 4 * item;
  if (w[2] != 0) return;
  const int sub = lane & 15;
  const AttVec v = att_init(a, sub);
  const int64_t row = (int64_t)w[0] * a.g.N + w[1];
  ColAcc r;
#pragma unroll
  for (int d = 0; d < 8; ++d) { r.ax[d] = 0.f; r.ac[d] = 0.f; }
  r.dsx = 0.f; r.dsc = 0.f;
  for (int p = 0; p < w[3]; ++p) {
    const float* rec = a.long_partial + (item + p) * kColsRec;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      r.ax[d] += rec[8 * sub + d];
      r.ac[d] += rec[kS + 8 * sub + d];
    }
    r.dsx += rec[256 + (sub >> 1)];
    r.dsc += rec[264 + (sub >> 1)];
  }
  const ColOwn o = col_own(a, row, sub);
  gat_bwd_col_finish<LO>(a, row, o, r, v, lane);
}

// Gradients of the attention vectors, a streaming pass over every vertex of the snapshots in use:
//   d a_dst^h += d s_dst_i^h z_i^h (covered rows, own projection),
//   d a_src^h += d s_srcX_i^h zX_i^h (covered rows) + d s_srcC_i^h zC_i^h (all rows).
// Lanes span the 128 features; each wave walks rows with a grid stride and leaves its sums in its
// own slot.
struct AttGradArgs {
  const int32_t* used_t; int32_t n_used; int64_t N;
  const int32_t* owner;
  const uint16_t* zX; const uint16_t* zC;
  const float4* st2; const float* dss;
  float* da_partial;    // [waves][2][128]: d a_src, d a_dst
};

__global__ __launch_bounds__(256) void k_att_grad(AttGradArgs a) {
  const int lane = threadIdx.x & 63, head = lane >> 3;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), n_waves = (int64_t)gridDim.x * 4;
  const int64_t n_rows = a.N * a.n_used;
  float gs0 = 0.f, gs1 = 0.f, gd0 = 0.f, gd1 = 0.f;
  for (int64_t r0 = wave * 8; r0 < n_rows; r0 += n_waves * 8) {
    // eight rows in flight: all loads first (rows past the end and the input-side data of rows no
    // chunk covers are read from a valid row and weighted by zero)
    uint32_t zc[8], zx[8];
    float dsc[8], dsx[8], dsd[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t idx = min(r0 + k, n_rows - 1);
      const int64_t row = (int64_t)a.used_t[idx / a.N] * a.N + idx % a.N;
      const float live = r0 + k < n_rows ? 1.f : 0.f;
      const float cov = a.owner[row] >= 0 ? live : 0.f;
      zc[k] = *reinterpret_cast<const uint32_t*>(a.zC + row * kS + 2 * lane);
      zx[k] = *reinterpret_cast<const uint32_t*>(a.zX + row * kS + 2 * lane);
      dsc[k] = live * a.dss[row * 16 + 8 + head];
      dsx[k] = cov * a.dss[row * 16 + head];
      dsd[k] = cov * a.st2[row * 8 + head].w;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      // 0 * (stale value) must stay 0: the input-side buffers of uncovered rows are never written
      const float x0 = dsx[k] != 0.f || dsd[k] != 0.f ? h_lo(zx[k]) : 0.f;
      const float x1 = dsx[k] != 0.f || dsd[k] != 0.f ? h_hi(zx[k]) : 0.f;
      gs0 += dsc[k] * h_lo(zc[k]) + dsx[k] * x0;
      gs1 += dsc[k] * h_hi(zc[k]) + dsx[k] * x1;
      gd0 += dsd[k] * x0;
      gd1 += dsd[k] * x1;
    }
  }
  float* o = a.da_partial + wave * 2 * kS;
  o[2 * lane] = gs0; o[2 * lane + 1] = gs1;
  o[kS + 2 * lane] = gd0; o[kS + 2 * lane + 1] = gd1;
}

// code of every stored non-zero (j, i) of snapshot t: see GatBwdColsArgs
__global__ void k_edge_code(GraphDev g, const int32_t* used_t, int32_t n_used, const int32_t* owner,
                            const int64_t* ecode_off, uint8_t* ecode) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= g.N * n_used) return;
  const int32_t t = used_t[idx / g.N];
  const int64_t j = idx % g.N, base = (int64_t)t * g.N;
  const int32_t oj = owner[base + j];
  const int32_t* col = g.colidx[t];
  uint8_t* out = ecode + ecode_off[t];
  for (int64_t e = g.rowptr[t][j]; e < g.rowptr[t][j + 1]; ++e) {
    const int32_t oi = owner[base + col[e]];
    out[e] = oi < 0 ? 0 : (oi == oj ? 1 : 2);
  }
}

// list of the split rows of the reverse-edge pass: count, then fill (the order of the rows in
// the list is arbitrary; the parts of a row are consecutive)
__global__ void k_cols_long(GraphDev g, const int32_t* used_t, int32_t n_used, int32_t long_nnz, int32_t part_nnz,
                            int32_t* counter, int32_t* list) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= g.N * n_used) return;
  const int32_t t = used_t[idx / g.N];
  const int64_t v = idx % g.N;
  const int64_t deg = g.rowptr[t][v + 1] - g.rowptr[t][v];
  if (deg <= long_nnz) return;
  const int32_t parts = (int32_t)((deg + part_nnz - 1) / part_nnz);
  const int32_t at = atomicAdd(counter, parts);
  if (!list) return;
  for (int32_t p = 0; p < parts; ++p) {
    list[4 * (at + p)] = t; list[4 * (at + p) + 1] = (int32_t)v;
    list[4 * (at + p) + 2] = p; list[4 * (at + p) + 3] = parts;
  }
}

}  // namespace

namespace {
constexpr int kDwGroups = 256;     // workgroups (slots) of the weight-gradient kernel
constexpr int kTbwdWaves = 2048;   // waves (slots) of the temporal backward kernel
constexpr int kColsBlocks = 1024;  // workgroups of the reverse-edge pass (4 slots each)

// Gradient of the input rows: the projection is z = W x, so dx = W^T dz, i.e. dX[row] = dzX[row] W for
// every covered row (a row no chunk covers is never an input row; it is not written).  Same
// tiling as the projection: a wave per 32 vertices of a snapshot in turn, dzX rows as the second operand
// straight from memory, fragments of W^T (both parts, 64 KB, staged in LDS once per workgroup) as the first.
// Bound by memory: 3.2 GB in 0.72 ms for 4 000 000 rows (1.02 ms with W^T from the caches,
// loads under a condition and 8-byte stores).
struct GatDxArgs {
  const uint16_t* dzX; const uint16_t* dzXlo;
  const uint4* WT; const uint4* WTlo;
  const int32_t* owner; const int32_t* used_t; int32_t n_used; int64_t N;
  uint16_t* dX; int64_t lddx;
};

__global__ __launch_bounds__(512, 4) void k_gat_dx(GatDxArgs a) {
  extern __shared__ uint4 wlds[];
  for (int i = threadIdx.x; i < kFragsPerW; i += 512) {
    wlds[i] = a.WT[i];
    wlds[kFragsPerW + i] = a.WTlo[i];
  }
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
    if (__ballot(covered) == 0ull) continue;
    const uint32_t keep = covered ? 0xffffffffu : 0u;
    // both operands as a bf16 value plus what it lost to rounding: a row's gradient is one sum of
    // 128 terms, nothing averages the roundings out as the sums over rows of the weight gradients do
    bf16x8 gf[8], gl[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      // rows no chunk covers hold no gradient (their dzX was never written): zeros.  Loaded all the same: loads under
      // a condition are each waited for
      gf[ks] = and_mask(as_frag(*reinterpret_cast<const uint4*>(a.dzX + row * kS + ks * 16 + 8 * hh)), keep);
      gl[ks] = and_mask(as_frag(*reinterpret_cast<const uint4*>(a.dzXlo + row * kS + ks * 16 + 8 * hh)), keep);
    }
#pragma unroll 1
    for (int ib = 0; ib < 4; ++ib) {
      floatx16 acc = {};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const bf16x8 wh = as_frag(wlds[(ib * 8 + ks) * 64 + lane]), wl = as_frag(wlds[kFragsPerW + (ib * 8 + ks) * 64 + lane]);
        acc = mfma(wl, gf[ks], acc);
        acc = mfma(wh, gl[ks], acc);
        acc = mfma(wh, gf[ks], acc);
      }
#pragma unroll
      for (int hd = 0; hd < 2; ++hd) {
        const uint4 o = head_order(__builtin_bit_cast(uint4, pack8v(acc, 8 * hd)));
        if (covered) *reinterpret_cast<uint4*>(a.dX + row * a.lddx + ib * 32 + 16 * hd + 8 * hh) = o;
      }
    }
  }
}

}  // namespace

// scratch layout: [weight-gradient slots | position-gradient slots | attention-vector slots]
int64_t dysat_partial_elems(const DysatWs& ws) {
  return (int64_t)kDwGroups * 3 * kS * kS + (int64_t)kTbwdWaves * ws.T * kS +
         (int64_t)kColsBlocks * 4 * 2 * kS;
}
int64_t dysat_long_partial_elems(const DysatWs& ws) {
  return std::max<int64_t>(ws.n_long * kLongRec, ws.n_cols_long * kColsRec);
}
void dysat_edge_code(const GraphDev& g, const int32_t* used_t, int32_t n_used, const int32_t* owner,
                     const int64_t* ecode_off, uint8_t* ecode, hipStream_t st) {
  hipLaunchKernelGGL(k_edge_code, blocks_for(g.N * n_used, 256), 256, 0, st, g, used_t, n_used, owner, ecode_off, ecode);
}
void dysat_cols_long(const GraphDev& g, const int32_t* used_t, int32_t n_used, int32_t long_nnz, int32_t part_nnz,
                     int32_t* counter, int32_t* list, hipStream_t st) {
  hipLaunchKernelGGL(k_cols_long, blocks_for(g.N * n_used, 256), 256, 0, st, g, used_t, n_used, long_nnz, part_nnz,
                     counter, list);
}
int64_t dysat_loss_partial_elems(const DysatWs&) { return kTbwdWaves; }

void dysat_backward(const DysatWs& ws, const void* Y, int64_t ldy, const void* dY, int64_t lddy, const void* target,
                    int64_t ldt, float* loss_out, void* dX, int64_t lddx, hipEvent_t* ev, hipStream_t st) {
  float* dw_slots = ws.partial;
  float* dpos_slots = dw_slots + (int64_t)kDwGroups * 3 * kS * kS;
  float* da_slots = dpos_slots + (int64_t)kTbwdWaves * ws.T * kS;
  const int64_t count = ws.total_rows * kS;
  const int64_t tiles32 = (ws.N + 31) / 32 * ws.n_used;
  const int groups = (int)std::min<int64_t>(kDwGroups, tiles32);

  // (1) temporal attention: dQ, dK, dV (+ loss), then dP -> dU and the position-table gradient
  const size_t lds = sizeof(uint4) * 3 * kFragsPerW;
  {
    // (if not allowed, the launch is an error)
    static std::atomic<uint64_t> ready[4] = {};
    (void)allow_lds(reinterpret_cast<const void*>(k_temporal_bwd<false>), lds, ready[0]);
    (void)allow_lds(reinterpret_cast<const void*>(k_temporal_bwd<true>), lds, ready[1]);
    (void)allow_lds(reinterpret_cast<const void*>(k_dw_bf16<3, true>), sizeof(uint4) * 2 * 64 * dw_frags<3, true>() + 65536,
                    ready[2]);   // and the position rows
    (void)allow_lds(reinterpret_cast<const void*>(k_temporal_bwd2), lds, ready[3]);
  }
  const int grid_a = (int)std::min<int64_t>(kTbwdWaves / 8, (ws.n_tiles + 7) / 8);
  const int grid_b = (int)std::min<int64_t>(kTbwdWaves / 8, (tiles32 + 7) / 8);
  const int n_tw = grid_b * 8;
  hipLaunchKernelGGL(k_fill_f32, blocks_for((int64_t)n_tw * ws.T * kS, 256), 256, 0, st, dpos_slots, 0.f,
                     (int64_t)n_tw * ws.T * kS);
  if (ev) (void)hipEventRecord(ev[0], st);
  TemporalBwdArgs ta{};
  ta.chunks = ws.chunks; ta.n_chunks = ws.n_chunks; ta.tile_ptr = ws.tile_ptr; ta.n_tiles = ws.n_tiles;
  ta.N = ws.N; ta.T = ws.T; ta.U = ws.U; ta.pos = ws.P[DY_POS];
  ta.Wq = ws.Wqp; ta.Wk = ws.Wkp; ta.Wv = ws.Wvp;
  ta.Y = static_cast<const uint16_t*>(Y); ta.ldy = ldy;
  ta.dY = static_cast<const uint16_t*>(dY); ta.lddy = lddy;
  ta.target = static_cast<const uint16_t*>(target); ta.ldt = ldt;
  ta.scale = 2.0f / (float)count;
  ta.dQ = ws.dQ; ta.dK = ws.dK; ta.dV = ws.dV;
  ta.loss_partial = ws.loss_partial;
  if (ws.wide) hipLaunchKernelGGL(k_temporal_bwd<true>, grid_a, 512, lds, st, ta);
  else hipLaunchKernelGGL(k_temporal_bwd<false>, grid_a, 512, lds, st, ta);
  if (target && loss_out)
    hipLaunchKernelGGL(k_reduce_slots, 1, 1024, 0, st, ws.loss_partial, (int64_t)grid_a * 8, (int64_t)1, (int64_t)1,
                       1.0f / (float)count, loss_out);
  TemporalBwd2Args tb{};
  tb.used_t = ws.used_t; tb.n_used = ws.n_used; tb.N = ws.N; tb.T = ws.T; tb.owner = ws.owner; tb.U = ws.U;
  tb.WqT = ws.WqT; tb.WkT = ws.WkT; tb.WvT = ws.WvT; tb.dQ = ws.dQ; tb.dK = ws.dK; tb.dV = ws.dV;
  tb.dU = ws.dU; tb.c = ws.dss; tb.dpos_partial = dpos_slots;
  hipLaunchKernelGGL(k_temporal_bwd2, grid_b, 512, lds, st, tb);
  hipLaunchKernelGGL(k_reduce_slots, blocks_for((int64_t)ws.T * kS, 64), 1024, 0, st, dpos_slots, (int64_t)n_tw,
                     (int64_t)ws.T * kS, (int64_t)ws.T * kS, 1.f, ws.G[DY_POS]);
  // (2) dW_q, dW_k, dW_v = sum over rows of d{q,k,v}^T P
  DwBf16Args da{};
  da.used_t = ws.used_t; da.n_used = ws.n_used; da.N = ws.N; da.owner = ws.owner; da.covered_only = 1;
  da.A = nullptr; da.lda = 0; da.Uf = ws.U; da.pos = ws.P[DY_POS];
  da.G[0] = ws.dQ; da.G[1] = ws.dK; da.G[2] = ws.dV;
  da.partial = dw_slots; da.n_groups = groups;
  {  // LDS: the position rows of the snapshots one workgroup's tile range can touch
    const int64_t tiles_per_t = (ws.N + 31) / 32, n_tiles = tiles_per_t * ws.n_used;
    const int64_t per = (n_tiles + groups - 1) / groups;
    const size_t pos_lds = sizeof(float) * kS * (size_t)((per + tiles_per_t - 1) / tiles_per_t + 1);
    hipLaunchKernelGGL((k_dw_bf16<3, true>), groups, 512, (sizeof(uint4) * 2 * 64 * dw_frags<3, true>()) + pos_lds, st, da, da);
  }
  for (int gi = 0; gi < 3; ++gi)
    hipLaunchKernelGGL(k_reduce_slots, blocks_for(kS * kS, 64), 1024, 0, st, dw_slots + (int64_t)gi * kS * kS,
                       (int64_t)groups, (int64_t)3 * kS * kS, (int64_t)kS * kS, 1.f, ws.G[DY_WQ + gi]);
  if (ev) (void)hipEventRecord(ev[1], st);
  // (3) graph attention, row pass
  GatBwdRowsArgs ra{};
  ra.g = ws.g; ra.segs = ws.segs; ra.work = ws.work_short; ra.n_work = ws.n_short;
  ra.zX = ws.zX; ra.zC = ws.zC; ra.sX = ws.sX; ra.sC = ws.sC; ra.dU = ws.dU; ra.c = ws.dss; ra.lse = ws.lse;
  ra.st2 = reinterpret_cast<float4*>(ws.st2);
  ra.work_long = ws.work_long; ra.n_long = ws.n_long; ra.long_nnz = ws.long_nnz; ra.part_nnz = ws.part_nnz;
  ra.long_partial = ws.long_partial;
  const int64_t long_blocks = (ws.n_long + 3) / 4;
  hipLaunchKernelGGL(k_gat_bwd_rows, (unsigned)(long_blocks + (ws.n_short + 3) / 4), 256, 0, st, ra, long_blocks);
  if (ws.n_long > 0) hipLaunchKernelGGL(k_gat_bwd_rows_merge, blocks_for(ws.n_long * 8, 256), 256, 0, st, ra);
  if (ev) (void)hipEventRecord(ev[2], st);
  // (4) reverse-edge pass, then the gradients of the attention vectors
  const int64_t items = (ws.N + 15) / 16 * ws.n_used;
  GatBwdColsArgs ca{};
  ca.g = ws.g; ca.used_t = ws.used_t; ca.n_used = ws.n_used; ca.owner = ws.owner;
  ca.ecode = ws.ecode; ca.ecode_off = ws.ecode_off;
  ca.zX = ws.zX; ca.zC = ws.zC; ca.sX = ws.sX; ca.sC = ws.sC; ca.dU = ws.dU;
  ca.st2 = reinterpret_cast<const float4*>(ws.st2);
  ca.a_src = ws.P[DY_ASRC]; ca.a_dst = ws.P[DY_ADST];
  ca.dzX = ws.dzX; ca.dzC = ws.dzC; ca.dss = ws.dss;
  ca.dzXlo = dX ? ws.dzXlo : nullptr;
  ca.cols_long = ws.cols_long; ca.n_cols_long = ws.n_cols_long; ca.long_nnz = ws.long_nnz; ca.part_nnz = ws.part_nnz;
  ca.long_partial = ws.long_partial;
  const int64_t quads = (ws.N + 3) / 4 * ws.n_used;
  if (dX) hipLaunchKernelGGL(k_gat_bwd_cols_slot<true>, blocks_for(quads, 4), 256, 0, st, ca);
  else hipLaunchKernelGGL(k_gat_bwd_cols_slot<false>, blocks_for(quads, 4), 256, 0, st, ca);
  const int64_t cols_long_blocks = (ws.n_cols_long + 3) / 4;
  const unsigned cols_blocks = (unsigned)(cols_long_blocks + (items + 3) / 4);
  if (dX) hipLaunchKernelGGL(k_gat_bwd_cols<true>, cols_blocks, 256, 0, st, ca, cols_long_blocks);
  else hipLaunchKernelGGL(k_gat_bwd_cols<false>, cols_blocks, 256, 0, st, ca, cols_long_blocks);
  if (ws.n_cols_long > 0) {
    if (dX) hipLaunchKernelGGL(k_gat_bwd_cols_merge<true>, blocks_for(ws.n_cols_long, 4), 256, 0, st, ca);
    else hipLaunchKernelGGL(k_gat_bwd_cols_merge<false>, blocks_for(ws.n_cols_long, 4), 256, 0, st, ca);
  }
  AttGradArgs ag{};
  ag.used_t = ws.used_t; ag.n_used = ws.n_used; ag.N = ws.N; ag.owner = ws.owner; ag.zX = ws.zX; ag.zC = ws.zC;
  ag.st2 = reinterpret_cast<const float4*>(ws.st2); ag.dss = ws.dss; ag.da_partial = da_slots;
  const int ablocks = (int)std::min<int64_t>(kColsBlocks, (ws.N * ws.n_used + 31) / 32);
  hipLaunchKernelGGL(k_att_grad, ablocks, 256, 0, st, ag);
  const int64_t da_n = (int64_t)ablocks * 4;
  hipLaunchKernelGGL(k_reduce_slots, 2, 1024, 0, st, da_slots, da_n, (int64_t)2 * kS, (int64_t)kS, 1.f, ws.G[DY_ASRC]);
  hipLaunchKernelGGL(k_reduce_slots, 2, 1024, 0, st, da_slots + kS, da_n, (int64_t)2 * kS, (int64_t)kS, 1.f,
                     ws.G[DY_ADST]);
  // (5) dW = sum over covered rows of dzX^T x  +  sum over all rows of dzC^T c
  DwBf16Args dx = da;
  dx.A = static_cast<const uint16_t*>(ws.X); dx.lda = ws.ldx; dx.Uf = nullptr; dx.covered_only = 1;
  dx.G[0] = ws.dzX; dx.partial = dw_slots;
  DwBf16Args dc = dx;
  dc.A = static_cast<const uint16_t*>(ws.C); dc.lda = ws.ldc; dc.covered_only = 0;
  dc.G[0] = ws.dzC; dc.partial = dw_slots + (int64_t)groups * kS * kS;
  hipLaunchKernelGGL((k_dw_bf16<1, false>), dim3(groups, 2), 512, (sizeof(uint4) * 2 * 64 * dw_frags<1, false>()), st, dx, dc);
  hipLaunchKernelGGL(k_reduce_slots, blocks_for(kS * kS, 64), 1024, 0, st, dw_slots, (int64_t)2 * groups,
                     (int64_t)kS * kS, (int64_t)kS * kS, 1.f, ws.G[DY_W]);
  // (6) optional: the gradient of the input rows, dX = dzX W (covered rows only)
  if (dX) {
    GatDxArgs xa{};
    xa.dzX = ws.dzX; xa.dzXlo = ws.dzXlo; xa.WT = ws.WT; xa.WTlo = ws.WTlo; xa.owner = ws.owner; xa.used_t = ws.used_t; xa.n_used = ws.n_used; xa.N = ws.N;
    xa.dX = static_cast<uint16_t*>(dX); xa.lddx = lddx;
    hipLaunchKernelGGL(k_gat_dx, (unsigned)std::min<int64_t>(512, (tiles32 + 7) / 8), 512, sizeof(uint4) * 2 * kFragsPerW, st, xa);
  }
  if (ev) (void)hipEventRecord(ev[3], st);
}

}  // namespace dgc
