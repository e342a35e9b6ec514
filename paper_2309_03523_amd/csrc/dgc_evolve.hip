// EvolveGCN-O support (the paper lists EvolveGCN among its DGNNs, Section 1; the "-O" variant of
// the cited work is used): the GCN weight matrix W [F][S] is the state of a matrix GRU,
//     Zg = sig(Uz W + Vz W + Bz)   Rg = sig(Ur W + Vr W + Br)
//     Wc = tanh(Uh W + Vh (Rg*W) + Bh)      W' = (1 - Zg)*W + Zg*Wc
// evolved once per snapshot over all T snapshots (global, independent of the chunk windows),
// Y[t,i] = relu(M[t,i] W_t), mean-squared-error loss, gradients of all ten parameter matrices.
//
// Kernels here: a double-precision MFMA kernel that fuses the small (F x F)(F x S) products of
// one step of the weight recurrence, or of its back-propagation through time, with the gate
// arithmetic that follows them (latency-bound), and the one large kernel of the backward pass,
// dW_t = M_t^T dP_t reduced over all rows of snapshot t across the fused chunks.
#include <algorithm>

#include "dgc_internal.h"
#include "dgc_split_dev.h"

namespace dgc {
namespace {

// ---------------------------------------------------------------------------------------------
// The weight recurrence and its back-propagation through time run in DOUBLE precision: W is the
// state of a 64-step recurrence whose rounding errors feed every output row of every snapshot,
// and the work is tiny (a handful of n x n x n products per step, n = F = S <= 256), so it is
// latency-bound whatever the precision: a chain of two dependent launches per snapshot each way.
// One kernel does every matrix step:
//   tile(C) = [C +] sum_p op(A_p) op(B_p)   followed by an elementwise epilogue,
// on v_mfma_f64_16x16x4f64 (lane l supplies A[l%16][l/16], B[l/16][l%16]; receives
// D[4*v + l/16][l%16], v = 0..3).  A workgroup of 4 waves owns one 16 x 16 tile; the waves
// split K, their partial tiles are added in wave order (reproducible), a quarter of the tile by each wave,
// which then applies the epilogue to it.  grid.z selects one of several independent jobs of a launch.
// A wave's whole share of a product is requested at once, the next product's behind it.
// (n = 64, 16 snapshots: the weights and their back-propagation took 490 us of device time as six launches per snapshot
// that read eight k at a time; 263 us like this.)
typedef double doublex4 __attribute__((ext_vector_type(4)));

struct EvProd { const double* A; const double* B; int ta, tb; };  // ta: A stored [K][M]; tb: B stored [N][K]
enum { EPI_ZR = 1, EPI_OUT = 2, EPI_BWD2 = 3, EPI_STEP = 4 };
struct EvJob {
  EvProd p[3];
  int np;
  double* C;           // STEP, jobs after the first: C += sum
  // operands of the epilogues (see k_ev_mm)
  const double* bias;  // ZR, OUT: gate bias
  const double* W;     // ZR, OUT, BWD2: previous weights
  const double* z;     // OUT: update gate      BWD2: reset gate r
  double* o0;          // ZR: gate out          OUT: Wc      BWD2: dAr     STEP: running gradient G
  double* o1;          // ZR(r job): Rg*W       OUT: W_t     BWD2: dWp (+=)   STEP: dWp (read)
  float* o2;           // OUT: W_t in fp32 (for the dense kernels)
  double* o3;          // BWD2: gradient of B_r (+=)
  int write_rw;        // ZR: this is the r job
};

// First elementwise half of a backward step, from G = dL/dW_t without the direct part.
struct EvBack {
  const float* dWd;              // direct gradient of W_t
  const double *z, *r, *c, *Wp;  // gates of step t, weights before it
  double *dWp, *dAh, *dAz, *rw;
  double *gBh, *gBz;
};
struct EvJobs { EvJob j[5]; EvBack back; };   // back: of the step that follows, dWd = NULL after the last one

__device__ __forceinline__ double sigmoidd(double x) { return 1.0 / (1.0 + exp(-x)); }

__device__ __forceinline__ void ev_back(const EvBack& b, double g, int64_t e) {
  g += (double)b.dWd[e];
  const double zz = b.z[e], cc = b.c[e], wp = b.Wp[e];
  const double dz = g * (cc - wp), dc = g * zz;
  b.dWp[e] = g * (1.0 - zz);
  const double ah = dc * (1.0 - cc * cc), azv = dz * zz * (1.0 - zz);
  b.dAh[e] = ah; b.dAz[e] = azv;
  b.rw[e] = b.r[e] * wp;
  b.gBh[e] += ah; b.gBz[e] += azv;
}

// KS: k-steps of 4 that a wave takes of a product (n = 16 KS)
template <int EPI, int KS>
__global__ __launch_bounds__(256) void k_ev_mm(EvJobs jobs) {
  constexpr int n = 16 * KS;
  __shared__ double part[4][64][4];
  const EvJob& J = jobs.j[blockIdx.z];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, kq = lane >> 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
  doublex4 acc = {0.0, 0.0, 0.0, 0.0};
  double a[2][KS], b[2][KS];
  auto request = [&](int p) {
    const int ak = J.p[p].ta ? n : 1, am = J.p[p].ta ? 1 : n;   // strides of A along k and m
    const int bk = J.p[p].tb ? 1 : n, bn = J.p[p].tb ? n : 1;
    const int k0 = wave * 4 * KS + kq;
    const double* A = J.p[p].A + (m0 + l16) * am + k0 * ak;
    const double* B = J.p[p].B + (n0 + l16) * bn + k0 * bk;
#pragma unroll
    for (int k = 0; k < KS; ++k) { a[p & 1][k] = A[4 * k * ak]; b[p & 1][k] = B[4 * k * bk]; }
  };
  request(0);
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (p >= J.np) break;
    if (p + 1 < 3 && p + 1 < J.np) request(p + 1);
#pragma unroll
    for (int k = 0; k < KS; ++k) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p & 1][k], b[p & 1][k], acc, 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) part[wave][lane][v] = acc[v];
  __syncthreads();
  const int v = wave;
  const double sum = ((part[0][lane][v] + part[1][lane][v]) + part[2][lane][v]) + part[3][lane][v];
  const int64_t e = (int64_t)(m0 + 4 * v + kq) * n + n0 + l16;
  if (EPI == EPI_ZR) {
    const double g = sigmoidd(sum + J.bias[e]);
    J.o0[e] = g;
    if (J.write_rw) J.o1[e] = g * J.W[e];
  } else if (EPI == EPI_OUT) {
    const double c = tanh(sum + J.bias[e]);
    const double zz = J.z[e];
    const double wn = (1.0 - zz) * J.W[e] + zz * c;
    J.o0[e] = c;
    J.o1[e] = wn;
    J.o2[e] = (float)wn;
  } else if (EPI == EPI_BWD2) {   // sum = Vh^T dAh = gradient of (Rg * W)
    const double rr = J.z[e];
    const double dar = sum * J.W[e] * rr * (1.0 - rr);
    J.o0[e] = dar;
    J.o1[e] += sum * rr;
    J.o3[e] += dar;
  } else if (blockIdx.z > 0) {    // a parameter gradient
    J.C[e] += sum;
  } else {                        // G_{t-1} = dWp + sum, and the first half of the step before
    const double g = J.o1[e] + sum;
    J.o0[e] = g;
    if (jobs.back.dWd) ev_back(jobs.back, g, e);
  }
}

// the first half of the last snapshot's step (G = 0)
__global__ void k_ev_back(EvBack b, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) ev_back(b, 0.0, e);
}

// The parameters widened to double, and the sums of those that multiply the same matrix (the input of the
// recurrence is its state): U_z + V_z, U_r + V_r.
struct EvParams { const float* P[EV_NPAR]; double* D[EV_NPAR]; double *zsum, *rsum; };
__global__ void k_ev_widen(EvParams p, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  for (int k = 0; k < EV_NPAR; ++k) p.D[k][e] = (double)p.P[k][e];
  p.zsum[e] = (double)p.P[EV_UZ][e] + (double)p.P[EV_VZ][e];
  p.rsum[e] = (double)p.P[EV_UR][e] + (double)p.P[EV_VR][e];
}
struct EvGrads { float* G[EV_NPAR]; double* D[EV_NPAR]; };
__global__ void k_ev_clear(EvGrads p, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  for (int k = 0; k < EV_NPAR; ++k) p.D[k][e] = 0.0;
}
// the input of the GRU is the state itself, so Uz, Vz (and Ur, Vr) receive identical gradients
__global__ void k_ev_round(EvGrads p, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  for (int k = 0; k < EV_NPAR; ++k) p.G[k][e] = (float)p.D[k == EV_VZ ? EV_UZ : k == EV_VR ? EV_UR : k][e];
}

// W_t [F][S] for all t -> fragment order of W_t^T [S][F] (the dense kernels take (out, in) weights)
__global__ void k_pack_weight_t(const float* Wt, int32_t T, int32_t F, int32_t S, float4* packed) {
  const int nkb = (F + 7) / 8;
  const int64_t per = (int64_t)(S / 32) * nkb * 64;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= per * T) return;
  const int64_t t = idx / per, i = idx - t * per;
  const int lane = (int)(i & 63);
  const int64_t f = i >> 6;
  const int kb = (int)(f % nkb), jb = (int)(f / nkb);
  const int out = jb * 32 + (lane & 31);      // column s of W_t
  const int k0 = kb * 8 + (lane >> 5) * 4;    // row f of W_t
  const float* W = Wt + t * (int64_t)F * S;
  float v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = (k0 + q < F) ? W[(int64_t)(k0 + q) * S + out] : 0.f;
  packed[idx] = make_float4(v[0], v[1], v[2], v[3]);
}

// ---------------------------------------------------------------------------------------------
// dW_t = sum over the rows (t, i) of the batch of M[row]^T dP[row],  dP = dL/d(pre-activation):
//   dP = [Y > 0] * dY                      (explicit upstream gradient), or
//   dP = [Y > 0] * 2 (Y - target) / count  (mean-squared-error loss, also summed into loss).
// 2 F S flops per row against (F + 2 S) floats read.  One workgroup of F/32 waves owns (snapshot t, split k) and
// walks every split-th 32-row tile of that snapshot, 16 rows at a time; wave w keeps rows [32w, 32w+32) x all S
// columns of the partial sum in its accumulators.  The products are sums of bf16 products on
// v_mfma_f32_32x32x16_bf16 (dgc_dense_split.hip); they contract over rows, so an operand fragment is eight rows of
// one column: a thread loads just these (a wave's load instruction is two lines of two rows), splits them once
// and leaves the parts in LDS in fragment order for every wave.  Two LDS buffers in turn, the next rows' loads
// in flight meanwhile.  With dP given, every tile's dP goes there over the rows of M that the tile has read (the
// input gradient starts from it): a pass of its own over Y and the target that is not needed.
// (64 snapshots x 62 500 rows, F = 256: 5.0 ms on the fp32 instruction and 2.1 ms for that pass; 4.8 ms here.)
// `split` workgroups per snapshot, as many as fill the chip (evolve_dw_split).
constexpr int kDwRows = 16;

struct DwArgs {
  const DenseTile* items;     // 32-row tiles ordered by snapshot
  const int64_t* item_ptr;    // [T+1]
  const ChunkInfo* chunks;
  int64_t N;
  float* M; int64_t ldm;
  const float* Y; int64_t ldy;
  const float* dY; int64_t lddy;       // or nullptr
  const float* target; int64_t ldt;    // or nullptr
  float inv_count2;                    // 2 / count
  int32_t split;
  bool keep_dp;                        // leave dP in the rows of M
  float* partial;                      // [T][split][F][S]
  float* loss_partial;                 // [T][split]
};

template <int NJB>  // F / 32 = S / 32
__global__ __launch_bounds__(64 * NJB) void k_dw_split(DwArgs a) {
  using namespace split;
  extern __shared__ __align__(16) uint4 lds[];
  constexpr int F = 32 * NJB;
  constexpr int kOperand = NJB * 3 * kFrag;            // uint4 of one operand of 16 rows
  float* red = reinterpret_cast<float*>(lds + 4 * kOperand);   // [NJB] loss partials
  const int t = blockIdx.x / a.split, ks = blockIdx.x % a.split;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = 32 * wave + l32;                     // this thread's column of both operands
  floatx16 acc[NJB];
#pragma unroll
  for (int jb = 0; jb < NJB; ++jb) acc[jb] = (floatx16)(0.f);
  float loss = 0.f;
  const int64_t i1 = table_entry(a.item_ptr, t + 1);
  const float* upstream = a.target ? a.target : a.dY;
  const int64_t ldu = a.target ? a.ldt : a.lddy;

  // Rows r0 .. r0 + 15 of tile `it`; this thread's are 8 * half + i.  A row past the tile's end is its last row,
  // and counts as zero.
  int64_t it = table_entry(a.item_ptr, t) + ks;
  int r0 = 0;
  struct Rows {
    float m[8], y[8], g[8];
    float* mp;       // this thread's first row of M
    int rows;        // of its eight that exist
    bool there;
  };
  auto request = [&](Rows& q) {
    q.there = it < i1;
    if (!q.there) return;
    const DenseTile tile = table_entry(a.items, it);
    const ChunkInfo ch = table_entry(a.chunks, tile.chunk);
    const int64_t vrow = (int64_t)t * a.N + ch.v_lo + tile.v0;
    const int first = r0 + 8 * half, last = tile.nrows - 1;
    q.rows = max(0, min(8, tile.nrows - first));
    float* m = a.M + (ch.row_off0 + (int64_t)tile.step * ch.nv + tile.v0) * a.ldm + col;
    q.mp = m + first * a.ldm;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t r = min(first + i, last);
      q.m[i] = m[r * a.ldm];
      q.y[i] = a.Y[(vrow + r) * a.ldy + col];
      q.g[i] = upstream[(vrow + r) * ldu + col];
    }
    if (r0 == 0 && tile.nrows > kDwRows) r0 = kDwRows;
    else { r0 = 0; it += a.split; }
  };
  uint4* buf = lds;
  auto step = [&](Rows& q) {
    float d[8];
    const int rows = q.rows;
    float* mp = q.mp;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool in = i < rows;
      const float diff = q.y[i] - q.g[i];
      d[i] = in && q.y[i] > 0.f ? (a.target ? diff * a.inv_count2 : q.g[i]) : 0.f;
      loss += in && a.target ? diff * diff : 0.f;
      q.m[i] = in ? q.m[i] : 0.f;
    }
    put(buf + wave * 3 * kFrag + lane, q.m);
    put(buf + kOperand + wave * 3 * kFrag + lane, d);
    request(q);
    __syncthreads();      // (also: every thread has read the rows of M that get dP)
    if (a.keep_dp) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (i < rows) mp[i * a.ldm] = d[i];
    }
    uint4 x[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) x[p] = buf[(wave * 3 + p) * kFrag + lane];
#pragma unroll
    for (int jb = 0; jb < NJB; ++jb) {
      uint4 y[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) y[p] = buf[kOperand + (jb * 3 + p) * kFrag + lane];
      // each link from zero, its small products apart, added up by rounding additions: hundreds of links would add up
      // the cut-off.  (16 x 3000 rows, width 64: U_r's gradient is 4.3e-8 off 64 bits, 8.4e-8 with the six in one sum.)
      floatx16 sum = (floatx16)(0.f);
      five(sum, x, y);
      acc[jb] += sum;
      acc[jb] += __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(x[0]), as_frag(y[0]), (floatx16)(0.f), 0, 0, 0);
    }
    buf = buf == lds ? lds + 2 * kOperand : lds;
  };
  // (two steps of rows on their way are no faster, 4.5 ms: the registers spill)
  Rows q;
  request(q);
  while (q.there) step(q);
  // partial sums: rows 32*wave .. of dW_t, standard accumulator layout (row by register, column = l%32)
  float* out = a.partial + ((int64_t)t * a.split + ks) * (int64_t)F * F;
#pragma unroll
  for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = wave * 32 + 8 * (v / 4) + 4 * half + (v % 4);
      out[(int64_t)row * F + jb * 32 + l32] = acc[jb][v];
    }
  // loss: wave sums in lane order, then the waves in order (fixed order, reproducible)
  for (int d = 32; d >= 1; d >>= 1) loss += __shfl_down(loss, d, 64);
  if (lane == 0) red[wave] = loss;
  __syncthreads();
  if (tid == 0) {
    float s = 0.f;
    for (int w = 0; w < NJB; ++w) s += red[w];
    a.loss_partial[(int64_t)t * a.split + ks] = s;
  }
}

__global__ void k_dw_reduce(const float* partial, float* dWd, int32_t split, int64_t n_per_t, int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int64_t t = e / n_per_t, i = e - t * n_per_t;
  double s = 0.0;
  for (int k = 0; k < split; ++k) s += (double)partial[(t * split + k) * n_per_t + i];
  dWd[e] = (float)s;
}

// loss = (sum of the partial sums, in index order) / count; one block
__global__ void k_loss_reduce(const float* loss_partial, int64_t n, float inv_count, float* loss_out) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) s += (double)loss_partial[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
    for (int i = 0; i < 256; ++i) tot += sh[i];
    *loss_out = (float)(tot * (double)inv_count);
  }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

// W_t [F][S] for all t -> fragment order of W_t itself as an (out = F, in = S) weight: the dense
// kernel then computes dM = dP W_t^T
__global__ void k_pack_weight_plain(const float* Wt, int32_t T, int32_t F, int32_t S, float4* packed) {
  const int nkb = (S + 7) / 8;
  const int64_t per = (int64_t)(F / 32) * nkb * 64;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= per * T) return;
  const int64_t t = idx / per, i = idx - t * per;
  const int lane = (int)(i & 63);
  const int64_t fr = i >> 6;
  const int kb = (int)(fr % nkb), jb = (int)(fr / nkb);
  const int out = jb * 32 + (lane & 31);      // row f of W_t
  const int k0 = kb * 8 + (lane >> 5) * 4;    // column s of W_t
  const float* W = Wt + t * (int64_t)F * S + (int64_t)out * S;
  float v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = (k0 + q < S) ? W[k0 + q] : 0.f;
  packed[idx] = make_float4(v[0], v[1], v[2], v[3]);
}

__global__ void k_ev_row_index(const ChunkInfo* chunks, int64_t N, int64_t* idx) {
  const ChunkInfo ch = chunks[blockIdx.z];
  const int32_t s = blockIdx.y;
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= ch.w || v >= ch.nv) return;
  idx[ch.row_off0 + (int64_t)s * ch.nv + v] = (int64_t)(ch.t_lo + s) * N + ch.v_lo + v;
}

template <int EPI>
void launch_mm(const EvJobs& jobs, int n_jobs, int n, hipStream_t st) {
  const dim3 grid(n / 16, n / 16, n_jobs);
  switch (n / 32) {
    case 1: hipLaunchKernelGGL((k_ev_mm<EPI, 2>), grid, 256, 0, st, jobs); break;
    case 2: hipLaunchKernelGGL((k_ev_mm<EPI, 4>), grid, 256, 0, st, jobs); break;
    case 3: hipLaunchKernelGGL((k_ev_mm<EPI, 6>), grid, 256, 0, st, jobs); break;
    case 4: hipLaunchKernelGGL((k_ev_mm<EPI, 8>), grid, 256, 0, st, jobs); break;
    case 5: hipLaunchKernelGGL((k_ev_mm<EPI, 10>), grid, 256, 0, st, jobs); break;
    case 6: hipLaunchKernelGGL((k_ev_mm<EPI, 12>), grid, 256, 0, st, jobs); break;
    case 7: hipLaunchKernelGGL((k_ev_mm<EPI, 14>), grid, 256, 0, st, jobs); break;
    case 8: hipLaunchKernelGGL((k_ev_mm<EPI, 16>), grid, 256, 0, st, jobs); break;
  }
}

}  // namespace

int32_t evolve_dw_split(int32_t T, int32_t F, int64_t most_tiles) {
  // about two rounds of workgroups of F/32 waves on 256 CUs of eight waves, at least 8 a snapshot (and at most one
  // a tile: the partial sums of every one are written and read)
  const int64_t n = std::min<int64_t>(64, 2 * 256 * 8 / ((int64_t)T * (F / 32)));
  return (int32_t)std::max<int64_t>(1, std::min(std::max<int64_t>(8, n), most_tiles));
}
int64_t evolve_partial_elems(const EvolveWs& ws) { return (int64_t)ws.T * ws.split_dw * ws.F * ws.S; }
int64_t evolve_loss_partial_elems(const EvolveWs& ws) { return (int64_t)ws.T * ws.split_dw; }

// Evolve W_t for t = 0..T-1 (ws.Wt, gates ws.Zg/Rg/Wc, all double) and pack every W_t, rounded
// to fp32, for the dense kernels.  Two launches per snapshot.
void evolve_forward_weights(const EvolveWs& ws, hipStream_t st) {
  const int n = ws.F;
  const int64_t nn = (int64_t)n * n;
  EvParams par{};
  for (int k = 0; k < EV_NPAR; ++k) { par.P[k] = ws.P[k]; par.D[k] = ws.Pd[k]; }
  par.zsum = ws.zsum; par.rsum = ws.rsum;
  hipLaunchKernelGGL(k_ev_widen, blocks_for(nn), 256, 0, st, par, nn);
  for (int t = 0; t < ws.T; ++t) {
    const double* W = t ? ws.Wt + (t - 1) * nn : ws.Pd[EV_W];
    double *z = ws.Zg + t * nn, *r = ws.Rg + t * nn, *c = ws.Wc + t * nn, *Wn = ws.Wt + t * nn;
    EvJobs zr{};
    zr.j[0].p[0] = {ws.zsum, W, 0, 0}; zr.j[0].np = 1;
    zr.j[0].bias = ws.Pd[EV_BZ]; zr.j[0].W = W; zr.j[0].o0 = z; zr.j[0].write_rw = 0;
    zr.j[1].p[0] = {ws.rsum, W, 0, 0}; zr.j[1].np = 1;
    zr.j[1].bias = ws.Pd[EV_BR]; zr.j[1].W = W; zr.j[1].o0 = r; zr.j[1].o1 = ws.tmp[1]; zr.j[1].write_rw = 1;
    launch_mm<EPI_ZR>(zr, 2, n, st);
    EvJobs out{};
    out.j[0].p[0] = {ws.Pd[EV_UH], W, 0, 0}; out.j[0].p[1] = {ws.Pd[EV_VH], ws.tmp[1], 0, 0}; out.j[0].np = 2;
    out.j[0].bias = ws.Pd[EV_BH]; out.j[0].W = W; out.j[0].z = z; out.j[0].o0 = c; out.j[0].o1 = Wn;
    out.j[0].o2 = ws.Wt_f32 + t * nn;
    launch_mm<EPI_OUT>(out, 1, n, st);
  }
  if (ws.split) {
    launch_pack_split(ws.Wt_f32, nn, 1, ws.S, ws.S, ws.F, ws.T, ws.Wt_packed, st);
    return;
  }
  const int64_t per = (int64_t)(ws.S / 32) * ((ws.F + 7) / 8) * 64;
  hipLaunchKernelGGL(k_pack_weight_t, blocks_for(per * ws.T), 256, 0, st, ws.Wt_f32, ws.T, ws.F, ws.S, ws.Wt_packed);
}

void evolve_row_index(const ChunkInfo* chunks, int32_t n_chunks, int64_t max_nv, int32_t max_w, int64_t N, int64_t* idx,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_ev_row_index, dim3(blocks_for(max_nv), (unsigned)max_w, (unsigned)n_chunks), 256, 0, st, chunks, N,
                     idx);
}

void evolve_pack_weights_plain(const EvolveWs& ws, float4* packed, hipStream_t st) {
  if (ws.split) {
    launch_pack_split(ws.Wt_f32, (int64_t)ws.F * ws.S, ws.S, 1, ws.F, ws.S, ws.T, packed, st);
    return;
  }
  const int64_t per = (int64_t)(ws.F / 32) * ((ws.S + 7) / 8) * 64;
  hipLaunchKernelGGL(k_pack_weight_plain, blocks_for(per * ws.T), 256, 0, st, ws.Wt_f32, ws.T, ws.F, ws.S, packed);
}

// dWd[t] for all t (and the loss), from the saved aggregated rows and the layer's output; keep_dp: the rows of M
// then hold dP.
bool evolve_backward_dw(const EvolveWs& ws, const EvolveBwdIn& in, bool keep_dp, hipStream_t st, std::string* why) {
  DwArgs a{};
  a.items = ws.items; a.item_ptr = ws.item_ptr; a.chunks = in.chunks; a.N = in.N;
  a.M = in.M; a.ldm = in.ldm; a.Y = in.Y; a.ldy = in.ldy; a.dY = in.dY; a.lddy = in.lddy;
  a.target = in.target; a.ldt = in.ldt;
  a.inv_count2 = 2.0f / (float)in.count;
  a.split = ws.split_dw; a.keep_dp = keep_dp; a.partial = ws.partial; a.loss_partial = ws.loss_partial;
  if (ws.F % 32 || ws.F > 256 || ws.S != ws.F) {
    if (why) *why = "the weight-gradient kernel needs F = S, a multiple of 32, at most 256";
    return false;
  }
  const int njb = ws.F / 32;
  const size_t lds = (size_t)4 * njb * 3 * split::kFrag * sizeof(uint4) + sizeof(float) * 16;
  const unsigned grid = (unsigned)ws.T * ws.split_dw;
  switch (njb) {
#define DGC_DW_CASE(NJB)                                                                               \
  case NJB: {                                                                                          \
    static std::atomic<uint64_t> ready{0};                                                             \
    if (!allow_lds(reinterpret_cast<const void*>(&k_dw_split<NJB>), 160 * 1024, ready, why)) return false;\
    hipLaunchKernelGGL((k_dw_split<NJB>), grid, 64 * NJB, lds, st, a);                                 \
    break;                                                                                             \
  }
    DGC_DW_CASE(1) DGC_DW_CASE(2) DGC_DW_CASE(3) DGC_DW_CASE(4) DGC_DW_CASE(5) DGC_DW_CASE(6) DGC_DW_CASE(7)
    DGC_DW_CASE(8)
#undef DGC_DW_CASE
    default:
      if (why) *why = "unsupported S";
      return false;
  }
  const int64_t n = (int64_t)ws.F * ws.S;
  hipLaunchKernelGGL(k_dw_reduce, blocks_for(n * ws.T), 256, 0, st, ws.partial, ws.dWd, ws.split_dw, n, n * ws.T);
  if (in.target && in.loss_out)
    hipLaunchKernelGGL(k_loss_reduce, 1, 256, 0, st, ws.loss_partial, (int64_t)ws.T * ws.split_dw, 1.0f / (float)in.count,
                       in.loss_out);
  return true;
}

// Back-propagation through time over the weight recurrence (double precision, two launches per
// snapshot); the gradients of the ten parameters end up in ws.G[k] as fp32.
void evolve_backward_bptt(const EvolveWs& ws, hipStream_t st) {
  const int n = ws.F;
  const int64_t nn = (int64_t)n * n;
  const unsigned nb = blocks_for(nn);
  EvGrads gr{};
  for (int k = 0; k < EV_NPAR; ++k) { gr.G[k] = ws.G[k]; gr.D[k] = ws.Gd[k]; }
  hipLaunchKernelGGL(k_ev_clear, nb, 256, 0, st, gr, nn);
  double* Gt = ws.Gd[EV_W];  // running dL/dW_t; ends as the gradient of W_init
  double *dWp = ws.tmp[0], *dAr = ws.tmp[2];
  // A step's launch leaves the first half of the step before it in the other one of two sets: its tiles still read
  // this step's.
  auto back = [&](int t) {
    EvBack b{};
    if (t < 0) return b;
    double* const* set = t % 2 ? ws.back1 : ws.back0;
    b.dWd = ws.dWd + t * nn;
    b.z = ws.Zg + t * nn; b.r = ws.Rg + t * nn; b.c = ws.Wc + t * nn;
    b.Wp = t ? ws.Wt + (t - 1) * nn : ws.Pd[EV_W];
    b.dWp = dWp; b.dAh = set[0]; b.dAz = set[1]; b.rw = set[2];
    b.gBh = ws.Gd[EV_BH]; b.gBz = ws.Gd[EV_BZ];
    return b;
  };
  hipLaunchKernelGGL(k_ev_back, nb, 256, 0, st, back(ws.T - 1), nn);
  for (int t = ws.T - 1; t >= 0; --t) {
    const EvBack cur = back(t);
    EvJobs b2{};   // Vh^T dAh -> dAr, dWp += ., dB_r += .
    b2.j[0].p[0] = {ws.Pd[EV_VH], cur.dAh, 1, 0}; b2.j[0].np = 1;
    b2.j[0].W = cur.Wp; b2.j[0].z = cur.r; b2.j[0].o0 = dAr; b2.j[0].o1 = dWp; b2.j[0].o3 = ws.Gd[EV_BR];
    launch_mm<EPI_BWD2>(b2, 1, n, st);
    EvJobs g{};    // G_{t-1} = dWp + Uh^T dAh + (Uz + Vz)^T dAz + (Ur + Vr)^T dAr
    g.j[0].p[0] = {ws.Pd[EV_UH], cur.dAh, 1, 0}; g.j[0].p[1] = {ws.zsum, cur.dAz, 1, 0}; g.j[0].p[2] = {ws.rsum, dAr, 1, 0};
    g.j[0].np = 3;
    g.j[0].o0 = Gt; g.j[0].o1 = dWp;
    // dUh += dAh Wp^T, dVh += dAh (Rg*Wp)^T, dUz += dAz Wp^T, dUr += dAr Wp^T
    g.j[1].p[0] = {cur.dAh, cur.Wp, 0, 1}; g.j[1].np = 1; g.j[1].C = ws.Gd[EV_UH];
    g.j[2].p[0] = {cur.dAh, cur.rw, 0, 1}; g.j[2].np = 1; g.j[2].C = ws.Gd[EV_VH];
    g.j[3].p[0] = {cur.dAz, cur.Wp, 0, 1}; g.j[3].np = 1; g.j[3].C = ws.Gd[EV_UZ];
    g.j[4].p[0] = {dAr, cur.Wp, 0, 1}; g.j[4].np = 1; g.j[4].C = ws.Gd[EV_UR];
    g.back = back(t - 1);
    launch_mm<EPI_STEP>(g, 5, n, st);
  }
  hipLaunchKernelGGL(k_ev_round, nb, 256, 0, st, gr, nn);
}

}  // namespace dgc
