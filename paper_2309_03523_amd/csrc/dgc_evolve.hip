// EvolveGCN-O support (the paper lists EvolveGCN among its DGNNs, Section 1; the "-O" variant of
// the cited work is used): the GCN weight matrix W [F][S] is the state of a matrix GRU,
//     Zg = sig(Uz W + Vz W + Bz)   Rg = sig(Ur W + Vr W + Br)
//     Wc = tanh(Uh W + Vh (Rg*W) + Bh)      W' = (1 - Zg)*W + Zg*Wc
// evolved once per snapshot over all T snapshots (global, independent of the chunk windows),
// Y[t,i] = relu(M[t,i] W_t), mean-squared-error loss, gradients of all ten parameter matrices.
//
// Kernels here: the weight recurrence and its back-propagation in double precision on f64 MFMA, one launch each that
// walks all snapshots, the parameter gradients as one launch after it, and the one large kernel of the backward pass,
// dW_t = M_t^T dP_t reduced over all rows of snapshot t across the fused chunks.
#include <algorithm>

#include "dgc_internal.h"
#include "dgc_split_dev.h"

namespace dgc {
namespace {

// ---------------------------------------------------------------------------------------------
// The weight recurrence and its back-propagation through time run in DOUBLE precision: W is the
// state of a 64-step recurrence whose rounding errors feed every output row of every snapshot,
// and the work is tiny (four n x n x n products per step, n = F = S <= 256), so it is bound by the
// serial chain whatever the precision.
// The columns of W never meet: every product multiplies W (or its gradient) from the left.  So a workgroup
// owns four columns and walks all snapshots by itself, one launch each way, and the only waits are its own two
// barriers a step.  Four columns, because v_mfma_f64_4x4x4_4b does as many products per cycle as the
// 16x16x4 form: a step's chain is as short as it gets and n / 4 workgroups share the work.
//   Wave w of the n / 16 that share a product owns rows 16 w .. +15.  The four 4x4 blocks of an instruction take four
//   quarters of a 16-wide stretch of the contraction, and four accumulators the four row groups: lane
//   (i = l / 16, blk = l / 4 % 4, j = l % 4) supplies A[4 g + i'][16 kc + 4 blk + k'] (i' = l % 4, k' = l / 16) and
//   B[16 kc + 4 blk + i][j].  After the four blocks' sums are added up the lane holds row 4 blk + i,
//   column j of the wave's sixteen rows: the layout of B, so a state goes to LDS and comes back one double a lane in order.
//   The small matrices stay in registers (n <= 64); larger ones are read from L2 at every step, a batch of 32 columns of
//   16 rows at a time, D batches ahead, which is what bounds them (2 MB a step for n = 256).
// Up to n = 128 two sets of waves share a step: the first gate (whose product with the state the last product waits
// for) is the second set's.
// Measured alone, per snapshot: n = 64 1.4 us forward and 1.2 back (8 and 10 us as two launches per snapshot of 16 x 16
// tiles, K split over four waves, with the gaps between them), n = 128 4.1 and 5.2, n = 256 17.7 and 21.4 (20 and 31).
// The matrices' batches take the registers to their limit in the widest walks: of a lane 12 (forward) and 18 (back) go to scratch
// for n = 224, 10 back for n = 256.
typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double sigmoidd(double x) { return 1.0 / (1.0 + exp(-x)); }

struct EvWalkArgs {
  int32_t T;
  const float* P[EV_NPAR];         // back: U and V are those kept
  float* kept;                     // forward, resident: ev_keep
  const doublex2* packed;          // streamed matrices (ev_packed_index); unused where they are resident
  double *Wt, *Zg, *Rg, *Wc;       // Wt[0] = W_init, Wt[t + 1] = W_t
  float* Wt_f32;
  const float* dWd;                // back: direct gradient of every W_t
  double *Ah, *Az, *Ar;            // back: gradients of the gates' arguments
  float *gW, *gBz, *gBr, *gBh;     // back: gradients of W_init and of the biases
};

// Matrix m of a step at [row][k].  Forward: U_r + V_r, U_z + V_z, U_h, V_h; back: V_h, U_z + V_z, U_h, U_r + V_r, transposed.
// (The input of the recurrence is its state, so U and V of a gate multiply the same matrix.)
template <bool BACK>
__device__ __forceinline__ double ev_weight(const float* const (&P)[EV_NPAR], int m, int n, int row, int k) {
  const int e = BACK ? k * n + row : row * n + k;
  switch (BACK && m != 1 && m != 2 ? 3 - m : m) {
    case 0: return (double)P[EV_UR][e] + (double)P[EV_VR][e];
    case 1: return (double)P[EV_UZ][e] + (double)P[EV_VZ][e];
    case 2: return (double)P[EV_UH][e];
    default: return (double)P[EV_VH][e];
  }
}

// The way back is that of the parameters which the forward pass used, whatever has been set since: the first launch of a forward
// keeps its U and V, [6][n][n], in the order of kKept (beside its loads of them; 1 us at most).
constexpr int kKept[6] = {EV_UZ, EV_VZ, EV_UR, EV_VR, EV_UH, EV_VH};
__device__ __forceinline__ void ev_keep(const float* const (&P)[EV_NPAR], float* kept, int n, int first, int stride) {
  const int quads = n * n / 4;
#pragma unroll
  for (int m = 0; m < 6; ++m)
    for (int i = first; i < quads; i += stride)
      reinterpret_cast<float4*>(kept)[m * quads + i] = reinterpret_cast<const float4*>(P[kKept[m]])[i];
}

// A batch is 32 columns of a wave's 16 rows: pair q of lane l holds row groups 2 (q % 2), + 1 of stretch 2 batch + q / 2.
struct EvElement { int row, k; };
__device__ __forceinline__ EvElement ev_element(int wave, int batch, int q, int half, int lane) {
  return {16 * wave + 4 * (2 * (q & 1) + half) + (lane & 3), 16 * (2 * batch + (q >> 1)) + (lane & 12) + (lane >> 4)};
}

struct EvPackArgs { const float* P[EV_NPAR]; float* kept; doublex2* packed; int32_t n; };
template <bool BACK>
__global__ __launch_bounds__(256) void k_ev_pack(EvPackArgs a) {
  const int nw = a.n / 16, nb = nw / 2;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;      // ((m * nw + wave) * nb + batch) * 256 + q * 64 + lane
  if (idx >= 4 * nw * nb * 256) return;
  if constexpr (!BACK) ev_keep(a.P, a.kept, a.n, idx, 4 * nw * nb * 256);
  const int lane = idx & 63, q = (idx >> 6) & 3;
  int r = idx >> 8;
  const int batch = r % nb; r /= nb;
  const int wave = r % nw, m = r / nw;
  const EvElement x = ev_element(wave, batch, q, 0, lane), y = ev_element(wave, batch, q, 1, lane);
  doublex2 v;
  v.x = ev_weight<BACK>(a.P, m, a.n, x.row, x.k);
  v.y = ev_weight<BACK>(a.P, m, a.n, y.row, y.k);
  a.packed[idx] = v;
}

template <int CTRL>
__device__ __forceinline__ double move_lanes(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}
// sum over the four blocks of the accumulator that a lane's own block stands for
__device__ __forceinline__ double add_blocks(const double (&acc)[4], int lane) {
  const bool b1 = lane & 8, b0 = lane & 4;
  const double k0 = (b1 ? acc[2] : acc[0]) + move_lanes<0x128>(b1 ? acc[0] : acc[2]);    // lane ^ 8: rotation by 8 of 16
  const double k1 = (b1 ? acc[3] : acc[1]) + move_lanes<0x128>(b1 ? acc[1] : acc[3]);
  return (b0 ? k1 : k0) + move_lanes<0x1b>(move_lanes<0x141>(b0 ? k0 : k1));             // lane ^ 4: ^ 7, then ^ 3
}

// One role's matrices, in the order of their use: resident in registers, or streamed through a ring of D batches.
template <int NW, int FIRST, int NM, bool RESIDENT, bool BACK>
struct EvMatrices {
  static constexpr int NB = NW / 2;
  static constexpr int D = RESIDENT ? NM * NB : (NM * NB) % 4 == 0 ? 4 : 3;
  static_assert((NM * NB) % D == 0, "the ring comes round with the step");
  doublex2 w[D][4];
  __amdgpu_buffer_rsrc_t rsrc;     // streamed: the place of a batch is a scalar, the lane's part of it a vector offset
  int first, lane16;
  __device__ __forceinline__ void fetch(int id) {
    const int at = first + ((id / NB) * NW * NB + id % NB) * 4096;
#pragma unroll
    for (int q = 0; q < 4; ++q) w[id % D][q] = __builtin_bit_cast(doublex2, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane16, at + q * 1024, 0));
  }
  __device__ __forceinline__ void start(const EvWalkArgs& a, int wave, int lane) {
    if constexpr (RESIDENT) {
#pragma unroll
      for (int id = 0; id < D; ++id)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const EvElement x = ev_element(wave, id % NB, q, 0, lane), y = ev_element(wave, id % NB, q, 1, lane);
          w[id][q].x = ev_weight<BACK>(a.P, FIRST + id / NB, 16 * NW, x.row, x.k);
          w[id][q].y = ev_weight<BACK>(a.P, FIRST + id / NB, 16 * NW, y.row, y.k);
        }
    } else {
      rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<doublex2*>(a.packed), 0, 4 * NW * NB * 4096, 0x00020000);
      first = (FIRST * NW + wave) * NB * 4096;
      lane16 = lane * 16;
#pragma unroll
      for (int id = 0; id < D; ++id) fetch(id);
    }
  }
  // acc += matrix m of this role's x the state in LDS
  __device__ __forceinline__ void product(int m, const double* state, double (&acc)[4]) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int id = m * NB + b;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double s = state[(2 * b + c) * 64];
        acc[0] = __builtin_amdgcn_mfma_f64_4x4x4f64(w[id % D][2 * c].x, s, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_4x4x4f64(w[id % D][2 * c].y, s, acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_4x4x4f64(w[id % D][2 * c + 1].x, s, acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f64_4x4x4f64(w[id % D][2 * c + 1].y, s, acc[3], 0, 0, 0);
      }
      if constexpr (!RESIDENT) {
        fetch((id + D) % (NM * NB));
        __builtin_amdgcn_sched_barrier(0);    // else all of the state is read ahead, and the registers spill
      }
    }
  }
};

// What the two sets of waves do, and in which order, is written once: ONE set does both, the first one FIRST..
template <int NW, int ROLE, bool BACK>   // ROLE 0: one set of waves does it all; 1: the first gate; 2: the rest
__device__ __forceinline__ void ev_walk(const EvWalkArgs& a, int wave, double* lds) {
  constexpr int n = 16 * NW;
  constexpr bool kGate = ROLE != 2, kRest = ROLE != 1;
  constexpr bool kResident = ROLE == 1 || NW <= 4;
  const int lane = threadIdx.x & 63;
  const int e = (16 * wave + (lane & 12) + (lane >> 4)) * n + 4 * blockIdx.x + (lane & 3);
  constexpr int64_t nn = (int64_t)n * n;
  // states that all waves read: S (and S2 back), Q between the step's two barriers, P back to the other set
  double *S = lds, *S2 = lds + n * 4, *Q = lds + 2 * n * 4, *P = lds + 3 * n * 4;
  const int own = wave * 64 + lane;
  EvMatrices<NW, ROLE == 2 ? 1 : 0, ROLE == 0 ? 4 : ROLE == 1 ? 1 : 3, kResident, BACK> mat;
  constexpr int m1 = ROLE == 0 ? 1 : 0;       // the rest's first matrix
  mat.start(a, wave, lane);
  if constexpr (!BACK) {
    double W = (double)a.P[EV_W][e];
    double bz = 0.0, br = 0.0, bh = 0.0;
    if constexpr (kGate) br = (double)a.P[EV_BR][e];
    if constexpr (kRest) {
      bz = (double)a.P[EV_BZ][e]; bh = (double)a.P[EV_BH][e];
      S[own] = W;
      a.Wt[e] = W;
    }
    for (int t = 0; t < a.T; ++t) {
      __syncthreads();
      if constexpr (kGate) {
        if (ROLE == 1) W = S[own];
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        mat.product(0, S + lane, acc);
        const double r = sigmoidd(add_blocks(acc, lane) + br);
        Q[own] = r * W;
        a.Rg[t * nn + e] = r;
      }
      double z = 0.0, acc[4] = {0.0, 0.0, 0.0, 0.0};
      if constexpr (kRest) {
        double az[4] = {0.0, 0.0, 0.0, 0.0};
        mat.product(m1, S + lane, az);
        z = sigmoidd(add_blocks(az, lane) + bz);
        mat.product(m1 + 1, S + lane, acc);
      }
      __syncthreads();
      if constexpr (kRest) {
        mat.product(m1 + 2, Q + lane, acc);
        const double c = tanh(add_blocks(acc, lane) + bh);
        W = (1.0 - z) * W + z * c;
        S[own] = W;
        a.Zg[t * nn + e] = z;
        a.Wc[t * nn + e] = c;
        a.Wt[(t + 1) * nn + e] = W;
        a.Wt_f32[t * nn + e] = (float)W;
      }
    }
  } else {
    // operands of a step's elementwise part, requested a step ahead
    double z = 0.0, c = 0.0, wp = 0.0, r = 0.0;
    float d = 0.f;
    auto request = [&](int t) {
      wp = a.Wt[t * nn + e];
      if constexpr (kGate) r = a.Rg[t * nn + e];
      if constexpr (kRest) { z = a.Zg[t * nn + e]; c = a.Wc[t * nn + e]; d = a.dWd[t * nn + e]; }
    };
    double G = 0.0, bz = 0.0, br = 0.0, bh = 0.0;
    request(a.T - 1);
    for (int t = a.T - 1; t >= 0; --t) {
      double direct = 0.0;                    // of dL/dW_{t-1}: the part that no matrix multiplies
      if constexpr (kRest) {
        const double g = G + (double)d;
        const double dz = g * (c - wp), dc = g * z;
        const double ah = dc * (1.0 - c * c), az = dz * z * (1.0 - z);
        direct = g * (1.0 - z);
        S[own] = ah; S2[own] = az;
        bh += ah; bz += az;
        a.Ah[t * nn + e] = ah;
        a.Az[t * nn + e] = az;
      }
      const double wp_t = wp, r_t = r;
      if (t > 0) request(t - 1);
      __syncthreads();
      if constexpr (kGate) {
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        mat.product(0, S + lane, acc);
        const double s = add_blocks(acc, lane);      // gradient of R * W
        const double ar = s * wp_t * r_t * (1.0 - r_t);
        Q[own] = ar;
        if constexpr (kRest) direct += s * r_t;
        else P[own] = s * r_t;
        br += ar;
        a.Ar[t * nn + e] = ar;
      }
      double acc[4] = {0.0, 0.0, 0.0, 0.0};
      if constexpr (kRest) {
        mat.product(m1, S2 + lane, acc);
        mat.product(m1 + 1, S + lane, acc);
      }
      __syncthreads();
      if constexpr (kRest) {
        mat.product(m1 + 2, Q + lane, acc);
        if constexpr (!kGate) direct += P[own];
        G = direct + add_blocks(acc, lane);
      }
    }
    if constexpr (kGate) a.gBr[e] = (float)br;
    if constexpr (kRest) {
      a.gW[e] = (float)G;
      a.gBz[e] = (float)bz;
      a.gBh[e] = (float)bh;
    }
  }
}

template <int NW, bool BACK>
__global__ __launch_bounds__(64 * (NW <= 8 ? 2 * NW : NW)) void k_ev_walk(EvWalkArgs a) {
  __shared__ double lds[4 * 16 * NW * 4];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (!BACK && NW <= 4) ev_keep(a.P, a.kept, 16 * NW, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
  if constexpr (NW <= 8) {
    if (wave >= NW) ev_walk<NW, 1, BACK>(a, wave - NW, lds);
    else ev_walk<NW, 2, BACK>(a, wave, lds);
  } else {
    ev_walk<NW, 0, BACK>(a, wave, lds);
  }
}

// Parameter gradients, sums over snapshots and columns of W (the contraction):
//   dU_h = sum Ah Wp^T   dV_h = sum Ah (R * Wp)^T   dU_z = dV_z = sum Az Wp^T   dU_r = dV_r = sum Ar Wp^T
// A workgroup of 8 waves owns a TM x TM tile of one of them; its waves split the contraction sixteen columns at a time and
// their partial tiles are added in wave order (reproducible).  TM = 32 halves what is read per product, TM = 16 gives a
// small matrix more workgroups.  v_mfma_f64_16x16x4f64: lane l supplies A[l%16][l/16], B[l/16][l%16] and receives
// D[4*v + l/16][l%16]; four consecutive columns of a lane are four instructions.
// Jobs 4 to 7 take the walk's own four gradients to where the caller reads them (the walk writes 16 bytes of a row at a
// time, which is no way to write to host memory).
struct EvGradArgs { int32_t T, n; const double *Wt, *Rg, *Ah, *Az, *Ar; const float* walk; float* G[EV_NPAR]; };

template <int TM>
__global__ __launch_bounds__(512) void k_ev_grads(EvGradArgs a) {
  constexpr int NT = TM / 16;
  __shared__ double part[8][TM * TM];
  const int n = a.n, job = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, kq = lane >> 4;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
  if (job >= 4) {
    float* G = a.G[job == 4 ? EV_W : job == 5 ? EV_BZ : job == 6 ? EV_BR : EV_BH];
    for (int i = tid; i < TM * TM; i += 512) {
      const int64_t e = (int64_t)(m0 + i / TM) * n + n0 + i % TM;
      G[e] = a.walk[(int64_t)(job - 4) * n * n + e];
    }
    return;
  }
  const double* A = job < 2 ? a.Ah : job == 2 ? a.Az : a.Ar;
  const int per_t = n / 16, units = a.T * per_t;
  const int64_t nn = (int64_t)n * n;
  doublex4 acc[NT][NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = (doublex4)(0.0);
  doublex2 x[NT][2], y[NT][2], r[NT][2];
  auto request = [&](int u) {
    const int t = u / per_t, s0 = (u - t * per_t) * 16 + 4 * kq;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t ea = t * nn + (m0 + 16 * i + l16) * n + s0 + 2 * h, eb = t * nn + (n0 + 16 * i + l16) * n + s0 + 2 * h;
        x[i][h] = *reinterpret_cast<const doublex2*>(A + ea);
        y[i][h] = *reinterpret_cast<const doublex2*>(a.Wt + eb);
        if (job == 1) r[i][h] = *reinterpret_cast<const doublex2*>(a.Rg + eb);
      }
  };
  if (wave < units) request(wave);
  for (int u = wave; u < units; u += 8) {
    doublex2 p[NT][2], q[NT][2];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) { p[i][h] = x[i][h]; q[i][h] = job == 1 ? y[i][h] * r[i][h] : y[i][h]; }
    if (u + 8 < units) request(u + 8);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[i][h][k], q[j][h][k], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[wave][(16 * i + 4 * v + kq) * TM + 16 * j + l16] = acc[i][j][v];
  __syncthreads();
  float* G = a.G[job == 0 ? EV_UH : job == 1 ? EV_VH : job == 2 ? EV_UZ : EV_UR];
  float* G2 = job < 2 ? nullptr : a.G[job == 2 ? EV_VZ : EV_VR];    // the input is the state: U and V get one gradient
  for (int i = tid; i < TM * TM; i += 512) {
    double sum = part[0][i];
#pragma unroll
    for (int w = 1; w < 8; ++w) sum += part[w][i];
    const int64_t e = (int64_t)(m0 + i / TM) * n + n0 + i % TM;
    G[e] = (float)sum;
    if (G2) G2[e] = (float)sum;
  }
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
  constexpr int kAhead = 8;        // partial sums requested together (past the last: the last one, not added)
  for (int k0 = 0; k0 < split; k0 += kAhead) {
    float v[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) v[k] = partial[(t * split + min(k0 + k, split - 1)) * n_per_t + i];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) s += k0 + k < split ? (double)v[k] : 0.0;
  }
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

template <bool BACK>
void launch_walk(const EvolveWs& ws, hipStream_t st) {
  const int n = ws.F;
  EvWalkArgs a{};
  a.T = ws.T;
  for (int k = 0; k < EV_NPAR; ++k) a.P[k] = ws.P[k];
  if (BACK)
    for (int k = 0; k < 6; ++k) a.P[kKept[k]] = ws.kept + (int64_t)k * n * n;
  a.kept = ws.kept;
  a.packed = reinterpret_cast<const doublex2*>(ws.walk_packed);
  a.Wt = ws.Wt; a.Zg = ws.Zg; a.Rg = ws.Rg; a.Wc = ws.Wc; a.Wt_f32 = ws.Wt_f32; a.dWd = ws.dWd;
  a.Ah = ws.Ah; a.Az = ws.Az; a.Ar = ws.Ar;
  const int64_t nn = (int64_t)n * n;
  a.gW = ws.walk_grads; a.gBz = a.gW + nn; a.gBr = a.gBz + nn; a.gBh = a.gBr + nn;
  if (n > 64) {
    EvPackArgs p{};
    for (int k = 0; k < EV_NPAR; ++k) p.P[k] = a.P[k];
    p.kept = ws.kept;
    p.packed = reinterpret_cast<doublex2*>(ws.walk_packed);
    p.n = n;
    hipLaunchKernelGGL((k_ev_pack<BACK>), blocks_for(evolve_walk_elems(ws) / 2), 256, 0, st, p);
  }
  switch (n / 32) {
    case 1: hipLaunchKernelGGL((k_ev_walk<2, BACK>), n / 4, 256, 0, st, a); break;
    case 2: hipLaunchKernelGGL((k_ev_walk<4, BACK>), n / 4, 512, 0, st, a); break;
    case 3: hipLaunchKernelGGL((k_ev_walk<6, BACK>), n / 4, 768, 0, st, a); break;
    case 4: hipLaunchKernelGGL((k_ev_walk<8, BACK>), n / 4, 1024, 0, st, a); break;
    case 5: hipLaunchKernelGGL((k_ev_walk<10, BACK>), n / 4, 640, 0, st, a); break;
    case 6: hipLaunchKernelGGL((k_ev_walk<12, BACK>), n / 4, 768, 0, st, a); break;
    case 7: hipLaunchKernelGGL((k_ev_walk<14, BACK>), n / 4, 896, 0, st, a); break;
    case 8: hipLaunchKernelGGL((k_ev_walk<16, BACK>), n / 4, 1024, 0, st, a); break;
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
// to fp32, for the dense kernels.
void evolve_forward_weights(const EvolveWs& ws, hipStream_t st) {
  const int64_t nn = (int64_t)ws.F * ws.S;
  launch_walk<false>(ws, st);
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

// Back-propagation through time over the weight recurrence (double precision); the gradients of the ten
// parameters end up in ws.G[k] as fp32.
void evolve_backward_bptt(const EvolveWs& ws, hipStream_t st) {
  launch_walk<true>(ws, st);
  EvGradArgs g{};
  g.T = ws.T; g.n = ws.F; g.Wt = ws.Wt; g.Rg = ws.Rg; g.Ah = ws.Ah; g.Az = ws.Az; g.Ar = ws.Ar; g.walk = ws.walk_grads;
  for (int k = 0; k < EV_NPAR; ++k) g.G[k] = ws.G[k];
  if (ws.F <= 128) hipLaunchKernelGGL((k_ev_grads<16>), dim3(ws.F / 16, ws.F / 16, 8), 512, 0, st, g);
  else hipLaunchKernelGGL((k_ev_grads<32>), dim3(ws.F / 32, ws.F / 32, 8), 512, 0, st, g);
}

}  // namespace dgc
