// Tensor product + neighbour sum of a scalar-output layer (only the paths
// (l, l, 0): the last layer, whose outputs only the readout reads): the FP32
// forward, and the adjoint from the senders' side, for 64 x CH channels (CH
// adjacent channels per lane, loaded as one vector).
//
// For an edge e = (i <- j) with direction d_e the forward gives
//   A[i,p,k] = nu^-1 sum_e R[e,p,k] T[e,p,k],  T[e,p,k] = sum_m C^p[m,m,0] h[j,k,l m] Y_e[l m],
// so the adjoint needs, per edge,
//   dR[e,p,k]  = nu^-1 dA[i,p,k] T[e,p,k]
//   dY[e,l m]  = nu^-1 sum_{p,k} C^p R[e,p,k] dA[i,p,k] h[j,k,l m]
// and per sender
//   dh[j,k,l m] = nu^-1 sum_{e: src(e) = j} C^p R[e,p,k] dA[i,p,k] Y_e[l m].
// A workgroup owns a sender j, holds h_j in registers and walks j's own
// incoming edges e' = (j <- i): each stands for j's outgoing edge e = rev(e') = (i <- j),
// with d_e = -d_e', R_e = R_e' (R depends on |d| only) and dA_i gathered
// (NP x C values, where a receiver-side pass gathers h_j, (L+1)^2 x C, per
// edge). dh_j is summed in registers in an order that j's row alone fixes, so
// the result does not depend on other structures in the batch.
//
// In FP32 R' comes with R, and the edge's dE/dr = sum dR_e R'_e takes
// the place of dR_e (and of the radial MLP's adjoint); it is stored as dY's
// first value, which the constant l = 0 harmonic leaves free. The BF16 mode
// writes dR_e for its radial adjoint on the BF16 matrix cores.
//
// dR_e and dY_e are stored in the slot of e' (j's own row, contiguous, and
// inside a receiver chunk when j is), dY_e with the sign (-1)^l: it is then the
// adjoint of the harmonics of e''s own direction (Y_l(-n) = (-1)^l Y_l(n)),
// and the radial adjoint of slot e' yields the gradient with respect to d_e'
// = -d_e, i.e. minus e's. Forces F_i = sum_{e in in(i)} (g_e - g_rev(e)) take
// each edge with both signs, so the forces are the same. An edge inside the
// cutoff whose reverse is not (its FP64 length within rounding of r_c, where
// the envelope and its derivatives vanish) gets zeros.
#include <type_traits>

#include "common.h"
#include "paths.h"
#include "runtime.h"

namespace e3mi {
namespace {

// dR and dY are streamed out with non-temporal stores (not kept in the
// caches), so that they do not evict the R rows this pass still has to read
template <int n>
__device__ __forceinline__ void str_nt(__bf16* p, const float* v) {
  typedef __bf16 bvec __attribute__((ext_vector_type(n)));
  bvec t;
#pragma unroll
  for (int q = 0; q < n; ++q) t[q] = (__bf16)v[q];
  __builtin_nontemporal_store(t, reinterpret_cast<bvec*>(p));
}

// Forward of the layer in FP32: a workgroup of C x S threads per receiver, a
// thread per channel and stream; stream s takes the edges s, s + S, ... of the
// row and the streams' sums meet in LDS, added in their order.
// Bound: the senders' rows (8 KB an edge in models of 128) out of the L2s; on
// small systems the chain of a row's edges. us with one, two and four streams:
// 24 atoms 10.5, 6.5, 5.0; 138 atoms 24, 14, 9; 1,205 atoms 34, 36, 31; 3,000
// atoms 99, 102, 95; 64 charged clusters 158, 154, 144; 20,000 atoms 1,275,
// 1,290, 1,310. Two adjacent channels a lane with the next edge's rows loaded
// ahead: 14 on 138 atoms, 134 on 3,000 (four streams).
template <int LMAX, int KIND, int S, bool WAVES>
__global__ void __launch_bounds__(128 * S) __attribute__((amdgpu_waves_per_eu(1, 3))) k_tps_fwd(
    const int* __restrict__ row_ptr, const int* __restrict__ src, const float4* __restrict__ dvec,
    const float* __restrict__ R, int r_stride, const float* __restrict__ h, int h_nc, float* __restrict__ A, int C,
    float inv_nu, int i0, int r_first, const int* __restrict__ r_row) {
  using PS = PathSet<LMAX, KIND>;
  constexpr int NP = PS::NP, NIN = PS::NIN, NY = PS::NY;
  static_assert(PS::NOUT == NP, "scalar outputs only");
  __shared__ float part[S][NP][128];
  const int i = i0 + xcd_contiguous(blockIdx.x, gridDim.x);
  const int k = threadIdx.x;
  // WAVES: whole waves per stream (C a multiple of 64)
  const int s = WAVES ? __builtin_amdgcn_readfirstlane(threadIdx.y) : threadIdx.y;
  float acc[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) acc[p] = 0.0f;
  const int e1 = row_ptr[i + 1];
  for (int e = row_ptr[i] + s; e < e1; e += S) {
    const float4 d = dvec[e];
    const float ir = 1.0f / d.w;
    float Y[NY], hv[NIN], rv[NP];
    real_sh<LMAX>(d.x * ir, d.y * ir, d.z * ir, Y);
    const float* Re = R + (long)(r_row ? r_row[e] : e - r_first) * r_stride;
    const float* hj = h + (long)src[e] * h_nc * C;
#pragma unroll
    for (int q = 0; q < NIN; ++q) hv[q] = hj[q * C + k];
#pragma unroll
    for (int p = 0; p < NP; ++p) rv[p] = Re[p * C + k];
    static_for<NP>([&](auto pi) {
      constexpr int g = PS::T.id[pi];
      constexpr int l1 = kL1[g], l2 = kL2[g];
      constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
      static_assert(one_coefficient(g), "paths (l, l, 0)");
      float t = 0.0f;
      static_for<nz>([&](auto z) {
        constexpr int q = z0 + z;
        t += hv[l1 * l1 + kM1[q]] * Y[l2 * l2 + kM2[q]];
      });
      acc[pi] += rv[pi] * t;
    });
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) part[s][p][k] = acc[p];
  __syncthreads();
  static_for<NP>([&](auto pi) {
    if (pi % S != s) return;
    constexpr int g = PS::T.id[pi];
    float sum = 0.0f;
#pragma unroll
    for (int x = 0; x < S; ++x) sum += part[x][pi][k];
    A[((long)i * NP + PS::T.rank[pi]) * C + k] = sum * (kC[kNzBegin[g]] * inv_nu);
  });
}

// FP32: W waves per sender, wave w taking the edges w, w + W, ... of the row,
// each CH adjacent channels per lane (lanes past the last channel, in models
// of 32, contribute nothing). One wave per sender leaves three waves per SIMD
// on a 3,000-atom system and a chain of 50 edges per wave; the waves' shares of
// dh_j meet in LDS at the end, added in the order of the waves. One, two and
// four waves cost the same on 3,000 atoms (125 us: the gathers bound it); on
// 138 atoms four take 16 us where one, writing dR, took 66.
template <int LMAX, int KIND, int CH, bool DH, int W>
__global__ void __launch_bounds__(64 * W) k_tps_sender(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                       const int* __restrict__ rev, const float4* __restrict__ dvec,
                                                       const float* __restrict__ R, const float* __restrict__ Rp,
                                                       const float* __restrict__ h,
                                                       int h_nc, const float* __restrict__ dA,
                                                       float* __restrict__ dY, float* __restrict__ dh, int dh_nc,
                                                       int dh_acc, int C, float inv_nu, int i0, int r_first,
                                                       const int* __restrict__ r_row) {
  using PS = PathSet<LMAX, KIND>;
  constexpr int NP = PS::NP, NIN = PS::NIN, NY = PS::NY;
  constexpr int NA = DH ? NIN : 1;
  static_assert(PS::NOUT == NP, "scalar outputs only");
  __shared__ float part[DH ? W : 1][DH ? NIN : 1][64 * CH];
  const int j = i0 + xcd_contiguous(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool on = lane * CH < C;
  const unsigned k0 = (on ? lane * CH : lane * CH - C) & 127;
  const float scale = on ? inv_nu : 0.0f;
  float hv[NIN][CH];
#pragma unroll
  for (int q = 0; q < NIN; ++q) ldr_n<CH>(h + ((long)j * h_nc + q) * C + k0, hv[q]);
  float acc[NA][CH];
#pragma unroll
  for (int q = 0; q < NA; ++q)
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[q][c] = 0.0f;
  // software pipeline: the indices of the edge after next and the R, R' and dA
  // rows of the next are in flight while an edge is processed (the rows of a
  // sender's edges lie far apart)
  const int eb = row_ptr[j] + w, e1 = row_ptr[j + 1];
  struct Idx {
    int rev, i, row;
    float4 d;
  };
  auto load_idx = [&](int e) {
    Idx x;
    x.rev = rev[e];
    x.i = src[e];
    x.row = r_row ? r_row[e] : e - r_first;
    x.d = dvec[e];
    return x;
  };
  auto load_rows = [&](const Idx& x, float (&oR)[2 * NP][CH], float (&oA)[NP][CH]) {
    if (x.rev < 0) return;
    const float* Re = R + (long)x.row * NP * C;
    const float* Rpe = Rp + (long)x.row * NP * C;
    const float* dAi = dA + (long)x.i * NP * C;
    static_for<NP>([&](auto pi) {
      ldr_n<CH>(Re + pi * C + k0, oR[pi]);
      ldr_n<CH>(Rpe + pi * C + k0, oR[NP + pi]);
      ldr_n<CH>(dAi + PS::T.rank[pi] * C + k0, oA[pi]);
    });
  };
  float nR[2 * NP][CH], nA[NP][CH];
  Idx nx{-1, 0, 0, make_float4(0.f, 0.f, 1.f, 1.f)}, nnx = nx;
  if (eb < e1) {
    nx = load_idx(eb);
    load_rows(nx, nR, nA);
  }
  if (eb + W < e1) nnx = load_idx(eb + W);
  for (int e2 = eb; e2 < e1; e2 += W) {
    const Idx cx = nx;
    float cR[2 * NP][CH], cA[NP][CH];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        cR[p][c] = nR[p][c];
        cR[NP + p][c] = nR[NP + p][c];
        cA[p][c] = nA[p][c];
      }
    if (e2 + W < e1) {
      nx = nnx;
      load_rows(nx, nR, nA);
      if (e2 + 2 * W < e1) nnx = load_idx(e2 + 2 * W);
    }
    if (cx.rev < 0) {  // the edge i <- j is not in i's list
      if (lane < 16) dY[(long)e2 * 16 + lane] = 0.0f;
      continue;
    }
    const float ir = -1.0f / cx.d.w;  // d_e = -d_e2
    float Y[NY], dyp[NY];
    real_sh<LMAX>(cx.d.x * ir, cx.d.y * ir, cx.d.z * ir, Y);
#pragma unroll
    for (int q = 0; q < NY; ++q) dyp[q] = 0.0f;
    static_for<NP>([&](auto pi) {
      constexpr int g = PS::T.id[pi];
      constexpr int l1 = kL1[g], l2 = kL2[g];
      constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
      static_assert(one_coefficient(g), "paths (l, l, 0)");
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const float dai = cA[pi][c] * (kC[z0] * scale);
        const float u = cR[pi][c] * dai;
        float t = 0.0f;
        static_for<nz>([&](auto z) {
          constexpr int q = z0 + z;
          constexpr int q1 = l1 * l1 + kM1[q], q2 = l2 * l2 + kM2[q];
          t += hv[q1][c] * Y[q2];
          if constexpr (l2 > 0) dyp[q2] += hv[q1][c] * u;
          if constexpr (DH) acc[q1][c] += u * Y[q2];
        });
        dyp[0] += (dai * t) * cR[NP + pi][c];
      }
    });
    const float tot = wave_sum_scatter16<NY>(dyp);
    const int q = lane >> 2;
    // (-1)^l for component q = l^2 + m + l: odd for q in 1..3 and 9..15
    const bool odd = (q >= 1 && q <= 3) || q >= 9;
    if ((lane & 3) == 0 && q < NY) dY[(long)e2 * 16 + q] = odd ? -tot : tot;
  }
  if constexpr (DH) {
#pragma unroll
    for (int q = 0; q < NIN; ++q) str_n<CH>(&part[w][q][lane * CH], acc[q]);
    __syncthreads();
    if (!on) return;
    // components below dh_acc (all when dh_acc <= 0) are added to, the others
    // written (zero past the paths' inputs); wave w takes components w, w + W, ...
#pragma unroll
    for (int q = 0; q < NIN; ++q) {
      if (q % W != w) continue;
      float* o = dh + ((long)j * dh_nc + q) * C + k0;
      float v[CH];
      const bool add = dh_acc <= 0 || q < dh_acc;
      if (add) ldr_n<CH>(o, v);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        float sum = add ? v[c] : 0.0f;
#pragma unroll
        for (int x = 0; x < W; ++x) sum += part[x][q][lane * CH + c];
        v[c] = sum;
      }
      str_n<CH>(o, v);
    }
    if (dh_acc > 0 && w == 0)
      for (int q = NIN; q < dh_nc; ++q)
        if (q >= dh_acc) {
          const float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
          str_n<CH>(dh + ((long)j * dh_nc + q) * C + k0, z);
        }
  }
}

// The BF16 mode's pass, one wave per sender.
template <int LMAX, int KIND, int CH, bool DH>
__global__ void __launch_bounds__(64) k_tps_bwd_sender(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                       const int* __restrict__ rev, const float4* __restrict__ dvec,
                                                       const __bf16* __restrict__ R, int r_stride,
                                                       const float* __restrict__ h, int h_nc,
                                                       const float* __restrict__ dA, __bf16* __restrict__ dR,
                                                       float* __restrict__ dY, float* __restrict__ dh, int dh_nc,
                                                       int dh_acc, int C, float inv_nu, int i0, int e_first,
                                                       const int* __restrict__ r_row, int r_first) {
  using PS = PathSet<LMAX, KIND>;
  constexpr int NP = PS::NP, NIN = PS::NIN, NY = PS::NY;
  constexpr int NA = DH ? NIN : 1;
  static_assert(PS::NOUT == NP, "scalar outputs only");
  const int j = i0 + xcd_contiguous(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x;
  const int k0 = lane * CH;
  float hv[NIN][CH];
  {
    const float* hj = h + (long)j * h_nc * C + k0;
#pragma unroll
    for (int q = 0; q < NIN; ++q) ldr_n<CH>(hj + q * C, hv[q]);
  }
  float acc[NA][CH];
#pragma unroll
  for (int q = 0; q < NA; ++q)
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[q][c] = 0.0f;
  // Software pipeline over j's row: the indices of edge e2 + 2 and the R and dA
  // rows of edge e2 + 1 are in flight while edge e2 is processed (the rows of
  // consecutive edges lie far apart, and a wave owns one sender).
  const int eb = row_ptr[j], e1 = row_ptr[j + 1];
  struct Idx {
    int rev, i, row;
    float4 d;
  };
  auto load_idx = [&](int e) {
    Idx x;
    x.rev = rev[e];
    x.i = src[e];
    x.row = r_row ? r_row[e] : e - r_first;
    x.d = dvec[e];
    return x;
  };
  auto load_rows = [&](const Idx& x, float (&oR)[NP][CH], float (&oA)[NP][CH]) {
    if (x.rev < 0) return;
    const __bf16* Re = R + (long)x.row * r_stride + k0;
    const float* dAi = dA + (long)x.i * NP * C + k0;
    static_for<NP>([&](auto pi) {
      ldr_n<CH>(Re + pi * C, oR[pi]);
      ldr_n<CH>(dAi + PS::T.rank[pi] * C, oA[pi]);
    });
  };
  float nR[NP][CH], nA[NP][CH];
  Idx nx{-1, 0, 0, make_float4(0.f, 0.f, 1.f, 1.f)}, nnx = nx;
  if (eb < e1) {
    nx = load_idx(eb);
    load_rows(nx, nR, nA);
  }
  if (eb + 1 < e1) nnx = load_idx(eb + 1);
  for (int e2 = eb; e2 < e1; ++e2) {
    const Idx cx = nx;
    float cR[NP][CH], cA[NP][CH];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        cR[p][c] = nR[p][c];
        cA[p][c] = nA[p][c];
      }
    if (e2 + 1 < e1) {
      nx = nnx;
      load_rows(nx, nR, nA);
      if (e2 + 2 < e1) nnx = load_idx(e2 + 2);
    }
    __bf16* dRe = dR + (long)(e2 - e_first) * r_stride + k0;
    if (cx.rev < 0) {  // the edge i <- j is not in i's list
      const float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      static_for<NP>([&](auto pi) { str_nt<CH>(dRe + pi * C, z); });
      if (lane < 16) __builtin_nontemporal_store(0.0f, dY + (long)e2 * 16 + lane);
      continue;
    }
    const float4 d = cx.d;
    const float ir = -1.0f / d.w;  // d_e = -d_e2
    float Y[NY];
    real_sh<LMAX>(d.x * ir, d.y * ir, d.z * ir, Y);
    float dyp[NY];
#pragma unroll
    for (int q = 0; q < NY; ++q) dyp[q] = 0.0f;
    static_for<NP>([&](auto pi) {
      constexpr int g = PS::T.id[pi];
      constexpr int l1 = kL1[g], l2 = kL2[g];
      constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
      float s[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const float dai = cA[pi][c] * inv_nu;
        const float u = cR[pi][c] * dai;
        float t = 0.0f;
        static_for<nz>([&](auto z) {
          constexpr int q = z0 + z;
          const float cy = kC[q] * Y[l2 * l2 + kM2[q]];
          t += hv[l1 * l1 + kM1[q]][c] * cy;
          dyp[l2 * l2 + kM2[q]] += kC[q] * (hv[l1 * l1 + kM1[q]][c] * u);
          if constexpr (DH) acc[l1 * l1 + kM1[q]][c] += u * cy;
        });
        s[c] = dai * t;
      }
      str_nt<CH>(dRe + pi * C, s);
    });
    const float tot = wave_sum_scatter16<NY>(dyp);
    const int q = lane >> 2;
    // (-1)^l for component q = l^2 + m + l: odd for q in 1..3 and 9..15
    const bool odd = (q >= 1 && q <= 3) || q >= 9;
    if ((lane & 3) == 0 && q < NY) __builtin_nontemporal_store(odd ? -tot : tot, dY + (long)e2 * 16 + q);
  }
  if constexpr (DH) {
    // components below dh_acc (all when dh_acc <= 0) are added to, the others
    // written (zero past the paths' inputs)
#pragma unroll
    for (int q = 0; q < NIN; ++q) {
      float* o = dh + ((long)j * dh_nc + q) * C + k0;
      float v[CH];
      const bool add = dh_acc <= 0 || q < dh_acc;
      if (add) ldr_n<CH>(o, v);
#pragma unroll
      for (int c = 0; c < CH; ++c) v[c] = (add ? v[c] : 0.0f) + acc[q][c];
      str_n<CH>(o, v);
    }
    if (dh_acc > 0)
      for (int q = NIN; q < dh_nc; ++q)
        if (q >= dh_acc) {
          const float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
          str_n<CH>(dh + ((long)j * dh_nc + q) * C + k0, z);
        }
  }
}

template <int LMAX, int KIND, int CH>
void sender_launch_bf16(const TpArgs& a, int nr, hipStream_t st) {
  const __bf16* R = reinterpret_cast<const __bf16*>(a.R);
  __bf16* dR = reinterpret_cast<__bf16*>(a.dR);
  if (a.dh)
    k_tps_bwd_sender<LMAX, KIND, CH, true><<<nr, 64, 0, st>>>(a.row_ptr, a.src, a.rev, a.dvec, R, a.r_stride, a.h,
                                                              a.h_nc, a.dA, dR, a.dY, a.dh, a.dh_nc, a.dh_acc, a.C,
                                                              a.inv_nu, a.i0, a.e_first, a.r_row, a.r_first);
  else
    k_tps_bwd_sender<LMAX, KIND, CH, false><<<nr, 64, 0, st>>>(a.row_ptr, a.src, a.rev, a.dvec, R, a.r_stride, a.h,
                                                               a.h_nc, a.dA, dR, a.dY, nullptr, 0, 0, a.C, a.inv_nu,
                                                               a.i0, a.e_first, a.r_row, a.r_first);
}

constexpr int kSenderWaves = 4, kFwdStreams = 4;

template <int LMAX, int KIND, int CH>
void sender_launch(const TpArgs& a, int nr, hipStream_t st) {
  constexpr int W = kSenderWaves;
  if (a.dh)
    k_tps_sender<LMAX, KIND, CH, true, W><<<nr, 64 * W, 0, st>>>(a.row_ptr, a.src, a.rev, a.dvec, a.R, a.Rp, a.h, a.h_nc,
                                                                 a.dA, a.dY, a.dh, a.dh_nc, a.dh_acc, a.C, a.inv_nu,
                                                                 a.i0, a.r_first, a.r_row);
  else
    k_tps_sender<LMAX, KIND, CH, false, W><<<nr, 64 * W, 0, st>>>(a.row_ptr, a.src, a.rev, a.dvec, a.R, a.Rp, a.h, a.h_nc,
                                                                  a.dA, a.dY, nullptr, 0, 0, a.C, a.inv_nu, a.i0,
                                                                  a.r_first, a.r_row);
}

template <int LMAX, int KIND>
void fwd_kind(const TpArgs& a, int nr, hipStream_t st) {
  constexpr int S = kFwdStreams;
  auto go = [&](auto waves) {
    k_tps_fwd<LMAX, KIND, S, decltype(waves)::value><<<nr, dim3(a.C, S), 0, st>>>(
        a.row_ptr, a.src, a.dvec, a.R, a.r_stride, a.h, a.h_nc, a.A, a.C, a.inv_nu, a.i0, a.r_first, a.r_row);
  };
  if (a.C == 128 || a.C == 64) go(std::true_type{});
  else if (a.C == 32) go(std::false_type{});
  else throw Error(E3MI_EUNSUPPORTED, "scalar-output tensor product: unsupported channels");
}

template <int LMAX, int KIND>
void tps_kind(const TpArgs& a, int nr, hipStream_t st) {
  if (a.r_bf16) {
    if (a.C == 64) return sender_launch_bf16<LMAX, KIND, 1>(a, nr, st);
    if (a.C == 128) return sender_launch_bf16<LMAX, KIND, 2>(a, nr, st);
  } else {
    if (a.C == 32 || a.C == 64) return sender_launch<LMAX, KIND, 1>(a, nr, st);
    if (a.C == 128) return sender_launch<LMAX, KIND, 2>(a, nr, st);
  }
  throw Error(E3MI_EUNSUPPORTED, "scalar-output tensor product: unsupported channels");
}

// One thread per edge: the position adjoint of its row.
template <int LMAX>
__global__ void __launch_bounds__(256) k_edge_geo(const int* __restrict__ row_ptr_x, int N,
                                                  const float4* __restrict__ dvec, const float* __restrict__ rows,
                                                  int accumulate, float4* __restrict__ g) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= row_ptr_x[N]) return;
  const float4 d = dvec[e];
  const float ir = 1.0f / d.w;
  const float nx = d.x * ir, ny = d.y * ir, nz = d.z * ir;
  float dy[16];
  ldr_n<16>(rows + (long)e * 16, dy);
  float Gx, Gy, Gz;
  real_sh_vjp<LMAX>(nx, ny, nz, dy, Gx, Gy, Gz);
  const float dot = Gx * nx + Gy * ny + Gz * nz;
  float gx = dy[0] * nx + (Gx - dot * nx) * ir;
  float gy = dy[0] * ny + (Gy - dot * ny) * ir;
  float gz = dy[0] * nz + (Gz - dot * nz) * ir;
  if (accumulate) {
    const float4 o = g[e];
    gx += o.x;
    gy += o.y;
    gz += o.z;
  }
  g[e] = make_float4(gx, gy, gz, 0.0f);
}

}  // namespace

bool tps_supported(const TpArgs& a) {
  return (a.kind == kLast || a.kind == kFirstLast) && ((a.C == 32 && !a.r_bf16) || a.C == 64 || a.C == 128) &&
         (a.lmax == 2 || a.lmax == 3);
}

void launch_tps_sender(const TpArgs& a, hipStream_t st) {
  if (a.N == 0) return;
  E3MI_REQUIRE(tps_supported(a), E3MI_EUNSUPPORTED, "sender-side adjoint: unsupported layer");
  E3MI_REQUIRE(a.rev, E3MI_EINVAL, "sender-side adjoint: needs the reverse edges");
  E3MI_REQUIRE((a.r_bf16 != 0) != (a.Rp != nullptr), E3MI_EINVAL, "sender-side adjoint: R' rows in FP32, dR in BF16");
  // senders i0 .. i0 + nr - 1: their rows hold the chunk's R
  const int nr = a.n_recv > 0 ? a.n_recv : a.N;
  if (a.n_recv == 0 && (a.i0 != 0 || a.e_first != 0 || a.r_first != 0))
    throw Error(E3MI_EINVAL, "tensor product: receiver offset without a receiver count");
  if (a.lmax == 2) {
    if (a.kind == kLast) return tps_kind<2, kLast>(a, nr, st);
    return tps_kind<2, kFirstLast>(a, nr, st);
  }
  if (a.kind == kLast) return tps_kind<3, kLast>(a, nr, st);
  return tps_kind<3, kFirstLast>(a, nr, st);
}

void launch_tps_fwd(const TpArgs& a, hipStream_t st) {
  if (a.N == 0) return;
  E3MI_REQUIRE(tps_supported(a) && !a.r_bf16, E3MI_EUNSUPPORTED, "scalar-output tensor product: unsupported layer");
  const int nr = a.n_recv > 0 ? a.n_recv : a.N;
  if (a.n_recv == 0 && (a.i0 != 0 || a.r_first != 0))
    throw Error(E3MI_EINVAL, "tensor product: receiver offset without a receiver count");
  if (a.lmax == 2) {
    if (a.kind == kLast) return fwd_kind<2, kLast>(a, nr, st);
    return fwd_kind<2, kFirstLast>(a, nr, st);
  }
  if (a.kind == kLast) return fwd_kind<3, kLast>(a, nr, st);
  return fwd_kind<3, kFirstLast>(a, nr, st);
}

void launch_edge_geo(int lmax, const int* row_ptr_x, int N, long e_cap, const float4* dvec, const float* rows,
                     int accumulate, float4* g, hipStream_t st) {
  if (e_cap == 0) return;
  const int grid = (int)((e_cap + 255) / 256);
  if (lmax == 3)
    k_edge_geo<3><<<grid, 256, 0, st>>>(row_ptr_x, N, dvec, rows, accumulate, g);
  else
    k_edge_geo<2><<<grid, 256, 0, st>>>(row_ptr_x, N, dvec, rows, accumulate, g);
}

}  // namespace e3mi
