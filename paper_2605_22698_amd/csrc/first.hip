// First interaction layer, factorised by species.
//
// The first layer's input features are the embedding h0_j = W_emb[z_j] (a
// function of the sender's species only), and its paths are (0, l, l). The
// neighbour sum then factorises exactly:
//   A_i[l, k, m] = nu^-1 sum_e R_e[l, k] W_emb[z_j, k] (C Y_e)[l m]
//                = nu^-1 sum_{s, q} W3[q, l C + k] W_emb[s, k] G_i[s, q, l m],
//   G_i[s, q, l m] = sum_{e in in(i), z_j = s} H2_e[q] (C Y_e)[l m],
// with H2 the radial MLP's second hidden layer. Folding in the channel mix,
//   h~_l = G_l U_l (+ h0 S_0 for l = 0),   U_l = nu^-1 (W3_l o W_emb) W_mix_l,
// so the per-edge output layer of the radial MLP (64 x P C multiply-adds and
// 4 P C bytes of R per edge) is never formed: per edge only the 8 -> 64 -> 64
// hidden layers and a 64 x 16 outer product remain, and U_l is a weight
// computed once per model.
//
// The hidden layers depend on the edge length only, so an edge and its
// reverse share them: the second hidden layer H2 = silu(silu(B W1) W2) and its
// derivative H2' in the length are computed once per edge pair (tiles of 64 pair
// owners, or of 64 edges without the pair list; in FP32 by k_radial_rows, in the
// BF16 mode by k_first_hidden), and both kernels below read them through the
// edge's pair index.
//
// With dG = dh~_l U_l^T the adjoint is one contraction over q, of H2 and of
// H2' with the receiver's rows of the sender's species:
//   d(CY)_e[c] = sum_q H2_e[q]  dG[c, z_j, q]
//   x_e[c]     = sum_q H2'_e[q] dG[c, z_j, q],   dE/dr_e = sum_c (CY)_e[c] x_e[c],
// so neither dH2 nor the hidden layers' own adjoint (a 64 x 64 product per
// edge) is formed.
//
// Kernels:
//   k_first_hidden  [H2 | H2'] [pairs, 128] (BF16 mode)
//   k_first_fwd  G_i [N, (L3+1)^2, S*64]
//   k_first_bwd  g_e = dE/dd_e (added to the other layers')
// The last two give a wave to each (receiver, sender species): it picks the
// species' edges out of the receiver's row (the order of the row is kept) and
// reads the hidden rows and dG straight into matrix-core operands, so no wave
// waits for another. Per launch on the 3,000-atom box (160k edges, 4 species):
// hidden layers 28 us by k_radial_rows, 32 by k_first_hidden (18 without the
// derivative), forward 18 us (23 with a workgroup per receiver and the tile's
// hidden rows in LDS), adjoint 37 us (94 with dH2 and the hidden layers' adjoint
// per edge).
#include "common.h"
#include "paths.h"
#include "runtime.h"

namespace e3mi {
namespace {

constexpr int kTile = 64;
constexpr int kH = 64;
constexpr int kLd = 65;

__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// (C Y)[l m3] = sum_m2 C^{(0,l,l)}[0, m2, m3] Y[l m2] for l <= L3 (and its transpose).
template <int L3>
__device__ __forceinline__ void cg_apply(const float* Y, float* CY) {
  static_for<L3 + 1>([&](auto l) {
    constexpr int lv = decltype(l)::value;
    constexpr int g = [] {
      for (int q = 0; q < kNumPaths; ++q)
        if (kL1[q] == 0 && kL2[q] == lv && kL3[q] == lv) return q;
      return -1;
    }();
    static_assert(g >= 0, "path (0,l,l) missing from the table");
#pragma unroll
    for (int m = 0; m < 2 * lv + 1; ++m) CY[lv * lv + m] = 0.0f;
    static_for<kNzBegin[g + 1] - kNzBegin[g]>([&](auto z) {
      constexpr int q = kNzBegin[g] + z;
      CY[lv * lv + kM3[q]] += kC[q] * Y[lv * lv + kM2[q]];
    });
  });
}
template <int L3>
__device__ __forceinline__ void cg_apply_t(const float* dCY, float* dY) {
  static_for<L3 + 1>([&](auto l) {
    constexpr int lv = decltype(l)::value;
    constexpr int g = [] {
      for (int q = 0; q < kNumPaths; ++q)
        if (kL1[q] == 0 && kL2[q] == lv && kL3[q] == lv) return q;
      return -1;
    }();
#pragma unroll
    for (int m = 0; m < 2 * lv + 1; ++m) dY[lv * lv + m] = 0.0f;
    static_for<kNzBegin[g + 1] - kNzBegin[g]>([&](auto z) {
      constexpr int q = kNzBegin[g] + z;
      dY[lv * lv + kM2[q]] += kC[q] * dCY[lv * lv + kM3[q]];
    });
  });
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// [H2 | H2'] of 64 pair owners (own: the pair list, P = *n_own) or of 64 edges
// (own NULL: every edge inside the cutoff, row_ptr_x[N]), row q for the
// tile's row q.
template <int NB>
__global__ void __launch_bounds__(256) k_first_hidden(const float4* __restrict__ dvec, const int* __restrict__ row_ptr_x,
                                                      int N, const int* __restrict__ own,
                                                      const int* __restrict__ n_own, const float* __restrict__ W1,
                                                      const float* __restrict__ W2, float rc, int p,
                                                      float* __restrict__ H) {
  __shared__ float Bs[kTile][NB + 1], dBs[kTile][NB + 1];
  __shared__ float X[kTile][kLd], dX[kTile][kLd];
  const int n = own ? *n_own : row_ptr_x[N];
  const int q0 = blockIdx.x * kTile;
  if (q0 >= n) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (t < kTile) {
    const int q = q0 + t;
    const int e = q < n ? (own ? own[q] : q) : -1;
    const float r = e >= 0 ? dvec[e].w : rc;
    float b[NB], db[NB];
    radial_basis<NB>(r, rc, p, b, db);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      Bs[t][k] = b[k];
      dBs[t][k] = db[k];
    }
  }
  __syncthreads();
  for (int o = t; o < kTile * kH; o += 256) {
    const int row = o >> 6, col = o & 63;
    float s = 0.0f, ds = 0.0f;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const float wv = W1[k * kH + col];
      s += Bs[row][k] * wv;
      ds += dBs[row][k] * wv;
    }
    X[row][col] = siluf(s);
    dX[row][col] = silu_grad(s) * ds;
  }
  __syncthreads();
  const int rb = (w >> 1) * 32, cb = (w & 1) * 32;
  f32x16 a = {}, da = {};
#pragma unroll 8
  for (int kk = 0; kk < kH; kk += 2) {
    const float wv = W2[(kk + (lane >> 5)) * kH + cb + (lane & 31)];
    a = __builtin_amdgcn_mfma_f32_32x32x2f32(X[rb + (lane & 31)][kk + (lane >> 5)], wv, a, 0, 0, 0);
    da = __builtin_amdgcn_mfma_f32_32x32x2f32(dX[rb + (lane & 31)][kk + (lane >> 5)], wv, da, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int q = q0 + rb + acc_row(r, lane);
    if (q < n) {
      float* row = H + (long)q * 2 * kH + cb + (lane & 31);
      row[0] = siluf(a[r]);
      row[kH] = silu_grad(a[r]) * da[r];
    }
  }
}

// A wave's share of a receiver's row: the edges e of the 64 from e0 on whose
// sender has species s, in row order. Lane k < n holds the k-th: its edge, its
// row of the hidden layers, its vector; (CY) of it is in CY[k] (LDS, the
// wave's own; 17 floats a row keep the column reads conflict-free).
struct SpeciesEdges {
  int n, e, row;
  float4 d;
};
template <int LMAX, int L3>
__device__ __forceinline__ SpeciesEdges species_edges(const float4* __restrict__ dvec, const int* __restrict__ src,
                                                      const int* __restrict__ species,
                                                      const int* __restrict__ pair_of, int e0, int e1, int s,
                                                      float (*CY)[17]) {
  constexpr int NC3 = (L3 + 1) * (L3 + 1);
  const int lane = threadIdx.x & 63;
  const bool mine = e0 + lane < e1 && species[src[e0 + lane]] == s;
  const unsigned long long m = __ballot(mine);
  SpeciesEdges x;
  x.n = __popcll(m);
  // the k-th set bit of m, found by every lane k < n: the set lanes send
  // their offset to their rank
  const int rank = __popcll(m & ((1ull << lane) - 1ull));
  const int to = mine ? rank : x.n + (lane - rank);  // a permutation of the lanes
  const int off = __builtin_amdgcn_ds_permute(to * 4, lane);
  x.e = lane < x.n ? e0 + off : -1;
  x.row = x.e >= 0 ? (pair_of ? pair_of[x.e] : x.e) : 0;
  x.d = x.e >= 0 ? dvec[x.e] : make_float4(0.f, 0.f, 1.f, 1.f);
  float Y[(LMAX + 1) * (LMAX + 1)], cy[NC3];
  const float ir = 1.0f / x.d.w;
  real_sh<LMAX>(x.d.x * ir, x.d.y * ir, x.d.z * ir, Y);
  cg_apply<L3>(Y, cy);
#pragma unroll
  for (int c = 0; c < NC3; ++c) CY[lane][c] = cy[c];
  return x;
}

// LDS written by some lanes of a wave and read by others of it: a wave's LDS
// accesses are done in order, so only the compiler must keep them so
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The (receiver, species) of a wave; false past the last.
__device__ __forceinline__ bool wave_item(int N, int S, int& i, int& s) {
  const int item = __builtin_amdgcn_readfirstlane(xcd_contiguous(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6));
  i = item / S;
  s = item % S;
  return i < N;
}

// Forward: G_i[n = (c, s), q] = sum_e [z_j(e) = s] (CY)_e[c] H2_e[q], a 16
// (component) x 64 (q) product over the species' edges on the matrix cores
// (16x16x4 steps over groups of 4 edges).
template <int LMAX, int L3>
__global__ void __launch_bounds__(256) k_first_fwd(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                   const float4* __restrict__ dvec, const int* __restrict__ species,
                                                   int N, int S, const int* __restrict__ pair_of,
                                                   const float* __restrict__ H, float* __restrict__ G) {
  constexpr int NC3 = (L3 + 1) * (L3 + 1);
  __shared__ float CYs[4][kTile][17];
  int i, s;
  if (!wave_item(N, S, i, s)) return;
  const int lane = threadIdx.x & 63;
  float(*CY)[17] = CYs[threadIdx.x >> 6];
  const int c = lane & 15, h = lane >> 4;
  f32x4 acc[4];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int e1 = row_ptr[i + 1];
  for (int e0 = row_ptr[i]; e0 < e1; e0 += kTile) {
    wave_fence();
    const SpeciesEdges x = species_edges<LMAX, L3>(dvec, src, species, pair_of, e0, e1, s, CY);
    wave_fence();
    for (int k0 = 0; k0 < x.n; k0 += 16) {
      float av[4], bv[4][4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int k = k0 + 4 * g + h;
        const bool on = k < x.n;
        const float* Hr = H + (long)__shfl(x.row, k & 63) * 2 * kH + c;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) bv[g][nb] = on ? Hr[nb * 16] : 0.0f;
        av[g] = on && c < NC3 ? CY[k & 63][c] : 0.0f;
      }
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[nb] = mfma16(av[g], bv[g][nb], acc[nb]);
    }
  }
  float* Gi = G + (long)i * NC3 * S * kH;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int cc = 4 * h + r;
    if (cc < NC3) {
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) Gi[(cc * S + s) * kH + nb * 16 + c] = acc[nb][r];
    }
  }
}

// Adjoint: blocks of 16 of the species' edges against the receiver's 16
// (component) x 64 (q) rows of dG, for H2 and for H2' (16x16x4 steps; lane
// group h takes q = 16 h .. 16 h + 15, so every lane's operands are 16
// consecutive floats of a row).
template <int LMAX, int L3>
__global__ void __launch_bounds__(256) k_first_bwd(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                   const float4* __restrict__ dvec, const int* __restrict__ species,
                                                   int N, int S, const int* __restrict__ pair_of,
                                                   const float* __restrict__ H, const float* __restrict__ dG,
                                                   const float* __restrict__ rows, float4* __restrict__ g,
                                                   int accumulate) {
  constexpr int NC3 = (L3 + 1) * (L3 + 1);
  __shared__ float CYs[4][kTile][17];
  int i, s;
  if (!wave_item(N, S, i, s)) return;
  const int lane = threadIdx.x & 63;
  float(*CY)[17] = CYs[threadIdx.x >> 6];
  const int c = lane & 15, h = lane >> 4;
  float u[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) u[q] = 0.0f;
  if (c < NC3) ldr_n<16>(dG + ((long)i * NC3 * S + c * S + s) * kH + h * 16, u);
  const int e1 = row_ptr[i + 1];
  for (int e0 = row_ptr[i]; e0 < e1; e0 += kTile) {
    wave_fence();
    const SpeciesEdges x = species_edges<LMAX, L3>(dvec, src, species, pair_of, e0, e1, s, CY);
    wave_fence();
    for (int k0 = 0; k0 < x.n; k0 += 16) {
      const float* Hr = H + (long)__shfl(x.row, k0 + c) * 2 * kH + h * 16;  // rows past the last: row 0, not used
      float v[16], dv[16];
      ldr_n<16>(Hr, v);
      ldr_n<16>(Hr + kH, dv);
      f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        a = mfma16(v[q], u[q], a);
        b = mfma16(dv[q], u[q], b);
      }
      // lane (h, c), register r: edge k0 + 4 h + r, component c
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float* cy = CY[k0 + 4 * h + r];
        float t = c < NC3 ? cy[c] * b[r] : 0.0f;
        t += lane_xor1(t);
        t += lane_xor2(t);
        t += lane_xor4(t);
        t += lane_xor8(t);
        wave_fence();
        if (c < NC3) cy[c] = a[r];
        if (c == 0) cy[16] = t;
      }
    }
    wave_fence();
    if (lane < x.n) {
      const float ir = 1.0f / x.d.w;
      const float nx = x.d.x * ir, ny = x.d.y * ir, nz = x.d.z * ir;
      float dcy[NC3], dy[16];
#pragma unroll
      for (int q = 0; q < NC3; ++q) dcy[q] = CY[lane][q];
      float dr = CY[lane][16];
#pragma unroll
      for (int q = 0; q < 16; ++q) dy[q] = 0.0f;
      cg_apply_t<L3>(dcy, dy);
      if (rows) {  // the later layers' share
        float later[16];
        ldr_n<16>(rows + (long)x.e * 16, later);
        dr += later[0];
#pragma unroll
        for (int q = 1; q < (LMAX + 1) * (LMAX + 1); ++q) dy[q] += later[q];
      }
      float Gx, Gy, Gz;
      real_sh_vjp<LMAX>(nx, ny, nz, dy, Gx, Gy, Gz);
      const float dot = Gx * nx + Gy * ny + Gz * nz;
      const float gx = dr * nx + (Gx - dot * nx) * ir;
      const float gy = dr * ny + (Gy - dot * ny) * ir;
      const float gz = dr * nz + (Gz - dot * nz) * ir;
      if (accumulate) {
        const float4 o = g[x.e];
        g[x.e] = make_float4(o.x + gx, o.y + gy, o.z + gz, 0.0f);
      } else {
        g[x.e] = make_float4(gx, gy, gz, 0.0f);
      }
    }
  }
}

}  // namespace

template <int LMAX, int L3>
static void first_launch(bool fwd, const int* row_ptr, const int* src, const float4* dvec, const int* species, int N,
                         int S, const int* pair_of, const float* H, float* G, const float* dG,
                         const float* rows, float4* g, int accumulate, hipStream_t st) {
  const int grid = (int)(((long)N * S + 3) / 4);
  if (fwd)
    k_first_fwd<LMAX, L3><<<grid, 256, 0, st>>>(row_ptr, src, dvec, species, N, S, pair_of, H, G);
  else
    k_first_bwd<LMAX, L3><<<grid, 256, 0, st>>>(row_ptr, src, dvec, species, N, S, pair_of, H, dG, rows, g, accumulate);
}

void launch_first_hidden(const float4* dvec, const int* row_ptr_x, int N, long e_cap, const int* own,
                         const int* n_own, const float* W1, const float* W2, float rc, int p, float* H,
                         hipStream_t st) {
  if (e_cap == 0) return;
  E3MI_REQUIRE((own == nullptr) == (n_own == nullptr), E3MI_EINVAL, "first layer: pair list without its count");
  k_first_hidden<8><<<(int)((e_cap + kTile - 1) / kTile), 256, 0, st>>>(dvec, row_ptr_x, N, own, n_own, W1, W2, rc,
                                                                         p, H);
}

void launch_first(bool fwd, int lmax, int l3max, const int* row_ptr, const int* src, const float4* dvec,
                  const int* species, int N, int S64, const int* pair_of, const float* H, float* G, const float* dG,
                  const float* rows, float4* g, int accumulate, hipStream_t st) {
  if (N == 0) return;
  E3MI_REQUIRE(H, E3MI_EINVAL, "first layer: hidden layers missing");
  const int S = S64 / kH;
  if (lmax == 3 && l3max == 3)
    first_launch<3, 3>(fwd, row_ptr, src, dvec, species, N, S, pair_of, H, G, dG, rows, g, accumulate, st);
  else if (lmax == 3 && l3max == 0)
    first_launch<3, 0>(fwd, row_ptr, src, dvec, species, N, S, pair_of, H, G, dG, rows, g, accumulate, st);
  else if (lmax == 2 && l3max == 2)
    first_launch<2, 2>(fwd, row_ptr, src, dvec, species, N, S, pair_of, H, G, dG, rows, g, accumulate, st);
  else if (lmax == 2 && l3max == 0)
    first_launch<2, 0>(fwd, row_ptr, src, dvec, species, N, S, pair_of, H, G, dG, rows, g, accumulate, st);
  else
    throw Error(E3MI_EUNSUPPORTED, "first-layer factorisation: unsupported orders");
}

}  // namespace e3mi
