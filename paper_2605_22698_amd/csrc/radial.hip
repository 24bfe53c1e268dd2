// Radial MLP per edge (NequIP table of Appendix F: 8 Bessel functions, a
// radial net of two hidden layers of 64 with swish, polynomial envelope; one
// output weight per (path, channel), no biases):
//   B = bessel(r) u(r/rc);  H1 = silu(B W1);  H2 = silu(H1 W2);  R = H2 W3
// FP32 takes R with its derivatives in the edge length (k_radial_rows), which
// make the MLP's adjoint a dot product. The BF16 mode evaluates R and the
// adjoint of the MLP, ending in the geometric gradient of every edge:
//   dr = dR . dR/dr  (through the MLP and the basis),
//   g_e = dE/dd_e = dr d^ + (I - d^ d^T)/r grad_Y(d^) . dY
// Weight gradients go back through the MLP from the adjoints of R and R'
// (k_radial_wgrad).
//
// One workgroup (4 waves) owns a tile of 64 consecutive rows (edges or pairs).
// The 64x64 hidden layer and the 64 x (P C) output layer are dense contractions
// and run on the matrix cores, each wave with 32x32 output blocks. The row
// count is read on the device (row_ptr_x[N], or the pair count); the grid is
// sized for the skin-list capacity and surplus tiles exit at once.
//
// An edge and its reverse have exactly opposite vectors, so equal lengths and
// equal R. With the pair owners of the pruned list given (own[0 .. P), P on
// the device), a tile holds 64 owners instead of 64 edges: R is computed once
// per pair and stored in the pair's row (the tensor-product kernels find an
// edge's row through its pair index), and the adjoint takes dR of the pair's
// two edges summed (E depends on the pair's length through both) through the
// MLP once; the length gradient goes to the owner's g and each edge keeps its
// own harmonics term. F_i sums g_e - g_rev(e) over i's edges, so the forces are
// those of the edge-by-edge adjoint (to rounding).
//
// MFMA 32x32x2 operand layout (wave64): lane l supplies A[l%32][l/32] and
// B[l/32][l%32]; accumulator register r of lane l holds
// D[8 (r/4) + 4 (l/32) + r%4][l%32].
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "runtime.h"

namespace e3mi {
namespace {

constexpr int kTile = 64;
constexpr int kH = 64;  // hidden width
constexpr int kLd = 65; // padded LDS row

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// H1 = silu(B W1) (K = NB) on the vector ALU; 256 threads x 16 outputs.
template <int NB>
__device__ __forceinline__ void layer1(const float (*Bs)[NB + 1], const float* __restrict__ W1, float (*H1)[kLd]) {
  const int t = threadIdx.x;
  const int row = t >> 2, cb = (t & 3) * 16;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    float s = 0.0f;
#pragma unroll
    for (int n = 0; n < NB; ++n) s += Bs[row][n] * W1[n * kH + cb + j];
    H1[row][cb + j] = siluf(s);
  }
}

// The BF16 mode's products: operands rounded to BF16 (nearest even) and
// multiplied on v_mfma_f32_32x32x16_bf16 (lane l supplies A[l%32][8 (l/32) ..
// +8] and B[8 (l/32) .. +8][l%32]), FP32 accumulation.
// BF16 operands already rounded and laid out for the 32x32x16 steps: rows of
// X in LDS as BF16 (row stride kLdb, 16-byte aligned), and the weights
// transposed so that each output column's K values are contiguous (WT[col *
// ldk + k]). Lane l then loads its 8 A and 8 B values with one 16-byte read
// each; the values are the ones the conversions at use produce (round to
// nearest even of the same FP32 numbers), so the results are the same.
constexpr int kLdb = 72;
__device__ __forceinline__ f32x16 block_64_bf(const __bf16 (*Xb)[kLdb], int rb, const __bf16* __restrict__ WT, int ldk,
                                              int cb) {
  const int lane = threadIdx.x & 63;
  f32x16 acc = {};
#pragma unroll
  for (int kb = 0; kb < kH; kb += 16) {
    const int k0 = kb + 8 * (lane >> 5);
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(&Xb[rb + (lane & 31)][k0]);
    const bf16x8 b = *reinterpret_cast<const bf16x8*>(WT + (long)(cb + (lane & 31)) * ldk + k0);
    acc = mfma_bf(a, b, acc);
  }
  return acc;
}

// rows 0-31 and 32-63 of Xb times the columns cc .. cc+31 of W (WT = W^T, K = 64)
__device__ __forceinline__ void block_64x2_bf(const __bf16 (*Xb)[kLdb], const __bf16* __restrict__ WT, int cc,
                                              f32x16& a0, f32x16& a1) {
  const int lane = threadIdx.x & 63;
  a0 = f32x16{};
  a1 = f32x16{};
#pragma unroll
  for (int kb = 0; kb < kH; kb += 16) {
    const int k0 = kb + 8 * (lane >> 5);
    const bf16x8 b = *reinterpret_cast<const bf16x8*>(WT + (long)(cc + (lane & 31)) * kH + k0);
    const bf16x8 x0 = *reinterpret_cast<const bf16x8*>(&Xb[lane & 31][k0]);
    const bf16x8 x1 = *reinterpret_cast<const bf16x8*>(&Xb[32 + (lane & 31)][k0]);
    a0 = mfma_bf(x0, b, a0);
    a1 = mfma_bf(x1, b, a1);
  }
}

// the 64 x 64 floats of X rounded into Xb (all 256 threads)
__device__ __forceinline__ void to_bf16_tile(const float (*X)[kLd], __bf16 (*Xb)[kLdb]) {
  for (int o = threadIdx.x; o < kTile * kH; o += 256) Xb[o >> 6][o & 63] = (__bf16)X[o >> 6][o & 63];
}

template <int NB, class RS, bool PAIR>
__global__ void __launch_bounds__(256) k_radial_fwd(const float4* __restrict__ dvec, const int* __restrict__ row_ptr_x,
                                                    int N, const float* __restrict__ W1, int PC,
                                                    RS* __restrict__ R, float rc, int p, int e_first, int e_end,
                                                    const __bf16* __restrict__ W2Tb,
                                                    const __bf16* __restrict__ W3Tb, const int* __restrict__ own,
                                                    const int* __restrict__ n_own) {
  // edges [e_first, e_end) (e_end < 0: every edge inside the cutoff); R is
  // indexed from e_first. W2Tb = W2^T and W3Tb = W3^T (used columns) in
  // BF16. PAIR: the tile's rows are pair owners (e_first = 0, e_end < 0) and R
  // is written to the pair's row
  __shared__ float Bs[kTile][NB + 1];
  __shared__ float H[kTile][kLd];
  __shared__ __align__(16) __bf16 Hb[kTile][kLdb];
  const int E = PAIR ? *n_own : e_end >= 0 ? e_end : row_ptr_x[N];
  const int e0 = (PAIR ? 0 : e_first) + blockIdx.x * kTile;
  if (e0 >= E) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (t < kTile) {
    const int q = e0 + t;
    const int e = q < E ? (PAIR ? own[q] : q) : -1;
    const float r = e >= 0 ? dvec[e].w : rc;
    float b[NB];
    radial_basis<NB>(r, rc, p, b, nullptr);
#pragma unroll
    for (int n = 0; n < NB; ++n) Bs[t][n] = b[n];
  }
  __syncthreads();
  layer1<NB>(Bs, W1, H);
  __syncthreads();
  to_bf16_tile(H, Hb);
  __syncthreads();
  {
    const int rb = (w >> 1) * 32, cb = (w & 1) * 32;
    const f32x16 acc = block_64_bf(Hb, rb, W2Tb, kH, cb);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) Hb[rb + acc_row(r, lane)][cb + (lane & 31)] = (__bf16)siluf(acc[r]);
  }
  __syncthreads();
  for (int cc = w * 32; cc < PC; cc += 128) {
    f32x16 a0, a1;
    block_64x2_bf(Hb, W3Tb, cc, a0, a1);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = acc_row(r, lane);
      const int ea = e0 + row, eb = e0 + 32 + row;  // rows in order: edges, or pair indices
      if (ea < E) str(R + (long)(ea - e_first) * PC + cc + (lane & 31), a0[r]);
      if (eb < E) str(R + (long)(eb - e_first) * PC + cc + (lane & 31), a1[r]);
    }
  }
}

template <int NB, int LMAX, class RS, bool PAIR>
__global__ void __launch_bounds__(256) k_radial_bwd(const float4* __restrict__ dvec, const int* __restrict__ row_ptr_x,
                                                    int N, const float* __restrict__ W1, int PC,
                                                    const RS* __restrict__ dR, const float* __restrict__ dY,
                                                    float4* __restrict__ g, int accumulate, float rc, int p,
                                                    int e_first, int e_end, const __bf16* __restrict__ W2Tb,
                                                    const __bf16* __restrict__ W2b,
                                                    const __bf16* __restrict__ W3ub, const int* __restrict__ own,
                                                    const int* __restrict__ n_own, const int* __restrict__ rev) {
  // W2Tb = W2^T, W2b = W2 and W3ub = W3 (used columns) in BF16, W3 in
  // slabs of 32 columns: W3ub[((c / 32) * 64 + q) * 32 + c % 32] = W3[q][c]
  __shared__ float Bs[kTile][NB + 1];
  __shared__ float dBs[kTile][NB + 1];
  __shared__ float P2[kTile][kLd];
  __shared__ float X[kTile][kLd];
  __shared__ __align__(16) __bf16 Xb[kTile][kLdb];
  __shared__ __align__(16) __bf16 Dsb[kTile][40];
  __shared__ int Es[PAIR ? kTile : 1], Ps[PAIR ? kTile : 1];  // owners and partners (-1: none)
  // edges [e_first, e_end) (e_end < 0: every edge inside the cutoff); dR is
  // indexed from e_first, dY and g by edge. PAIR: the tile's rows are pair
  // owners (e_first = 0, e_end < 0)
  const int E = PAIR ? *n_own : e_end >= 0 ? e_end : row_ptr_x[N];
  const int e0 = (PAIR ? 0 : e_first) + blockIdx.x * kTile;
  if (e0 >= E) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int rb = (w >> 1) * 32, cb = (w & 1) * 32;
  // the row's edge and (pair mode) its partner
  auto row_edge = [&](int row) { return PAIR ? Es[row] : (e0 + row < E ? e0 + row : -1); };
  auto row_partner = [&](int row) { return PAIR ? Ps[row] : -1; };
  if (t < kTile) {
    const int q = e0 + t;
    const int e = q < E ? (PAIR ? own[q] : q) : -1;
    if constexpr (PAIR) {
      Es[t] = e;
      Ps[t] = e >= 0 ? rev[e] : -1;
    }
    const float r = e >= 0 ? dvec[e].w : rc;
    float b[NB], db[NB];
    radial_basis<NB>(r, rc, p, b, db);
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      Bs[t][n] = b[n];
      dBs[t][n] = db[n];
    }
  }
  __syncthreads();
  layer1<NB>(Bs, W1, X);  // X = H1 (pre1 is recomputed at the end)
  __syncthreads();
  to_bf16_tile(X, Xb);
  __syncthreads();
  {
    const f32x16 acc = block_64_bf(Xb, rb, W2Tb, kH, cb);
#pragma unroll
    for (int r = 0; r < 16; ++r) P2[rb + acc_row(r, lane)][cb + (lane & 31)] = acc[r];
  }
  // dH2 = dR W3^T, K = PC, dR staged through LDS in slabs of 32 columns; the
  // next slab is loaded into registers while the current one is multiplied.
  // In pair mode a row's dR is the sum of its two edges' rows; the partner's
  // slab is loaded beside the owner's and added when the slab is staged.
  f32x16 acc = {};
  const int srow = t >> 2, sc8 = (t & 3) * 8;
  const int se = row_edge(srow), sp = row_partner(srow);
  const bool sval = se >= 0;
  const RS* dRrow = dR + (long)(sval ? se - e_first : 0) * PC + sc8;
  const RS* dRpart = dR + (long)(sp >= 0 ? sp : 0) * PC + sc8;
  float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f), p1 = p0, q0 = p0, q1 = p0;
  auto load_slab = [&](int kc) {
    if (sval) {
      float v[8];
      ldr_n<8>(dRrow + kc, v);
      p0 = make_float4(v[0], v[1], v[2], v[3]);
      p1 = make_float4(v[4], v[5], v[6], v[7]);
    }
    if (sp >= 0) {
      float v[8];
      ldr_n<8>(dRpart + kc, v);
      q0 = make_float4(v[0], v[1], v[2], v[3]);
      q1 = make_float4(v[4], v[5], v[6], v[7]);
    }
  };
  load_slab(0);
  for (int kc = 0; kc < PC; kc += 32) {
    __syncthreads();
    if (sp >= 0) {
      p0 = make_float4(p0.x + q0.x, p0.y + q0.y, p0.z + q0.z, p0.w + q0.w);
      p1 = make_float4(p1.x + q1.x, p1.y + q1.y, p1.z + q1.z, p1.w + q1.w);
    }
    const float v[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
    bf16x8 vb;
#pragma unroll
    for (int k = 0; k < 8; ++k) vb[k] = (__bf16)v[k];
    *reinterpret_cast<bf16x8*>(&Dsb[srow][sc8]) = vb;
    __syncthreads();
    if (kc + 32 < PC) load_slab(kc + 32);
#pragma unroll
    for (int kb = 0; kb < 32; kb += 16) {
      const int k0 = kb + 8 * (lane >> 5);
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(&Dsb[rb + (lane & 31)][k0]);
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(W3ub + ((long)(kc >> 5) * kH + cb + (lane & 31)) * 32 + k0);
      acc = mfma_bf(a, b, acc);
    }
  }
  __syncthreads();
  // dpre2 = dH2 * silu'(pre2) -> Xb
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = rb + acc_row(r, lane), col = cb + (lane & 31);
    Xb[row][col] = (__bf16)(acc[r] * silu_grad(P2[row][col]));
  }
  __syncthreads();
  {
    // dH1 = dpre2 W2^T ; dpre1 = dH1 * silu'(pre1) -> P2
    const f32x16 a2 = block_64_bf(Xb, rb, W2b, kH, cb);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = rb + acc_row(r, lane), col = cb + (lane & 31);
      float p1 = 0.0f;
#pragma unroll
      for (int n = 0; n < NB; ++n) p1 += Bs[row][n] * W1[n * kH + col];
      P2[row][col] = a2[r] * silu_grad(p1);
    }
  }
  __syncthreads();
  // threads 0-63: the rows' edges (length gradient and harmonics term);
  // threads 64-127 in pair mode: the partners (their harmonics term only)
  if (t < (PAIR ? 2 : 1) * kTile) {
    const bool partner = t >= kTile;
    const int row = t & (kTile - 1);
    const int e = partner ? row_partner(row) : row_edge(row);
    if (e >= 0) {
      float dr = 0.0f;
      if (!partner) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          float s = 0.0f;
          for (int q = 0; q < kH; ++q) s += P2[row][q] * W1[n * kH + q];
          dr += s * dBs[row][n];
        }
      }
      const float4 d = dvec[e];
      const float ir = 1.0f / d.w;
      const float nx = d.x * ir, ny = d.y * ir, nz = d.z * ir;
      float gx = dr * nx, gy = dr * ny, gz = dr * nz;
      if (dY) {
        float dy[16];
#pragma unroll
        for (int q = 0; q < (LMAX + 1) * (LMAX + 1); ++q) dy[q] = dY[(long)e * 16 + q];
        float Gx, Gy, Gz;
        real_sh_vjp<LMAX>(nx, ny, nz, dy, Gx, Gy, Gz);
        const float dot = Gx * nx + Gy * ny + Gz * nz;
        gx += (Gx - dot * nx) * ir;
        gy += (Gy - dot * ny) * ir;
        gz += (Gz - dot * nz) * ir;
      }
      if (accumulate) {
        const float4 o = g[e];
        g[e] = make_float4(o.x + gx, o.y + gy, o.z + gz, 0.0f);
      } else {
        g[e] = make_float4(gx, gy, gz, 0.0f);
      }
    }
  }
}


// R and its first ND - 1 derivatives in the edge length, FP32.
// ND 2, for energies and forces: since R depends on the length alone, the
// adjoint of the whole radial MLP is the dot product dE/dr_e = sum dR_e R'_e,
// which the tensor product's adjoint takes while it forms dR_e. So dR never
// goes to memory and no adjoint of the MLP is evaluated. R' is streamed past
// the caches: the forward pass reads only R, which then stays in the
// last-level cache (a call of 3,000 atoms 5 % faster, of 1,205, where both fit,
// 1 % slower). ND 1 (the same R): the forward pass of receiver chunks.
// ND 3, for Hessian-vector products and weight gradients: the tangent of R
// along any direction is R' r_dot, and the adjoint of the MLP a dot product
// with R' and R'', so that one evaluation serves every direction of a call.
// One row of each per pair owner or, without the pair list, per edge of
// [e_first, e_end) (e_end < 0: every edge inside the cutoff), from row 0;
// output s starts at out + s out_gap, rows out_ld apart.
// With each activation x: s = silu(x), s' = silu'(x) x', s'' = silu''(x) x'^2 + silu'(x) x''.
//
// The products with W2 and W3 run on the BF16 matrix cores with every operand
// split in three (gemm.hip's scheme: the error is below the FP32 instruction's,
// K = 64 5.0e-8 against 1.4e-7). The hidden layers are split once, on their way
// into LDS in operand order; the second layer is formed transposed (columns in
// the accumulator's rows), so that a lane holds four neighbouring columns of
// one pair and writes their parts as one piece. A wave then takes 32 columns
// of W3 for the tile's 64 rows and every output: each W3 operand feeds 2 ND
// rows' products.
// Bound: the stores (write rate 3.5 to 4.2 TB/s); small calls, the chain of
// the hidden layers (12 us). us per launch, this and the same on
// v_mfma_f32_32x32x2_f32: ND 2, 3,000 atoms (80,132 pairs, P C = 512) 92 and
// 142; 64 charged clusters 138 and 182; 138 atoms 17 and 31; 20,000 atoms, P C =
// 2,944 and 512 together 6,000 and 8,120. ND 3, 3,000 atoms 160 and 268.
struct RadialJobs {
  RadialJob j[kMaxRadialJobs];
};
template <int ND>
__global__ void __launch_bounds__(256, 2) k_radial_rows(const float4* __restrict__ dvec, const int* __restrict__ row_ptr_x,
                                                        int N, RadialJobs jobs, float rc, int p, int e_first, int e_end,
                                                        const int* __restrict__ own, const int* __restrict__ n_own) {
  constexpr int NB = 8;
  __shared__ bf16x8 X[ND][2][kH / 16][3][64];  // [output][32 rows][16 K][part][lane]
  const RadialJob& job = jobs.j[blockIdx.z];
  const float* __restrict__ W1 = job.W1;
  const __bf16 *__restrict__ W2 = job.W2, *__restrict__ W3 = job.W3;
  const int PC = job.PC, out_ld = job.out_ld;
  const long out_gap = job.out_gap;
  float* __restrict__ out = job.out;
  const int E = own ? *n_own : e_end >= 0 ? e_end : row_ptr_x[N];
  const int e0 = (own ? 0 : e_first) + blockIdx.x * kTile;
  if (e0 >= E || (PC == 0 ? blockIdx.y > 0 : blockIdx.y * 128 >= (unsigned)PC)) return;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  // the weights' operands of one product, on their way while the rows before are formed
  bf16x8 y[kH / 16][3];
  auto load_w = [&](const __bf16* __restrict__ W, int blocks, int block) {
    const bf16x8* __restrict__ f = reinterpret_cast<const bf16x8*>(W) + (long)block * 192;
#pragma unroll
    for (int j = 0; j < kH / 16; ++j)
#pragma unroll
      for (int i = 0; i < 3; ++i) y[j][i] = f[(long)j * blocks * 192 + i * 64 + lane];
  };
  const int c0 = 32 * (w + 4 * blockIdx.y), stride = 128 * gridDim.y;
  load_w(W2, 2, w & 1);
  {
    // a lane's row, 16 columns of the first layer per wave
    const int q = e0 + lane;
    const float r = q < E ? dvec[own ? own[q] : q].w : rc;
    float b[3][NB];
    if constexpr (ND == 3) radial_basis_d2<NB>(r, rc, p, b[0], b[1], b[2]);
    else radial_basis<NB>(r, rc, p, b[0], ND == 2 ? b[1] : nullptr);
#pragma unroll 1  // code size: what a small call waits for
    for (int h = 0; h < 2; ++h) {
      float v[ND][8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float x[3] = {};
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const float wv = W1[n * kH + 16 * w + 8 * h + j];
#pragma unroll
          for (int s = 0; s < ND; ++s) x[s] += b[s][n] * wv;
        }
        v[0][j] = siluf(x[0]);
        if constexpr (ND > 1) {
          const float g = silu_grad(x[0]);
          v[1][j] = g * x[1];
          if constexpr (ND > 2) v[2][j] = silu_grad2(x[0]) * x[1] * x[1] + g * x[2];
        }
      }
#pragma unroll
      for (int s = 0; s < ND; ++s) {
        bf16x8* f = &X[s][lane >> 5][w][0][(lane & 31) + 32 * h];
        split_bf16(v[s], f[0], f[64], f[128]);
      }
    }
  }
  __syncthreads();
  f32x16 hi[ND], lo[ND];
  {
    const int rb = w >> 1, cb = w & 1;
#pragma unroll
    for (int s = 0; s < ND; ++s) hi[s] = lo[s] = f32x16{};
#pragma unroll
    for (int j = 0; j < kH / 16; ++j) {
      __builtin_amdgcn_sched_barrier(0);  // few operands in flight: registers
      bf16x8 x[ND][3];
#pragma unroll
      for (int s = 0; s < ND; ++s)
#pragma unroll
        for (int i = 0; i < 3; ++i) x[s][i] = X[s][rb][j][i][lane];
#pragma unroll
      for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int s = 0; s < ND; ++s) {
          f32x16& acc = i < 5 ? lo[s] : hi[s];
          acc = mfma_bf(y[j][kSplitB[i]], x[s][kSplitA[i]], acc);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (c0 < PC) load_w(W3, PC / 32, c0 / 32);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      // columns 32 cb + 8 g + 4 (lane / 32) .. + 4 of row lane % 32
      float v[ND][4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float x = hi[0][4 * g + k] + lo[0][4 * g + k];
        v[0][k] = siluf(x);
        if constexpr (ND > 1) {
          const float d = silu_grad(x), x1 = hi[1][4 * g + k] + lo[1][4 * g + k];
          v[1][k] = d * x1;
          if constexpr (ND > 2) v[2][k] = silu_grad2(x) * x1 * x1 + d * (hi[2][4 * g + k] + lo[2][4 * g + k]);
        }
      }
      if (PC == 0) {
        const int row = 32 * rb + (lane & 31);
        if (e0 + row < E)
#pragma unroll
          for (int s = 0; s < ND; ++s)
            str_n<4>(out + (long)(e0 - (own ? 0 : e_first) + row) * out_ld + s * out_gap + 32 * cb + 8 * g + 4 * (lane >> 5),
                     v[s]);
        continue;
      }
#pragma unroll
      for (int s = 0; s < ND; ++s) {
        bf16x4* f = reinterpret_cast<bf16x4*>(&X[s][rb][2 * cb + g / 2][0][(lane & 31) + 32 * (g & 1)]) + (lane >> 5);
        split_bf16(v[s], f[0], f[128], f[256]);
      }
    }
  }
  __syncthreads();
  // lane part of an output's address, in bytes: rows 4 (lane / 32) on
  const unsigned oo = 4u * (4 * (lane >> 5) * out_ld + (lane & 31));
  for (int cc = c0; cc < PC; cc += stride) {
    float* __restrict__ o = out + (long)(e0 - (own ? 0 : e_first)) * out_ld + cc;
    auto store = [&](int h, const f32x16* v) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * h + 8 * (r >> 2) + (r & 3);  // + 4 (lane / 32)
        if (e0 + row + 4 * (lane >> 5) < E) {
          float* d = o + (long)row * out_ld;
          *at_off(d, oo) = v[0][r];
          if constexpr (ND == 2) __builtin_nontemporal_store(v[1][r], at_off(d + out_gap, oo));
          if constexpr (ND == 3) {
            *at_off(d + out_gap, oo) = v[1][r];
            *at_off(d + 2 * out_gap, oo) = v[2][r];
          }
        }
      }
    };
    f32x16 sum[2][ND];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int s = 0; s < ND; ++s) hi[s] = lo[s] = f32x16{};
#pragma unroll
      for (int j = 0; j < kH / 16; ++j) {
        __builtin_amdgcn_sched_barrier(0);  // few LDS operands in flight: registers
        bf16x8 x[ND][3];
#pragma unroll
        for (int s = 0; s < ND; ++s)
#pragma unroll
          for (int i = 0; i < 3; ++i) x[s][i] = X[s][h][j][i][lane];
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
          for (int s = 0; s < ND; ++s) {
            f32x16& acc = i < 5 ? lo[s] : hi[s];
            acc = mfma_bf(x[s][kSplitA[i]], y[j][kSplitB[i]], acc);
          }
      }
#pragma unroll
      for (int s = 0; s < ND; ++s) sum[h][s] = hi[s] + lo[s];
      if (ND == 3 && h == 0) store(0, sum[0]);  // no registers to hold them
      __builtin_amdgcn_sched_barrier(0);
    }
    // the next columns' operands before the stores: loads and stores complete
    // in order, a load behind the stores would wait for them
    __builtin_amdgcn_sched_barrier(0);
    if (cc + stride < PC) load_w(W3, PC / 32, (cc + stride) / 32);
    __builtin_amdgcn_sched_barrier(0);
    if (ND < 3) store(0, sum[0]);
    store(1, sum[1]);
  }
}

// Weight gradients of a loss on energies and forces: back from the adjoints Rb
// of R = H2 W3 and Rc of R' = H2' W3 (primes: derivatives in the edge length),
// per tile of 64 pair owners (edges without the pair list):
//   H2b = Rb W3^T, H2c = Rc W3^T
//   P2b = H2b silu'(P2) + H2c silu''(P2) P2',  P2c = H2c silu'(P2)
//   H1b = P2b W2^T, H1c = P2c W2^T
//   P1b = H1b silu'(P1) + H1c silu''(P1) P1',  P1c = H1c silu'(P1)
// with the hidden layers evaluated again (two 64 x 64 products; keeping them
// from the forward pass would write and read 2 KB per pair and layer). A pair's
// two rows of Rb (Rc) are added on the way in and the sum is left in the
// owner's row for the gradient of W3; the other operands of the weights'
// products go to Bd, H1d, H2d, P1g and P2g. The next slab of 32 columns is in
// flight while one is multiplied. Bound: its streams (two rows of Rb and Rc in
// and one out per pair, 2.1 KB of operands out). Per launch on 7,032 atoms
// (64 channels, P C = 256): 444 us, where the tangent and its reverse per edge
// took 960 + 747 us.
__global__ void __launch_bounds__(256, 2)
k_radial_wgrad(const float4* __restrict__ dvec, const int* __restrict__ row_ptr_x, int N, const float* __restrict__ W1,
               const float* __restrict__ W2, const float* __restrict__ W2T, const float* __restrict__ W3T, int PC,
               float* __restrict__ Rb, float* __restrict__ Rc, float rcut, int p, const int* __restrict__ own,
               const int* __restrict__ n_own, const int* __restrict__ rev, float* __restrict__ Bd,
               float* __restrict__ H1d, float* __restrict__ H2d, float* __restrict__ P1g, float* __restrict__ P2g) {
  constexpr int NB = 8;
  __shared__ float Bs[2][kTile][NB + 1];
  __shared__ float X[2][kTile][kLd];
  __shared__ __align__(16) float Ds[2][kTile][36];
  const int E = own ? *n_own : row_ptr_x[N];
  const int e0 = blockIdx.x * kTile;
  if (e0 >= E) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int rb = (w >> 1) * 32, cb = (w & 1) * 32;
  if (t < kTile) {
    const int q = e0 + t;
    const float r = q < E ? dvec[own ? own[q] : q].w : rcut;
    float b[NB], db[NB];
    radial_basis<NB>(r, rcut, p, b, db);
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      Bs[0][t][n] = b[n];
      Bs[1][t][n] = db[n];
      if (q < E) {
        Bd[(long)q * 16 + n] = b[n];
        Bd[(long)q * 16 + 8 + n] = db[n];
      }
    }
  }
  __syncthreads();
  for (int o = t; o < kTile * kH; o += 256) {
    const int row = o >> 6, col = o & 63;
    float x = 0.0f, x1 = 0.0f;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const float wv = W1[n * kH + col];
      x += Bs[0][row][n] * wv;
      x1 += Bs[1][row][n] * wv;
    }
    const float h = siluf(x), h1 = silu_grad(x) * x1;
    X[0][row][col] = h;
    X[1][row][col] = h1;
    if (e0 + row < E) {
      H1d[(long)(e0 + row) * 128 + col] = h;
      H1d[(long)(e0 + row) * 128 + 64 + col] = h1;
    }
  }
  __syncthreads();
  f32x16 p2 = {}, p2d = {};  // the wave's block of P2 and P2'
#pragma unroll 8
  for (int kk = 0; kk < kH; kk += 2) {
    const float b = W2[(kk + (lane >> 5)) * kH + cb + (lane & 31)];
    p2 = mfma32(X[0][rb + (lane & 31)][kk + (lane >> 5)], b, p2);
    p2d = mfma32(X[1][rb + (lane & 31)][kk + (lane >> 5)], b, p2d);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int q = e0 + rb + acc_row(r, lane);
    if (q < E) {
      H2d[(long)q * 128 + cb + (lane & 31)] = siluf(p2[r]);
      H2d[(long)q * 128 + 64 + cb + (lane & 31)] = silu_grad(p2[r]) * p2d[r];
    }
  }
  // H2b and H2c, slab by slab: a thread stages 8 columns of one row
  const int srow = t >> 2, sc8 = (t & 3) * 8;
  const int se = e0 + srow < E ? (own ? own[e0 + srow] : e0 + srow) : -1;
  const int sp = own && se >= 0 ? rev[se] : -1;
  float vb[8], vc[8], qb[8], qc[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) vb[q] = vc[q] = qb[q] = qc[q] = 0.0f;
  auto load = [&](int kc) {
    if (se >= 0) {
      ldr_n<8>(Rb + (long)se * PC + kc + sc8, vb);
      ldr_n<8>(Rc + (long)se * PC + kc + sc8, vc);
    }
    if (sp >= 0) {
      ldr_n<8>(Rb + (long)sp * PC + kc + sc8, qb);
      ldr_n<8>(Rc + (long)sp * PC + kc + sc8, qc);
    }
  };
  f32x16 ab = {}, ac = {};
  load(0);
  for (int kc = 0; kc < PC; kc += 32) {
    if (sp >= 0) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        vb[q] += qb[q];
        vc[q] += qc[q];
      }
    }
    __syncthreads();  // the previous slab has been read
    str_n<8>(&Ds[0][srow][sc8], vb);
    str_n<8>(&Ds[1][srow][sc8], vc);
    float ob[8], oc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      ob[q] = vb[q];
      oc[q] = vc[q];
    }
    __syncthreads();
    if (kc + 32 < PC) load(kc + 32);
    if (sp >= 0) {
      str_n<8>(Rb + (long)se * PC + kc + sc8, ob);
      str_n<8>(Rc + (long)se * PC + kc + sc8, oc);
    }
#pragma unroll
    for (int kk = 0; kk < 32; kk += 2) {
      const float b = W3T[(kc + kk + (lane >> 5)) * kH + cb + (lane & 31)];
      ab = mfma32(Ds[0][rb + (lane & 31)][kk + (lane >> 5)], b, ab);
      ac = mfma32(Ds[1][rb + (lane & 31)][kk + (lane >> 5)], b, ac);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = rb + acc_row(r, lane), col = cb + (lane & 31), q = e0 + row;
    const float g1 = silu_grad(p2[r]);
    const float pb = ab[r] * g1 + ac[r] * silu_grad2(p2[r]) * p2d[r], pc = ac[r] * g1;
    X[0][row][col] = pb;
    X[1][row][col] = pc;
    if (q < E) {
      P2g[(long)q * 128 + col] = pb;
      P2g[(long)q * 128 + 64 + col] = pc;
    }
  }
  __syncthreads();
  f32x16 hb = {}, hc = {};
#pragma unroll 8
  for (int kk = 0; kk < kH; kk += 2) {
    const float b = W2T[(kk + (lane >> 5)) * kH + cb + (lane & 31)];
    hb = mfma32(X[0][rb + (lane & 31)][kk + (lane >> 5)], b, hb);
    hc = mfma32(X[1][rb + (lane & 31)][kk + (lane >> 5)], b, hc);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = rb + acc_row(r, lane), col = cb + (lane & 31), q = e0 + row;
    if (q >= E) continue;
    float x = 0.0f, x1 = 0.0f;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const float wv = W1[n * kH + col];
      x += Bs[0][row][n] * wv;
      x1 += Bs[1][row][n] * wv;
    }
    const float g1 = silu_grad(x);
    P1g[(long)q * 128 + col] = hb[r] * g1 + hc[r] * silu_grad2(x) * x1;
    P1g[(long)q * 128 + 64 + col] = hc[r] * g1;
  }
}

inline int tiles(long n) { return (int)((n + kTile - 1) / kTile); }

}  // namespace

void launch_radial_fwd(int n_basis, const float4* dvec, const int* row_ptr_x, int N, long e_cap, const float* W1,
                       int PC, void* R, bool r_bf16, float rc, int p, hipStream_t st, int e_first, int e_end,
                       const RadialBf16* wb, const EdgePairs* pairs) {
  if (e_cap == 0) return;
  if (n_basis != 8) throw Error(E3MI_EUNSUPPORTED, "n_basis must be 8");
  if (PC % 32) throw Error(E3MI_EUNSUPPORTED, "paths x channels must be a multiple of 32");
  if (!(wb && wb->W2T && wb->W3T)) throw Error(E3MI_EINVAL, "BF16 mode: BF16 radial weights missing");
  if (pairs && (e_first != 0 || e_end >= 0 || !pairs->own || !pairs->n_own || !pairs->rev))
    throw Error(E3MI_EINVAL, "radial MLP per edge pair: needs the whole edge list and the pair owners");
  const int grid = tiles(e_end >= 0 ? (long)e_end - e_first : e_cap);
  if (grid == 0) return;
  const int* own = pairs ? pairs->own : nullptr;
  const int* n_own = pairs ? pairs->n_own : nullptr;
  auto go = [&](auto pc) {
    constexpr bool PAIR = decltype(pc)::value;
    if (r_bf16)
      k_radial_fwd<8, __bf16, PAIR><<<grid, 256, 0, st>>>(dvec, row_ptr_x, N, W1, PC, static_cast<__bf16*>(R), rc, p,
                                                          e_first, e_end, wb->W2T, wb->W3T, own, n_own);
    else
      k_radial_fwd<8, float, PAIR><<<grid, 256, 0, st>>>(dvec, row_ptr_x, N, W1, PC, static_cast<float*>(R), rc, p,
                                                         e_first, e_end, wb->W2T, wb->W3T, own, n_own);
  };
  if (pairs) go(std::true_type{});
  else go(std::false_type{});
}

void launch_radial_bwd(int n_basis, int lmax, const float4* dvec, const int* row_ptr_x, int N, long e_cap,
                       const float* W1, int PC, const void* dR, bool r_bf16, const float* dY, float4* g, int accumulate,
                       float rc, int p, hipStream_t st, int e_first, int e_end, const RadialBf16* wb,
                       const EdgePairs* pairs) {
  if (e_cap == 0) return;
  if (n_basis != 8) throw Error(E3MI_EUNSUPPORTED, "n_basis must be 8");
  if (lmax != 2 && lmax != 3) throw Error(E3MI_EUNSUPPORTED, "lmax must be 2 or 3");
  if (!(wb && wb->W2T && wb->W2 && wb->W3u)) throw Error(E3MI_EINVAL, "BF16 mode: BF16 radial weights missing");
  if (pairs && (e_first != 0 || e_end >= 0 || !pairs->own || !pairs->n_own || !pairs->rev))
    throw Error(E3MI_EINVAL, "radial adjoint per edge pair: needs the whole edge list and the pair owners");
  const int grid = tiles(e_end >= 0 ? (long)e_end - e_first : e_cap);
  if (grid == 0) return;
  auto go = [&](auto l, auto pc, auto rs) {
    using RS = decltype(rs);
    k_radial_bwd<8, decltype(l)::value, RS, decltype(pc)::value><<<grid, 256, 0, st>>>(
        dvec, row_ptr_x, N, W1, PC, static_cast<const RS*>(dR), dY, g, accumulate, rc, p, e_first, e_end, wb->W2T,
        wb->W2, wb->W3u, pairs ? pairs->own : nullptr, pairs ? pairs->n_own : nullptr, pairs ? pairs->rev : nullptr);
  };
  auto go_l = [&](auto pc, auto rs) {
    if (lmax == 3) go(std::integral_constant<int, 3>{}, pc, rs);
    else go(std::integral_constant<int, 2>{}, pc, rs);
  };
  auto go_p = [&](auto rs) {
    if (pairs) go_l(std::true_type{}, rs);
    else go_l(std::false_type{}, rs);
  };
  if (r_bf16) go_p(__bf16{});
  else go_p(float{});
}

void launch_radial_wgrad(const float4* dvec, const int* row_ptr_x, int N, long e_cap, const float* W1,
                         const float* W2, const float* W2T, const float* W3T, int PC, float* Rb, float* Rc, float rc,
                         int p, const int* own, const int* n_own, const int* rev, float* Bd, float* H1d, float* H2d,
                         float* P1g, float* P2g, hipStream_t st) {
  if (e_cap == 0) return;
  if (PC % 32) throw Error(E3MI_EUNSUPPORTED, "paths x channels must be a multiple of 32");
  k_radial_wgrad<<<tiles(e_cap), 256, 0, st>>>(dvec, row_ptr_x, N, W1, W2, W2T, W3T, PC, Rb, Rc, rc, p, own, n_own,
                                               rev, Bd, H1d, H2d, P1g, P2g);
}
void launch_radial_rows(int n_basis, const float4* dvec, const int* row_ptr_x, int N, long e_cap,
                        const RadialJob* jobs, int n_jobs, int n_out, float rc, int p, int e_first, int e_end,
                        const int* own, const int* n_own, hipStream_t st) {
  if (e_cap == 0) return;
  if (n_basis != 8) throw Error(E3MI_EUNSUPPORTED, "n_basis must be 8");
  if (n_jobs < 1 || n_jobs > kMaxRadialJobs) throw Error(E3MI_EINVAL, "internal: radial rows of too many layers");
  RadialJobs jj{};
  int PC = 0;
  for (int k = 0; k < n_jobs; ++k) {
    if (jobs[k].PC % 32) throw Error(E3MI_EUNSUPPORTED, "paths x channels must be a multiple of 32");
    jj.j[k] = jobs[k];
    PC = std::max(PC, jobs[k].PC);
  }
  if (own && (e_first != 0 || e_end >= 0 || !n_own))
    throw Error(E3MI_EINVAL, "radial MLP per edge pair: needs the whole edge list and the pair owners");
  const int grid = tiles(e_end >= 0 ? (long)e_end - e_first : e_cap);
  if (grid == 0) return;
  // A tile's columns over several workgroups, each with the hidden layers of its
  // own (the same bits), while they fit the chip at two a compute unit twice
  // over (the grid is sized for the list's capacity, about twice the pairs).
  // Both measured (us, split and not): 138 atoms 17 and 28, 64 molecules of 10
  // to 31 atoms 25 and 30, 1,205 atoms (no split left) 40 and 40.
  const int split = std::max(1, std::min((PC + 127) / 128, 1024 / (grid * n_jobs)));
  auto go = [&](auto nd) {
    k_radial_rows<decltype(nd)::value><<<dim3(grid, split, n_jobs), 256, 0, st>>>(dvec, row_ptr_x, N, jj, rc, p, e_first,
                                                                             e_end, own, n_own);
  };
  if (n_out == 1) go(std::integral_constant<int, 1>{});
  else if (n_out == 2) go(std::integral_constant<int, 2>{});
  else if (n_out == 3) go(std::integral_constant<int, 3>{});
  else throw Error(E3MI_EINVAL, "internal: outputs of the radial MLP");
}
}  // namespace e3mi
