// Per-atom dense contractions (channel mixes, self connections, the product
// block's linear layers and their adjoints): C = A0 B0 + A1 B1, B a weight.
//
// FP32 on the BF16 matrix cores: a float is the sum of three BF16 numbers to
// within 2^-27 of itself, x = x1 + x2 + x3, and
//   x y = x1 y1 + (x1 y2 + x2 y1) + (x1 y3 + x2 y2 + x3 y1) + O(2^-26 |x y|),
// six products of v_mfma_f32_32x32x16_bf16 (32 cycles for K = 16) in place of
// eight v_mfma_f32_32x32x2_f32 (64 cycles for K = 2): 192 against 512 cycles.
// The products are exact in the FP32 accumulators; x1 y1 and the five small
// ones have one each, added at the end. RMS error against 64 bits over
// Gaussian operands, this and the FP32 instruction: K = 64 5.0e-8 and 1.4e-7,
// K = 256 9.0e-8 and 2.8e-7, K = 640 1.4e-7 and 4.5e-7 (three products, without
// the last bracket, 4.4e-6: not FP32).
// A value that BF16 cannot hold, infinite or past 3.39e38, has parts that are
// not numbers: what it reaches is NaN, where the FP32 instruction's sums were
// infinite or NaN. Energies and forces of an overflow are NaN either way.
//
// The weights are split once, when they are laid out (kFragments), in the order
// the operands are loaded in: for every 16 K and 32 columns, per part, lane l
// holds B[8 (l / 32) .. + 8][l % 32]. A is split in registers on the way in;
// each lane loads its own operand (row l % 32, K 8 (l / 32) .. + 8) straight
// from the row, so A passes through no LDS.
//
// Both kernels add an output's products in the same order: an atom's result
// does not depend on which of them a batch takes.
//
// The mixed mode (BF) takes the first product of one accumulator over all K.
#include <algorithm>
#include <climits>

#include "common.h"
#include "runtime.h"

namespace e3mi {

namespace {

constexpr int kStep = 32;  // K per step: two matrix-core steps of 16

// Row r = (atom, m) of a matrix (the three of a product have as many rows per atom)
struct Row {
  int atom, m;
  __device__ __forceinline__ Row(int r, int g) : atom(r / g), m(r - atom * g) {}
  __device__ __forceinline__ long off(const RowMap& x) const { return (long)atom * x.s_atom + (long)m * x.s_m; }
};
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// Independent products of one group share a launch: workgroup b (after the
// XCD-contiguous remapping, so that the column blocks of a row tile and
// neighbouring row tiles meet in one L2) takes tile b - tile0[k] of product k,
// column blocks fastest.
struct GemmGroup {
  GemmArgs g[kMaxGemmGroup];
  int tile0[kMaxGemmGroup];
  int ncb[kMaxGemmGroup];
};

// The product of workgroup b (unused tile0 are past every tile)
__device__ __forceinline__ int gemm_product(const GemmGroup& gg, int b) {
  int gi = 0;
#pragma unroll
  for (int k = 1; k < kMaxGemmGroup; ++k) gi += b >= gg.tile0[k];
  return gi;
}

// A lane's part of a step of its row (p: the row + 8 (lane / 32))
struct ARow {
  float4 v[kStep / 8];
  __device__ __forceinline__ void load(const float* __restrict__ p) {
#pragma unroll
    for (int j = 0; j < kStep / 16; ++j) {
      v[2 * j] = *reinterpret_cast<const float4*>(p + 16 * j);
      v[2 * j + 1] = *reinterpret_cast<const float4*>(p + 16 * j + 4);
    }
  }
  // the operand of 16 K in PARTS BF16 parts
  template <int PARTS>
  __device__ __forceinline__ void split(int j, bf16x8* x) const {
    const float f[8] = {v[2 * j].x,     v[2 * j].y,     v[2 * j].z,     v[2 * j].w,
                        v[2 * j + 1].x, v[2 * j + 1].y, v[2 * j + 1].z, v[2 * j + 1].w};
    if constexpr (PARTS == 3) {
      split_bf16(f, x[0], x[1], x[2]);
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) x[0][q] = (__bf16)f[q];
    }
  }
};
// per column block hi += x1 y1; lo += the five small products (PARTS 1: hi alone)
template <int PARTS, int NB>
__device__ __forceinline__ void mul_split(const bf16x8* x, const bf16x8* y, f32x16* hi, f32x16* lo) {
#pragma unroll
  for (int i = PARTS == 3 ? 0 : 5; i < 6; ++i)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      f32x16& acc = i < 5 ? lo[n] : hi[n];
      acc = mfma_bf(x[kSplitA[i]], y[n * PARTS + kSplitB[i]], acc);
    }
}

// A wave's 32 rows from bm and NB column blocks from cb; lanes hold the offsets
// of the rows they loaded
template <bool BF, int NB>
__device__ __forceinline__ void store_rows(const GemmArgs& a, const Row& row, int bm, int cb, int lane,
                                           const f32x16* hi, const f32x16* lo) {
  const long mine = row.off(a.c);
  const long first = (long)(unsigned)__builtin_amdgcn_readfirstlane((int)mine) |
                     (long)__builtin_amdgcn_readfirstlane((int)(mine >> 32)) << 32;
  const int rel = (int)(mine - first);  // 32 rows
  float* __restrict__ C = a.c.base + first + cb * 32 + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int k = acc_row(r, lane), o = __shfl(rel, k);
    if (bm + k < a.M) {
#pragma unroll
      for (int n = 0; n < NB; ++n) C[o + 32 * n] = BF ? hi[n][r] : hi[n][r] + lo[n][r];
    }
  }
}

// Many rows: a workgroup takes 128 rows and NB 32-column blocks, each wave 32
// of the rows; a step's weights are staged through LDS for the four waves and
// the next step's operands are in flight while one is multiplied. A's operand
// loads touch 32 rows each and take four times the cycles of a contiguous
// load: with two column blocks per pass over A they were the bound, with four
// the streams of A and C are.
template <bool BF, int NB>
__global__ void __launch_bounds__(256, 2) k_gemm(GemmGroup gg) {
  constexpr int PARTS = BF ? 1 : 3;
  constexpr int kQ = NB * PARTS * 64;        // 16-byte pieces of the weights per 16 K
  constexpr int kPieces = kStep / 16 * kQ;   // a step
  constexpr int kW = (kPieces + 255) / 256;  // and per thread
  __shared__ bf16x8 Bs[2][kPieces];
  const int b = xcd_contiguous(blockIdx.x, gridDim.x);
  const int gi = gemm_product(gg, b);
  const GemmArgs a = gg.g[gi];
  const int ncb = gg.ncb[gi], local = b - gg.tile0[gi];
  const int bm = (local / ncb) * 128, cb = (local % ncb) * NB, nb = a.Nc / 32;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int s0 = a.k0 / kStep, ns = s0 + a.k1 / kStep;
  // rows past M read the last row and store nothing
  const Row row(min(bm + 32 * w + (lane & 31), a.M - 1), a.c.g);
  const float* p0 = a.a0.base + row.off(a.a0) + 8 * (lane >> 5);
  const float* p1 = a.k1 > 0 ? a.a1.base + row.off(a.a1) + 8 * (lane >> 5) : p0;
  // this thread's pieces of a step's weights, in bytes from the step's first
  unsigned wo[kW];
#pragma unroll
  for (int i = 0; i < kW; ++i) {
    const int idx = t + 256 * i, j = idx / kQ, q = idx % kQ;  // PARTS 1: of each block the first part
    wo[i] = 16u * (unsigned)(j * nb * 192 + (PARTS == 3 ? q : (q / 64) * 192 + q % 64));
  }
  auto mine = [&](int i) { return kPieces % 256 == 0 || t + 256 * i < kPieces; };
  const __bf16* bw = (s0 > 0 ? a.b0 : a.b1) + (long)cb * 1536;
  const float* pa = s0 > 0 ? p0 : p1;
  ARow next;
  bf16x8 wt[kW];
  auto load = [&] {
    next.load(pa);
#pragma unroll
    for (int i = 0; i < kW; ++i)
      if (mine(i)) wt[i] = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(bw) + wo[i]);
  };
  f32x16 hi[NB] = {}, lo[NB] = {};
  if (ns > 0) load();
  for (int s = 0; s < ns; ++s) {
    bf16x8* Bt = Bs[s & 1];
#pragma unroll
    for (int i = 0; i < kW; ++i)
      if (mine(i)) Bt[t + 256 * i] = wt[i];
    bf16x8 x[kStep / 16][PARTS];
#pragma unroll
    for (int j = 0; j < kStep / 16; ++j) next.split<PARTS>(j, x[j]);
    __syncthreads();
    if (s + 1 < ns) {
      const bool sw = s + 1 == s0;
      pa = sw ? p1 : pa + kStep;
      bw = sw ? a.b1 + (long)cb * 1536 : bw + (long)(kStep / 16) * nb * 1536;
      load();
    }
    // one column block's operands at a time, the next ones on their way from LDS
    constexpr int kG = NB * (kStep / 16);
    bf16x8 y[2][PARTS];
    auto fetch = [&](int g) {
#pragma unroll
      for (int i = 0; i < PARTS; ++i) y[g & 1][i] = Bt[(g * PARTS + i) * 64 + lane];
    };
    fetch(0);
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      if (g + 1 < kG) fetch(g + 1);
      __builtin_amdgcn_sched_barrier(0);
      const int j = g / NB, n = g % NB;
      mul_split<PARTS, 1>(x[j], y[g & 1], hi + n, lo + n);
    }
  }
  store_rows<BF, NB>(a, row, bm + 32 * w, cb, lane, hi, lo);
}

// Few rows: every wave takes a 32 x 32 block of its own and loads the weights
// straight into registers, two steps in flight; a row of workgroups per
// product, so that its arguments are read at once. Bound: the chain of
// instruction fetches, loads and matrix-core steps of one block. The code runs
// once, so its size counts: the first layer's mix of 138 atoms (K = 256) 11.4
// us, with four steps in flight (twice the code) 12.5, with a division per
// stored row on top 14.0, k_gemm 20.4.
template <int PARTS>
struct FewStep {
  ARow a;
  bf16x8 y[kStep / 16][PARTS];
};
template <bool BF>
__global__ void __launch_bounds__(256, 1) k_gemm_few(GemmGroup gg) {
  constexpr int PARTS = BF ? 1 : 3, kRing = 2;
  const GemmArgs& a = gg.g[blockIdx.y];
  const int t = threadIdx.x, lane = t & 63, nb = a.Nc / 32;
  const int blk = 4 * xcd_contiguous(blockIdx.x, gridDim.x) + __builtin_amdgcn_readfirstlane(t >> 6);
  const int bm = (blk / nb) * 32, cb = blk % nb;
  if (bm >= a.M) return;  // past the last block
  const int s0 = a.k0 / kStep, ns = s0 + a.k1 / kStep;
  const Row row(min(bm + (lane & 31), a.M - 1), a.c.g);
  const float* p0 = a.a0.base + row.off(a.a0) + 8 * (lane >> 5);
  const float* p1 = a.k1 > 0 ? a.a1.base + row.off(a.a1) + 8 * (lane >> 5) : p0;
  FewStep<PARTS> ring[kRing];
  auto load = [&](int s, FewStep<PARTS>& f) {
    const bool second = s >= s0;
    const int k = (second ? s - s0 : s) * kStep;
    const __bf16* bw = (second ? a.b1 : a.b0) + ((long)(k / 16) * nb + cb) * 1536 + lane * 8;
#pragma unroll
    for (int j = 0; j < kStep / 16; ++j)
#pragma unroll
      for (int i = 0; i < PARTS; ++i)
        f.y[j][i] = *reinterpret_cast<const bf16x8*>(bw + (long)j * nb * 1536 + i * 512);
    f.a.load((second ? p1 : p0) + k);
  };
#pragma unroll
  for (int q = 0; q < kRing; ++q)
    if (q < ns) load(q, ring[q]);
  f32x16 hi[1] = {}, lo[1] = {};
  for (int s = 0; s < ns; s += kRing) {
#pragma unroll
    for (int q = 0; q < kRing; ++q) {
      if (s + q >= ns) break;
#pragma unroll
      for (int j = 0; j < kStep / 16; ++j) {
        bf16x8 x[PARTS];
        ring[q].a.template split<PARTS>(j, x);
        mul_split<PARTS, 1>(x, ring[q].y[j], hi, lo);
      }
      if (s + q + kRing < ns) load(s + q + kRing, ring[q]);
    }
  }
  store_rows<BF, 1>(a, row, bm, cb, lane, hi, lo);
}

// k_gemm_few up to this many 32 x 32 blocks, one wave per SIMD of the chip: a
// wave per block then is all the parallelism there is. Both measured (us, few
// and many): 276 blocks 11.4 and 20.4, 820 blocks 9.6 and 10.3, 1,880 blocks
// 14.8 and 13.1, 2,600 blocks 36 and 23.
constexpr int kFewBlocks = 1024;

}  // namespace

template <bool BF>
static void gemm_launch(const GemmGroup& gg, int tiles, int nb, hipStream_t st) {
  if (nb == 4) k_gemm<BF, 4><<<tiles, 256, 0, st>>>(gg);
  else if (nb == 2) k_gemm<BF, 2><<<tiles, 256, 0, st>>>(gg);
  else k_gemm<BF, 1><<<tiles, 256, 0, st>>>(gg);
}

void launch_gemm_group(const GemmArgs* a, int n, hipStream_t st, bool bf16) {
  if (n < 1 || n > kMaxGemmGroup) throw Error(E3MI_EINVAL, "GEMM group size out of range");
  int nb = 4;  // column blocks of a workgroup
  for (int k = 0; k < n; ++k) {
    if ((a[k].k0 % 32) || (a[k].k1 % 32) || (a[k].Nc % 32))
      throw Error(E3MI_EUNSUPPORTED, "GEMM dimensions must be multiples of 32");
    if (a[k].a0.g != a[k].c.g || (a[k].k1 && a[k].a1.g != a[k].c.g))
      throw Error(E3MI_EINVAL, "internal: GEMM rows per atom differ");
    while (a[k].Nc % (32 * nb)) nb /= 2;
  }
  GemmGroup gg{};
  int tiles = 0, m = 0;
  long total = 0, most = 0;  // 32 x 32 blocks
  for (int k = 0; k < n; ++k) {
    if (a[k].M == 0 || a[k].Nc == 0) continue;
    gg.g[m] = a[k];
    gg.tile0[m] = tiles;
    gg.ncb[m] = a[k].Nc / (32 * nb);
    tiles += (a[k].M + 127) / 128 * gg.ncb[m];
    const long blocks = (long)((a[k].M + 31) / 32) * (a[k].Nc / 32);
    total += blocks;
    most = std::max(most, blocks);
    ++m;
  }
  if (m == 0) return;
  for (int k = m; k < kMaxGemmGroup; ++k) gg.tile0[k] = INT_MAX;
  if (total <= kFewBlocks) {
    const dim3 grid((unsigned)((most + 31) / 32 * 8), m);  // a multiple of the 8 XCDs per product
    if (bf16) k_gemm_few<true><<<grid, 256, 0, st>>>(gg);
    else k_gemm_few<false><<<grid, 256, 0, st>>>(gg);
  } else if (bf16) {
    gemm_launch<true>(gg, tiles, nb, st);
  } else {
    gemm_launch<false>(gg, tiles, nb, st);
  }
}

}  // namespace e3mi
