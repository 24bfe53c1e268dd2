// Clebsch-Gordan tensor product + neighbour sum (the operation the paper's
// backend accelerates, Section 4), and its two adjoints.
//
// Receiver-centric: one workgroup owns one receiver atom i and walks its CSR
// row of edges e = (i <- j), so the neighbour sum accumulates in registers and
// needs no global atomics. Threads map to channels (channel-contiguous h, R and
// A make every load and store coalesced); each thread handles CPT channels.
//
//   forward   A[i,p,k,m3]  = nu^-1 sum_e R[e,p,k] sum_{m1 m2} C^p[m1,m2,m3] h[j,k,l1 m1] Y_e[l2 m2]
//   edge adj  dR[e,p,k]    = nu^-1 sum_m3 dA[i,p,k,m3] T[e,p,k,m3]   (T = the inner CG sum)
//             dY[e,l2 m2]  = nu^-1 sum_{p,k,m1,m3} C R dA h           (reduced over channels)
//   node adj  dh[j,k,l1 m1] = nu^-1 sum_{e: src(e) = j} sum_p R sum C Y_e dA[dst(e)]
//             computed for atom j from its own incoming edges e' via the reverse
//             edge: dst(rev e') = src(e'), R is a function of |d| only, and
//             Y(-d) = (-1)^l Y(d), so no other row is read except dA[src(e')].
//
// A layout (consumed by the channel-mix GEMM): for each output order l3 a
// block [N, 2 l3 + 1, P_l3, C].
#include "common.h"
#include "paths.h"
#include "runtime.h"

namespace e3mi {
namespace {

template <int W>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int off = W / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, W);
  return v;
}

// The scalar-output layer's forward (here in the BF16 mode; in FP32 k_tps_fwd)
// is compiled for at most three waves per SIMD: the compiler then schedules its
// edge loop with 88 registers instead of 72 (the hardware still holds five
// waves) and it runs faster (0.134 ms against 0.141 on the 3,000-atom step).
// Holding residency at three or two waves for real, by reserving LDS, is slower
// (0.167, 0.196 ms).
template <int LMAX, int KIND, int CPT, class RS, bool IDX>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, KIND == kLast ? 3 : 10))) k_tp_fwd(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                const float4* __restrict__ dvec, const RS* __restrict__ R,
                                                int r_stride, const float* __restrict__ h, int h_nc,
                                                float* __restrict__ A, int N, int C, float inv_nu, int i0,
                                                int r_first, const int* __restrict__ r_row) {
  using PS = PathSet<LMAX, KIND>;
  constexpr int NP = PS::NP, NOUT = PS::NOUT, NIN = PS::NIN, NY = PS::NY;
  const int i = i0 + xcd_contiguous(blockIdx.x, gridDim.x);
  const int tpr = blockDim.x;
  float acc[CPT][NOUT];
#pragma unroll
  for (int c = 0; c < CPT; ++c)
#pragma unroll
    for (int o = 0; o < NOUT; ++o) acc[c][o] = 0.0f;
  const int e1 = row_ptr[i + 1];
  for (int e = row_ptr[i]; e < e1; ++e) {
    const int j = src[e];
    const float4 d = dvec[e];
    const float ir = 1.0f / d.w;
    float Y[NY];
    real_sh<LMAX>(d.x * ir, d.y * ir, d.z * ir, Y);
    const RS* Re = R + (long)(IDX ? r_row[e] : e - r_first) * r_stride;
    const float* hj = h + (long)j * h_nc * C;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int k = threadIdx.x + c * tpr;
      float hv[NIN], rv[NP];
#pragma unroll
      for (int q = 0; q < NIN; ++q) hv[q] = hj[q * C + k];
      // every path's weight of the edge in one batch of loads
#pragma unroll
      for (int q = 0; q < NP; ++q) rv[q] = ldr(Re + q * C + k);
      static_for<NP>([&](auto pi) {
        constexpr int g = PS::T.id[pi];
        constexpr int l1 = kL1[g], l2 = kL2[g], l3 = kL3[g];
        constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
        constexpr int off = PS::T.off[pi];
        const float rp = rv[pi];
        float tm[2 * l3 + 1];
#pragma unroll
        for (int m = 0; m < 2 * l3 + 1; ++m) tm[m] = 0.0f;
        static_for<nz>([&](auto z) {
          constexpr int q = z0 + z;
          tm[kM3[q]] += hv[l1 * l1 + kM1[q]] * (kC[q] * Y[l2 * l2 + kM2[q]]);
        });
#pragma unroll
        for (int m = 0; m < 2 * l3 + 1; ++m) acc[c][off + m] += rp * tm[m];
      });
    }
  }
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int k = threadIdx.x + c * tpr;
    static_for<NP>([&](auto pi) {
      constexpr int g = PS::T.id[pi];
      constexpr int l3 = kL3[g];
      constexpr int off = PS::T.off[pi], rank = PS::T.rank[pi];
      constexpr int P3 = PS::T.np_l3[l3];
      float* base = A + a_group_base<PS>(l3, N, C);
#pragma unroll
      for (int m = 0; m < 2 * l3 + 1; ++m)
        base[(((long)i * (2 * l3 + 1) + m) * P3 + rank) * C + k] = acc[c][off + m] * inv_nu;
    });
  }
}

// MSG: also write each edge's share of its sender's gradient,
//   msg[e, l1 m1, k] = nu^-1 sum_p R[e,p,k] sum_{m2 m3} C^p Y_e[l2 m2] dA[i,p,k,m3],
// at row e - e_first, for k_tp_msg_node to add up per sender.
// Layers with every path hold 99 adjoint values per channel: the compiler is
// asked for two waves per SIMD (at most 256 registers); one wave per SIMD
// halves the kernel's speed.
// DER: R' is given (Rp); instead of dR the edge's dE/dr = sum dR R' is
// formed, in place of dY's first value (the l = 0 harmonic is constant).
template <int LMAX, int KIND, int CPT, bool MSG, class RS, bool IDX, bool DER>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KIND == kFull ? 2 : 1, 10))) k_tp_bwd_edge(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                     const float4* __restrict__ dvec, const RS* __restrict__ R,
                                                     const float* __restrict__ Rp, int r_stride,
                                                     const float* __restrict__ h, int h_nc,
                                                     const float* __restrict__ dA, RS* __restrict__ dR,
                                                     float* __restrict__ dY, int N, int C, float inv_nu, int i0,
                                                     int e_first, float* __restrict__ msg, int* __restrict__ touched,
                                                     int tag, const int* __restrict__ r_row, int r_first,
                                                     int row_add) {
  using PS = PathSet<LMAX, KIND>;
  constexpr int NP = PS::NP, NOUT = PS::NOUT, NIN = PS::NIN, NY = PS::NY;
  __shared__ float red[4][16];
  const int i = i0 + xcd_contiguous(blockIdx.x, gridDim.x);
  const int tpr = blockDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float dai[CPT][NOUT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int k = threadIdx.x + c * tpr;
    static_for<NP>([&](auto pi) {
      constexpr int g = PS::T.id[pi];
      constexpr int l3 = kL3[g];
      constexpr int off = PS::T.off[pi], rank = PS::T.rank[pi];
      constexpr int P3 = PS::T.np_l3[l3];
      const float* base = dA + a_group_base<PS>(l3, N, C);
#pragma unroll
      for (int m = 0; m < 2 * l3 + 1; ++m)
        dai[c][off + m] = base[(((long)i * (2 * l3 + 1) + m) * P3 + rank) * C + k] * inv_nu;
    });
  }
  const int e1 = row_ptr[i + 1];
  for (int e = row_ptr[i]; e < e1; ++e) {
    const int j = src[e];
    if (MSG && threadIdx.x == 0) touched[j] = tag;  // j receives a message from this chunk
    const float4 d = dvec[e];
    const float ir = 1.0f / d.w;
    float Y[NY];
    real_sh<LMAX>(d.x * ir, d.y * ir, d.z * ir, Y);
    const RS* Re = R + (long)(IDX ? r_row[e] : e - r_first) * r_stride;
    const float* Rpe = DER ? Rp + (long)(IDX ? r_row[e] : e - r_first) * r_stride : nullptr;
    RS* dRe = DER ? nullptr : dR + (long)(e - e_first) * r_stride;
    const float* hj = h + (long)j * h_nc * C;
    float dyp[NY];
#pragma unroll
    for (int q = 0; q < NY; ++q) dyp[q] = 0.0f;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int k = threadIdx.x + c * tpr;
      float hv[NIN], mv[MSG ? NIN : 1], rv[NP];
#pragma unroll
      for (int q = 0; q < NIN; ++q) hv[q] = hj[q * C + k];
#pragma unroll
      for (int q = 0; q < NP; ++q) rv[q] = ldr(Re + q * C + k);
#pragma unroll
      for (int q = 0; q < (MSG ? NIN : 1); ++q) mv[q] = 0.0f;
      static_for<NP>([&](auto pi) {
        constexpr int g = PS::T.id[pi];
        constexpr int l1 = kL1[g], l2 = kL2[g], l3 = kL3[g];
        constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
        constexpr int off = PS::T.off[pi];
        const float rp = rv[pi];
        float tm[2 * l3 + 1];
#pragma unroll
        for (int m = 0; m < 2 * l3 + 1; ++m) tm[m] = 0.0f;
        static_for<nz>([&](auto z) {
          constexpr int q = z0 + z;
          const float cy = kC[q] * Y[l2 * l2 + kM2[q]];
          const float rd = rp * dai[c][off + kM3[q]];
          tm[kM3[q]] += hv[l1 * l1 + kM1[q]] * cy;
          if constexpr (!DER || l2 > 0) dyp[l2 * l2 + kM2[q]] += kC[q] * (hv[l1 * l1 + kM1[q]] * rd);
          if constexpr (MSG) mv[l1 * l1 + kM1[q]] += rd * cy;
        });
        float s = 0.0f;
#pragma unroll
        for (int m = 0; m < 2 * l3 + 1; ++m) s += dai[c][off + m] * tm[m];
        if constexpr (DER)
          dyp[0] += s * Rpe[pi * C + k];
        else
          str(dRe + pi * C + k, s);
      });
      if constexpr (MSG) {
        float* me = msg + (long)(e - e_first) * NIN * C + k;
#pragma unroll
        for (int q = 0; q < NIN; ++q) me[q * C] = mv[q];
      }
    }
    // reduce dY over the channels of the workgroup
    auto put = [&](int q, float v) {
      float* o = dY + (long)e * 16 + q;
      *o = DER && row_add ? *o + v : v;
    };
    if (tpr >= 64) {
      const float tot = wave_sum_scatter16<NY>(dyp);
      const int q = lane >> 2;
      if (tpr == 64) {
        if ((lane & 3) == 0 && q < NY) put(q, tot);
      } else {
        if ((lane & 3) == 0) red[wave][q] = tot;
        __syncthreads();
        if (threadIdx.x < NY) {
          float v = 0.0f;
          for (int w = 0; w < tpr / 64; ++w) v += red[w][threadIdx.x];
          put(threadIdx.x, v);
        }
        __syncthreads();
      }
    } else {
#pragma unroll
      for (int q = 0; q < NY; ++q) dyp[q] = group_sum<32>(dyp[q]);
      if (lane < NY) {
        float v = 0.0f;
#pragma unroll
        for (int q = 0; q < NY; ++q) v = lane == q ? dyp[q] : v;
        put(lane, v);
      }
    }
  }
}

template <int LMAX, int KIND, int CPT, class RS, bool IDX>
__global__ void __launch_bounds__(256) k_tp_bwd_node(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                     const float4* __restrict__ dvec, const RS* __restrict__ R,
                                                     int r_stride, const float* __restrict__ dA,
                                                     float* __restrict__ dh, int dh_nc, int N, int C, float inv_nu,
                                                     int i0, int r_first, int dh_acc, const int* __restrict__ r_row) {
  using PS = PathSet<LMAX, KIND>;
  constexpr int NP = PS::NP, NIN = PS::NIN, NY = PS::NY;
  const int j = i0 + xcd_contiguous(blockIdx.x, gridDim.x);
  const int tpr = blockDim.x;
  float acc[CPT][NIN];
#pragma unroll
  for (int c = 0; c < CPT; ++c)
#pragma unroll
    for (int q = 0; q < NIN; ++q) acc[c][q] = 0.0f;
  const int e1 = row_ptr[j + 1];
  for (int e = row_ptr[j]; e < e1; ++e) {
    const int i2 = src[e];  // receiver of the reverse edge
    const float4 d = dvec[e];
    const float ir = -1.0f / d.w;  // direction of the reverse edge
    float Y[NY];
    real_sh<LMAX>(d.x * ir, d.y * ir, d.z * ir, Y);
    const RS* Re = R + (long)(IDX ? r_row[e] : e - r_first) * r_stride;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int k = threadIdx.x + c * tpr;
      static_for<NP>([&](auto pi) {
        constexpr int g = PS::T.id[pi];
        constexpr int l1 = kL1[g], l2 = kL2[g], l3 = kL3[g];
        constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
        constexpr int rank = PS::T.rank[pi];
        constexpr int P3 = PS::T.np_l3[l3];
        const float rp = ldr(Re + pi * C + k);
        const float* base = dA + a_group_base<PS>(l3, N, C);
        float dav[2 * l3 + 1];
#pragma unroll
        for (int m = 0; m < 2 * l3 + 1; ++m)
          dav[m] = rp * base[(((long)i2 * (2 * l3 + 1) + m) * P3 + rank) * C + k];
        static_for<nz>([&](auto z) {
          constexpr int q = z0 + z;
          acc[c][l1 * l1 + kM1[q]] += dav[kM3[q]] * (kC[q] * Y[l2 * l2 + kM2[q]]);
        });
      });
    }
  }
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int k = threadIdx.x + c * tpr;
    // components below dh_acc (all when dh_acc <= 0) are added to, the others
    // written (zero past the paths' inputs)
#pragma unroll
    for (int q = 0; q < NIN; ++q) {
      float* o = dh + ((long)j * dh_nc + q) * C + k;
      *o = (dh_acc <= 0 || q < dh_acc) ? *o + acc[c][q] * inv_nu : acc[c][q] * inv_nu;
    }
    if (dh_acc > 0)
      for (int q = NIN; q < dh_nc; ++q)
        if (q >= dh_acc) dh[((long)j * dh_nc + q) * C + k] = 0.0f;
  }
}

// Sender gradient from the edges' messages: dh[j] continues from its stored
// value (from init, the first chunk, or the previous chunk) and adds msg of
// j's outgoing edges e = rev(e2), e2 over the run of j's row whose senders
// (the receivers of e) lie in this chunk's receivers [c0, c1), in row order.
// Rows are sorted by sender, so the runs of successive chunks follow each
// other along the row and every sender's sum is the same sequence of
// additions whatever the chunking. init: components below dh_acc (all when
// dh_acc <= 0) start from dh, the others from zero (components NIN..dh_nc-1
// past dh_acc are zeroed). Block b is sender b (no XCD remapping): the
// senders a chunk touches are a compact index range (atoms are spatially
// sorted), and consecutive blocks go to different XCDs, so that range
// spreads over the whole chip. Messages are read four edges at a time (64
// loads in flight per lane) and added in row order.
template <int NIN>
__global__ void __launch_bounds__(256) k_tp_msg_node(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                     const int* __restrict__ rev, const float* __restrict__ msg,
                                                     float* __restrict__ dh, int dh_nc, int C, int c0, int c1,
                                                     int e_first, int init, int dh_acc,
                                                     const int* __restrict__ touched, int tag) {
  const int j = blockIdx.x;
  // after the first chunk, only senders this chunk's edge adjoint sent to
  // (touched carries the chunk's tag; another value can only add an empty run)
  if (!init && touched[j] != tag) return;
  const int a = row_ptr[j], b = row_ptr[j + 1];
  // the run: first entry with src >= c0 .. first entry with src >= c1
  auto lower = [&](int v) {
    int lo = a, hi = b;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (src[mid] < v) lo = mid + 1; else hi = mid;
    }
    return lo;
  };
  const int r0 = lower(c0), r1 = lower(c1);
  for (int k = threadIdx.x; k < C; k += blockDim.x) {
    float acc[NIN];
#pragma unroll
    for (int q = 0; q < NIN; ++q) {
      const bool keep = !init || dh_acc <= 0 || q < dh_acc;
      acc[q] = keep ? dh[((long)j * dh_nc + q) * C + k] : 0.0f;
    }
    int e2 = r0;
    for (; e2 + 4 <= r1; e2 += 4) {
      int ev[4];
      float mv[4][NIN];
#pragma unroll
      for (int u = 0; u < 4; ++u) ev[u] = rev[e2 + u];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        // an edge without a reverse reads the chunk's first message, unused
        const float* me = msg + (ev[u] >= 0 ? (long)(ev[u] - e_first) : 0L) * NIN * C + k;
#pragma unroll
        for (int q = 0; q < NIN; ++q) mv[u][q] = me[q * C];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < NIN; ++q)
          if (ev[u] >= 0) acc[q] += mv[u][q];
    }
    for (; e2 < r1; ++e2) {
      const int e = rev[e2];
      if (e < 0) continue;
      const float* me = msg + (long)(e - e_first) * NIN * C + k;
#pragma unroll
      for (int q = 0; q < NIN; ++q) acc[q] += me[q * C];
    }
#pragma unroll
    for (int q = 0; q < NIN; ++q) dh[((long)j * dh_nc + q) * C + k] = acc[q];
    if (init && dh_acc > 0)
      for (int q = NIN; q < dh_nc; ++q)
        if (q >= dh_acc) dh[((long)j * dh_nc + q) * C + k] = 0.0f;
  }
}

// ---- layers with every path, FP32 ---------------------------------------------
// One channel per thread, 99 outputs (l_max 3) per channel in registers. An
// edge costs about 350 coefficient terms per channel, so the vector ALU bounds
// both kernels once the loads are hidden; with two or three waves per SIMD they
// have to be requested far ahead: the weights of a path are loaded kRing paths
// before their use, across the edge's end into the next edge's row, the next
// edge's features during the current edge, and the indices an edge earlier
// still. The order of a path's work is fixed by scheduling barriers; without
// them the compiler moves the loads to their uses and keeps products of
// coefficients and harmonics alive across paths. On the 3,000-atom box with the
// product block (160k edges, 128 channels): forward 1,165 -> 517 us, edge
// adjoint 1,192 -> 1,164 us while it also takes the radial adjoint's place
// (529 us).
constexpr int kRing = 8;
struct FullEdge {
  int j, row;
  float4 d;
};
__device__ __forceinline__ FullEdge full_edge(const int* __restrict__ src, const float4* __restrict__ dvec,
                                              const int* __restrict__ r_row, int r_first, int e) {
  return FullEdge{src[e], r_row ? r_row[e] : e - r_first, dvec[e]};
}

template <int LMAX>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2, 10)))
k_tp_full_fwd(const int* __restrict__ row_ptr, const int* __restrict__ src, const float4* __restrict__ dvec,
              const float* __restrict__ R, int r_stride, const float* __restrict__ h, float* __restrict__ A, int N,
              int C, float inv_nu, int i0, int r_first, const int* __restrict__ r_row) {
  using PS = PathSet<LMAX, kFull>;
  constexpr int NP = PS::NP, NOUT = PS::NOUT, NIN = PS::NIN, NY = PS::NY;
  constexpr int STEPS = (NP + kRing - 1) / kRing * kRing;
  const int i = i0 + xcd_contiguous(blockIdx.x, gridDim.x);
  const unsigned k = threadIdx.x;
  const int e0 = row_ptr[i], e1 = row_ptr[i + 1];
  float acc[NOUT];
#pragma unroll
  for (int o = 0; o < NOUT; ++o) acc[o] = 0.0f;
  if (e0 < e1) {
    FullEdge cur = full_edge(src, dvec, r_row, r_first, e0);
    FullEdge nxt = full_edge(src, dvec, r_row, r_first, min(e0 + 1, e1 - 1));
    float ring[kRing], hv[NIN];
#pragma unroll
    for (int p = 0; p < kRing; ++p) ring[p] = (R + (long)cur.row * r_stride + p * C)[k];
#pragma unroll
    for (int q = 0; q < NIN; ++q) hv[q] = (h + ((long)cur.j * NIN + q) * C)[k];
    for (int e = e0; e < e1; ++e) {
      const FullEdge after = full_edge(src, dvec, r_row, r_first, min(e + 2, e1 - 1));
      const float* Re = R + (long)cur.row * r_stride;
      const float* Rn = R + (long)nxt.row * r_stride;
      float Y[NY], hn[NIN];
      const float ir = 1.0f / cur.d.w;
      real_sh<LMAX>(cur.d.x * ir, cur.d.y * ir, cur.d.z * ir, Y);
#pragma unroll
      for (int q = 0; q < NIN; ++q) hn[q] = (h + ((long)nxt.j * NIN + q) * C)[k];
      static_for<STEPS>([&](auto pi) {
        __builtin_amdgcn_sched_barrier(0);
        const float rp = ring[pi % kRing];
        constexpr int nextp = pi + kRing < STEPS ? pi + kRing : pi + kRing - STEPS;
        if constexpr (nextp < NP) ring[pi % kRing] = ((pi + kRing < STEPS ? Re : Rn) + nextp * C)[k];
        if constexpr (pi < NP) {
          constexpr int g = PS::T.id[pi];
          constexpr int l1 = kL1[g], l2 = kL2[g], l3 = kL3[g];
          constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
          constexpr int off = PS::T.off[pi];
          constexpr bool ONE = one_coefficient(g);
#pragma unroll
          for (int m = 0; m < 2 * l2 + 1; ++m) asm volatile("" : "+v"(Y[l2 * l2 + m]));
          float tm[2 * l3 + 1];
#pragma unroll
          for (int m = 0; m < 2 * l3 + 1; ++m) tm[m] = 0.0f;
          static_for<nz>([&](auto z) {
            constexpr int q = z0 + z;
            const float y = Y[l2 * l2 + kM2[q]];
            tm[kM3[q]] += hv[l1 * l1 + kM1[q]] * (ONE ? y : kC[q] * y);
          });
          const float rv = ONE ? kC[z0] * rp : rp;
#pragma unroll
          for (int m = 0; m < 2 * l3 + 1; ++m) acc[off + m] += rv * tm[m];
        }
      });
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < NIN; ++q) hv[q] = hn[q];
      cur = nxt;
      nxt = after;
    }
  }
  static_for<NP>([&](auto pi) {
    constexpr int g = PS::T.id[pi];
    constexpr int l3 = kL3[g];
    constexpr int off = PS::T.off[pi], rank = PS::T.rank[pi];
    constexpr int P3 = PS::T.np_l3[l3];
    float* base = A + a_group_base<PS>(l3, N, C);
#pragma unroll
    for (int m = 0; m < 2 * l3 + 1; ++m)
      (base + (((long)i * (2 * l3 + 1) + m) * P3 + rank) * C)[k] = acc[off + m] * inv_nu;
  });
}

// Edge adjoint, with R' given (Rp). Per edge the row [dE/dr, dY 1..]
// (dE/dr = sum dR R'; the l = 0 harmonic is constant) and the message to its
// sender (see k_tp_bwd_edge).
template <int LMAX>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2, 10)))
k_tp_full_bwd(const int* __restrict__ row_ptr, const int* __restrict__ src, const float4* __restrict__ dvec,
              const float* __restrict__ R, const float* __restrict__ Rp, const float* __restrict__ h,
              const float* __restrict__ dA, float* __restrict__ dY, int N, int C, float inv_nu, int i0, int e_first, float* __restrict__ msg,
              int* __restrict__ touched, int tag, int r_first, const int* __restrict__ r_row, int row_add) {
  using PS = PathSet<LMAX, kFull>;
  constexpr int NP = PS::NP, NOUT = PS::NOUT, NIN = PS::NIN, NY = PS::NY;
  constexpr int STEPS = (NP + kRing - 1) / kRing * kRing;
  __shared__ float red[2][2][16];
  const int i = i0 + xcd_contiguous(blockIdx.x, gridDim.x);
  const unsigned k = threadIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e0 = row_ptr[i], e1 = row_ptr[i + 1];
  if (e0 >= e1) return;
  const int r_stride = NP * C;
  float dai[NOUT];
  static_for<NP>([&](auto pi) {
    constexpr int g = PS::T.id[pi];
    constexpr int l3 = kL3[g];
    constexpr int off = PS::T.off[pi], rank = PS::T.rank[pi];
    constexpr int P3 = PS::T.np_l3[l3];
    const float* base = dA + a_group_base<PS>(l3, N, C);
#pragma unroll
    for (int m = 0; m < 2 * l3 + 1; ++m)
      dai[off + m] = (base + (((long)i * (2 * l3 + 1) + m) * P3 + rank) * C)[k] * inv_nu;
  });
  FullEdge cur = full_edge(src, dvec, r_row, r_first, e0);
  FullEdge nxt = full_edge(src, dvec, r_row, r_first, min(e0 + 1, e1 - 1));
  float ring[kRing], ring1[kRing], hv[NIN];
#pragma unroll
  for (int p = 0; p < kRing; ++p) {
    ring[p] = (R + (long)cur.row * r_stride + p * C)[k];
    ring1[p] = (Rp + (long)cur.row * r_stride + p * C)[k];
  }
#pragma unroll
  for (int q = 0; q < NIN; ++q) hv[q] = (h + ((long)cur.j * NIN + q) * C)[k];
  for (int e = e0; e < e1; ++e) {
    if (threadIdx.x == 0) touched[cur.j] = tag;  // j receives a message from this chunk
    const FullEdge after = full_edge(src, dvec, r_row, r_first, min(e + 2, e1 - 1));
    const float* Re = R + (long)cur.row * r_stride;
    const float* Rn = R + (long)nxt.row * r_stride;
    float Y[NY], hn[NIN], dyp[NY], mv[NIN];
    const float ir = 1.0f / cur.d.w;
    real_sh<LMAX>(cur.d.x * ir, cur.d.y * ir, cur.d.z * ir, Y);
#pragma unroll
    for (int q = 0; q < NIN; ++q) {
      hn[q] = (h + ((long)nxt.j * NIN + q) * C)[k];
      mv[q] = 0.0f;
    }
#pragma unroll
    for (int q = 0; q < NY; ++q) dyp[q] = 0.0f;
    static_for<STEPS>([&](auto pi) {
      __builtin_amdgcn_sched_barrier(0);
      const float rp = ring[pi % kRing], r1 = ring1[pi % kRing];
      constexpr int nextp = pi + kRing < STEPS ? pi + kRing : pi + kRing - STEPS;
      if constexpr (nextp < NP) {
        ring[pi % kRing] = ((pi + kRing < STEPS ? Re : Rn) + nextp * C)[k];
        ring1[pi % kRing] = (Rp + (long)(pi + kRing < STEPS ? cur.row : nxt.row) * r_stride + nextp * C)[k];
      }
      if constexpr (pi < NP) {
        constexpr int g = PS::T.id[pi];
        constexpr int l1 = kL1[g], l2 = kL2[g], l3 = kL3[g];
        constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
        constexpr int off = PS::T.off[pi];
        constexpr bool ONE = one_coefficient(g);
#pragma unroll
        for (int m = 0; m < 2 * l2 + 1; ++m) asm volatile("" : "+v"(Y[l2 * l2 + m]));
        float tm[2 * l3 + 1], rd[2 * l3 + 1];
        const float rv = ONE ? kC[z0] * rp : rp;
#pragma unroll
        for (int m = 0; m < 2 * l3 + 1; ++m) {
          tm[m] = 0.0f;
          rd[m] = rv * dai[off + m];
        }
        static_for<nz>([&](auto z) {
          constexpr int q = z0 + z;
          constexpr int q1 = l1 * l1 + kM1[q], q2 = l2 * l2 + kM2[q], m = kM3[q];
          const float cy = ONE ? Y[q2] : kC[q] * Y[q2];
          tm[m] += hv[q1] * cy;
          mv[q1] += rd[m] * cy;
          if constexpr (l2 > 0) {
            const float t = hv[q1] * rd[m];
            dyp[q2] += ONE ? t : kC[q] * t;
          }
        });
        float s = 0.0f;
#pragma unroll
        for (int m = 0; m < 2 * l3 + 1; ++m) s += dai[off + m] * tm[m];
        dyp[0] += s * (ONE ? kC[z0] * r1 : r1);
      }
    });
    __builtin_amdgcn_sched_barrier(0);
    float* me = msg + (long)(e - e_first) * NIN * C;
#pragma unroll
    for (int q = 0; q < NIN; ++q) (me + q * C)[k] = mv[q];
    // sums over the channels: a half, one or two waves
    auto put = [&](int q, float v) {
      float* o = dY + (long)e * 16 + q;
      *o = row_add ? *o + v : v;
    };
    if (blockDim.x >= 64) {
      const float tot = wave_sum_scatter16<NY>(dyp);
      const int q = lane >> 2;
      if (blockDim.x == 64) {
        if ((lane & 3) == 0 && q < NY) put(q, tot);
      } else {  // one barrier per edge, the exchange buffer alternates
        float(*buf)[16] = red[e & 1];
        if ((lane & 3) == 0) buf[wave][q] = tot;
        __syncthreads();
        if (threadIdx.x < NY) put(threadIdx.x, buf[0][threadIdx.x] + buf[1][threadIdx.x]);
      }
    } else {
#pragma unroll
      for (int q = 0; q < NY; ++q) dyp[q] = group_sum<32>(dyp[q]);
      if (lane < NY) {
        float v = 0.0f;
#pragma unroll
        for (int q = 0; q < NY; ++q) v = lane == q ? dyp[q] : v;
        put(lane, v);
      }
    }
#pragma unroll
    for (int q = 0; q < NIN; ++q) hv[q] = hn[q];
    cur = nxt;
    nxt = after;
  }
}

}  // namespace

// ---- dispatch ---------------------------------------------------------------

// the first-order passes (0 forward, 1 edge adjoint, 2 node adjoint); IDX:
// R rows through the edges' pair indices. FP32 adjoints take R' (a.Rp), the BF16 mode's write dR (in FP32 in layers with every path); the
// node adjoint is left to scalar-output layers of the BF16 mode that the
// sender-side adjoint does not take.
template <int LMAX, int KIND, int CPT, bool IDX>
static void first_order_launch(int which, const TpArgs& a, int nr, int tpr, hipStream_t st) {
  const __bf16* Rb = reinterpret_cast<const __bf16*>(a.R);
  __bf16* dRb = reinterpret_cast<__bf16*>(a.dR);
  const int rf = a.r_first;
  if (which == 0) {
    if constexpr (KIND != kFull) {
      if (a.r_bf16) {
        k_tp_fwd<LMAX, KIND, CPT, __bf16, IDX><<<nr, tpr, 0, st>>>(a.row_ptr, a.src, a.dvec, Rb, a.r_stride, a.h,
                                                                    a.h_nc, a.A, a.N, a.C, a.inv_nu, a.i0, rf,
                                                                    a.r_row);
        return;
      }
    }
    if constexpr (KIND == kFull) {
      if (a.fp32) {
        k_tp_full_fwd<LMAX><<<nr, tpr, 0, st>>>(a.row_ptr, a.src, a.dvec, a.R, a.r_stride, a.h, a.A, a.N, a.C,
                                                a.inv_nu, a.i0, rf, a.r_row);
        return;
      }
    }
    if constexpr (KIND == kLast || KIND == kFirstLast)
      throw Error(E3MI_EINVAL, "tensor product: scalar-output layers in FP32 take launch_tps_fwd");
    else
      k_tp_fwd<LMAX, KIND, CPT, float, IDX><<<nr, tpr, 0, st>>>(a.row_ptr, a.src, a.dvec, a.R, a.r_stride, a.h, a.h_nc,
                                                                 a.A, a.N, a.C, a.inv_nu, a.i0, rf, a.r_row);
    return;
  }
  constexpr bool MSG = KIND == kFull;
  if (which == 1 && (a.msg != nullptr) != MSG)
    throw Error(E3MI_EINVAL, "tensor product: messages go with layers with every path");
  if (which == 1 && a.Rp) {
    if (a.r_bf16) throw Error(E3MI_EINVAL, "tensor product: R' rows are FP32");
    if constexpr (KIND == kFull)
      k_tp_full_bwd<LMAX><<<nr, tpr, 0, st>>>(a.row_ptr, a.src, a.dvec, a.R, a.Rp, a.h, a.dA, a.dY, a.N, a.C, a.inv_nu,
                                              a.i0, a.e_first, a.msg, a.touched, a.tag, rf, a.r_row, a.row_add);
    else if constexpr (KIND == kFirst)
      k_tp_bwd_edge<LMAX, KIND, CPT, MSG, float, IDX, true><<<nr, tpr, 0, st>>>(
          a.row_ptr, a.src, a.dvec, a.R, a.Rp, a.r_stride, a.h, a.h_nc, a.dA, nullptr, a.dY, a.N, a.C, a.inv_nu, a.i0,
          a.e_first, a.msg, a.touched, a.tag, a.r_row, rf, a.row_add);
    else
      throw Error(E3MI_EINVAL, "tensor product: scalar-output layers take the sender-side adjoint");
  } else if (which == 1) {
    if constexpr (KIND == kFull) {
      if (a.r_bf16) throw Error(E3MI_EINVAL, "tensor product: layers with every path keep FP32 R");
      k_tp_bwd_edge<LMAX, KIND, CPT, true, float, IDX, false><<<nr, tpr, 0, st>>>(
          a.row_ptr, a.src, a.dvec, a.R, nullptr, a.r_stride, a.h, a.h_nc, a.dA, a.dR, a.dY, a.N, a.C, a.inv_nu, a.i0,
          a.e_first, a.msg, a.touched, a.tag, a.r_row, rf, 0);
    } else {
      if (!a.r_bf16) throw Error(E3MI_EINVAL, "tensor product: FP32 adjoints take R' rows");
      k_tp_bwd_edge<LMAX, KIND, CPT, false, __bf16, IDX, false><<<nr, tpr, 0, st>>>(
          a.row_ptr, a.src, a.dvec, Rb, nullptr, a.r_stride, a.h, a.h_nc, a.dA, dRb, a.dY, a.N, a.C, a.inv_nu, a.i0, a.e_first,
          nullptr, nullptr, 0, a.r_row, rf, 0);
    }
  } else if constexpr (KIND == kLast) {
    if (!a.r_bf16) throw Error(E3MI_EINVAL, "tensor product: FP32 adjoints take R' rows");
    k_tp_bwd_node<LMAX, KIND, CPT, __bf16, IDX><<<nr, tpr, 0, st>>>(a.row_ptr, a.src, a.dvec, Rb, a.r_stride, a.dA,
                                                                     a.dh, a.dh_nc, a.N, a.C, a.inv_nu, a.i0, rf,
                                                                     a.dh_acc, a.r_row);
  } else {
    throw Error(E3MI_EINVAL, "tensor product: node adjoint of a layer that has none");
  }
}

template <int LMAX, int KIND, int CPT>
static void tp_launch(int which, const TpArgs& a, hipStream_t st) {
  const int tpr = a.C / CPT;
  if (a.N == 0) return;
  const int nr = a.n_recv > 0 ? a.n_recv : a.N;  // receivers of this launch
  if (which <= 2 && a.n_recv == 0 && (a.i0 != 0 || a.e_first != 0 || a.r_first != 0))
    throw Error(E3MI_EINVAL, "tensor product: receiver offset without a receiver count");
  if (which <= 2) {
    if (a.r_row)
      first_order_launch<LMAX, KIND, CPT, true>(which, a, nr, tpr, st);
    else
      first_order_launch<LMAX, KIND, CPT, false>(which, a, nr, tpr, st);
  }
  else if (which == 7) {
    using PS = PathSet<LMAX, KIND>;
    const int c1 = a.n_recv > 0 ? a.i0 + a.n_recv : a.N;
    k_tp_msg_node<PS::NIN><<<a.N, 128, 0, st>>>(a.row_ptr, a.src, a.rev, a.msg, a.dh, a.dh_nc, a.C, a.i0, c1,
                                                 a.e_first, a.i0 == 0 ? 1 : 0, a.dh_acc, a.touched, a.tag);
  }
  else
    throw Error(E3MI_EINVAL, "tensor product: unknown pass");
}

template <int LMAX, int KIND>
static void tp_cpt(int which, const TpArgs& a, hipStream_t st) {
  // Layers with every path keep one channel per thread (the accumulators of
  // 99 outputs already fill the register file). The others run one channel
  // per thread too (twice the workgroups: one receiver per workgroup leaves
  // few waves per SIMD) except in the kernels that reduce over the
  // workgroup's channels once per edge (the first-order edge adjoint's dY),
  // which take the requested two.
  if constexpr (KIND == kFull) {
    if (a.cpt == 1) return tp_launch<LMAX, KIND, 1>(which, a, st);
  } else {
    const bool reduces_per_edge = which == 1;
    if (a.cpt == 1 || (a.cpt == 2 && !reduces_per_edge)) return tp_launch<LMAX, KIND, 1>(which, a, st);
    if (a.cpt == 2) return tp_launch<LMAX, KIND, 2>(which, a, st);
  }
  throw Error(E3MI_EUNSUPPORTED, "channels per thread not supported for this layer");
}

template <int LMAX>
static void tp_kind(int which, const TpArgs& a, hipStream_t st) {
  switch (a.kind) {
    case kFirst: return tp_cpt<LMAX, kFirst>(which, a, st);
    case kFull: return tp_cpt<LMAX, kFull>(which, a, st);
    case kLast: return tp_cpt<LMAX, kLast>(which, a, st);
    case kFirstLast: return tp_cpt<LMAX, kFirstLast>(which, a, st);
    default: throw Error(E3MI_EINVAL, "bad layer kind");
  }
}

void launch_tp(int which, const TpArgs& a, hipStream_t st) {
  switch (a.lmax) {
    case 2: return tp_kind<2>(which, a, st);
    case 3: return tp_kind<3>(which, a, st);
    default: throw Error(E3MI_EUNSUPPORTED, "lmax must be 2 or 3");
  }
}

}  // namespace e3mi
