// Per-atom stages of the interaction besides its dense contractions (gemm.hip):
//   gate (MACE table of Appendix F: gate_nodes):
//     h[0] = silu(h~[0]),  h[l>0] = h~[l] sigmoid(h~[0])
//   readout E_i = w2 . silu(W_r^T h[0]) + E0[z_i]
//   (Section 5.3 readout with one head), fused with its adjoint dE/dh[0]
//   energy reduction per structure in FP64, fixed summation order
//   force assembly F_i = sum_{e in in(i)} (g_e - g_rev(e))
#include "common.h"
#include "runtime.h"

namespace e3mi {

namespace {

// NC components of a channel per thread, all loads in flight at once. Bound: the
// streams, and on small systems the launch. us forward and back, with a loop
// over the components before: 138 atoms 3 and 3.5 (6.5 and 6.8), 3,000 atoms
// 8.8 and 12.5 (9.6 and 15.6; 49 and 74 MB), 20,000 atoms 47 and 72 (68 and 82).
template <int NC>
__global__ void __launch_bounds__(256) k_gate_fwd(const float* __restrict__ ht, float* __restrict__ h, int N, int C) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)N * C) return;
  const long at = idx / C * NC * C + idx % C;
  float x[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) x[c] = ht[at + (long)c * C];
  const float s = sigmoidf(x[0]);
#pragma unroll
  for (int c = 0; c < NC; ++c) h[at + (long)c * C] = x[c] * s;
}

// Scalar-only layer whose channel mix was split over K: h~ = the sum of the
// partial products in order, then h = silu(h~).
__global__ void k_gate_fwd_sum(const float* __restrict__ part, int n_parts, float* __restrict__ ht,
                               float* __restrict__ h, long NC) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= NC) return;
  float s0 = part[idx];
  for (int p = 1; p < n_parts; ++p) s0 += part[p * NC + idx];
  ht[idx] = s0;
  h[idx] = s0 * sigmoidf(s0);
}

template <int NC>
__global__ void __launch_bounds__(256) k_gate_bwd(const float* __restrict__ ht, const float* __restrict__ dh,
                                                  float* __restrict__ dht, int N, int C) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)N * C) return;
  const long at = idx / C * NC * C + idx % C;
  float x[NC], g[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    x[c] = ht[at + (long)c * C];
    g[c] = dh[at + (long)c * C];
  }
  const float s = sigmoidf(x[0]);
  float acc = 0.0f;
#pragma unroll
  for (int c = 1; c < NC; ++c) {
    acc += g[c] * x[c];
    dht[at + (long)c * C] = g[c] * s;
  }
  // (the contraction is fixed: the BF16 mode rounds what follows)
  dht[at] = __builtin_fmaf(acc * s, 1.0f - s, g[0] * silu_grad(x[0]));
}

// One wave per atom; readout_hidden = 16.
__global__ void __launch_bounds__(256) k_readout(const float* __restrict__ h, int nc, const int* __restrict__ species,
                                                 const float* __restrict__ Wr, const float* __restrict__ w2,
                                                 const float* __restrict__ e0, int N, int C,
                                                 double* __restrict__ e_atom, float* __restrict__ dh,
                                                 const float* __restrict__ wq, const float* __restrict__ bq,
                                                 float* __restrict__ q_raw) {
  const int i = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (i >= N) return;
  const float* hi = h + (long)i * nc * C;
  float pre[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) pre[q] = 0.0f;
  float qa = 0.0f;
  for (int k = lane; k < C; k += 64) {
    const float x = hi[k];
#pragma unroll
    for (int q = 0; q < 16; ++q) pre[q] += x * Wr[k * 16 + q];
    if (wq) qa += x * wq[k];
  }
  if (wq) {
    qa = wave_sum(qa);
    if (lane == 0) q_raw[i] = qa + bq[species[i]];
  }
  float e = 0.0f;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    pre[q] = wave_sum(pre[q]);
    e += w2[q] * siluf(pre[q]);
  }
  if (lane == 0) e_atom[i] = (double)e + (double)e0[species[i]];
  float gq[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) gq[q] = w2[q] * silu_grad(pre[q]);
  for (int k = lane; k < C; k += 64) {
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) s += Wr[k * 16 + q] * gq[q];
    dh[(long)i * C + k] = s;
  }
}

// Readout of a scalar-only last layer straight from its pre-gate values x (the
// sum of n_parts partial products [n_parts, N, C], or h~ itself when n_parts
// is 0), with the gate and its adjoint folded in: h = silu(x),
// E_i = w2 . silu(W_r^T h) + E0[z_i], dh~ = (W_r g) o silu'(x).
__global__ void __launch_bounds__(256) k_readout_gated(const float* __restrict__ xt, int n_parts,
                                                       const int* __restrict__ species, const float* __restrict__ Wr,
                                                       const float* __restrict__ w2, const float* __restrict__ e0,
                                                       int N, int C, double* __restrict__ e_atom,
                                                       float* __restrict__ dht) {
  const int i = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (i >= N) return;
  // every partial product of the lane's channels in flight at once (a loop over
  // them, once forward and once back: 138 atoms 7.4 us for 5.0, 3,000 9.2 for 7.3)
  const long NC = (long)N * C;
  float part[2][kMaxGemmGroup], x[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int p = 0; p < kMaxGemmGroup; ++p)
      part[u][p] = lane + 64 * u < C && (p == 0 || p < n_parts) ? xt[p * NC + (long)i * C + lane + 64 * u] : 0.0f;
  float pre[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) pre[q] = 0.0f;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int k = lane + 64 * u;
    if (k >= C) break;
    x[u] = part[u][0];
#pragma unroll
    for (int p = 1; p < kMaxGemmGroup; ++p)
      if (p < n_parts) x[u] += part[u][p];
    const float hv = x[u] * sigmoidf(x[u]);
#pragma unroll
    for (int q = 0; q < 16; ++q) pre[q] += hv * Wr[k * 16 + q];
  }
  // lane L holds the pre-activation of hidden unit L / 4
  const float pq = wave_sum_scatter16<16>(pre);
  const int q0 = lane >> 2;
  float e = (lane & 3) == 0 ? w2[q0] * siluf(pq) : 0.0f;
#pragma unroll
  for (int off = 4; off < 64; off <<= 1) e += __shfl_xor(e, off);
  if (lane == 0) e_atom[i] = (double)e + (double)e0[species[i]];
  const float gl = w2[q0] * silu_grad(pq);
  float gq[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) gq[q] = __shfl(gl, 4 * q);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int k = lane + 64 * u;
    if (k >= C) break;
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) s += Wr[k * 16 + q] * gq[q];
    dht[(long)i * C + k] = s * silu_grad(x[u]);
  }
}

// Energy of structure s, by one workgroup
__device__ __forceinline__ void sum_energy(const EnergySum& es, int s) {
  __shared__ double red[256];
  const int64_t a = es.off[s], b = es.off[s + 1];
  double acc = 0.0;
  for (int64_t i = a + threadIdx.x; i < b; i += 256) acc += es.e_atom[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) es.energy[s] = red[0];
}

// One wave per atom: the lanes take the row's edges in turn, then a fixed
// reduction tree over the wave (bitwise repeatable). The workgroups past the
// atoms' add up the structures' energies, which need a launch of their own
// otherwise (2 us of a 24-atom call, 5 of a 3,000-atom step).
__global__ void __launch_bounds__(256) k_forces(const int* __restrict__ row_ptr, const int* __restrict__ rev,
                                                const float4* __restrict__ g, int N, const float* __restrict__ extra,
                                                float* __restrict__ F, long e_stride, EnergySum es) {
  const int atom_blocks = (N + 3) / 4;
  if ((int)blockIdx.x >= atom_blocks) return sum_energy(es, blockIdx.x - atom_blocks);
  g += blockIdx.y * e_stride;
  F += 3L * blockIdx.y * N;
  const int i = (int)(((long)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= N) return;
  float fx = 0.f, fy = 0.f, fz = 0.f;
  const int b = row_ptr[i + 1];
  for (int e = row_ptr[i] + lane; e < b; e += 64) {
    const int re = rev[e];
    const float4 a = g[e];
    const float4 r = re >= 0 ? g[re] : make_float4(0.f, 0.f, 0.f, 0.f);
    fx += a.x - r.x;
    fy += a.y - r.y;
    fz += a.z - r.z;
  }
  fx = wave_sum(fx);
  fy = wave_sum(fy);
  fz = wave_sum(fz);
  if (extra) {
    fx += extra[3 * i];
    fy += extra[3 * i + 1];
    fz += extra[3 * i + 2];
  }
  if (lane == 0) {
    F[3 * i] = fx;
    F[3 * i + 1] = fy;
    F[3 * i + 2] = fz;
  }
}

inline int blocks(long n, int t) { return (int)((n + t - 1) / t); }

}  // namespace

void launch_gate_fwd(const float* ht, float* h, int N, int nc, int C, hipStream_t st) {
  if (N == 0) return;
  with_components(nc, [&](auto n) {
    k_gate_fwd<decltype(n)::value><<<blocks((long)N * C, 256), 256, 0, st>>>(ht, h, N, C);
  });
}
void launch_gate_fwd_sum(const float* part, int n_parts, float* ht, float* h, int N, int C, hipStream_t st) {
  if (N == 0) return;
  k_gate_fwd_sum<<<blocks((long)N * C, 256), 256, 0, st>>>(part, n_parts, ht, h, (long)N * C);
}
void launch_gate_bwd(const float* ht, const float* dh, float* dht, int N, int nc, int C, hipStream_t st) {
  if (N == 0) return;
  with_components(nc, [&](auto n) {
    k_gate_bwd<decltype(n)::value><<<blocks((long)N * C, 256), 256, 0, st>>>(ht, dh, dht, N, C);
  });
}
void launch_readout(const float* h, int nc, const int* species, const float* Wr, const float* w2, const float* e0,
                    int N, int C, double* e_atom, float* dh, hipStream_t st, const float* wq, const float* bq,
                    float* q_raw) {
  if (N == 0) return;
  k_readout<<<blocks((long)N * 64, 256), 256, 0, st>>>(h, nc, species, Wr, w2, e0, N, C, e_atom, dh, wq, bq, q_raw);
}
void launch_readout_gated(const float* xt, int n_parts, const int* species, const float* Wr, const float* w2,
                          const float* e0, int N, int C, double* e_atom, float* dht, hipStream_t st) {
  if (N == 0) return;
  k_readout_gated<<<blocks((long)N * 64, 256), 256, 0, st>>>(xt, n_parts, species, Wr, w2, e0, N, C, e_atom, dht);
}
void launch_forces(const int* row_ptr, const int* rev, const float4* g, int N, float* F, hipStream_t st,
                   const float* extra, int B, long e_stride, const EnergySum& es) {
  if (N == 0) return;
  k_forces<<<dim3(blocks(N, 4) + es.S, B), 256, 0, st>>>(row_ptr, rev, g, N, extra, F, e_stride, es);
}

}  // namespace e3mi
