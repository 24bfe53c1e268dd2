// Device copies of a model's weights, laid out from the flat FP64 vector on the
// device: the kernels' FP32 tensors, their transposes, the BF16 copies (rounded
// to nearest even from the FP32 values), the three-part BF16 operands of the
// per-atom contractions and the first layer's U_l. A training
// step replaces the weights every time: laid out on the host and sent tensor by
// tensor (41 copies, 10 M multiply-adds for U at 64 channels and 5 species) that
// took 1.4 ms of a 6.5 ms step.
#include "common.h"
#include "runtime.h"

namespace e3mi {
namespace {

// Rounded to FP32, and whatever is rounded to BF16 next from that value: the
// compiler otherwise rounds the FP64 one to BF16 directly, which differs at ties
__device__ __forceinline__ float to_f32(double x) {
  float v = (float)x;
  asm volatile("" : "+v"(v));
  return v;
}

__device__ __forceinline__ void put_fragment(__bf16* __restrict__ f, float v) {
  __bf16 x[3];
  split_bf16(v, x[0], x[1], x[2]);
#pragma unroll
  for (int p = 0; p < 3; ++p) f[512 * p] = x[p];
}

// *bad = 1 when a value is not finite. Everything below leaves the weights
// alone when *bad is set.
__global__ void __launch_bounds__(256) k_weights_check(const double* __restrict__ w, long n, int* __restrict__ bad) {
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256)
    if (!isfinite(w[i])) *bad = 1;
}

__global__ void __launch_bounds__(256) k_weights_layout(const double* __restrict__ w,
                                                        const WeightCopy* __restrict__ copies,
                                                        const int* __restrict__ bad) {
  if (*bad) return;
  const WeightCopy c = copies[blockIdx.y];
  const long n = (long)c.rows * c.cols;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) {
    const int r = (int)(i / c.cols), k = (int)(i % c.cols);
    const float v = to_f32(w[c.src + (long)r * c.ld + k]);
    const long t = (long)k * c.rows + r;  // transposed
    switch (c.kind) {
      case kCopyF32: static_cast<float*>(c.dst)[i] = v; break;
      case kTransposeF32: static_cast<float*>(c.dst)[t] = v; break;
      case kCopyBf16: static_cast<__bf16*>(c.dst)[i] = (__bf16)v; break;
      case kTransposeBf16: static_cast<__bf16*>(c.dst)[t] = (__bf16)v; break;
      case kFragments: put_fragment(static_cast<__bf16*>(c.dst) + fragment_at(r, k, c.cols), v); break;
      case kFragmentsT: put_fragment(static_cast<__bf16*>(c.dst) + fragment_at(k, r, c.rows), v); break;
      default:  // slabs of 32 columns
        static_cast<__bf16*>(c.dst)[((long)(k / 32) * c.rows + r) * 32 + k % 32] = (__bf16)v;
    }
  }
}

// U_l[(s, q), k'] = nu^-1 sum_k (W3[q, l C + k] W_emb[s, k]) W_mix_l[k, k'] in
// FP64, and its transpose. One workgroup per row (s, q) and order l, a thread
// per k'.
__global__ void __launch_bounds__(128) k_weights_u(const double* __restrict__ w, FirstWeights f,
                                                   const int* __restrict__ bad) {
  __shared__ double V[128];
  if (*bad) return;
  const int l = blockIdx.y, row = blockIdx.x, s = row / f.H, q = row % f.H, k = threadIdx.x, C = f.C;
  if (k < C) V[k] = w[f.rad3 + (long)q * f.ld3 + (long)l * C + k] * w[f.emb + (long)s * C + k] / f.nu;
  __syncthreads();
  if (k >= C) return;
  const double* Wm = w + f.mix[l] + k;
  double u = 0.0;
#pragma unroll 8
  for (int j = 0; j < C; ++j) u += V[j] * Wm[(long)j * C];
  const float v = to_f32(u);
  put_fragment(f.U[l] + fragment_at(row, k, C), v);
  put_fragment(f.UT[l] + fragment_at(k, row, gridDim.x), v);
}

}  // namespace

void launch_weights(const double* w, long n, const WeightCopy* copies, int n_copies, const FirstWeights& f,
                    bool check, int* bad, hipStream_t st) {
  launch_zero(bad, sizeof(int), st);
  if (check) k_weights_check<<<256, 256, 0, st>>>(w, n, bad);
  k_weights_layout<<<dim3(32, n_copies), 256, 0, st>>>(w, copies, bad);
  k_weights_u<<<dim3(f.n_species * f.H, f.n_orders), 128, 0, st>>>(w, f, bad);
}

}  // namespace e3mi
