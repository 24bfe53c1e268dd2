// Parameter gradients of a loss that depends on energies and forces.
//
// For upstream gradients gE (per structure) and gF (per atom), the gradient
// with respect to the weights theta is
//   dL/dtheta = d/dtheta [ sum_s gE_s E_s  -  D_v E ],   v = gF,
// where D_v E = sum_i v_i . dE/dr_i is the change of E when the atoms move
// along v (forces are -dE/dr; the paper trains on force labels and, in §5.2,
// on Hessian rows obtained by differentiating forces). D_v E is computed by a
// tangent (forward-mode) pass through the interaction and the whole scalar by
// a reverse pass over both the primal and the tangent values. This file holds
// the per-atom and per-edge kernels of those passes that are not tensor
// products or radial MLPs, and the reductions over edges and atoms that give
// the weight gradients, in a fixed order (no atomics).
#include <algorithm>

#include "common.h"
#include "runtime.h"

namespace e3mi {
namespace {

inline int blocks(long n, int t) { return (int)((n + t - 1) / t); }

// h_dot = gate'(h~) h~_dot; NC components of a channel per thread, all loads in
// flight at once. Bound: the streams. 17,043 rows (a batch of 13 directions) 52 us
// and back 120, with a loop over the components 66 and 124.
template <int NC>
__global__ void __launch_bounds__(256) k_gate_dual_fwd(const float* __restrict__ x, const float* __restrict__ xd,
                                                       float* __restrict__ hd, int N, int C, int B) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)B * N * C) return;
  const long u = idx / C, k = idx % C;
  const long base = u * NC * C + k, bx = (u % N) * NC * C + k;
  float xv[NC], xdv[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    xv[c] = x[bx + (long)c * C];
    xdv[c] = xd[base + (long)c * C];
  }
  const float s = sigmoidf(xv[0]), s1 = s * (1.0f - s);
  hd[base] = silu_grad(xv[0]) * xdv[0];
#pragma unroll
  for (int c = 1; c < NC; ++c) hd[base + (long)c * C] = xdv[c] * s + xv[c] * s1 * xdv[0];
}

// Reverse of (h, h_dot) = gate(h~), gate'(h~) h~_dot:
//   xc_l = hc_l s                       xc_0 = hc_0 silu'(x0) + sum_l hc_l x_l s'
//   xb_l = hb_l s + hc_l s' xd0          xb_0 = hb_0 silu'(x0) + hc_0 silu''(x0) xd0
//                                              + sum_l [hb_l x_l s' + hc_l (xd_l s' + x_l s'' xd0)]
template <int NC>
__global__ void __launch_bounds__(256) k_gate_dual_bwd(const float* __restrict__ x, const float* __restrict__ xd,
                                                       const float* __restrict__ hb, const float* __restrict__ hc,
                                                       float* __restrict__ xb, float* __restrict__ xc, int N, int C,
                                                       int B) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)B * N * C) return;
  const long u = idx / C, k = idx % C;
  const long base = u * NC * C + k, bx = (u % N) * NC * C + k;
  float xv[NC], xdv[NC], bv[NC], cv[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    xv[c] = x[bx + (long)c * C];
    xdv[c] = xd[base + (long)c * C];
    bv[c] = hb[base + (long)c * C];
    cv[c] = hc[base + (long)c * C];
  }
  const float x0 = xv[0], xd0 = xdv[0];
  const float s = sigmoidf(x0), s1 = s * (1.0f - s), s2 = s1 * (1.0f - 2.0f * s);
  float b0 = bv[0] * silu_grad(x0) + cv[0] * silu_grad2(x0) * xd0;
  float c0 = cv[0] * silu_grad(x0);
#pragma unroll
  for (int c = 1; c < NC; ++c) {
    xc[base + (long)c * C] = cv[c] * s;
    xb[base + (long)c * C] = bv[c] * s + cv[c] * s1 * xd0;
    c0 += cv[c] * xv[c] * s1;
    b0 += bv[c] * xv[c] * s1 + cv[c] * (xdv[c] * s1 + xv[c] * s2 * xd0);
  }
  xb[base] = b0;
  xc[base] = c0;
}

// Readout E_i = w2 . silu(P), P = h0 W_r, with tangent E_dot_i = w2 . (silu'(P) P_dot),
// P_dot = h0_dot W_r, reversed for the scalar sum_i [gE_{s(i)} E_i - E_dot_i].
// One wave per atom. Writes the adjoints of P and P_dot ([N,16] each), the
// per-atom terms of the w2 gradient ([N,16]), the adjoints of h0 and h0_dot
// ([N, nc, C], component 0) and gE_{s(i)} per atom (for the E0 gradient).
__global__ void __launch_bounds__(256) k_readout_dual(const float* __restrict__ h, const float* __restrict__ hd, int nc,
                                                      const int* __restrict__ owner, const double* __restrict__ gE,
                                                      const float* __restrict__ Wr, const float* __restrict__ w2,
                                                      int N, int C, float* __restrict__ Pb, float* __restrict__ Pc,
                                                      float* __restrict__ w2c, float* __restrict__ hb,
                                                      float* __restrict__ hc, float* __restrict__ eb) {
  const int i = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (i >= N) return;
  float P[16], Pd[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) P[q] = Pd[q] = 0.0f;
  for (int k = lane; k < C; k += 64) {
    const float a = h[(long)i * nc * C + k], ad = hd[(long)i * nc * C + k];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      P[q] += a * Wr[k * 16 + q];
      Pd[q] += ad * Wr[k * 16 + q];
    }
  }
  const float Eb = (float)gE[owner[i]];
  const float Ec = -1.0f;
  float pb[16], pc[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    P[q] = wave_sum(P[q]);
    Pd[q] = wave_sum(Pd[q]);
    const float s1 = silu_grad(P[q]), s2 = silu_grad2(P[q]);
    pc[q] = Ec * w2[q] * s1;
    pb[q] = Eb * w2[q] * s1 + Ec * w2[q] * s2 * Pd[q];
    if (lane == q) {
      Pb[(long)i * 16 + q] = pb[q];
      Pc[(long)i * 16 + q] = pc[q];
      w2c[(long)i * 16 + q] = Eb * siluf(P[q]) + Ec * s1 * Pd[q];
    }
  }
  if (lane == 0) eb[i] = Eb;
  for (int k = lane; k < C; k += 64) {
    float sb = 0.0f, sc = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      sb += Wr[k * 16 + q] * pb[q];
      sc += Wr[k * 16 + q] * pc[q];
    }
    hb[(long)i * nc * C + k] = sb;
    hc[(long)i * nc * C + k] = sc;
  }
}

// Sums over atoms by group, in two passes of fixed order, in FP64: partials
// over chunks of kSumAtoms atoms, then over the chunks. part[chunk, g, c] =
// sum over the chunk's atoms i with species[i] == g (all when species is NULL)
// of X[i * ld + c]. One pass over all atoms per output leaves as many threads
// as outputs (16 to a few hundred), each with a chain of N loads: 1.0-1.3 ms on
// 7,000 atoms, against 20 us for both passes.
constexpr int kSumAtoms = 64;
__global__ void __launch_bounds__(256) k_group_partial(const float* __restrict__ X, long ld,
                                                       const int* __restrict__ species, int n_groups, int N,
                                                       int ncols, double* __restrict__ part) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n_groups * ncols) return;
  const int g = t / ncols, c = t % ncols;
  const int i0 = blockIdx.y * kSumAtoms, n = min(kSumAtoms, N - i0);
  double acc = 0.0;
#pragma unroll 8
  for (int i = 0; i < n; ++i) {
    const float v = X[(long)(i0 + i) * ld + c];
    if (!species || species[i0 + i] == g) acc += (double)v;
  }
  part[(long)blockIdx.y * n_groups * ncols + t] = acc;
}
__global__ void __launch_bounds__(256) k_group_total(const double* __restrict__ part, int chunks, int n_groups,
                                                     int ncols, double* __restrict__ out, long ld_out) {
  // 32 outputs x 8 shares of the chunks
  __shared__ double red[8][32];
  const int total = n_groups * ncols;
  const int t = blockIdx.x * 32 + (threadIdx.x & 31), w = threadIdx.x >> 5;
  double acc = 0.0;
  if (t < total) {
#pragma unroll 4
    for (int q = w; q < chunks; q += 8) acc += part[(long)q * total + t];
  }
  red[w][threadIdx.x & 31] = acc;
  __syncthreads();
  if (w == 0 && t < total) {
    for (int q = 1; q < 8; ++q) acc += red[q][threadIdx.x];
    out[(long)(t / ncols) * ld_out + t % ncols] = acc;
  }
}

// Weight gradients: products X1^T Y1 + X2^T Y2 over rows (X: [rows, mo], Y:
// [rows, no], rows addressed through RowMaps), several in one launch. A
// workgroup takes a 64 x 64 output tile and a chunk of the rows, kTnRows at a
// time through LDS, the next ones in flight; its partial sum goes to memory and
// k_tn_reduce adds the chunks in order in FP64. FP32 as six BF16 products
// (gemm.hip): a lane loads eight rows of one column, which is an operand's eight
// K, and splits them on the way into LDS. Bound: the streams of X and Y (W3, W2
// and W1 of 183,000 pairs, P C = 256, 760 MB: 204 us, 3.7 TB/s). The products of a
// training step of 7,032 atoms 510 us and 45 for the sums of the chunks (640 and
// fewer with half the chunks, on the FP32 matrix cores 750); those with rows
// (atom, m), whose addresses take longer, 49.
struct TnGroup {
  TnArgs g[kMaxTnGroup];
  int block0[kMaxTnGroup + 1];  // first workgroup
  int tiles[kMaxTnGroup], ncol[kMaxTnGroup], chunks[kMaxTnGroup];
  long part0[kMaxTnGroup];      // first float of the partials
  int red0[kMaxTnGroup + 1];    // first workgroup of the reduction
  int n;
};
constexpr int kTnRows = 32;

__device__ __forceinline__ const float* tn_row(const RowMap& m, int r) {
  const int a = m.g == 1 ? r : r / m.g;
  return m.base + a * m.s_atom + (r - a * m.g) * m.s_m;
}

__global__ void __launch_bounds__(256) k_gemm_tn(TnGroup gg, float* __restrict__ partial) {
  __shared__ bf16x8 B[2][kTnRows / 16][2][3][64];  // [X, Y][16 rows][32 columns][part][lane]
  int gi = 0;
  while (gi + 1 < gg.n && (int)blockIdx.x >= gg.block0[gi + 1]) ++gi;
  const TnArgs& a = gg.g[gi];
  const int local = blockIdx.x - gg.block0[gi];
  const int chunk = local / gg.tiles[gi], tile = local % gg.tiles[gi];
  const int bm = tile / gg.ncol[gi] * 64, bn = tile % gg.ncol[gi] * 64;
  const int R = a.rows_dev ? min((int)a.rows, *a.rows_dev) : (int)a.rows;
  const int per = ((R + gg.chunks[gi] - 1) / gg.chunks[gi] + kTnRows - 1) / kTnRows * kTnRows;
  const int r0 = min(R, chunk * per), r1 = min(R, r0 + per);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int rb = w >> 1, cb = w & 1;
  const bool in_m = bm + lane < a.mo, in_n = bn + lane < a.no;
  const int terms = a.x2.base ? 2 : 1;
  const int steps = (r1 - r0 + kTnRows - 1) / kTnRows * terms;
  // a wave stages eight rows, a lane one column of each: an operand's eight K;
  // the rows' indices in Y come one step earlier
  const int* __restrict__ y_row = a.y_row;
  float xv[8], yv[8];
  int ahead = 0;
  auto index = [&](int s) {
    if (y_row && s < steps) ahead = y_row[min(r0 + s / terms * kTnRows + 8 * w + (lane & 7), R - 1)];
  };
  auto load = [&](int s) {
    const RowMap X = s % terms ? a.x2 : a.x1, Y = s % terms ? a.y2 : a.y1;
    const int r = r0 + s / terms * kTnRows + 8 * w, n = r1 - r;
    const int yi = ahead;
    index(s + 1);
    if (n >= 8 && X.g == 1 && Y.g == 1) {
      const float* px = X.base + (long)r * X.s_atom + bm + lane;
#pragma unroll
      for (int q = 0; q < 8; ++q) xv[q] = in_m ? px[(long)q * X.s_atom] : 0.0f;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int ry = y_row ? __builtin_amdgcn_readlane(yi, q) : r + q;
        yv[q] = in_n ? Y.base[(long)ry * Y.s_atom + bn + lane] : 0.0f;
      }
      return;
    }
    // the last rows, and rows (atom, m)
    int xa = r / X.g, xm = r - xa * X.g, ya = r / Y.g, ym = r - ya * Y.g;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      xv[q] = q < n && in_m ? X.base[xa * X.s_atom + xm * X.s_m + bm + lane] : 0.0f;
      if (++xm == X.g) {
        xm = 0;
        ++xa;
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int ry = __builtin_amdgcn_readlane(yi, q);
      yv[q] = q < n && in_n ? (y_row ? tn_row(Y, ry) : Y.base + ya * Y.s_atom + ym * Y.s_m)[bn + lane] : 0.0f;
      if (++ym == Y.g) {
        ym = 0;
        ++ya;
      }
    }
  };
  index(0);
  f32x16 hi = {}, lo = {};
  if (steps > 0) load(0);
  for (int s = 0; s < steps; ++s) {
    if (s > 0) __syncthreads();
    const int slot = (lane & 31) + 32 * (w & 1);
    split_bf16(xv, B[0][w >> 1][lane >> 5][0][slot], B[0][w >> 1][lane >> 5][1][slot], B[0][w >> 1][lane >> 5][2][slot]);
    split_bf16(yv, B[1][w >> 1][lane >> 5][0][slot], B[1][w >> 1][lane >> 5][1][slot], B[1][w >> 1][lane >> 5][2][slot]);
    __syncthreads();
    if (s + 1 < steps) load(s + 1);
#pragma unroll
    for (int j = 0; j < kTnRows / 16; ++j) {
      bf16x8 x[3], y[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        x[p] = B[0][j][rb][p][lane];
        y[p] = B[1][j][cb][p][lane];
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        f32x16& acc = i < 5 ? lo : hi;
        acc = mfma_bf(x[kSplitA[i]], y[kSplitB[i]], acc);
      }
    }
  }
  float* P = partial + gg.part0[gi] + (long)chunk * a.mo * a.no;
  const int col = bn + 32 * cb + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = bm + 32 * rb + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    if (row < a.mo && col < a.no) P[(long)row * a.no + col] = hi[r] + lo[r];
  }
}

// out[i * ld_out + j] = sum over chunks of partial[c][i][j] in FP64: 32 outputs
// x 8 shares of the chunks per workgroup, each in order.
__global__ void __launch_bounds__(256) k_tn_reduce(TnGroup gg, const float* __restrict__ partial) {
  __shared__ double red[8][32];
  int gi = 0;
  while (gi + 1 < gg.n && (int)blockIdx.x >= gg.red0[gi + 1]) ++gi;
  const TnArgs& a = gg.g[gi];
  const int total = a.mo * a.no, chunks = gg.chunks[gi];
  const int idx = (blockIdx.x - gg.red0[gi]) * 32 + (threadIdx.x & 31), w = threadIdx.x >> 5;
  const float* P = partial + gg.part0[gi];
  const int per = (chunks + 7) / 8, c1 = min(chunks, (w + 1) * per);
  double s = 0.0;
  if (idx < total) {
#pragma unroll 8
    for (int c = w * per; c < c1; ++c) s += (double)P[(long)c * total + idx];
  }
  red[w][threadIdx.x & 31] = s;
  __syncthreads();
  if (w == 0 && idx < total) {
    for (int q = 1; q < 8; ++q) s += red[q][threadIdx.x];
    a.out[(long)(idx / a.no) * a.ld_out + idx % a.no] = s;
  }
}

}  // namespace

void launch_gate_dual_fwd(const float* x, const float* xd, float* hd, int N, int nc, int C, hipStream_t st, int B) {
  if (N == 0) return;
  with_components(nc, [&](auto n) {
    k_gate_dual_fwd<decltype(n)::value><<<blocks((long)B * N * C, 256), 256, 0, st>>>(x, xd, hd, N, C, B);
  });
}
void launch_gate_dual_bwd(const float* x, const float* xd, const float* hb, const float* hc, float* xb, float* xc,
                          int N, int nc, int C, hipStream_t st, int B) {
  if (N == 0) return;
  with_components(nc, [&](auto n) {
    k_gate_dual_bwd<decltype(n)::value><<<blocks((long)B * N * C, 256), 256, 0, st>>>(x, xd, hb, hc, xb, xc, N, C, B);
  });
}
void launch_readout_dual(const float* h, const float* hd, int nc, const int* owner, const double* gE, const float* Wr,
                         const float* w2, int N, int C, float* Pb, float* Pc, float* w2c, float* hb, float* hc,
                         float* eb, hipStream_t st) {
  if (N == 0) return;
  k_readout_dual<<<blocks((long)N * 64, 256), 256, 0, st>>>(h, hd, nc, owner, gE, Wr, w2, N, C, Pb, Pc, w2c, hb, hc,
                                                             eb);
}
void launch_group_sum(const float* X, long ld, const int* species, int n_groups, int N, int ncols, double* part,
                      double* out, long ld_out, hipStream_t st) {
  const int total = n_groups * ncols, chunks = group_chunks(N);
  if (total == 0) return;
  if (N > 0)
    k_group_partial<<<dim3(blocks(total, 256), chunks), 256, 0, st>>>(X, ld, species, n_groups, N, ncols, part);
  k_group_total<<<blocks(total, 32), 256, 0, st>>>(part, N > 0 ? chunks : 0, n_groups, ncols, out, ld_out);
}
int group_chunks(int N) { return std::max(1, blocks(N, kSumAtoms)); }

// Chunks of a product's rows. A chunk is one sum in FP32, the chunks are added
// up in FP64: as many as it takes for chunks of at most kTnChunkRows rows (up to
// kTnChunks, and as many as the partial sums have room for), and no fewer than
// make about four workgroups per CU, without chunks of fewer than 128 rows, which
// do not pay for their partial sums. The gradient of W3 of a layer with every path
// (64 x 2,944 out of 183,000 rows) was off by 8e-7 with 11 chunks, now 1e-7 with
// 89; a training step of 7,032 atoms (64 x 256) 4.72 ms with 128 chunks, now 4.34.
constexpr int kTnChunkRows = 1024, kTnChunks = 256;
static int tn_chunks(long rows, int tiles, long mo_no) {
  const long exact = std::min<long>((rows + kTnChunkRows - 1) / kTnChunkRows, kTnChunks);
  const long fill = std::min<long>((rows + 127) / 128, 1024 / tiles);
  return (int)std::max<long>(1, std::min(std::max(exact, fill), kTnPartial / mo_no));
}

// The products share a launch while their partial sums fit the buffer together.
void launch_gemm_tn(const TnArgs* args, int n, float* partial, hipStream_t st) {
  E3MI_REQUIRE(n >= 0 && n <= kMaxTnGroup, E3MI_EINVAL, "weight-gradient group size out of range");
  TnGroup gg{};
  int m = 0, nblocks = 0, nred = 0;
  long part = 0;
  auto launch = [&] {
    if (m == 0) return;
    gg.block0[m] = nblocks;
    gg.red0[m] = nred;
    gg.n = m;
    k_gemm_tn<<<nblocks, 256, 0, st>>>(gg, partial);
    k_tn_reduce<<<nred, 256, 0, st>>>(gg, partial);
    m = nblocks = nred = 0;
    part = 0;
  };
  for (int k = 0; k < n; ++k) {
    const TnArgs& a = args[k];
    if (a.mo == 0 || a.no == 0 || a.rows <= 0) continue;
    E3MI_REQUIRE(a.mo % 4 == 0 && a.no % 4 == 0 && a.rows < (1L << 31), E3MI_EUNSUPPORTED,
                 "weight gradients: dimensions must be multiples of 4");
    const long mo_no = (long)a.mo * a.no;
    const int ncol = blocks(a.no, 64), tiles = blocks(a.mo, 64) * ncol, chunks = tn_chunks(a.rows, tiles, mo_no);
    if (part + chunks * mo_no > kTnPartial) launch();
    gg.g[m] = a;
    gg.ncol[m] = ncol;
    gg.tiles[m] = tiles;
    gg.chunks[m] = chunks;
    gg.block0[m] = nblocks;
    gg.part0[m] = part;
    gg.red0[m] = nred;
    nblocks += tiles * chunks;
    part += chunks * mo_no;
    nred += blocks(mo_no, 32);
    ++m;
  }
  launch();
}

size_t tn_partial_floats(long mo_no_max) { return (size_t)std::max(kTnPartial, mo_no_max); }

}  // namespace e3mi
