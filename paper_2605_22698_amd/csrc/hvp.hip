// Hessian-vector products: the tangent pass along position directions v_b and
// the reverse pass over primal and tangent values, continued to the positions.
// The primal values (features, R and its derivatives) are computed once per
// call; everything here carries a direction index b, and one launch takes a
// batch of directions (rows (b, atom) and (b, edge)), so that small systems
// fill the GPU and the launches are shared.
//
// For an edge e = (i <- j) with vector d, tangent d_dot = v_j - v_i and
// rho = n . d_dot (n = d / r), R_dot = R'(r) rho, so
//   A      = nu^-1 sum_e R T(h_j, Y)
//   A_dot  = nu^-1 sum_e [R' rho T(h_j, Y) + R (T(h_dot_j, Y) + T(h_j, Y_dot))].
// With ab, ac the adjoints of A and A_dot (times nu^-1), per path and channel
//   sb = ab T(h, Y) + ac (T(h_dot, Y) + T(h, Y_dot)),   sc = ac T(h, Y)
//   ds/dr += sb R' + sc rho R'',                        ds/drho += sc R'
//   eb = ab R + ac R' rho,                              ec = ac R
//   Yb += C (eb h + ec h_dot),                          Yc += C ec h
//   hb_j += C (eb Y + ec Y_dot),                        hc_j += C ec Y.
// Yb, Yc, ds/dr and ds/drho are summed over paths and channels into one row
// per edge ("geo row"), which k_hvp_geo turns into the edge's position
// adjoint; neither R_dot nor the adjoints of R go to memory.
//
// The weight gradient of a loss on energies and forces runs the same kernels
// along one direction (W variants); it stops at the adjoints of R and R' = dR/dr,
// sb and rho sc, which radial.hip takes back through the radial MLP.
//
// Bound: the feature and adjoint gathers from L2 (16 x C values each) and, in
// the adjoints, the vector ALU. Measured (l_max 3, 128 channels, 2 layers): the
// full Hessians of 64 molecules of 10-31 atoms (93 products, 13 directions at
// once) 90.5 -> 13.7 ms, one product on a 3,000-atom box 5.35 -> 1.96 ms,
// against one direction at a time with the radial MLP's tangent and adjoint
// formed per direction and R_dot and the adjoints of R in memory. Per 13
// directions of the molecules: sender adjoint 420 us, receiver-side adjoint of
// the first layer 302 us, tangent sums 325 and 116 us (402 and 149 us with one
// direction per workgroup).
#include "common.h"
#include "paths.h"
#include "runtime.h"

namespace e3mi {
namespace {

constexpr int kGeo = kHvpGeoRow;  // [Yb 16][Yc 16][ds/dr][ds/drho][2 unused]

// element (row, m, path rank) of an order's block in the grouped layout, channel 0
__device__ __forceinline__ long a_index(int l3, int C, int P3, long row, int m, int rank, long gb) {
  return gb + ((row * (2 * l3 + 1) + m) * P3 + rank) * C;
}

// The lane's CH channels start at k0; lanes past the last channel (32-channel
// models) read the first channels again and contribute zeros.
// Loads are written as (uniform address)[k0] with k0 unsigned, so that the
// address stays in scalar registers (64-bit vector addresses of an edge's
// rows would take half the register file).
struct Lane {
  unsigned k0;
  bool on;
};
template <int CH>
__device__ __forceinline__ Lane lane_channels(int C) {
  const unsigned k = threadIdx.x * CH;
  return Lane{(k < (unsigned)C ? k : k - C) & 127, k < (unsigned)C};  // & 127: a known range

}

// ---- tangent of the neighbour sum ---------------------------------------------
// One workgroup per (ND directions, receiver), CH channels per lane. The
// senders' features and R are the same for every direction, and the gathers
// bound the kernel (L2), so layers whose accumulators are few take two
// directions at once. An odd last direction is computed twice by its workgroup
// (the same values to the same place).
template <int LMAX, int KIND, int CH, int ND>
__global__ void __launch_bounds__(KIND == kFull ? 128 : 64) k_hvp_fwd(HvpArgs a) {
  using PS = PathSet<LMAX, KIND>;
  constexpr bool H = KIND == kFull || KIND == kLast;  // h_dot is not zero
  constexpr int NP = PS::NP, NOUT = PS::NOUT, NIN = PS::NIN, NY = PS::NY;
  const int w = xcd_contiguous(blockIdx.x, gridDim.x);
  const int i = w % a.N, C = a.C;
  const long rows = (long)a.B * a.N;
  const Lane ln = lane_channels<CH>(C);
  long u[ND];  // row (direction, receiver)
  const float4* dd[ND];
  const float* hd[ND];
#pragma unroll
  for (int n = 0; n < ND; ++n) {
    const int b = min(w / a.N * ND + n, a.B - 1);
    u[n] = (long)b * a.N + i;
    dd[n] = a.dd + b * a.e_stride;
    hd[n] = H ? a.hd + (long)b * a.N * NIN * C : nullptr;
  }
  float acc[ND][NOUT][CH];
#pragma unroll
  for (int n = 0; n < ND; ++n)
#pragma unroll
    for (int o = 0; o < NOUT; ++o)
#pragma unroll
      for (int c = 0; c < CH; ++c) acc[n][o][c] = 0.0f;
  const int e1 = a.row_ptr[i + 1];
  for (int e = a.row_ptr[i]; e < e1; ++e) {
    const int j = a.src[e];
    const float4 d = a.dvec[e];
    float4 t[ND];
    float Y[NY], Yd[ND][NY];
#pragma unroll
    for (int n = 0; n < ND; ++n) {
      t[n] = dd[n][e];
      real_sh_dual<LMAX>(d, t[n], Y, Yd[n]);
    }
    const long ro = (long)(a.r_row ? a.r_row[e] : e) * a.r_stride;
    float hv[NIN][CH], hdv[ND][H ? NIN : 1][CH];
#pragma unroll
    for (int q = 0; q < NIN; ++q) {
      ldr_n<CH>(a.h + ((long)j * a.h_nc + q) * C + ln.k0, hv[q]);
      if constexpr (H) {
#pragma unroll
        for (int n = 0; n < ND; ++n) ldr_n<CH>(hd[n] + ((long)j * NIN + q) * C + ln.k0, hdv[n][q]);
      }
    }
    float r0[NP][CH], r1[NP][CH];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      ldr_n<CH>(a.R + ro + q * C + ln.k0, r0[q]);
      ldr_n<CH>(a.Rp + ro + q * C + ln.k0, r1[q]);
    }
    static_for<NP>([&](auto pi) {
      constexpr int g = PS::T.id[pi];
      constexpr int l1 = kL1[g], l2 = kL2[g], l3 = kL3[g];
      constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
      constexpr int off = PS::T.off[pi];
      constexpr bool ONE = one_coefficient(g);
      float tm[2 * l3 + 1][CH], td[ND][2 * l3 + 1][CH];
#pragma unroll
      for (int m = 0; m < 2 * l3 + 1; ++m)
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          tm[m][c] = 0.0f;
#pragma unroll
          for (int n = 0; n < ND; ++n) td[n][m][c] = 0.0f;
        }
      static_for<nz>([&](auto z) {
        constexpr int q = z0 + z;
        constexpr int q1 = l1 * l1 + kM1[q], q2 = l2 * l2 + kM2[q], m = kM3[q];
        const float cy = ONE ? Y[q2] : kC[q] * Y[q2];
#pragma unroll
        for (int c = 0; c < CH; ++c) tm[m][c] += hv[q1][c] * cy;
#pragma unroll
        for (int n = 0; n < ND; ++n) {
          const float cyd = ONE ? Yd[n][q2] : kC[q] * Yd[n][q2];
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            td[n][m][c] += hv[q1][c] * cyd;
            if constexpr (H) td[n][m][c] += hdv[n][q1][c] * cy;
          }
        }
      });
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const float rv = ONE ? kC[z0] * r0[pi][c] : r0[pi][c], rp = ONE ? kC[z0] * r1[pi][c] : r1[pi][c];
#pragma unroll
        for (int n = 0; n < ND; ++n) {
          const float rd = rp * t[n].w;
#pragma unroll
          for (int m = 0; m < 2 * l3 + 1; ++m) acc[n][off + m][c] += rd * tm[m][c] + rv * td[n][m][c];
        }
      }
    });
  }
  if (!ln.on) return;
  static_for<NP>([&](auto pi) {
    constexpr int g = PS::T.id[pi];
    constexpr int l3 = kL3[g];
    constexpr int off = PS::T.off[pi], rank = PS::T.rank[pi];
    constexpr int P3 = PS::T.np_l3[l3];
    const long gb = a_group_base<PS>(l3, rows, C);
#pragma unroll
    for (int n = 0; n < ND; ++n)
#pragma unroll
      for (int m = 0; m < 2 * l3 + 1; ++m) {
        float v[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) v[c] = acc[n][off + m][c] * a.inv_nu;
        str_n<CH>(a.Ad + a_index(l3, C, P3, u[n], m, rank, gb) + ln.k0, v);
      }
  });
}

// Offset of the first output of order l3 in a channel's accumulator (paths are
// ordered by l3).
template <class PS>
constexpr int first_output(int l3) {
  int o = 0;
  for (int l = 0; l < l3 && l <= PS::L3MAX; ++l) o += (2 * l + 1) * PS::T.np_l3[l];
  return o;
}

// ab and ac (times nu^-1) of row u for the output orders LO..HI; zero on lanes
// past the last channel.
template <class PS, int LO, int HI, int CH>
__device__ __forceinline__ void load_adjoints(const HvpArgs& a, long u, Lane ln, float (*ab)[CH], float (*ac)[CH]) {
  const long bn = (long)a.B * a.N, rows = 2 * bn;  // ab of every direction, then ac
  const float scale = ln.on ? a.inv_nu : 0.0f;
  static_for<PS::NP>([&](auto pi) {
    constexpr int g = PS::T.id[pi];
    constexpr int l3 = kL3[g];
    if constexpr (l3 >= LO && l3 <= HI) {
      constexpr int off = PS::T.off[pi] - first_output<PS>(LO), rank = PS::T.rank[pi];
      constexpr int P3 = PS::T.np_l3[l3];
      const long gb = a_group_base<PS>(l3, rows, a.C);
#pragma unroll
      for (int m = 0; m < 2 * l3 + 1; ++m) {
        ldr_n<CH>(a.Ab + a_index(l3, a.C, P3, u, m, rank, gb) + ln.k0, ab[off + m]);
        ldr_n<CH>(a.Ab + a_index(l3, a.C, P3, u + bn, m, rank, gb) + ln.k0, ac[off + m]);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          ab[off + m][c] *= scale;
          ac[off + m][c] *= scale;
        }
      }
    }
  });
}

// One path's share of an edge: the sums above for CH channels (ab and ac from
// output O0 on). HD: h_dot is not zero, and its adjoint is wanted; HB: the
// adjoint of h is wanted. W (weight gradients): instead of the geo sums, rb and
// rc get the adjoints of R and of R' (rho times that of R_dot).
template <class PS, int PI, int O0, bool HD, bool HB, bool W, int CH, int NY>
__device__ __forceinline__ void path_adjoint(const float (*hv)[CH], const float (*hdv)[CH], const float* Y,
                                             const float* Yd, float rho, const float* r0, const float* r1,
                                             const float* r2, const float (*ab)[CH], const float (*ac)[CH],
                                             float& sr, float& sd, float* yb, float* yc, float (*hb)[CH],
                                             float (*hc)[CH], float* rb = nullptr, float* rc = nullptr) {
  constexpr int g = PS::T.id[PI];
  constexpr int l1 = kL1[g], l2 = kL2[g], l3 = kL3[g];
  constexpr int z0 = kNzBegin[g], nz = kNzBegin[g + 1] - kNzBegin[g];
  constexpr int off = PS::T.off[PI] - O0;
  constexpr bool ONE = one_coefficient(g);
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    float tm[2 * l3 + 1], td[2 * l3 + 1], eb[2 * l3 + 1], ec[2 * l3 + 1];
    // the path's one coefficient, if it has one, goes into R and its derivatives
    const float c0 = ONE ? kC[z0] : 1.0f;
    const float s0 = c0 * r0[c], s1 = c0 * r1[c], rd = s1 * rho;
#pragma unroll
    for (int m = 0; m < 2 * l3 + 1; ++m) {
      tm[m] = td[m] = 0.0f;
      eb[m] = ab[off + m][c] * s0 + ac[off + m][c] * rd;
      ec[m] = ac[off + m][c] * s0;
    }
    static_for<nz>([&](auto z) {
      constexpr int q = z0 + z;
      constexpr int q1 = l1 * l1 + kM1[q], q2 = l2 * l2 + kM2[q], m = kM3[q];
      const float cy = ONE ? Y[q2] : kC[q] * Y[q2], cyd = ONE ? Yd[q2] : kC[q] * Yd[q2];
      const float x = hv[q1][c], cx = ONE ? x : kC[q] * x;
      tm[m] += x * cy;
      td[m] += x * cyd;
      if constexpr (!W) {
        yb[q2] += eb[m] * cx;
        yc[q2] += ec[m] * cx;
      }
      if constexpr (HD) {
        const float xd = hdv[q1][c];
        td[m] += xd * cy;
        if constexpr (!W) yb[q2] += ec[m] * (ONE ? xd : kC[q] * xd);
        hc[q1][c] += ec[m] * cy;
      }
      if constexpr (HB) hb[q1][c] += eb[m] * cy + ec[m] * cyd;
    });
    float sb = 0.0f, sc = 0.0f;
#pragma unroll
    for (int m = 0; m < 2 * l3 + 1; ++m) {
      sb += ab[off + m][c] * tm[m] + ac[off + m][c] * td[m];
      sc += ac[off + m][c] * tm[m];
    }
    if constexpr (W) {
      rb[c] = c0 * sb;
      rc[c] = c0 * sc * rho;
    } else {
      sr += sb * s1 + sc * (rho * (c0 * r2[c]));
      sd += sc * s1;
    }
  }
}

// Sums a wave's per-lane geo values over its lanes and hands value q to `put`
// on one lane each.
template <int NY, class F>
__device__ __forceinline__ void reduce_geo(const float* yb, const float* yc, float sr, float sd, F&& put) {
  const int lane = threadIdx.x & 63;
  const float tb = wave_sum_scatter16<NY>(yb), tc = wave_sum_scatter16<NY>(yc);
  const float ts = wave_sum_scatter2(sr, sd);
  if ((lane & 3) == 0) {
    put(lane >> 2, tb);
    put(16 + (lane >> 2), tc);
  }
  if ((lane & 31) == 1) put(32 + (lane >> 5), ts);
}

// ---- receiver-side edge adjoint --------------------------------------------------
// Scalar-input layers: one wave per (direction, receiver), ab_i and ac_i in
// registers (h_dot is zero). W false: one geo row per edge (nothing depends on
// h). W true (weight gradients, one direction): the edges' adjoints of R and
// R', and the edge's share of its sender's embedding gradient, msg [E, C].
template <int LMAX, int KIND, int CH, bool W>
__global__ void __launch_bounds__(64) k_hvp_edge(HvpArgs a) {
  using PS = PathSet<LMAX, KIND>;
  constexpr int NP = PS::NP, NOUT = PS::NOUT, NIN = PS::NIN, NY = PS::NY;
  static_assert(NIN == 1, "scalar inputs");
  const long u = xcd_contiguous(blockIdx.x, gridDim.x);
  const int b = (int)(u / a.N), i = (int)(u % a.N), C = a.C;
  const Lane ln = lane_channels<CH>(C);
  const float4* dd = a.dd + (long)b * a.e_stride;
  float* geo = W ? nullptr : a.geo + (long)b * a.e_stride * kGeo;
  float ab[NOUT][CH], ac[NOUT][CH];
  load_adjoints<PS, 0, 3, CH>(a, u, ln, ab, ac);
  const int e1 = a.row_ptr[i + 1];
  for (int e = a.row_ptr[i]; e < e1; ++e) {
    const float4 t = dd[e];
    float Y[NY], Yd[NY], yb[NY], yc[NY];
    real_sh_dual<LMAX>(a.dvec[e], t, Y, Yd);
#pragma unroll
    for (int q = 0; q < NY; ++q) yb[q] = yc[q] = 0.0f;
    const long ro = (long)(a.r_row ? a.r_row[e] : e) * a.r_stride;
    float hv[1][CH], hb[1][CH], none[1][CH];
    ldr_n<CH>(a.h + (long)a.src[e] * a.h_nc * C + ln.k0, hv[0]);
#pragma unroll
    for (int c = 0; c < CH; ++c) hb[0][c] = 0.0f;
    float sr = 0.0f, sd = 0.0f;
    static_for<NP>([&](auto pi) {
      float r0[CH], r1[CH], r2[CH], rb[CH], rc[CH];
      ldr_n<CH>(a.R + ro + pi * C + ln.k0, r0);
      ldr_n<CH>(a.Rp + ro + pi * C + ln.k0, r1);
      if constexpr (!W) ldr_n<CH>(a.Rpp + ro + pi * C + ln.k0, r2);
      path_adjoint<PS, pi, 0, false, W, W, CH, NY>(hv, none, Y, Yd, t.w, r0, r1, r2, ab, ac, sr, sd, yb, yc, hb, none,
                                                   rb, rc);
      if constexpr (W) {
        if (ln.on) {
          str_n<CH>(a.Rb + ((long)e * NP + pi) * C + ln.k0, rb);
          str_n<CH>(a.Rc + ((long)e * NP + pi) * C + ln.k0, rc);
        }
      }
    });
    if constexpr (W) {
      if (ln.on) str_n<CH>(a.msg + (long)e * C + ln.k0, hb[0]);
    } else {
      reduce_geo<NY>(yb, yc, sr, sd, [&](int q, float v) { geo[(long)e * kGeo + q] = v; });
    }
  }
}

// Layers with every path: besides the geo row, the edge's share of its
// sender's adjoints, [2][NIN][C] (of h, then of h_dot), which k_hvp_msg_node
// adds up per sender (gathering the receivers' 198 adjoint values per channel
// from the senders' side would read six times as much). One channel per lane,
// up to two waves. For l_max 3 the 198 adjoint values, the features, the
// messages and the harmonics do not fit a lane's 512 registers, so the output
// orders LO..HI are taken in three launches (l3 < 2, l3 = 2, l3 = 3), each
// adding to the messages and geo rows of the one before (in one or two
// launches the compiler spills 139 or 11 registers to memory).
// W (weight gradients): the adjoints of R and R' instead of geo rows.
template <int LMAX, int LO, int HI, bool W>
__global__ void __launch_bounds__(128) k_hvp_edge_full(HvpArgs a) {
  using PS = PathSet<LMAX, kFull>;
  constexpr int NP = PS::NP, NIN = PS::NIN, NY = PS::NY;
  constexpr int O0 = first_output<PS>(LO), O1 = first_output<PS>(HI + 1);
  __shared__ float red[2][2][kGeo];
  const long u = xcd_contiguous(blockIdx.x, gridDim.x);
  const int b = (int)(u / a.N), i = (int)(u % a.N), C = a.C;
  const Lane ln = lane_channels<1>(C);
  const float4* dd = a.dd + (long)b * a.e_stride;
  const float* hd = a.hd + (long)b * a.N * NIN * C;
  float* geo = W ? nullptr : a.geo + (long)b * a.e_stride * kGeo;
  float* msg = a.msg + (long)b * a.e_stride * 2 * NIN * C;
  float ab[O1 - O0][1], ac[O1 - O0][1];
  load_adjoints<PS, LO, HI, 1>(a, u, ln, ab, ac);
  const int e1 = a.row_ptr[i + 1];
  for (int e = a.row_ptr[i]; e < e1; ++e) {
    const int j = a.src[e];
    const float4 t = dd[e];
    float Y[NY], Yd[NY], yb[NY], yc[NY];
    real_sh_dual<LMAX>(a.dvec[e], t, Y, Yd);
#pragma unroll
    for (int q = 0; q < NY; ++q) yb[q] = yc[q] = 0.0f;
    const long ro = (long)(a.r_row ? a.r_row[e] : e) * a.r_stride;
    float* me = msg + (long)e * 2 * NIN * C;
    float hv[NIN][1], hdv[NIN][1], hb[NIN][1], hc[NIN][1];
#pragma unroll
    for (int q = 0; q < NIN; ++q) {
      hv[q][0] = (a.h + ((long)j * NIN + q) * C)[ln.k0];
      hdv[q][0] = (hd + ((long)j * NIN + q) * C)[ln.k0];
      hb[q][0] = LO > 0 ? (me + q * C)[ln.k0] : 0.0f;
      hc[q][0] = LO > 0 ? (me + (NIN + q) * C)[ln.k0] : 0.0f;
    }
    float sr = 0.0f, sd = 0.0f;
    float r0[NP], r1[NP], r2[NP];
    static_for<NP>([&](auto pi) {
      if constexpr (kL3[PS::T.id[pi]] >= LO && kL3[PS::T.id[pi]] <= HI) {
        r0[pi] = (a.R + ro + pi * C)[ln.k0];
        r1[pi] = (a.Rp + ro + pi * C)[ln.k0];
        if constexpr (!W) r2[pi] = (a.Rpp + ro + pi * C)[ln.k0];
      }
    });
    // one path after the other, none keeping the products of coefficients and
    // harmonics of another (Y and Yd are opaque between paths): they would spill
    static_for<NP>([&](auto pi) {
      if constexpr (kL3[PS::T.id[pi]] >= LO && kL3[PS::T.id[pi]] <= HI) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < NY; ++q) asm volatile("" : "+v"(Y[q]), "+v"(Yd[q]));
        float rb, rc;
        path_adjoint<PS, pi, O0, true, true, W, 1, NY>(hv, hdv, Y, Yd, t.w, &r0[pi], &r1[pi], &r2[pi], ab, ac, sr, sd,
                                                       yb, yc, hb, hc, &rb, &rc);
        if constexpr (W) {
          if (ln.on) {
            (a.Rb + ((long)e * NP + pi) * C)[ln.k0] = rb;
            (a.Rc + ((long)e * NP + pi) * C)[ln.k0] = rc;
          }
        }
      }
    });
    __builtin_amdgcn_sched_barrier(0);
    if (ln.on) {
#pragma unroll
      for (int q = 0; q < NIN; ++q) {
        (me + q * C)[ln.k0] = hb[q][0];
        (me + (NIN + q) * C)[ln.k0] = hc[q][0];
      }
    }
    if constexpr (W) continue;
    float* row = geo + (long)e * kGeo;
    if (blockDim.x == 64) {
      reduce_geo<NY>(yb, yc, sr, sd, [&](int q, float v) { row[q] = LO > 0 ? row[q] + v : v; });
    } else {
      // two waves: one barrier per edge, the exchange buffer alternates
      float(*buf)[kGeo] = red[e & 1];
      reduce_geo<NY>(yb, yc, sr, sd, [&](int q, float v) { buf[threadIdx.x >> 6][q] = v; });
      __syncthreads();
      if (threadIdx.x < 34) {
        const float v = buf[0][threadIdx.x] + buf[1][threadIdx.x];
        row[threadIdx.x] = LO > 0 ? row[threadIdx.x] + v : v;
      }
    }
  }
}

// Sender gradients from the edges' messages: hb_j, hc_j (+)= the messages of
// j's outgoing edges, in the order of j's row (HC false: of h alone).
template <int NIN, bool HC>
__global__ void __launch_bounds__(128) k_hvp_msg_node(HvpArgs a) {
  constexpr int NM = HC ? 2 * NIN : NIN;
  const long u = xcd_contiguous(blockIdx.x, gridDim.x);
  const int b = (int)(u / a.N), j = (int)(u % a.N), C = a.C;
  const unsigned k = threadIdx.x;
  if (k >= (unsigned)C) return;
  const float* msg = a.msg + (long)b * a.e_stride * NM * C;
  float acc[NM];
#pragma unroll
  for (int q = 0; q < NM; ++q) {
    acc[q] = q % NIN < a.dh_acc ? ((q < NIN ? a.hb : a.hc) + (u * NIN + q % NIN) * C)[k] : 0.0f;
  }
  const int e1 = a.row_ptr[j + 1];
  for (int e2 = a.row_ptr[j]; e2 < e1; ++e2) {
    const int e = a.rev[e2];
    if (e < 0) continue;
    const float* me = msg + (long)e * NM * C;
#pragma unroll
    for (int q = 0; q < NM; ++q) acc[q] += (me + q * C)[k];
  }
#pragma unroll
  for (int q = 0; q < NM; ++q) ((q < NIN ? a.hb : a.hc) + (u * NIN + q % NIN) * C)[k] = acc[q];
}

// ---- scalar-output layer, from the senders' side ---------------------------------
// A wave owns (direction, sender j): h_j, h_dot_j, hb_j and hc_j in registers.
// It walks j's own row: the edge e2 = (j <- i) stands for e = rev(e2) =
// (i <- j), whose vector and tangent are the opposite, so Y_e = (-1)^l Y_e2,
// and with R_l replaced by (-1)^l R_l everything is a function of e2's own
// geometry. The geo row in slot e2 then gives the gradient with respect to
// d_e2 = -d_e, i.e. minus e's, and since the forces take g_e - g_rev(e) over
// i's edges they come out the same. Per edge only the receiver's 2 x NP x C
// adjoint values are gathered (a receiver-side pass gathers 2 x 16 x C).
// W (weight gradients): the adjoints of R and R' of e in slot e2 (a pair's two
// edges are added up later, so either slot will do) instead of the geo row.
template <int LMAX, int CH, bool W>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 10))) k_hvp_sender(HvpArgs a) {
  using PS = PathSet<LMAX, kLast>;
  constexpr int NP = PS::NP, NIN = PS::NIN, NY = PS::NY;
  static_assert(PS::NOUT == NP, "scalar outputs only");
  const long u = xcd_contiguous(blockIdx.x, gridDim.x);
  const int b = (int)(u / a.N), j = (int)(u % a.N), C = a.C;
  const long BN = (long)a.B * a.N;
  const Lane ln = lane_channels<CH>(C);
  const float scale = ln.on ? a.inv_nu : 0.0f;
  const float4* dd = a.dd + (long)b * a.e_stride;
  float* geo = W ? nullptr : a.geo + (long)b * a.e_stride * kGeo;
  float hv[NIN][CH], hdv[NIN][CH], hb[NIN][CH], hc[NIN][CH];
#pragma unroll
  for (int q = 0; q < NIN; ++q) {
    ldr_n<CH>(a.h + ((long)j * a.h_nc + q) * C + ln.k0, hv[q]);
    ldr_n<CH>(a.hd + (u * a.h_nc + q) * C + ln.k0, hdv[q]);
#pragma unroll
    for (int c = 0; c < CH; ++c) hb[q][c] = hc[q][c] = 0.0f;
  }
  const int e1 = a.row_ptr[j + 1];
  for (int e2 = a.row_ptr[j]; e2 < e1; ++e2) {
    if (a.rev[e2] < 0) {  // the edge i <- j is not in i's list
      if constexpr (W) {
        const float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int q = 0; q < NP && ln.on; ++q) {
          str_n<CH>(a.Rb + ((long)e2 * NP + q) * C + ln.k0, z);
          str_n<CH>(a.Rc + ((long)e2 * NP + q) * C + ln.k0, z);
        }
      } else {
        if (threadIdx.x < kGeo) geo[(long)e2 * kGeo + threadIdx.x] = 0.0f;
      }
      continue;
    }
    const long ro = (long)(a.r_row ? a.r_row[e2] : e2) * a.r_stride;
    const float* Ai = a.Ab + ((long)b * a.N + a.src[e2]) * NP * C;
    float r0[NP][CH], r1[NP][CH], r2[NP][CH], ab[NP][CH], ac[NP][CH];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      ldr_n<CH>(a.R + ro + q * C + ln.k0, r0[q]);
      ldr_n<CH>(a.Rp + ro + q * C + ln.k0, r1[q]);
      if constexpr (!W) ldr_n<CH>(a.Rpp + ro + q * C + ln.k0, r2[q]);
    }
    static_for<NP>([&](auto pi) {
      constexpr int g = PS::T.id[pi];
      ldr_n<CH>(Ai + PS::T.rank[pi] * C + ln.k0, ab[pi]);
      ldr_n<CH>(Ai + (BN * NP + PS::T.rank[pi]) * C + ln.k0, ac[pi]);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const float s = kL2[g] & 1 ? -scale : scale;  // (-1)^l of R, folded into ab and ac
        ab[pi][c] *= s;
        ac[pi][c] *= s;
      }
    });
    const float4 t = dd[e2];
    float Y[NY], Yd[NY], yb[NY], yc[NY];
    real_sh_dual<LMAX>(a.dvec[e2], t, Y, Yd);
#pragma unroll
    for (int q = 0; q < NY; ++q) yb[q] = yc[q] = 0.0f;
    float sr = 0.0f, sd = 0.0f;
    static_for<NP>([&](auto pi) {
      float rb[CH], rc[CH];
      path_adjoint<PS, pi, 0, true, true, W, CH, NY>(hv, hdv, Y, Yd, t.w, r0[pi], r1[pi], r2[pi], ab, ac, sr, sd, yb,
                                                     yc, hb, hc, rb, rc);
      if constexpr (W) {
        if (ln.on) {
          str_n<CH>(a.Rb + ((long)e2 * NP + pi) * C + ln.k0, rb);
          str_n<CH>(a.Rc + ((long)e2 * NP + pi) * C + ln.k0, rc);
        }
      }
    });
    if constexpr (!W) reduce_geo<NY>(yb, yc, sr, sd, [&](int q, float v) { geo[(long)e2 * kGeo + q] = v; });
  }
  if (!ln.on) return;
  // components below dh_acc are added to, the others written
#pragma unroll
  for (int q = 0; q < NIN; ++q) {
    float* ob = a.hb + (u * NIN + q) * C + ln.k0;
    float* oc = a.hc + (u * NIN + q) * C + ln.k0;
    float vb[CH], vc[CH];
    if (q < a.dh_acc) {
      ldr_n<CH>(ob, vb);
      ldr_n<CH>(oc, vc);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        hb[q][c] += vb[c];
        hc[q][c] += vc[c];
      }
    }
    str_n<CH>(ob, hb[q]);
    str_n<CH>(oc, hc[q]);
  }
}

// ---- edges -----------------------------------------------------------------------
// d_dot = v_j - v_i and r_dot = n . d_dot of every edge and direction. One
// wave per (direction, row).
__global__ void __launch_bounds__(256) k_hvp_tangent(const int* __restrict__ row_ptr, const int* __restrict__ src,
                                                     const float4* __restrict__ dvec, const float* __restrict__ v,
                                                     int N, int B, long e_stride, float4* __restrict__ dd) {
  const long u = ((long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (u >= (long)B * N) return;
  const int b = (int)(u / N), i = (int)(u % N);
  const float* vb = v + 3L * b * N;
  const float vx = vb[3 * i], vy = vb[3 * i + 1], vz = vb[3 * i + 2];
  const int e1 = row_ptr[i + 1];
  for (int e = row_ptr[i] + lane; e < e1; e += 64) {
    const int j = src[e];
    const float4 d = dvec[e];
    const float x = vb[3 * j] - vx, y = vb[3 * j + 1] - vy, z = vb[3 * j + 2] - vz;
    dd[b * e_stride + e] = make_float4(x, y, z, (d.x * x + d.y * y + d.z * z) / d.w);
  }
}

// Per-edge position adjoint of the second-order scalar s = -D_v E through the
// edge geometry of one layer, from its geo row. With n = d/r, P = I - n n^T,
// and u = P d_dot / r:
//   harmonics  Y = P_c(n), Y_dot = grad P_c(n) . u, adjoints Yb, Yc:
//     g += P G1 / r + P (H u) / r - r_dot/r^2 P G2 - (G2 . n)/r^2 P d_dot - (G2 . P d_dot)/r^2 n
//     G1 = sum Yb grad P, G2 = sum Yc grad P, H = sum Yc hess P
//   lengths    g += ds/dr n + ds/drho P d_dot / r
// One thread per (direction, edge); g accumulates over the layers.
template <int LMAX>
__global__ void __launch_bounds__(256) k_hvp_geo(const int* __restrict__ row_ptr_x, int N,
                                                 const float4* __restrict__ dvec, const float4* __restrict__ dd,
                                                 const float* __restrict__ geo, long e_stride, int accumulate,
                                                 float4* __restrict__ g) {
  const int E = row_ptr_x[N];
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= E) return;
  constexpr int NY = (LMAX + 1) * (LMAX + 1);
  const long o = blockIdx.y * e_stride + e;
  const float4 d = dvec[e], t = dd[o];
  const float ir = 1.0f / d.w;
  const float nx = d.x * ir, ny = d.y * ir, nz = d.z * ir;
  const float rd = t.w;
  const float px = t.x - nx * rd, py = t.y - ny * rd, pz = t.z - nz * rd;  // P d_dot
  const float* row = geo + o * kGeo;
  float yb[16], yc[16], s[4];
  ldr_n<16>(row, yb);
  ldr_n<16>(row + 16, yc);
  ldr_n<4>(row + 32, s);
  (void)NY;
  float g1x, g1y, g1z, g2x, g2y, g2z, hx, hy, hz;
  real_sh_vjp<LMAX>(nx, ny, nz, yb, g1x, g1y, g1z);
  real_sh_vjp<LMAX>(nx, ny, nz, yc, g2x, g2y, g2z);
  real_sh_vjp_jvp<LMAX>(nx, ny, nz, px * ir, py * ir, pz * ir, yc, hx, hy, hz);
  // P applied to (G1 + H u) / r - r_dot / r^2 G2
  const float ax = (g1x + hx) * ir - rd * ir * ir * g2x;
  const float ay = (g1y + hy) * ir - rd * ir * ir * g2y;
  const float az = (g1z + hz) * ir - rd * ir * ir * g2z;
  const float an = ax * nx + ay * ny + az * nz;
  const float g2n = g2x * nx + g2y * ny + g2z * nz;
  const float g2p = g2x * px + g2y * py + g2z * pz;
  float gx = ax - an * nx - g2n * ir * ir * px - g2p * ir * ir * nx + s[0] * nx + s[1] * px * ir;
  float gy = ay - an * ny - g2n * ir * ir * py - g2p * ir * ir * ny + s[0] * ny + s[1] * py * ir;
  float gz = az - an * nz - g2n * ir * ir * pz - g2p * ir * ir * nz + s[0] * nz + s[1] * pz * ir;
  if (accumulate) {
    const float4 q = g[o];
    gx += q.x;
    gy += q.y;
    gz += q.z;
  }
  g[o] = make_float4(gx, gy, gz, 0.0f);
}

// ---- readout ---------------------------------------------------------------------
// The last layer's gate, the readout and their reverse for s = -E_dot, from
// the pre-gate values x [N, C] and their tangents xd [B, N, C]: with
// h = silu(x), P = h W_r, E_dot = w2 . (silu'(P) P_dot), writes the adjoints xb
// and xc of x and x_dot. One wave per (direction, atom).
__global__ void __launch_bounds__(256) k_hvp_readout(const float* __restrict__ x, const float* __restrict__ xd,
                                                     const float* __restrict__ Wr, const float* __restrict__ w2,
                                                     int N, int B, int C, float* __restrict__ xb,
                                                     float* __restrict__ xc) {
  const long u = ((long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (u >= (long)B * N) return;
  const long i = u % N;
  float P[16], Pd[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) P[q] = Pd[q] = 0.0f;
  for (int k = lane; k < C; k += 64) {
    const float xv = x[i * C + k];
    const float h = siluf(xv), hd = silu_grad(xv) * xd[u * C + k];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      P[q] += h * Wr[k * 16 + q];
      Pd[q] += hd * Wr[k * 16 + q];
    }
  }
  // lane L holds hidden unit L / 4
  const float p = wave_sum_scatter16<16>(P), pd = wave_sum_scatter16<16>(Pd);
  const float w = w2[lane >> 2];
  const float cl = -w * silu_grad(p), bl = -w * silu_grad2(p) * pd;
  float pb[16], pc[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    pb[q] = __shfl(bl, 4 * q);
    pc[q] = __shfl(cl, 4 * q);
  }
  for (int k = lane; k < C; k += 64) {
    float hb = 0.0f, hc = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      hb += Wr[k * 16 + q] * pb[q];
      hc += Wr[k * 16 + q] * pc[q];
    }
    const float xv = x[i * C + k], g1 = silu_grad(xv);
    xb[u * C + k] = hb * g1 + hc * silu_grad2(xv) * xd[u * C + k];
    xc[u * C + k] = hc * g1;
  }
}

inline int blocks(long n, int t) { return (int)((n + t - 1) / t); }

template <int LMAX, int KIND, int CH>
void hvp_launch(int which, const HvpArgs& a, hipStream_t st) {
  const int grid = a.B * a.N, threads = a.C / CH < 64 ? 64 : a.C / CH;
  if (which == 0) {
    if (KIND != kFull && a.B > 1)
      k_hvp_fwd<LMAX, KIND, CH, KIND == kFull ? 1 : 2><<<(a.B + 1) / 2 * a.N, threads, 0, st>>>(a);
    else
      k_hvp_fwd<LMAX, KIND, CH, 1><<<grid, threads, 0, st>>>(a);
    return;
  }
  auto adjoint = [&](auto wc) {
    constexpr bool W = decltype(wc)::value;
    constexpr int NIN = PathSet<LMAX, KIND>::NIN;
    if constexpr (KIND == kLast) {
      k_hvp_sender<LMAX, CH, W><<<grid, threads, 0, st>>>(a);
    } else if constexpr (KIND == kFull) {
      if constexpr (LMAX == 3) {
        k_hvp_edge_full<LMAX, 0, 1, W><<<grid, threads, 0, st>>>(a);
        k_hvp_edge_full<LMAX, 2, 2, W><<<grid, threads, 0, st>>>(a);
        k_hvp_edge_full<LMAX, 3, 3, W><<<grid, threads, 0, st>>>(a);
      } else {
        k_hvp_edge_full<LMAX, 0, LMAX, W><<<grid, threads, 0, st>>>(a);
      }
      k_hvp_msg_node<NIN, true><<<grid, 128, 0, st>>>(a);
    } else {
      k_hvp_edge<LMAX, KIND, CH, W><<<grid, threads, 0, st>>>(a);
      if constexpr (W) k_hvp_msg_node<NIN, false><<<grid, 128, 0, st>>>(a);
    }
  };
  if (a.Rb) adjoint(std::true_type{});
  else adjoint(std::false_type{});
}

// Channels per lane: layers with every path keep one (99 outputs per channel);
// the others run one wave, which holds all of an edge's channel sums (no
// exchange between waves).
template <int LMAX, int KIND>
void hvp_channels(int which, const HvpArgs& a, hipStream_t st) {
  if constexpr (KIND == kFull) return hvp_launch<LMAX, KIND, 1>(which, a, st);
  else {
    if (a.C <= 64) return hvp_launch<LMAX, KIND, 1>(which, a, st);
    return hvp_launch<LMAX, KIND, 2>(which, a, st);
  }
}

template <int LMAX>
void hvp_kind(int which, const HvpArgs& a, hipStream_t st) {
  switch (a.kind) {
    case kFirst: return hvp_channels<LMAX, kFirst>(which, a, st);
    case kFull: return hvp_channels<LMAX, kFull>(which, a, st);
    case kLast: return hvp_channels<LMAX, kLast>(which, a, st);
    default: return hvp_channels<LMAX, kFirstLast>(which, a, st);
  }
}

}  // namespace

static void hvp_layer(int which, const HvpArgs& a, hipStream_t st) {
  if (a.N == 0 || a.B == 0) return;
  E3MI_REQUIRE(a.C == 32 || a.C == 64 || a.C == 128, E3MI_EUNSUPPORTED, "channels must be 32, 64 or 128");
  if (a.lmax == 2) return hvp_kind<2>(which, a, st);
  if (a.lmax == 3) return hvp_kind<3>(which, a, st);
  throw Error(E3MI_EUNSUPPORTED, "lmax must be 2 or 3");
}

void launch_hvp_tangent_sum(const HvpArgs& a, hipStream_t st) { hvp_layer(0, a, st); }
void launch_hvp_adjoint(const HvpArgs& a, hipStream_t st) { hvp_layer(1, a, st); }

void launch_hvp_edge_tangent(const int* row_ptr, const int* src, const float4* dvec, const float* v, int N, int B,
                             long e_stride, float4* dd, hipStream_t st) {
  if (N == 0) return;
  k_hvp_tangent<<<blocks((long)N * B * 64, 256), 256, 0, st>>>(row_ptr, src, dvec, v, N, B, e_stride, dd);
}

void launch_hvp_geo(const HvpArgs& a, long e_cap, int accumulate, float4* g, hipStream_t st) {
  if (e_cap == 0) return;
  const dim3 grid(blocks(e_cap, 256), a.B);
  if (a.lmax == 3)
    k_hvp_geo<3><<<grid, 256, 0, st>>>(a.row_ptr, a.N, a.dvec, a.dd, a.geo, a.e_stride, accumulate, g);
  else
    k_hvp_geo<2><<<grid, 256, 0, st>>>(a.row_ptr, a.N, a.dvec, a.dd, a.geo, a.e_stride, accumulate, g);
}

void launch_hvp_readout(const float* x, const float* xd, const float* Wr, const float* w2, int N, int B, int C,
                        float* xb, float* xc, hipStream_t st) {
  if (N == 0) return;
  k_hvp_readout<<<blocks((long)N * B * 64, 256), 256, 0, st>>>(x, xd, Wr, w2, N, B, C, xb, xc);
}

}  // namespace e3mi
