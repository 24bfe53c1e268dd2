// Host-side runtime pieces shared by the library's translation units:
// error type, allocator wrapper, device buffers, and the launchers each
// kernel file exports.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <stdexcept>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/e3mi.h"

namespace e3mi {

struct Error : std::runtime_error {
  int code;
  Error(int c, const std::string& m) : std::runtime_error(m), code(c) {}
};

#define E3MI_HIP(call)                                                                       \
  do {                                                                                       \
    hipError_t e3mi_err_ = (call);                                                           \
    if (e3mi_err_ != hipSuccess)                                                             \
      throw ::e3mi::Error(E3MI_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e3mi_err_)); \
  } while (0)

#define E3MI_REQUIRE(cond, code, msg)                  \
  do {                                                 \
    if (!(cond)) throw ::e3mi::Error((code), (msg));   \
  } while (0)

struct Allocator {
  e3mi_alloc_fn alloc = nullptr;
  e3mi_free_fn free_fn = nullptr;
  void* ctx = nullptr;
  // arena mode (arena not NULL): hand out consecutive 256-byte aligned pieces
  // of [arena, arena + arena_bytes) and never free; nothing is allocated
  char* arena = nullptr;
  size_t arena_bytes = 0, arena_used = 0;
  void* get(size_t bytes) {
    if (bytes == 0) bytes = 256;
    if (arena) {
      const size_t need = (bytes + 255) & ~(size_t)255;
      if (need > arena_bytes - arena_used)
        throw Error(E3MI_ENOMEM, "the evaluation needs more than the static scratch of " +
                                     std::to_string(arena_bytes) + " bytes");
      void* p = arena + arena_used;
      arena_used += need;
      return p;
    }
    void* p = nullptr;
    if (alloc) {
      p = alloc(bytes, ctx);
    } else if (hipMalloc(&p, bytes) != hipSuccess) {
      p = nullptr;
    }
    if (!p) throw Error(E3MI_ENOMEM, "device allocation of " + std::to_string(bytes) + " bytes failed");
    return p;
  }
  void put(void* p) {
    if (!p || arena) return;
    if (free_fn) {
      free_fn(p, ctx);
    } else if (!alloc) {
      (void)hipFree(p);
    }
  }
};

// A device allocation that can only grow. Contents are not preserved on growth.
struct DevBuf {
  Allocator* a = nullptr;
  void* p = nullptr;
  size_t bytes = 0;
  DevBuf() = default;
  explicit DevBuf(Allocator* al) : a(al) {}
  DevBuf(const DevBuf&) = delete;
  DevBuf& operator=(const DevBuf&) = delete;
  ~DevBuf() { release(); }
  void release() {
    if (p && a) a->put(p);
    p = nullptr;
    bytes = 0;
  }
  void* ensure(size_t n) {
    if (n > bytes || !p) {
      release();
      p = a->get(n);
      bytes = n == 0 ? 256 : n;
    }
    return p;
  }
  template <class T>
  T* as() const {
    return static_cast<T*>(p);
  }
};


// Optional per-stage timing with HIP events recorded on the launch stream.
struct Profiler {
  struct Pending {
    int stage;
    hipEvent_t a, b;
  };
  bool on = false;
  // record only this stage (-1: every stage) and, when >= 0, only this layer
  int only_stage = -1, only_layer = -1;
  bool wants(int stage_layer) const {
    if (!on) return false;
    if (only_stage >= 0 && stage_layer / 8 != only_stage) return false;
    return only_layer < 0 || stage_layer % 8 == only_layer;
  }
  std::vector<Pending> pending;
  std::vector<hipEvent_t> pool;
  std::vector<double> ms;
  std::vector<int64_t> count;
  hipEvent_t get() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e;
    E3MI_HIP(hipEventCreate(&e));
    return e;
  }
  void drain() {
    for (auto& p : pending) {
      E3MI_HIP(hipEventSynchronize(p.b));
      float t = 0.f;
      E3MI_HIP(hipEventElapsedTime(&t, p.a, p.b));
      if ((int)ms.size() <= p.stage) {
        ms.resize(p.stage + 1, 0.0);
        count.resize(p.stage + 1, 0);
      }
      ms[p.stage] += t;
      count[p.stage] += 1;
      pool.push_back(p.a);
      pool.push_back(p.b);
    }
    pending.clear();
  }
  void reset() {
    drain();
    ms.assign(ms.size(), 0.0);
    count.assign(count.size(), 0);
  }
  ~Profiler() {
    for (auto& p : pending) {
      (void)hipEventDestroy(p.a);
      (void)hipEventDestroy(p.b);
    }
    for (auto e : pool) (void)hipEventDestroy(e);
  }
};

struct ProfScope {
  Profiler* p;
  int stage;
  hipStream_t st;
  hipEvent_t a = nullptr;
  ProfScope(Profiler* prof, int s, hipStream_t stream) : p(prof), stage(s), st(stream) {
    if (p && p->wants(stage)) {
      a = p->get();
      E3MI_HIP(hipEventRecord(a, st));
    }
  }
  ~ProfScope() {
    if (a) {
      hipEvent_t b = p->get();
      if (hipEventRecord(b, st) == hipSuccess) p->pending.push_back({stage, a, b});
    }
  }
};

// Per-structure cell-list plan (orthorhombic periodic axes or open axes).
struct GridPlan {
  double lo[3];      // grid origin: 0 on periodic axes, bounding-box minimum on open axes
  double len[3];     // box length on periodic axes
  double inv_cw[3];  // 1 / cell width
  int nb[3];         // cells per axis
  int periodic[3];
  int cell_base;     // index of the structure's first cell in the global cell array
  int pad;
};

// ---- launchers exported by graph.hip -------------------------------------
void launch_owner(const int64_t* offsets, int S, int* owner, hipStream_t st);
void launch_bbox(const double* pos, const int64_t* offsets, int S, double* bbox, hipStream_t st);
void launch_exclusive_scan(const int* in, int* out, int n, hipStream_t st);
void launch_bin(const double* pos, const int* owner, const GridPlan* plan, int N, int* atom_cell,
                int* wrap, int* cell_count, hipStream_t st);
void launch_bin_fill(const int* atom_cell, const int* cell_start, int N, int* cell_fill,
                     int* cell_atoms, hipStream_t st);
void launch_edges(bool fill, const double* pos, const int* owner, const GridPlan* plan,
                  const int* atom_cell, const int* wrap, const int* cell_start, const int* cell_atoms,
                  const int* row_ptr, int N, double rc2, int* count, uint64_t* keys, int* err,
                  hipStream_t st);
void launch_sort_rows(const int* row_ptr, int N, uint64_t* keys, int* src, int* shift, hipStream_t st);
void launch_reverse(const int* row_ptr, const uint64_t* keys, int N, int* rev, int* err, hipStream_t st);
void launch_unpack_shift(const int* shift_packed, int E, int* shift3, hipStream_t st);
// The edges inside the cutoff (rc2: its square) out of the skin list (row_ptr,
// src, shift, rev): row_ptr_x [N + 1], src_x, dvec_x and rev_x, the skin edge of
// each (old_idx) and back (new_idx, -1: not selected), the pair owners in edge
// order (own_ptr [N + 1], own; own_ptr[N] is their count on the device) and each
// edge's pair index (pair_of); cnt and own_cnt are scratch [N]
struct PruneArgs {
  const double *pos, *box;
  const int *owner, *row_ptr, *src, *shift, *rev;
  int N;
  double rc2;
  int *cnt, *own_cnt, *row_ptr_x, *own_ptr, *src_x;
  float4* dvec_x;
  int *old_idx, *new_idx, *rev_x, *own, *pair_of;
  // the embedding h0 = W_emb[species] [N, C], in the first launch
  const int* species;
  const float* emb;
  float* h0;
  int C;
};
void launch_prune(const PruneArgs& a, hipStream_t st);

// ---- tensor product (tp.hip) ---------------------------------------------------
struct TpArgs {
  int lmax, kind, cpt;
  const int* row_ptr;
  const int* src;
  const float4* dvec;
  const float* R;
  int r_stride;
  const float* h;
  int h_nc;
  float* A;
  const float* dA;
  float* dR;
  float* dY;
  float* dh;
  int dh_nc;
  int dh_acc;  // node adjoint: components below dh_acc are accumulated, the rest written (<= 0: all accumulated)
  int N, C;
  float inv_nu;
  // receiver chunk (first-order kernels 0-2): receivers i0 .. i0 + n_recv - 1
  // (n_recv 0: all N from i0 = 0), R and dR indexed from edge e_first
  int i0, n_recv, e_first;
  const int* rev;  // reverse edge of each edge (-1: pruned), for the sender-side adjoint and pass 7
  float* msg;      // per-edge sender-gradient messages [edges of the chunk, NIN, C] (passes 1 and 7), or NULL
  int r_bf16;      // R and dR stored as BF16 (passes 0 and 1, and the sender-side adjoint)
  int* touched;    // with msg: per atom, set to `tag` for every sender of the chunk's edges (pass 1), read by pass 7
  int tag;
  // R rows (passes 0-2 and the sender-side adjoint): edge e's weights in row
  // r_row[e] (its pair index; NULL: row e - r_first); dR stays per edge
  const int* r_row;
  int r_first;
  // FP32 energies and forces: R' in rows like R's. The adjoints then write no
  // dR; dY's first value (the l = 0 harmonic is constant) is dE/dr instead, and
  // row_add adds to dY's rows
  const float* Rp;
  int row_add;
  int fp32;  // pass 0: FP32 model (layers with every path then need not give the BF16 mode's bits)
};
// which: 0 forward, 1 edge adjoint (dR, dY), 2 node adjoint (dh += ...),
//        7 node adjoint from the messages that pass 1 wrote (msg set), for the
//          chunk's receivers [i0, i0 + n_recv) as senders' partners
void launch_tp(int which, const TpArgs& a, hipStream_t st);
// scalar-output layer (tps.hip): the sender-side adjoint, dY (and in the BF16
// mode dR) of pass 1 and, when a.dh is set, dh of pass 2
bool tps_supported(const TpArgs& a);
void launch_tps_sender(const TpArgs& a, hipStream_t st);
// pass 0 in FP32
void launch_tps_fwd(const TpArgs& a, hipStream_t st);
// g (+)= the position adjoint of the edges' rows [dE/dr, dY 1..] (tps.hip)
void launch_edge_geo(int lmax, const int* row_ptr_x, int N, long e_cap, const float4* dvec, const float* rows,
                     int accumulate, float4* g, hipStream_t st);

// ---- per-atom stages (node.hip) -----------------------------------------------------
// Rows of a matrix whose row r lives at base + (r / g) * s_atom + (r % g) * s_m
// (an atom block of g = 2l + 1 rows); the row itself is contiguous.
struct RowMap {
  float* base;
  long s_atom;
  long s_m;
  int g;
};
// C[M x Nc] = A0[M x k0] B0[k0 x Nc] + A1[M x k1] B1[k1 x Nc]; k0, k1 and Nc
// multiples of 32, the weights B laid out by kFragments
struct GemmArgs {
  RowMap a0;
  const __bf16* b0;
  int k0;
  RowMap a1;  // optional second product (k1 = 0: none)
  const __bf16* b1;
  int k1;
  RowMap c;
  int M, Nc;
};
// Up to kMaxGemmGroup independent products (no output read or written by
// another of the group) in one launch. With l_max <= 3 a layer's groups hold
// at most 4 + 4 products (one per output order, plus the self connection's).
constexpr int kMaxGemmGroup = 8;
void launch_gemm_group(const GemmArgs* a, int n, hipStream_t st, bool bf16 = false);
// go(components) for the (l + 1)^2 that features have
template <class F>
inline void with_components(int nc, F go) {
  if (nc == 1) go(std::integral_constant<int, 1>{});
  else if (nc == 4) go(std::integral_constant<int, 4>{});
  else if (nc == 9) go(std::integral_constant<int, 9>{});
  else if (nc == 16) go(std::integral_constant<int, 16>{});
  else throw Error(E3MI_EINVAL, "internal: components of the gate");
}
void launch_gate_fwd(const float* ht, float* h, int N, int nc, int C, hipStream_t st);
void launch_gate_bwd(const float* ht, const float* dh, float* dht, int N, int nc, int C, hipStream_t st);
// h~ [N, C] = sum of n_parts partial products [n_parts, N, C] in order; h = silu(h~)
void launch_gate_fwd_sum(const float* part, int n_parts, float* ht, float* h, int N, int C, hipStream_t st);
void launch_readout(const float* h, int nc, const int* species, const float* Wr, const float* w2, const float* e0,
                    int N, int C, double* e_atom, float* dh, hipStream_t st, const float* wq = nullptr,
                    const float* bq = nullptr, float* q_raw = nullptr);
// Readout of a scalar-only last layer from its pre-gate values (the sum of
// n_parts partial products [n_parts, N, C], or h~ [N, C] when n_parts is 0),
// the gate and its adjoint folded in: writes E_i and dE/dh~ [N, C]
void launch_readout_gated(const float* xt, int n_parts, const int* species, const float* Wr, const float* w2,
                          const float* e0, int N, int C, double* e_atom, float* dht, hipStream_t st);
// energy[s] = the sum of e_atom over structure s (S 0: none)
struct EnergySum {
  const double* e_atom = nullptr;
  const int64_t* off = nullptr;
  int S = 0;
  double* energy = nullptr;
};
// (B > 1: g [B, e_stride] -> F [B, N, 3])
void launch_forces(const int* row_ptr, const int* rev, const float4* g, int N, float* F, hipStream_t st,
                   const float* extra = nullptr, int B = 1, long e_stride = 0, const EnergySum& es = EnergySum{});

// ---- Hessian-vector products (hvp.hip) ------------------------------------------------
// One layer's tangent or adjoint for a batch of B directions: atom rows are
// (b, i) = b N + i, edge rows b e_stride + e.
constexpr int kHvpGeoRow = 36;  // floats of an edge's geo row
struct HvpArgs {
  int lmax, kind, N, C, B;
  const int* row_ptr;
  const int* src;
  const int* rev;
  const float4* dvec;
  const float4* dd;   // per direction and edge: d_dot, r_dot
  long e_stride;
  const float *R, *Rp, *Rpp;  // rows [P, C] of R, R' and (not for weight gradients) R''
  long r_stride;      // floats from row to row
  const int* r_row;   // row of edge e (NULL: e)
  const float* h;     // layer input [N, h_nc, C]
  const float* hd;    // its tangents [B N, h_nc, C] (not read by the first layer)
  int h_nc;
  float inv_nu;
  float* Ad;          // tangent pass out: A_dot, grouped layout of B N atoms
  const float* Ab;    // adjoint pass in: adjoints of A (B N atoms), then of A_dot (B N atoms), grouped layout of 2 B N atoms
  float* geo;         // adjoint pass out, per direction and edge
  float* msg;         // scratch [B e_stride, 2, h_nc, C] of layers with every path after the first
  float* hb;          // adjoint pass out [B N, h_nc, C]: adjoint of h and of h_dot; components
  float* hc;          // below dh_acc are added to, the others written (not written by the first layer)
  int dh_acc;
  // weight gradients (B = 1; Rb not NULL): instead of geo, the adjoints of R
  // and R' per edge [E, P, C]; the first layer then writes hb too, through msg [E, C]
  float *Rb, *Rc;
};
void launch_hvp_tangent_sum(const HvpArgs& a, hipStream_t st);
void launch_hvp_adjoint(const HvpArgs& a, hipStream_t st);
void launch_hvp_edge_tangent(const int* row_ptr, const int* src, const float4* dvec, const float* v, int N, int B,
                             long e_stride, float4* dd, hipStream_t st);
// g [B, e_stride] (+)= the position adjoint of a layer's geo rows
void launch_hvp_geo(const HvpArgs& a, long e_cap, int accumulate, float4* g, hipStream_t st);
// from the last layer's pre-gate values x [N, C] and tangents xd [B N, C]: adjoints xb, xc [B N, C]
void launch_hvp_readout(const float* x, const float* xd, const float* Wr, const float* w2, int N, int B, int C,
                        float* xb, float* xc, hipStream_t st);
// FP32 rows of R and its first n_out - 1 derivatives in the edge length (output
// s from out + s out_gap, rows out_ld apart; W2 and W3 by kFragments), or with PC
// 0 of the second hidden layer [., 64] and its derivatives instead
struct RadialJob {
  const float* W1;
  const __bf16 *W2, *W3;
  int PC;
  float* out;
  long out_gap;
  int out_ld;
};
constexpr int kMaxRadialJobs = 4;
// up to kMaxRadialJobs of them in one launch, for every edge pair (own, n_own) or
// the edges [e_first, e_end) (e_end < 0: all)
void launch_radial_rows(int n_basis, const float4* dvec, const int* row_ptr_x, int N, long e_cap,
                        const RadialJob* jobs, int n_jobs, int n_out, float rc, int p, int e_first, int e_end,
                        const int* own, const int* n_own, hipStream_t st);

// ---- product block of body order 2 (product.hip) -------------------------------------
struct ProductArgs {
  int lmax = 0, lout = 0, N = 0, C = 0;
  int B_dirs = 1;                  // second-order pass: directions; tangents and adjoints have B N atoms, A~ N
  const float* at = nullptr;       // A~ [N, (lmax+1)^2, C]
  const int* species = nullptr;    // [N]
  const float* w1 = nullptr;       // [S, lout+1, C]
  const float* w2 = nullptr;       // [S, pairs, C]
  float* B = nullptr;              // forward output [N, (lout+1)^2, C]
  const float* dB = nullptr;       // adjoint input  [N, (lout+1)^2, C]
  float* dat = nullptr;            // adjoint output [N, (lmax+1)^2, C] (overwritten)
  // second-order pass: tangent A~_dot and B_dot, adjoints of B and B_dot, of
  // A~ and A~_dot, and (optional) per-atom weight-gradient rows
  const float* atd = nullptr;      // [N, (lmax+1)^2, C]
  float* Bd = nullptr;             // [N, (lout+1)^2, C] (overwritten)
  const float* Bb = nullptr;       // [N, (lout+1)^2, C]
  const float* Bc = nullptr;       // [N, (lout+1)^2, C]
  float* atb = nullptr;            // [N, (lmax+1)^2, C] (overwritten)
  float* atc = nullptr;            // [N, (lmax+1)^2, C] (overwritten)
  float* dw = nullptr;             // [N, lout+1+pairs, C]: d/dw1 then d/dw2 of atom i (overwritten)
};
int product_pair_count(int lmax, int lout);
void launch_product(bool fwd, const ProductArgs& p, hipStream_t st);
void launch_product_jvp(const ProductArgs& p, hipStream_t st);
void launch_product_dual_bwd(const ProductArgs& p, hipStream_t st);

// ---- electrostatics of open structures (coulomb.hip) ---------------------------------
// q~ = q - (sum_s q - Q_s) / N_s per structure
void launch_charge_fix(const float* q_raw, const int64_t* off, const double* Q, int S, float* q, hipStream_t st);
// soft-core Coulomb over all pairs of each structure: e_atom += 1/2 k q~_i phi_i,
// pot = k phi, fc = Coulomb forces [N, 3]; tiles = (structure, first receiver) per 64 receivers;
// waves (1, 2, 4, 8, 16) split each tile's senders
void launch_coulomb(const int2* tiles, int n_tiles, int waves, const int64_t* off, const double* pos, const float* q,
                    float r0, double* e_atom, float* pot, float* fc, hipStream_t st);
// dh[i, k] += (pot_i - mean_s pot) wq[k]; mean: scratch [S]; owner: structure of each atom
void launch_coulomb_dq(const int64_t* off, const int* owner, int S, int N, const float* pot, float* mean,
                       const float* wq, int C, float* dh, hipStream_t st);

// ---- radial MLP (radial.hip) ---------------------------------------------------------
// The BF16 mode's R and the adjoint of its MLP; R and dR are FP32, or BF16 when
// r_bf16 is set. BF16 copies of a layer's radial weights (rounded to nearest
// even), laid out for the BF16 matrix-core steps: W2^T and W2 [64][64], W3^T
// [PC][64] and W3 (used columns) in slabs of 32 columns, [PC / 32][64][32].
struct RadialBf16 {
  const __bf16* W2T = nullptr;
  const __bf16* W2 = nullptr;
  const __bf16* W3T = nullptr;
  const __bf16* W3u = nullptr;
};
// The pair owners of the pruned list (own [P], P = *n_own on the device) and
// its reverse index: given, the radial MLP and its adjoint run once per edge
// pair (whole edge list only): R once per pair, at row p for the owner own[p]
// (consumers find edge e's row through the pair index).
struct EdgePairs {
  const int* own = nullptr;
  const int* n_own = nullptr;
  const int* rev = nullptr;
};
void launch_radial_fwd(int n_basis, const float4* dvec, const int* row_ptr_x, int N, long e_cap, const float* W1,
                       int PC, void* R, bool r_bf16, float rc, int p, hipStream_t st, int e_first, int e_end,
                       const RadialBf16* wb, const EdgePairs* pairs = nullptr);
void launch_radial_bwd(int n_basis, int lmax, const float4* dvec, const int* row_ptr_x, int N, long e_cap,
                       const float* W1, int PC, const void* dR, bool r_bf16, const float* dY, float4* g, int accumulate,
                       float rc, int p, hipStream_t st, int e_first, int e_end, const RadialBf16* wb,
                       const EdgePairs* pairs);

// ---- second-order passes (radial.hip, grad.hip) -------------------------------------
// Radial MLP of weight gradients: from the adjoints Rb, Rc of R and R' per edge,
// the operands of the weights' products, per pair (own, n_own, rev) or edge row:
// [B | B'] [., 16], [H1 | H1'], [H2 | H2'] [., 128] and the adjoints [P1b | P1c],
// [P2b | P2c] [., 128] of the pre-activations; a pair's Rb, Rc rows are added
// up in its owner's row.
void launch_radial_wgrad(const float4* dvec, const int* row_ptr_x, int N, long e_cap, const float* W1,
                         const float* W2, const float* W2T, const float* W3T, int PC, float* Rb, float* Rc, float rc,
                         int p, const int* own, const int* n_own, const int* rev, float* Bd, float* H1d, float* H2d,
                         float* P1g, float* P2g, hipStream_t st);
// B directions: x has N atoms, the tangents and adjoints B N
void launch_gate_dual_fwd(const float* x, const float* xd, float* hd, int N, int nc, int C, hipStream_t st, int B = 1);
void launch_gate_dual_bwd(const float* x, const float* xd, const float* hb, const float* hc, float* xb, float* xc,
                          int N, int nc, int C, hipStream_t st, int B = 1);
void launch_readout_dual(const float* h, const float* hd, int nc, const int* owner, const double* gE, const float* Wr,
                         const float* w2, int N, int C, float* Pb, float* Pc, float* w2c, float* hb, float* hc,
                         float* eb, hipStream_t st);
// out[g, c] = sum over atoms of X[i * ld + c] by species (all atoms in group 0
// when species is NULL), FP64; part: group_chunks(N) * n_groups * ncols doubles
int group_chunks(int N);
void launch_group_sum(const float* X, long ld, const int* species, int n_groups, int N, int ncols, double* part,
                      double* out, long ld_out, hipStream_t st);
// out (FP64 [mo, no], row stride ld_out) = X1^T Y1 + X2^T Y2 over `rows` rows
// (capped at *rows_dev when given; x2.base NULL: one term); rows 16-byte aligned
struct TnArgs {
  RowMap x1, y1, x2, y2;
  long rows;
  const int* rows_dev;
  int mo, no;
  const int* y_row;  // rows of y1 and y2 (NULL: in order)
  double* out;
  long ld_out;
};
constexpr int kMaxTnGroup = 8;
constexpr long kTnPartial = 16L << 20;  // floats of partial sums per launch
// floats of `partial` for products of up to mo_no_max outputs
size_t tn_partial_floats(long mo_no_max);
void launch_gemm_tn(const TnArgs* args, int n, float* partial, hipStream_t st);

// ---- weights (weights.hip) ------------------------------------------------------------
// A device tensor taken from a [rows, cols] block (row stride ld) at `src` of
// the flat FP64 vector
enum WeightLayout : int { kCopyF32, kTransposeF32, kCopyBf16, kTransposeBf16, kSlabsBf16, kFragments, kFragmentsT };
// kFragments(T): the matrix B (its transpose) as operands of the BF16 matrix
// cores, split into three BF16 parts that add up to the FP32 value (gemm.hip):
// element (k, c) at fragment_at(k, c, columns), its parts 512 apart
__host__ __device__ constexpr long fragment_at(int k, int c, int cols) {
  return ((long)(k / 16) * (cols / 32) + c / 32) * 1536 + ((k % 16) / 8 * 32 + c % 32) * 8 + k % 8;
}
struct WeightCopy {
  int kind, rows, cols, ld;
  long src;
  void* dst;
};
// What U_l is formed from: offsets of W_emb, the first layer's W3 (row stride
// ld3) and mixes, and the outputs per order
struct FirstWeights {
  int C, H, n_species, n_orders, ld3;
  double nu;
  long emb, rad3, mix[4];
  __bf16 *U[4], *UT[4];  // kFragments
};
// *bad (device) = 1, and no weight written, when `check` finds a value of the
// n that is not finite
void launch_weights(const double* w, long n, const WeightCopy* copies, int n_copies, const FirstWeights& f,
                    bool check, int* bad, hipStream_t st);

// ---- species-factorised first layer (first.hip) ---------------------------------------
// H = [H2 | H2'] [rows, 128] of the first layer, the second hidden layer and
// its derivative in the edge length: per pair owner (own, P = *n_own on the
// device) or per edge (own and n_own NULL); e_cap bounds the rows
void launch_first_hidden(const float4* dvec, const int* row_ptr_x, int N, long e_cap, const int* own,
                         const int* n_own, const float* W1, const float* W2, float rc, int p, float* H,
                         hipStream_t st);
// forward (G) or adjoint (g) of the factorised first layer; edge e's row of H
// is pair_of[e] (or e when pair_of is NULL). The adjoint takes the later
// layers' edge rows [dE/dr, dY 1..] (rows, or NULL) into its own
void launch_first(bool fwd, int lmax, int l3max, const int* row_ptr, const int* src, const float4* dvec,
                  const int* species, int N, int S64, const int* pair_of, const float* H, float* G, const float* dG,
                  const float* rows, float4* g, int accumulate, hipStream_t st);

// ---- fused last layer (last.hip) ----------------------------------------------------------
struct LastArgs {
  int lmax, C, N;
  const int* row_ptr;
  const int* src;
  const float4* dvec;
  const float* h;    // layer input [N, (lmax+1)^2, C]
  const float* W1;   // [8, 64]
  const float* W2;   // [64, 64]
  const float* W2T;  // [64, 64]
  const float* W3;   // [64, ldw3], scalar-output paths in the first (lmax+1) C columns
  int ldw3;
  const float* W3T;  // [(lmax+1) C, 64]
  float* A;          // forward out: [N, lmax+1, C], nu^-1 applied
  const float* dA;   // adjoint in: [N, lmax+1, C] (without nu^-1)
  float4* g;         // adjoint out: per-edge dE/dd (+= when accumulate)
  int accumulate;
  float* dh;         // adjoint out (+=): [N, (lmax+1)^2, C]
  float rc, inv_nu;
  int p;
};
bool last_supported(int lmax, int C);
void launch_last(bool fwd, const LastArgs& a, hipStream_t st);

// ---- MD (md.hip) -----------------------------------------------------------------------
void launch_kick(double* v, const float* F, const int* species, const double* inv_mass, double half_dt_kappa, int N,
                 hipStream_t st);
// the drifts raise *flag to `stamp` when an atom is more than sqrt(limit2) from
// x_ref, and (probe not NULL) raise *probe to the bits of the largest
// |x - x_ref| + dt_next |v| over the atoms
void launch_drift(double* x, const double* v, const double* x_ref, double dt, double limit2, int N,
                  unsigned long long* flag, unsigned long long stamp, unsigned long long* probe, double dt_next,
                  hipStream_t st);
// k_kick then k_drift in one pass (same arithmetic)
void launch_kick_drift(double* v, const float* F, const int* species, const double* inv_mass, double half_dt_kappa,
                       double* x, const double* x_ref, double dt, double limit2, int N, unsigned long long* flag,
                       unsigned long long stamp, unsigned long long* probe, double dt_next, hipStream_t st);
// k_kick, with the n_copy structure energies copied e_src -> e_dst in the same
// launch; v_prev (may be NULL) receives the velocities before the kick;
// probe_clear (may be NULL) is set to 0
void launch_kick_copy(double* v, const float* F, const int* species, const double* inv_mass, double half_dt_kappa,
                      int N, const double* e_src, double* e_dst, int n_copy, double* v_prev,
                      unsigned long long* probe_clear, hipStream_t st);
void launch_nonfinite(const double* x, int n, int* flag, hipStream_t st);
// zero `bytes` (a multiple of 4) at p with a kernel (no memset node in a captured graph)
void launch_zero(void* p, size_t bytes, hipStream_t st);
void launch_species_range(const int* species, int n, int n_species, int* flag, hipStream_t st);
void launch_scale_positions(double* x, const int* owner, const double* lam, int N, hipStream_t st);
void launch_restore_rows(double* x, const double* x_save, const int* owner, const int* keep, int N, hipStream_t st);
void launch_ou(double* v, const int* species, const double* inv_mass, const int* owner, const int64_t* offsets,
               const uint64_t* seeds, const int64_t* step0, int64_t step, double c1, double c2, double kT_kappa, int N,
               hipStream_t st);
void launch_rekey(const int* src, const int* shift, int E, uint64_t* keys, hipStream_t st);

}  // namespace e3mi
