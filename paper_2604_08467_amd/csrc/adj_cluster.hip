// Cluster form of the adjoint passes (tiles of 8..11 qubits with qubit 0 at tile bit
// 0, windows from build_adj_clusters).  A window's gates run as a few clusters, each
// the product of up to 13 gates on four tile positions: a 16 x 16 complex matrix per
// trajectory, built once per call in 64 bits and rounded once, applied to the LDS tile
// on v_mfma_f32_16x16x4f32.
//
// The derivatives of a cluster's rotations need no state inside the cluster: with M_k =
// sum_cols psi_k lambda_k^dag (16 x 16, the states between gates k and k + 1),
//   d f / d theta_k = Im <lambda_{k-1}|P|psi_{k-1}> = Im tr(P M_{k-1}),
// and M_{k-1} follows from one 16 x 16 sum Q over the tiles: with unitary gates Q = M_0 and
// M_k = A_k M_{k-1} A_k^dag; with non-unitary ones Q = sum psi_0 lambda_L^dag and M_{k-1} =
// A_{k-1} .. A_1 Q A_L .. A_k.  So the backward window applies U^dag to psi and lambda and
// sums Q (three MFMA products per cluster instead of two matrix products and a reduction
// per gate), and adj_cl_grad_kernel walks the gates in 64 bits on 16 x 16 matrices.
//
// Measured on the 20-qubit, 10-layer ansatz, 64 trajectories (590 gates, here 76 clusters
// in 26 windows; 1.07 GB read or written per state and window): a forward window took 670
// us with each gate on its own and takes 285 (3.8 TB/s), a backward window 1650 and takes
// 690 (MFMA busy 0.72 of the SIMD cycles), a value in 64 bits 430 per window; value and
// gradient together 81 ms and now 40.  Relative error of the gradient against 64 bits 6.7e-7
// before, 3.2e-7 now: each cluster rounds its matrix once, not every gate.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_util.h"
#include "internal.h"
#include "sv_tile.h"

namespace ptsbe {
namespace {

// Column addressing of a cluster on tile positions cp[0..3]: cluster-local state
// v sits at offset soff(v); the other tile bits (the column) are deposited around
// the four positions (cs: cp ascending).
struct ClusterCols {
  int cp[4], cs[4];
  __device__ explicit ClusterCols(uint32_t pos) {    // byte i: position of cluster-local bit i
#pragma unroll
    for (int i = 0; i < 4; ++i) cp[i] = cs[i] = (int)((pos >> (8 * i)) & 0xffu);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (cs[k] > cs[k + 1]) { const int t = cs[k]; cs[k] = cs[k + 1]; cs[k + 1] = t; }
  }
  __device__ uint32_t soff(int v) const {
    return ((uint32_t)(v & 1) << cp[0]) | ((uint32_t)((v >> 1) & 1) << cp[1]) |
           ((uint32_t)((v >> 2) & 1) << cp[2]) | ((uint32_t)((v >> 3) & 1) << cp[3]);
  }
  __device__ uint32_t colbase(uint32_t col) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t lo = col & ((1u << cs[i]) - 1u);
      col = ((col >> cs[i]) << (cs[i] + 1)) | lo;
    }
    return col;
  }
};

__device__ inline double2 zfma(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}

// Column c of the merged gate of (trajectory, gate) in 64 bits: the bare gate's or
// rotation's column, then the inserted operators, later sites on the left.
__device__ void merged_column(const AdjClBuildArgs& b, int64_t traj, int gate, int c, double2* out) {
  const DeviceGate* G = b.g.gates + gate;
  const int d = G->arity == 2 ? 4 : 2;
  if (c >= d) return;
  double2 m[4], t[4];
  const int prm = b.gate_param[gate];
  if (prm >= 0) {                     // exp(-i theta P / 2) = cos I - i sin P
    double sn, cs;
    sincos(0.5 * b.theta[prm], &sn, &cs);
    const int axis = b.gate_axis[gate];
    m[0] = c == 0 ? make_double2(cs, axis == 2 ? -sn : 0.0)
                  : (axis == 0 ? make_double2(0.0, -sn) : make_double2(axis == 1 ? -sn : 0.0, 0.0));
    m[1] = c == 1 ? make_double2(cs, axis == 2 ? sn : 0.0)
                  : (axis == 0 ? make_double2(0.0, -sn) : make_double2(axis == 1 ? sn : 0.0, 0.0));
    m[2] = m[3] = make_double2(0.0, 0.0);
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] = r < d ? b.mats[gate * 16 + r * d + c] : make_double2(0.0, 0.0);
  }
  const uint8_t* kr = b.g.kraus + traj * b.g.S;
  for (int s = G->site_begin; s < G->site_end; ++s) {
    const int site = b.g.gate_site_list[s];
    const double2* op = b.site_ops + ((int64_t)site * b.g.max_kraus + kr[site]) * 16;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      t[r] = make_double2(0.0, 0.0);
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (r < d && x < d) t[r] = zfma(op[r * d + x], m[x], t[r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] = t[r];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (r < d) out[r * d + c] = m[r];
}

// Row (left) product U <- A U on cluster bits, entry (r, c) of a 16 x 16 matrix in LDS.
__device__ inline double2 left_entry(const AdjClOp& op, const double2* A, const double2* U, int r, int c) {
  double2 acc = make_double2(0.0, 0.0);
  if (op.kind == kSvOpGate1) {
    const int n = (r >> op.b0) & 1, r0 = r & ~(1 << op.b0);
#pragma unroll
    for (int k = 0; k < 2; ++k) acc = zfma(A[op.idx[n * 2 + k]], U[(r0 | (k << op.b0)) * 16 + c], acc);
  } else {
    const int n = ((r >> op.b0) & 1) | (((r >> op.b1) & 1) << 1), r0 = r & ~((1 << op.b0) | (1 << op.b1));
#pragma unroll
    for (int k = 0; k < 4; ++k)
      acc = zfma(A[op.idx[n * 4 + k]], U[(r0 | ((k & 1) << op.b0) | ((k >> 1) << op.b1)) * 16 + c], acc);
  }
  return acc;
}

// Column (right) product T <- T A on cluster bits, entry (r, c).
__device__ inline double2 right_entry(const AdjClOp& op, const double2* A, const double2* T, int r, int c) {
  double2 acc = make_double2(0.0, 0.0);
  if (op.kind == kSvOpGate1) {
    const int n = (c >> op.b0) & 1, c0 = c & ~(1 << op.b0);
#pragma unroll
    for (int k = 0; k < 2; ++k) acc = zfma(T[r * 16 + (c0 | (k << op.b0))], A[op.idx[k * 2 + n]], acc);
  } else {
    const int n = ((c >> op.b0) & 1) | (((c >> op.b1) & 1) << 1), c0 = c & ~((1 << op.b0) | (1 << op.b1));
#pragma unroll
    for (int k = 0; k < 4; ++k)
      acc = zfma(T[r * 16 + (c0 | ((k & 1) << op.b0) | ((k >> 1) << op.b1))], A[op.idx[k * 4 + n]], acc);
  }
  return acc;
}

// T A^dag on cluster bits, entry (r, c).
__device__ inline double2 right_entry_dagger(const AdjClOp& op, const double2* A, const double2* T, int r, int c) {
  double2 acc = make_double2(0.0, 0.0);
  const int d = op.kind == kSvOpGate1 ? 2 : 4;
  const int n = ((c >> op.b0) & 1) | (d == 4 ? ((c >> op.b1) & 1) << 1 : 0);
  const int c0 = c & ~((1 << op.b0) | (d == 4 ? 1 << op.b1 : 0));
  for (int k = 0; k < d; ++k) {
    const double2 g = A[op.idx[n * d + k]];
    acc = zfma(T[r * 16 + (c0 | ((k & 1) << op.b0) | ((k >> 1) << op.b1))], make_double2(g.x, -g.y), acc);
  }
  return acc;
}

// Merged gates (kept for the derivatives when b.A is set) and their product, the cluster
// matrix, one workgroup per (trajectory, cluster).
__global__ void __launch_bounds__(256) adj_cl_build_kernel(AdjClBuildArgs b) {
  __shared__ double2 Ua[2][256];
  __shared__ double2 As[kAdjClOps * 16];
  const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
  for (int64_t bid = blockIdx.x; bid < b.n_jobs * b.n_cl; bid += gridDim.x) {
    const int64_t job = bid / b.n_cl;
    const AdjCl cl = b.cls[bid % b.n_cl];
    if (tid < 4 * cl.n) merged_column(b, b.traj_base + job, b.ops[cl.first + (tid >> 2)].gate, tid & 3, As + 16 * (tid >> 2));
    Ua[0][tid] = make_double2(r == c ? 1.0 : 0.0, 0.0);
    __syncthreads();
    if (b.A && tid < 16 * cl.n) b.A[(job * b.n_ops + cl.first) * 16 + tid] = As[tid];
    int cur = 0;
    for (int k = 0; k < cl.n; ++k) {
      Ua[cur ^ 1][tid] = left_entry(b.ops[cl.first + k], As + 16 * k, Ua[cur], r, c);
      __syncthreads();
      cur ^= 1;
    }
    const double2 u = Ua[cur][tid];
    if (b.U64) b.U64[bid * 256 + tid] = u;
    else b.U[bid * 256 + tid] = make_float2((float)u.x, (float)u.y);
    __syncthreads();   // Ua and As are reused by the next (trajectory, cluster)
  }
}

// ------------------------------------------------------------- tile passes
// What bounds a pass: the HBM round trip of the states and the MFMA rate of the clusters,
// in turn, so the next tile's loads are issued before the current tile's clusters.  Loads
// complete in order: the cluster matrices are therefore staged in LDS in fragment order
// once per workgroup (a workgroup stays on one trajectory) and the cluster positions come
// with the kernel arguments, so that no wait inside a tile covers the next tile's loads.
template <int NP> constexpr int kPairs = NP > 9 ? 1 << (NP - 9) : 1;
// 16-byte amplitude pairs of a tile: pair tid + 256 i (2^8 amplitudes: 128 threads)
template <int NP> __device__ inline bool has_pair() { return NP > 8 || threadIdx.x < 128; }

// LDS layout: entry l at l ^ bits 4..7 ^ bits 8..11 folded into the low four (the bank slot
// of an amplitude), so that 16 lanes that step along any four neighbouring tile bits, a
// cluster's states or its columns, spread over the slots.  Linear, as swz.
__device__ inline uint32_t cl_swz(uint32_t l) { return l ^ ((l >> 4) & 15u) ^ ((l >> 8) & 15u); }

// The pairs of the tile at `base` of a state (null: the state |0 .. 0>, nothing is read);
// entries with a tile position of `fresh` set are zero and not read.
template <int NP>
__device__ inline void cl_load(const float2* state, uint32_t base, const int* P, uint32_t lo, uint32_t fresh,
                               floatx4_t (&v)[kPairs<NP>]) {
  if (!state) {
#pragma unroll
    for (int i = 0; i < kPairs<NP>; ++i)
      v[i] = floatx4_t{(base | lo | pair_hi<NP>(P, i)) == 0u ? 1.f : 0.f, 0.f, 0.f, 0.f};
    return;
  }
  if (fresh) {
    uint32_t e = 2u * threadIdx.x;
    asm volatile("" : "+v"(e));        // the conditions are worked out here, not kept over the tiles
    if (has_pair<NP>())
#pragma unroll
      for (int i = 0; i < kPairs<NP>; ++i) {
        v[i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        if (((e + 512u * i) & fresh) == 0)
          v[i] = *reinterpret_cast<const floatx4_t*>(state + (base | lo | pair_hi<NP>(P, i)));
      }
    return;
  }
  if (has_pair<NP>())
#pragma unroll
    for (int i = 0; i < kPairs<NP>; ++i) v[i] = *reinterpret_cast<const floatx4_t*>(state + (base | lo | pair_hi<NP>(P, i)));
}

typedef double doublex4_t __attribute__((ext_vector_type(4)));
template <typename T> struct ClNum;
template <> struct ClNum<float> {
  typedef float2 C;
  typedef floatx4_t V;
  // accumulator register i of lane 16 q + j holds row 4 q + i of column j
  static __device__ int row(int q, int i) { return 4 * q + i; }
};
template <> struct ClNum<double> {
  typedef double2 C;
  typedef doublex4_t V;
  static __device__ int row(int q, int i) { return 4 * i + q; }
};

// Pair tid + 256 i holds the entries e0 = 2 (tid + 256 i) and e0 + 1, at slots e = cl_swz(e0)
// and e ^ 1 (for 8-byte entries one 16-byte slot, halves swapped when e is odd).
__device__ inline void cl_put1(float2* tile, uint32_t e, floatx4_t v) {
  reinterpret_cast<floatx4_t*>(tile)[e >> 1] = (e & 1u) ? floatx4_t{v[2], v[3], v[0], v[1]} : v;
}
__device__ inline void cl_put1(double2* tile, uint32_t e, floatx4_t v) {
  tile[e] = make_double2(v[0], v[1]);
  tile[e ^ 1u] = make_double2(v[2], v[3]);
}
__device__ inline floatx4_t cl_get1(const float2* tile, uint32_t e) {
  const floatx4_t v = reinterpret_cast<const floatx4_t*>(tile)[e >> 1];
  return (e & 1u) ? floatx4_t{v[2], v[3], v[0], v[1]} : v;
}
__device__ inline floatx4_t cl_get1(const double2* tile, uint32_t e) {
  const double2 x = tile[e], y = tile[e ^ 1u];
  return floatx4_t{(float)x.x, (float)x.y, (float)y.x, (float)y.y};
}
template <int NP, typename C>
__device__ inline void cl_put(C* tile, uint32_t pt2, const floatx4_t (&v)[kPairs<NP>]) {
  if (has_pair<NP>())
#pragma unroll
    for (int i = 0; i < kPairs<NP>; ++i) cl_put1(tile, pt2 ^ cl_swz(512u * (uint32_t)i), v[i]);
}
template <int NP, typename C>
__device__ inline void cl_store(float2* A, const int* P, uint32_t lo, const C* tile, uint32_t pt2) {
  if (has_pair<NP>())
#pragma unroll
    for (int i = 0; i < kPairs<NP>; ++i)
      *reinterpret_cast<floatx4_t*>(A + (lo | pair_hi<NP>(P, i))) = cl_get1(tile, pt2 ^ cl_swz(512u * (uint32_t)i));
}

// Cluster matrices in fragment order: entry s 64 + lane is row j, column 4 s + q of the
// matrix (or of its adjoint), lane = 16 q + j.
template <typename C>
__device__ inline void cl_stage(const C* __restrict__ U, int n_cl, bool dagger, C* Us) {
  for (int i = threadIdx.x; i < 256 * n_cl; i += 256) {
    const int s = (i >> 6) & 3, q = (i >> 4) & 3, j = i & 15;
    C u = U[(i & ~255) + (dagger ? (4 * s + q) * 16 + j : j * 16 + 4 * s + q)];
    if (dagger) u.y = -u.y;
    Us[i] = u;
  }
}

// A cluster's byte addresses in a tile for lane 16 q + j.  rd[s]: state 4 s + q of column j
// (an operand of Y = U X); wr[i]: state j of column 4 q + i.  The product is taken as Y^T =
// X^T U^T, so that its result sits with the state along the lanes and the columns along q
// and the registers: the operand layout of a product over columns.  They are the same for
// every tile and wavefront: tabulated once per workgroup (16 bits each), because computed
// in place they are most of a cluster's VALU instructions; a column tile's part is XORed in.
template <typename T>
__device__ inline void cl_addresses(const uint32_t* pos, int n_cl, int n_tiles, uint4* tab, uint32_t* col) {
  constexpr uint32_t B = sizeof(typename ClNum<T>::C);
  for (int i = threadIdx.x; i < 64 * n_cl; i += 256) {
    const ClusterCols cc(pos[i >> 6]);
    const int q = (i >> 4) & 3, j = i & 15;
    const uint32_t cj = cl_swz(cc.colbase((uint32_t)j)), sj = cl_swz(cc.soff(j));
    uint32_t a[8];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      a[s] = B * (cj ^ cl_swz(cc.soff(4 * s + q)));
      a[4 + s] = B * (sj ^ cl_swz(cc.colbase((uint32_t)ClNum<T>::row(q, s))));
    }
    tab[i] = make_uint4(a[0] | a[1] << 16, a[2] | a[3] << 16, a[4] | a[5] << 16, a[6] | a[7] << 16);
  }
  for (int i = threadIdx.x; i < n_tiles * n_cl; i += 256)
    col[i] = B * cl_swz(ClusterCols(pos[i / n_tiles]).colbase((uint32_t)(16 * (i % n_tiles))));
}
struct ClAddr {
  uint32_t rd[4], wr[4];
  __device__ explicit ClAddr(const uint4* tab) {
    const uint4 a = tab[threadIdx.x & 63];
    rd[0] = a.x & 0xffffu; rd[1] = a.x >> 16; rd[2] = a.y & 0xffffu; rd[3] = a.y >> 16;
    wr[0] = a.z & 0xffffu; wr[1] = a.z >> 16; wr[2] = a.w & 0xffffu; wr[3] = a.w >> 16;
  }
};
template <typename C> __device__ inline C& cl_at(C* tile, uint32_t bytes) {
  return *reinterpret_cast<C*>(reinterpret_cast<char*>(tile) + bytes);
}
// Column tiles (16 columns each) of a wavefront: wave + 4 k, k < kColTiles.
template <int NP> constexpr int kColTiles = NP > 10 ? 1 << (NP - 10) : 1;
template <int NP> __device__ inline bool has_columns() { return NP > 9 || (int)(threadIdx.x >> 6) < (1 << (NP - 8)); }
// A window's tables in LDS: matrices, addresses and column parts of each cluster.
template <int NP, typename C> struct ClTables {
  C* U;                                            // [n_cl][256] in fragment order
  uint4* tab;                                      // [n_cl][64]
  uint32_t* col;                                   // [n_cl][column tiles]
  __device__ ClTables(C* at, int n_cl) : U(at), tab(reinterpret_cast<uint4*>(at + 256 * n_cl)),
                                         col(reinterpret_cast<uint32_t*>(tab + 64 * n_cl)) {}
  __device__ uint32_t column(int c, int k) const { return col[(c << (NP - 8)) + (threadIdx.x >> 6) + 4 * k]; }
};

// One column tile of Y^T = X^T U^T (u: this lane's fragment of U).  In 64 bits with three
// real products instead of four: yr = k1 - k3, yi = k1 + k2 with k1 = (xr + xi) ur, k2 = xr
// (ui - ur), k3 = xi (ur + ui); its cancellation costs 1e-16 there, but a bit in 32.
__device__ inline void cl_product(const float2 (&u)[4], const float2 (&x)[4], floatx4_t& yr, floatx4_t& yi) {
  yr = yi = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    yr = __builtin_amdgcn_mfma_f32_16x16x4f32(x[s].x, u[s].x, yr, 0, 0, 0);
    yi = __builtin_amdgcn_mfma_f32_16x16x4f32(x[s].x, u[s].y, yi, 0, 0, 0);
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    yr = __builtin_amdgcn_mfma_f32_16x16x4f32(x[s].y, -u[s].y, yr, 0, 0, 0);
    yi = __builtin_amdgcn_mfma_f32_16x16x4f32(x[s].y, u[s].x, yi, 0, 0, 0);
  }
}
__device__ inline void cl_product(const double2 (&u)[4], const double2 (&x)[4], doublex4_t& yr, doublex4_t& yi) {
  doublex4_t k1 = {0, 0, 0, 0}, k2 = k1, k3 = k1;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    k1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[s].x + x[s].y, u[s].x, k1, 0, 0, 0);
    k2 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[s].x, u[s].y - u[s].x, k2, 0, 0, 0);
    k3 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[s].y, u[s].x + u[s].y, k3, 0, 0, 0);
  }
  yr = k1 - k3;
  yi = k1 + k2;
}

template <typename T>
__device__ inline void cl_write(typename ClNum<T>::C* tile, uint32_t pc, const ClAddr& ad,
                                const typename ClNum<T>::V& yr, const typename ClNum<T>::V& yi) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    typename ClNum<T>::C y;
    y.x = yr[i];
    y.y = yi[i];
    cl_at(tile, pc ^ ad.wr[i]) = y;
  }
}

// Y = U X on this wavefront's columns, in place (a wavefront touches only its own columns;
// all of its reads are issued before its first product).
template <int NP, typename T>
__device__ inline void cl_apply(const ClTables<NP, typename ClNum<T>::C>& tb, int c, const typename ClNum<T>::C* U,
                                typename ClNum<T>::C* tile) {
  typedef ClNum<T> N;
  constexpr int PER = kColTiles<NP>;
  if (!has_columns<NP>()) return;
  const ClAddr ad(tb.tab + 64 * c);
  uint32_t pc[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) pc[k] = tb.column(c, k);
  typename N::C u[4], x[PER][4];
#pragma unroll
  for (int s = 0; s < 4; ++s) u[s] = U[256 * c + 64 * s + (threadIdx.x & 63)];
#pragma unroll
  for (int k = 0; k < PER; ++k)
#pragma unroll
    for (int s = 0; s < 4; ++s) x[k][s] = cl_at(tile, pc[k] ^ ad.rd[s]);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    typename N::V yr, yi;
    cl_product(u, x[k], yr, yi);
    cl_write<T>(tile, pc[k], ad, yr, yi);
  }
}

// sum over columns of a b^dag, both with the state along the lanes and column 4 q + i in
// register i: (qr, qi) += .
__device__ inline void cl_outer(const floatx4_t& ar, const floatx4_t& ai, const floatx4_t& br, const floatx4_t& bi,
                                floatx4_t& qr, floatx4_t& qi) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    qr = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[i], br[i], qr, 0, 0, 0);
    qi = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[i], br[i], qi, 0, 0, 0);
    qr = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[i], bi[i], qr, 0, 0, 0);
    qi = __builtin_amdgcn_mfma_f32_16x16x4f32(-ar[i], bi[i], qi, 0, 0, 0);
  }
}

// A cluster of a backward window.  UNITARY: psi and lambda walk back through U^dag in
// their tiles, and Q sums psi_in lambda_in^dag from the products' registers.  Otherwise
// `psi` holds the state before the cluster and stays, and Q sums psi_in lambda_out^dag.
template <int NP, bool UNITARY>
__device__ inline void cl_back(const ClTables<NP, float2>& tb, int c, float2* psi, float2* lam, floatx4_t& qr,
                               floatx4_t& qi) {
  constexpr int PER = kColTiles<NP>;
  if (!has_columns<NP>()) return;
  const ClAddr ad(tb.tab + 64 * c);
  uint32_t pc[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) pc[k] = tb.column(c, k);
  float2 u[4], x[PER][4], l[PER][4], lo[PER][4];
#pragma unroll
  for (int s = 0; s < 4; ++s) u[s] = tb.U[256 * c + 64 * s + (threadIdx.x & 63)];
#pragma unroll
  for (int k = 0; k < PER; ++k)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      x[k][s] = cl_at(psi, pc[k] ^ (UNITARY ? ad.rd[s] : ad.wr[s]));
      l[k][s] = cl_at(lam, pc[k] ^ ad.rd[s]);
      if (!UNITARY) lo[k][s] = cl_at(lam, pc[k] ^ ad.wr[s]);
    }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    floatx4_t pr, pi, lr, li;
    if (UNITARY) {
      cl_product(u, x[k], pr, pi);
      cl_product(u, l[k], lr, li);
      cl_write<float>(psi, pc[k], ad, pr, pi);
      cl_write<float>(lam, pc[k], ad, lr, li);
      cl_outer(pr, pi, lr, li, qr, qi);
    } else {
      cl_product(u, l[k], lr, li);
      cl_write<float>(lam, pc[k], ad, lr, li);
#pragma unroll
      for (int i = 0; i < 4; ++i) { pr[i] = x[k][i].x; pi[i] = x[k][i].y; lr[i] = lo[k][i].x; li[i] = lo[k][i].y; }
      cl_outer(pr, pi, lr, li, qr, qi);
    }
  }
}

// The tiles [b0, b1) of this workgroup within its trajectory.
__device__ inline void cl_range(const AdjClArgs& a, int64_t& job, uint32_t& b0, uint32_t& b1) {
  job = blockIdx.x / a.wpj;
  const uint32_t part = blockIdx.x % a.wpj, tiles = 1u << __popc(a.live);
  b0 = (uint32_t)((uint64_t)tiles * part / a.wpj);
  b1 = (uint32_t)((uint64_t)tiles * (part + 1) / a.wpj);
}

// Forward window: psi_out = U_C .. U_1 psi_in per tile.  T double (value-only calls): the
// window's arithmetic and tile in 64 bits, the states between windows in 32, so that the
// value's rounding error is the windows' stores alone.  Calls with a gradient take T float and
// return that pass's value.  Ansatz circuits of 8 to 16 qubits and 2 to 8 layers, error of the
// value per ZZ term (root mean square, worst of 252): gate by gate 9.6e-8 and 2.4e-7, float
// 7.0e-9 and 2.8e-8, double 7.3e-10; a value near zero, the usual one of a deep circuit, is a
// difference of large terms: relative error 1.0e-5 gate by gate, 1.3e-6 float.
template <int NP, typename T>
__global__ void __launch_bounds__(256) adj_cl_fwd_kernel(AdjClArgs a, const typename ClNum<T>::C* __restrict__ Uall) {
  typedef typename ClNum<T>::C C;
  extern __shared__ floatx4_t cl_lds[];
  C* tile = reinterpret_cast<C*>(cl_lds);
  const ClTables<NP, C> tb(tile + (1 << NP), a.n_cl);
  const uint32_t lo = pair_lo(a.P), pt2 = cl_swz(2u * threadIdx.x);
  int64_t job;
  uint32_t b0, b1;
  cl_range(a, job, b0, b1);
  const float2* in = a.psi_in ? a.psi_in + (job << a.n) : nullptr;
  float2* out = a.psi_out + (job << a.n);
  uint32_t base = deposit_other(b0, a.live);
  floatx4_t v[kPairs<NP>];
  cl_load<NP>(in, base, a.P, lo, a.fresh, v);
  cl_stage(Uall + (job * a.n_cl_total + a.cl_off) * 256, a.n_cl, false, tb.U);
  cl_addresses<T>(a.pos, a.n_cl, 1 << (NP - 8), tb.tab, tb.col);
  for (uint32_t t = b0; t < b1; ++t) {
    const uint32_t next = ((base | ~a.live) + 1u) & a.live;   // the next tile's other bits
    cl_put<NP>(tile, pt2, v);
    __syncthreads();
    if (t + 1 < b1) cl_load<NP>(in, next, a.P, lo, a.fresh, v);
    for (int c = 0; c < a.n_cl; ++c) {
      cl_apply<NP, T>(tb, c, tb.U, tile);
      __syncthreads();
    }
    cl_store<NP>(out + base, a.P, lo, tile, pt2);
    base = next;
    __syncthreads();   // every thread has read its part of the tile
  }
}

// Backward window.  RECOMPUTE false: psi_in is the state after the window, walked back
// by U^dag; true (non-unitary operators): the state before the window, psi before each
// cluster recomputed in a third tile.  Q of every cluster is summed over the tile's
// columns in FP32 on MFMA, over the wavefronts and tiles in FP64 registers (two entries
// of each cluster's Q per thread), in a fixed order.
template <int NP, bool RECOMPUTE>
__global__ void __launch_bounds__(256, 3) adj_cl_bwd_kernel(AdjClArgs a, const float2* __restrict__ Uall) {
  extern __shared__ floatx4_t cl_lds[];
  float2* psi = reinterpret_cast<float2*>(cl_lds);
  float2* lam = psi + (1 << NP);
  float2* work = lam + (1 << NP);                  // RECOMPUTE only
  float* stage = reinterpret_cast<float*>(work + (RECOMPUTE ? 1 << NP : 0));   // [4][512] wavefront sums
  const ClTables<NP, float2> tb(reinterpret_cast<float2*>(stage + 2048), a.n_cl);   // adjoints
  float2* Uf = reinterpret_cast<float2*>(tb.col + (a.n_cl << (NP - 8)));   // [n_cl][256], RECOMPUTE only
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t lo = pair_lo(a.P), pt2 = cl_swz(2u * tid);
  int64_t job;
  uint32_t b0, b1;
  cl_range(a, job, b0, b1);
  const float2* in = a.psi_in ? a.psi_in + (job << a.n) : nullptr;
  float2* lg = a.lam + (job << a.n);
  uint32_t base = deposit_other(b0, a.live);
  floatx4_t v[kPairs<NP>], w[kPairs<NP>];
  cl_load<NP>(in, base, a.P, lo, a.fresh, v);
  cl_load<NP>(lg, base, a.P, lo, 0u, w);
  {
    const float2* U = Uall + (job * a.n_cl_total + a.cl_off) * 256;
    cl_stage(U, a.n_cl, true, tb.U);
    if (RECOMPUTE) cl_stage(U, a.n_cl, false, Uf);
    cl_addresses<float>(a.pos, a.n_cl, 1 << (NP - 8), tb.tab, tb.col);
  }
  double sum[kAdjClMax][2];
#pragma unroll
  for (int k = 0; k < kAdjClMax; ++k) sum[k][0] = sum[k][1] = 0.0;
  for (uint32_t t = b0; t < b1; ++t) {
    cl_put<NP>(psi, pt2, v);
    cl_put<NP>(lam, pt2, w);
    __syncthreads();
    const uint32_t next = ((base | ~a.live) + 1u) & a.live;   // the next tile's other bits
    if (t + 1 < b1) {
      cl_load<NP>(in, next, a.P, lo, a.fresh, v);
      cl_load<NP>(lg, next, a.P, lo, 0u, w);
    }
    for (int c = a.n_cl - 1; c >= 0; --c) {
      floatx4_t qr = floatx4_t{0.f, 0.f, 0.f, 0.f}, qi = qr;
      if (RECOMPUTE && c > 0) {
        if (has_pair<NP>())
#pragma unroll
          for (int i = 0; i < kPairs<NP>; ++i) {
            const uint32_t e = (pt2 ^ cl_swz(512u * (uint32_t)i)) >> 1;
            reinterpret_cast<floatx4_t*>(work)[e] = reinterpret_cast<const floatx4_t*>(psi)[e];
          }
        __syncthreads();
        for (int k = 0; k < c; ++k) {
          cl_apply<NP, float>(tb, k, Uf, work);
          __syncthreads();
        }
      }
      cl_back<NP, !RECOMPUTE>(tb, c, RECOMPUTE && c > 0 ? work : psi, lam, qr, qi);
      float* st = stage + 512 * wave;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = (4 * (lane >> 4) + i) * 16 + (lane & 15);   // (psi state, lambda state)
        st[e] = qr[i];
        st[256 + e] = qi[i];
      }
      __syncthreads();   // the cluster's tiles and wavefront sums are complete
      const double dr = ((double)stage[tid] + (double)stage[512 + tid]) +
                        ((double)stage[1024 + tid] + (double)stage[1536 + tid]);
      const double di = ((double)stage[256 + tid] + (double)stage[768 + tid]) +
                        ((double)stage[1280 + tid] + (double)stage[1792 + tid]);
#pragma unroll
      for (int k = 0; k < kAdjClMax; ++k)
        if (k == c) {                  // uniform
          sum[k][0] += dr;
          sum[k][1] += di;
        }
      __syncthreads();   // every thread has read the sums
    }
    cl_store<NP>(lg + base, a.P, lo, lam, pt2);
    base = next;
    __syncthreads();   // every thread has read its part of the tile
  }
  double* out = a.q + (int64_t)blockIdx.x * a.n_cl * 512;
#pragma unroll
  for (int k = 0; k < kAdjClMax; ++k)
    if (k < a.n_cl) {
      out[k * 512 + tid] = sum[k][0];
      out[k * 512 + 256 + tid] = sum[k][1];
    }
}

// Im tr(P M) of a rotation about axis on the cluster bit with mask `bit`: the term of
// thread (r, c), m = M[row][r] for row = r (Z) or r ^ bit (X, Y), as <r|P|row> m.
__device__ inline double cl_rot_term(int axis, bool one, double2 m) {
  if (axis == 0) return m.y;                       // X[0][1] = X[1][0] = 1
  if (axis == 1) return one ? m.x : -m.x;          // Y[1][0] = i, Y[0][1] = -i
  return one ? -m.y : m.y;                         // Z = diag(1, -1)
}

// Derivatives of a cluster's rotations, one workgroup per (trajectory, cluster), in 64
// bits; Q is summed over the trajectory's workgroups in order.  UNITARY: Q = M before the
// first gate, then M <- A M A^dag gate by gate.  Otherwise F[k] = A_k .. A_1 forward, then
// T_k = Q A_L .. A_k backward and M = F_{k-1} T_k.
template <bool UNITARY>
__global__ void __launch_bounds__(256) adj_cl_grad_kernel(AdjClArgs a, const AdjCl* __restrict__ cls,
                                                          const AdjClOp* __restrict__ ops, int n_ops_total,
                                                          const double2* __restrict__ A,
                                                          const int32_t* __restrict__ gate_param,
                                                          const int32_t* __restrict__ gate_axis,
                                                          double* __restrict__ gop) {
  __shared__ double2 F[UNITARY ? 1 : kAdjClOps - 1][256];   // F[k - 1] = A_k .. A_1, k = 1 .. n - 1
  __shared__ double2 T[256];
  __shared__ double2 As[kAdjClOps * 16];
  __shared__ double red[2][4];
  const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
  const int64_t job = blockIdx.x / a.n_cl;
  const int ci = (int)(blockIdx.x % a.n_cl);
  const AdjCl cl = cls[a.cl_off + ci];
  if (tid < 16 * cl.n) As[tid] = A[(job * n_ops_total + cl.first) * 16 + tid];
  double2 q = make_double2(0.0, 0.0);
  {
    const double* src = a.q + (job * a.wpj * a.n_cl + ci) * 512 + tid;
    const int64_t step = (int64_t)a.n_cl * 512;
#pragma unroll 4
    for (int w = 0; w < a.wpj; ++w) {
      q.x += src[w * step];
      q.y += src[w * step + 256];
    }
  }
  T[tid] = q;
  __syncthreads();
  if (!UNITARY)
    for (int k = 1; k < cl.n; ++k) {
      const AdjClOp& op = ops[cl.first + k - 1];
      if (k == 1) {
        // A_1 itself: the product with the identity
        const int mask = (1 << op.b0) | (op.kind == kSvOpGate1 ? 0 : 1 << op.b1);
        double2 v = make_double2(0.0, 0.0);
        if ((r & ~mask) == (c & ~mask)) {
          const int d = op.kind == kSvOpGate1 ? 2 : 4;
          const int n = ((r >> op.b0) & 1) | (d == 4 ? ((r >> op.b1) & 1) << 1 : 0);
          const int m = ((c >> op.b0) & 1) | (d == 4 ? ((c >> op.b1) & 1) << 1 : 0);
          v = As[op.idx[n * d + m]];
        }
        F[0][tid] = v;
      } else {
        F[k - 1][tid] = left_entry(op, As + 16 * (k - 1), F[k - 2], r, c);
      }
      __syncthreads();
    }
  for (int i = 0; i < cl.n; ++i) {
    const int k = UNITARY ? i + 1 : cl.n - i;
    const AdjClOp& op = ops[cl.first + k - 1];
    const bool rot = gate_param[op.gate] >= 0;
    const int axis = gate_axis[op.gate], bit = 1 << op.b0;
    const int row = axis == 2 ? r : r ^ bit;
    double part = 0.0;
    if (UNITARY) {
      if (rot && c == 0) part = cl_rot_term(axis, (r & bit) != 0, T[row * 16 + r]);   // M before gate k
      if (i + 1 < cl.n) {
        // M <- A M A^dag: rows, then columns with the conjugate
        const double2 v = left_entry(op, As + 16 * (k - 1), T, r, c);
        __syncthreads();
        T[tid] = v;
        __syncthreads();
        const double2 w = right_entry_dagger(op, As + 16 * (k - 1), T, r, c);
        __syncthreads();
        T[tid] = w;
      }
    } else {
      const double2 v = right_entry(op, As + 16 * (k - 1), T, r, c);
      __syncthreads();                 // every thread has read T
      T[tid] = v;
      __syncthreads();
      if (rot) {                       // this thread: the term F[row][c] T[c][r] of M[row][r]
        const double2 f = k == 1 ? make_double2(row == c ? 1.0 : 0.0, 0.0) : F[k - 2][row * 16 + c];
        const double2 tv = T[c * 16 + r];
        part = cl_rot_term(axis, (r & bit) != 0, make_double2(f.x * tv.x - f.y * tv.y, f.x * tv.y + f.y * tv.x));
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
    if ((tid & 63) == 0) red[i & 1][tid >> 6] = part;
    __syncthreads();
    if (tid == 0 && rot) {
      const double* rd = red[i & 1];
      gop[job * n_ops_total + cl.first + k - 1] = (rd[0] + rd[1]) + (rd[2] + rd[3]);
    }
  }
}

// Derivative of each angle: its rotations' terms over all jobs, one wavefront per angle,
// strided partial sums and a fixed tree.
__global__ void __launch_bounds__(64) adj_cl_params_kernel(const double* __restrict__ gop, int64_t n_jobs,
                                                           int n_ops_total, const int32_t* __restrict__ off,
                                                           const int32_t* __restrict__ ops, int n_params, bool add,
                                                           double* __restrict__ grad) {
  for (int k = blockIdx.x; k < n_params; k += gridDim.x) {
    double sum = 0.0;
    for (int o = off[k]; o < off[k + 1]; ++o)
      for (int64_t j = threadIdx.x; j < n_jobs; j += 64) sum += gop[j * n_ops_total + ops[o]];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    if (threadIdx.x == 0) grad[k] = add ? grad[k] + sum : sum;
  }
}

template <template <int> class K, typename Go>
hipError_t by_np(int np, Go go) {
  switch (np) {
    case 8: return go(K<8>::f);
    case 9: return go(K<9>::f);
    case 10: return go(K<10>::f);
    case 11: return go(K<11>::f);
    default: return hipErrorInvalidValue;
  }
}
template <int NP> struct Fwd { static constexpr auto f = adj_cl_fwd_kernel<NP, float>; };
template <int NP> struct Fwd64 { static constexpr auto f = adj_cl_fwd_kernel<NP, double>; };
template <int NP> struct Bwd { static constexpr auto f = adj_cl_bwd_kernel<NP, false>; };
template <int NP> struct BwdR { static constexpr auto f = adj_cl_bwd_kernel<NP, true>; };

size_t cl_lds_bytes(AdjClPass pass, int np, int n_cl) {
  const size_t nt = (size_t)1 << np, m = (size_t)n_cl * 256;
  const size_t tab = (size_t)n_cl * (1024 + ((size_t)4 << (np - 8)));
  switch (pass) {
    case AdjClPass::value: return (nt + m) * sizeof(double2) + tab;
    case AdjClPass::forward: return (nt + m) * sizeof(float2) + tab;
    case AdjClPass::backward: return (2 * nt + m) * sizeof(float2) + tab + 8192;
    default: return (3 * nt + 2 * m) * sizeof(float2) + tab + 8192;
  }
}
template <typename Go>
hipError_t by_pass(AdjClPass pass, int np, Go go) {
  switch (pass) {
    case AdjClPass::value: return by_np<Fwd64>(np, go);
    case AdjClPass::forward: return by_np<Fwd>(np, go);
    case AdjClPass::backward: return by_np<Bwd>(np, go);
    default: return by_np<BwdR>(np, go);
  }
}

}  // namespace

hipError_t launch_adj_cl_build(const AdjClBuildArgs& b, hipStream_t stream) {
  if (b.n_jobs <= 0 || b.n_cl <= 0) return hipSuccess;
  hipLaunchKernelGGL(adj_cl_build_kernel, dim3(grid_blocks(b.n_jobs * b.n_cl)), dim3(256), 0, stream, b);
  return hipGetLastError();
}

int adj_cl_wpj(AdjClPass pass, int np, int n_cl, int64_t n_jobs, int tile_bits) {
  if (tile_bits == 0) return 1;        // one tile per trajectory
  int per_cu = 0, dev = 0, cus = 0;
  const hipError_t e = by_pass(pass, np, [&](auto k) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, 256, cl_lds_bytes(pass, np, n_cl));
  });
  if (e != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  const int64_t resident = (int64_t)std::max(per_cu, 1) * std::max(cus, 1);
  return (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)1 << tile_bits, resident / std::max<int64_t>(n_jobs, 1)));
}

hipError_t launch_adj_cl_pass(AdjClPass pass, const AdjClArgs& a, int np, hipStream_t stream) {
  if (a.n_jobs <= 0) return hipSuccess;
  if (np < 8 || np > 11 || np > a.n || a.P[0] != 0 || a.wpj < 1 || a.n_cl < 1 || a.n_cl > kAdjClMax)
    return hipErrorInvalidValue;
  const size_t lds = cl_lds_bytes(pass, np, a.n_cl);
  const dim3 grid((unsigned)(a.n_jobs * a.wpj));
  if (pass == AdjClPass::value)
    return by_np<Fwd64>(np, [&](auto k) {
      hipLaunchKernelGGL(k, grid, dim3(256), lds, stream, a, a.U64);
      return hipGetLastError();
    });
  auto go = [&](auto k) {
    hipLaunchKernelGGL(k, grid, dim3(256), lds, stream, a, a.U);
    return hipGetLastError();
  };
  return pass == AdjClPass::forward ? by_np<Fwd>(np, go)
                                    : (pass == AdjClPass::backward ? by_np<Bwd>(np, go) : by_np<BwdR>(np, go));
}

hipError_t launch_adj_cl_grad(const AdjClArgs& a, bool unitary, const AdjCl* cls, const AdjClOp* ops, int n_ops_total,
                              const double2* A, const int32_t* gate_param, const int32_t* gate_axis,
                              double* gop, hipStream_t stream) {
  if (a.n_jobs <= 0 || a.n_cl <= 0) return hipSuccess;
  hipLaunchKernelGGL(unitary ? adj_cl_grad_kernel<true> : adj_cl_grad_kernel<false>,
                     dim3((unsigned)(a.n_jobs * a.n_cl)), dim3(256), 0, stream, a, cls, ops, n_ops_total, A,
                     gate_param, gate_axis, gop);
  return hipGetLastError();
}

hipError_t launch_adj_cl_params(const double* gop, int64_t n_jobs, int n_ops_total, const int32_t* off,
                                const int32_t* ops, int n_params, bool add, double* grad, hipStream_t stream) {
  if (n_params <= 0) return hipSuccess;
  hipLaunchKernelGGL(adj_cl_params_kernel, dim3((unsigned)std::min(n_params, 4096)), dim3(64), 0, stream, gop, n_jobs,
                     n_ops_total, off, ops, n_params, add, grad);
  return hipGetLastError();
}

}  // namespace ptsbe
