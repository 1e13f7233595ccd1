// Gate windows of the statevector method (the ket network of a trajectory
// contracted in circuit order, Sec. III-A: one schedule shared by every
// trajectory, each applying its own UPV-merged gates).  A window is a set of at
// most 12 qubits, qubit 0 among them; every 2^np-amplitude tile of a state whose
// other bits are fixed is read from HBM once, all of the window's gates are
// applied to it in LDS, and it is written back.
//
// States start as |0...0>, so the first windows see few nonzero amplitudes: the
// first makes tile 0 out of nothing, and each later one reads what its
// predecessors wrote and writes as far as its own qubits reach (SvArgs live,
// fresh), until every qubit was in a window.  The amplitudes left out are zeros
// that a gate maps to zeros.  25 qubits x 48 states, 11 windows on one 12.9 GB
// set: a sampling call 136.4 -> 104.2 ms.
//
// The ops of a window are read through the scalar cache (uniform loads), the gate
// matrices of a trajectory and its gate-cluster matrices are staged in LDS when
// a workgroup reaches a new trajectory, and tiles move as 16-byte pairs of
// amplitudes (qubit 0 is tile bit 0).  The next tile's loads are issued before
// the current tile's ops, so that they are in flight during its LDS work.
//
// A gate cluster (a 16 x 16 complex matrix on four tile positions, the product
// of several gates built once per trajectory) is a real 32 x 32 by 32 x 2^(np-4)
// product on MFMA: FP32 (v_mfma_f32_16x16x4f32), or with hi + lo 16-bit operands
// (v_mfma_f32_16x16x32_bf16 / _f16, three products hi*hi + hi*lo + lo*hi, FP32
// accumulation; fp16 scales every column by a power of two).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "internal.h"
#include "sv_tile.h"

namespace ptsbe {
namespace {

template <int PREC, int NP, bool FRESH>
__global__ void __launch_bounds__(kSvwThreads, 4) sv_window_kernel(SvwArgs a, const SvOp* __restrict__ ops,
                                                               const float2* __restrict__ merged,
                                                               const float2* __restrict__ Ucl,
                                                               float2* __restrict__ psi) {
  extern __shared__ floatx4_t svw_lds[];
  const int64_t total = a.n_jobs << __popc(a.live);
  const int64_t per = (total + gridDim.x - 1) / gridDim.x;
  const int64_t b0 = (int64_t)blockIdx.x * per, b1 = b0 + per < total ? b0 + per : total;
  if (b0 < b1) window_tiles<PREC, NP, FRESH>(a, ops, merged, Ucl, psi, b0, b1, svw_lds);
}

// One resident generation of workgroups, each walking a contiguous range of the tiles.
template <class K, class... Args>
hipError_t resident_launch(K kernel, int64_t total, size_t lds, hipStream_t stream, const Args&... args) {
  int per_cu = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kSvwThreads, lds);
  if (e != hipSuccess) return e;
  int dev = 0, cus = 0;
  e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int64_t resident = (int64_t)std::max(per_cu, 1) * std::max(cus, 1);
  const dim3 grid((unsigned)std::min<int64_t>(total, resident));
  hipLaunchKernelGGL(kernel, grid, dim3(kSvwThreads), lds, stream, args...);
  return hipGetLastError();
}

}  // namespace

size_t sv_window_lds_bytes(const SvWin& w) {
  if (w.np < 10 || w.np > kFuseMax || w.P[0] != 0) return 0;
  const size_t b = ((size_t)1 << w.np) * sizeof(float2) + (size_t)w.n_plain * 16 * sizeof(float2) +
                   (size_t)w.n_cl * 256 * sizeof(float2);
  return b > 64 * 1024 ? 0 : b + (size_t)w.n_plain * sizeof(uint32_t);
}

hipError_t launch_sv_window(const SvWin& w, const SvOp* d_ops, const float2* merged, int G, const float2* Ucl,
                            int n_cl_total, int64_t n_jobs, int32_t traj_base, float2* psi, int n, int precision,
                            bool grow, hipStream_t stream) {
  if (n_jobs <= 0 || (w.n_ops == 0 && !grow)) return hipSuccess;
  const size_t lds = sv_window_lds_bytes(w);
  if (lds == 0) return hipErrorInvalidValue;
  SvwArgs a{};
  a.n = n;
  a.n_ops = w.n_ops;
  a.n_plain = w.n_plain;
  a.n_cl = w.n_cl;
  a.cl_first = w.cl_first;
  a.n_cl_total = n_cl_total;
  a.G = G;
  for (int k = 0; k < kFuseMax; ++k) a.P[k] = w.P[k];
  a.live = grow ? w.live : w.other;
  a.fresh = grow ? w.fresh : 0u;
  a.n_jobs = n_jobs;
  a.traj_base = traj_base;
  const int64_t total = n_jobs << __builtin_popcount(a.live);
  const SvOp* ops = d_ops + w.op_off;
  auto go = [&](auto kernel) { return resident_launch(kernel, total, lds, stream, a, ops, merged, Ucl, psi); };
  auto by_np = [&](auto k10, auto k11, auto k12) { return w.np == 10 ? go(k10) : w.np == 11 ? go(k11) : go(k12); };
  auto by_prec = [&](auto fresh) -> hipError_t {
    constexpr bool F = decltype(fresh)::value;
    if (precision == PTSBE_SPLIT_BF16)
      return by_np(sv_window_kernel<PTSBE_SPLIT_BF16, 10, F>, sv_window_kernel<PTSBE_SPLIT_BF16, 11, F>,
                   sv_window_kernel<PTSBE_SPLIT_BF16, 12, F>);
    if (precision == PTSBE_SPLIT_F16)
      return by_np(sv_window_kernel<PTSBE_SPLIT_F16, 10, F>, sv_window_kernel<PTSBE_SPLIT_F16, 11, F>,
                   sv_window_kernel<PTSBE_SPLIT_F16, 12, F>);
    return by_np(sv_window_kernel<PTSBE_C64, 10, F>, sv_window_kernel<PTSBE_C64, 11, F>,
                 sv_window_kernel<PTSBE_C64, 12, F>);
  };
  return a.fresh ? by_prec(std::true_type{}) : by_prec(std::false_type{});
}

// Runs of gates on a network tensor of rank 13 and more: the plain windows' tiles and
// register groups.  The generic pass over the same tile costs an LDS pass and a barrier a
// gate.  A call of 4 amplitude rows of a 100-qubit chain (4 tensors of rank 22, 3 to 7
// gates a run) took about 2.9 ms with that pass and takes 2.4 ms; the runs of a 50-qubit
// sampling call in batches of ten (384 tensors of rank 13 to 19, most runs with a gate
// picked by hyper legs) 7.6 ms and 3.2 ms.
hipError_t launch_part_window(const SvWin& w, const SvOp* d_ops, const float2* merged, int G, int64_t n_jobs,
                              const int32_t* job_traj, int32_t traj_base, float2* A, int r, hipStream_t stream) {
  if (n_jobs <= 0) return hipSuccess;
  const size_t lds = sv_window_lds_bytes(w);
  if (lds == 0 || w.np != kFuseMax) return hipErrorInvalidValue;
  SvwArgs a{};
  a.n = r;
  a.n_ops = w.n_ops;
  a.n_plain = w.n_plain;
  a.G = G;
  for (int k = 0; k < kFuseMax; ++k) a.P[k] = w.P[k];
  a.live = w.live;
  a.n_jobs = n_jobs;
  a.traj_base = traj_base;
  a.job_traj = job_traj;
  const int64_t total = n_jobs << __builtin_popcount(a.live);
  const float2* Ucl = nullptr;
  auto go = [&](auto kernel) {
    return resident_launch(kernel, total, lds, stream, a, d_ops + w.op_off, merged, Ucl, A);
  };
  return w.n_hyper ? go(sv_window_kernel<kSvwHyper, kFuseMax, false>) : go(sv_window_kernel<kSvwPlain, kFuseMax, false>);
}

}  // namespace ptsbe
