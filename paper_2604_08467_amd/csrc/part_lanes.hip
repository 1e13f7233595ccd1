// Sweeps of small tensors with one job a lane (gfx950).
//
// The per-element parts that continue an earlier batch's tensor keep their rank
// from end to end: 15 steps on 2^5 amplitudes for a chain of depth 6, for some
// 10^5 .. 10^6 elements a batch.  A lane holds its job's whole tensor in registers
// and takes the steps one after the other; 64 jobs, mostly of one or two
// trajectories, share the gates of a step in LDS as broadcasts, and tensors come and
// go through LDS so that memory sees whole rows.  A two-leg step is then 512 products
// a lane and eight 16-byte LDS reads, where part_vm_kernel (a thread per four
// amplitudes) also reads and writes the tensors in LDS, works out their addresses and
// meets at a barrier: 320000 elements x 15 steps 195 us there, 91 us here.  Bound by the
// products (VALU: 67 us of the 91).  Products are summed in the order of part_vm_kernel: the same
// results bit for bit.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "internal.h"

namespace ptsbe {
namespace {

constexpr int kPlPart = 16;                  // entries of a tensor in LDS at a time
constexpr int kPlRow = kPlPart + 1;          // LDS row of a job: one entry more, over the banks
constexpr int kPlGates = 64 * kPlRow / 16;   // staged gates (step, trajectory slot) in the same LDS

// Two contracted and two new legs in place on register bits I < J (gate bit 0: I).
template <int R, int I, int J>
__device__ __forceinline__ void lane_step2(float2 (&x)[1 << R], const float2* G) {
  float2 g[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) g[i] = G[i];
#pragma unroll
  for (int l = 0; l < (1 << R); ++l)
    if (!(l >> I & 1) && !(l >> J & 1)) {
      const float2 a[4] = {x[l], x[l | 1 << I], x[l | 1 << J], x[l | 1 << I | 1 << J]};
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        float2 acc = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc = cfma(a[k], g[4 * n + k], acc);
        x[l | (n & 1) << I | (n >> 1) << J] = acc;
      }
      __builtin_amdgcn_sched_barrier(0);     // one quad at a time: few registers
    }
}

// One contracted and one new leg in place on register bit I; entries g[2 n + k].
template <int R, int I>
__device__ __forceinline__ void lane_step1(float2 (&x)[1 << R], const float2 (&g)[4]) {
#pragma unroll
  for (int l = 0; l < (1 << R); ++l)
    if (!(l >> I & 1)) {
      const float2 a0 = x[l], a1 = x[l | 1 << I];
      const float2 zero = make_float2(0.f, 0.f);
      x[l] = cfma(a1, g[1], cfma(a0, g[0], zero));
      x[l | 1 << I] = cfma(a1, g[3], cfma(a0, g[2], zero));
    }
}

// Entries [16 PART, 16 PART + 16) of the output of a last step that contracts register bit
// I and makes bits I (value l) and R (value t): entry (l, t, k) of its gate is g[4 t + 2 l + k].
template <int R, int PART, int I>
__device__ __forceinline__ void lane_raise(const float2 (&x)[1 << R], const float2 (&g)[8], float2* to) {
#pragma unroll
  for (int e = 0; e < kPlPart; ++e) {
    const int o = PART * kPlPart + e, t = o >> R, l = o >> I & 1, i = o & ((1 << R) - 1) & ~(1 << I);
    to[e] = cfma(x[i | 1 << I], g[4 * t + 2 * l + 1], cfma(x[i], g[4 * t + 2 * l], make_float2(0.f, 0.f)));
  }
}

// Output entries [16 PART, ...) of every job, through LDS to whole rows of memory.
template <int R, bool RAISE, int PART>
__device__ __forceinline__ void lane_store(const float2 (&x)[1 << R], const float2 (&g)[8], int bit, float2* buf,
                                           float2* __restrict__ out, int64_t job0, int64_t n_jobs) {
  constexpr int ROUT = RAISE ? R + 1 : R;
  if constexpr (PART < (1 << ROUT) / kPlPart) {
    const int lane = threadIdx.x;
    float2* to = buf + lane * kPlRow;
    if constexpr (RAISE) {
      switch (bit) {
        case 0: lane_raise<R, PART, 0>(x, g, to); break;
        case 1: lane_raise<R, PART, 1>(x, g, to); break;
        case 2: lane_raise<R, PART, 2>(x, g, to); break;
        case 3: lane_raise<R, PART, 3>(x, g, to); break;
        default: if constexpr (R > 4) lane_raise<R, PART, 4>(x, g, to); break;
      }
    } else {
#pragma unroll
      for (int e = 0; e < kPlPart; ++e) to[e] = x[PART * kPlPart + e];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int j = 4 * i + (lane >> 4);
      if (job0 + j < n_jobs) out[((job0 + j) << ROUT) + PART * kPlPart + (lane & 15)] = buf[j * kPlRow + (lane & 15)];
    }
    __syncthreads();
    lane_store<R, RAISE, PART + 1>(x, g, bit, buf, out, job0, n_jobs);
  }
}

template <int R, bool RAISE>
__global__ void __launch_bounds__(64, 3) part_lanes_kernel(const AbsorbStep* __restrict__ steps, int n_steps, GateCtx g,
                                                           int64_t n_jobs, const int32_t* __restrict__ job_traj,
                                                           int32_t traj_base, const uint64_t* __restrict__ job_prefix,
                                                           int NW, InitArgs init, float2* __restrict__ out) {
  extern __shared__ __align__(16) float2 pl_lds[];
  float2* buf = pl_lds;                                              // tensors' parts, or staged gates
  int64_t* row_off = reinterpret_cast<int64_t*>(buf + 64 * kPlRow);  // [64] the jobs' initial tensors
  int4* stab = reinterpret_cast<int4*>(row_off + 64);                // [n_steps] gate | conj << 31, gperm
  int* slot_traj = reinterpret_cast<int*>(stab + n_steps);           // [64]
  const int lane = threadIdx.x;
  constexpr int N = 1 << R;
  for (int s = lane; s < n_steps; s += 64)
    stab[s] = make_int4(steps[s].gate | (steps[s].conj ? (int)0x80000000 : 0), (int)steps[s].gperm[0],
                        (int)steps[s].gperm[1], 0);
  const int64_t job0 = (int64_t)blockIdx.x * 64;
  const int64_t job = job0 + lane < n_jobs ? job0 + lane : n_jobs - 1;   // idle lanes repeat the last job
  const int traj = job_traj ? job_traj[job] : traj_base + (int)job;
  const uint64_t* pj = job_prefix ? job_prefix + job * NW : nullptr;
  // a slot per run of equal trajectories
  const int tprev = __shfl_up(traj, 1);
  const bool start = lane == 0 || tprev != traj;
  const uint64_t starts = __ballot(start);
  const int slot = __popcll(starts & ((2ull << lane) - 1ull)) - 1;
  const int n_slots = __popcll(starts);
  if (start) slot_traj[slot] = traj;
  int64_t off = (init.parent ? (int64_t)init.parent[job] : job) * init.stride;
  for (int i = 0; i < init.nsl; ++i) off += (int64_t)bit_of_prefix(pj, init.q[i]) << init.pos[i];
  row_off[lane] = off;
  __syncthreads();
  float2 x[N];
#pragma unroll
  for (int part = 0; part < N / kPlPart; ++part) {
    // entry m of a part (its sliced positions free) of 4 jobs per load
    uint32_t m = (uint32_t)(part * kPlPart + (lane & 15));
    for (int i = 0; i < init.nsl; ++i) {
      const uint32_t low = (1u << init.pos[i]) - 1u;
      m = ((m & ~low) << 1) | (m & low);
    }
    float2 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = init.Vprev[row_off[4 * i + (lane >> 4)] + m];
#pragma unroll
    for (int i = 0; i < 16; ++i) buf[(4 * i + (lane >> 4)) * kPlRow + (lane & 15)] = v[i];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPlPart; ++e) x[part * kPlPart + e] = buf[lane * kPlRow + e];
    __syncthreads();
  }
  const int chunk = kPlGates / n_slots;    // steps staged at a time: at least one
  int cs = -chunk;
  for (int s = 0; s < n_steps; ++s) {
    if (s == cs + chunk) {
      cs = s;
      const int E = (n_steps - cs < chunk ? n_steps - cs : chunk) * n_slots * 16;
      __syncthreads();                     // the previous chunk's gates are no longer read
      for (int e0 = 0; e0 < E; e0 += 256) {
        float2 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e = e0 + 64 * u + lane, ec = e < E ? e : E - 1;
          const int q = ec >> 4, gi = ec & 15, si = q / n_slots, sl = q - si * n_slots;
          const int4 sd = stab[cs + si];
          const uint32_t src = ((uint32_t)(gi < 8 ? sd.y : sd.z) >> (4 * (gi & 7))) & 15u;
          v[u] = g.merged[((int64_t)slot_traj[sl] * g.G + (sd.x & 0x7fffffff)) * 16 + src];
          if (sd.x < 0) v[u].y = -v[u].y;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (e0 + 64 * u + lane < E) buf[e0 + 64 * u + lane] = v[u];
      }
      __syncthreads();
    }
    if (RAISE && s == n_steps - 1) break;
    const AbsorbStep& st = steps[s];
    const float2* G = buf + ((s - cs) * n_slots + slot) * 16;
    const int k0 = st.kpos[0];
    if (st.nK == 2) {                      // four legs: none hyper or sliced, entries in (n, k) order
      const int k1 = st.kpos[1];
      switch (k0 * 8 + k1) {
#define PL_TWO(I, J) case I * 8 + J: if constexpr (J < R) lane_step2<R, I, J>(x, G); break;
        PL_TWO(0, 1) PL_TWO(0, 2) PL_TWO(0, 3) PL_TWO(0, 4) PL_TWO(1, 2) PL_TWO(1, 3) PL_TWO(1, 4)
        PL_TWO(2, 3) PL_TWO(2, 4) PL_TWO(3, 4)
#undef PL_TWO
        default: break;                    // not reached: lane_sweep takes these positions only
      }
    } else {
      int h = 0;
      for (int i = 0; i < st.nS; ++i) h += (int)bit_of_prefix(pj, st.sq[i]) * st.sw[i];
      float2 e[4];
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int k = 0; k < 2; ++k) e[2 * n + k] = st.nS == 0 ? G[2 * n + k] : G[h + st.nB[n] + st.kB[k]];
      switch (k0) {
        case 0: lane_step1<R, 0>(x, e); break;
        case 1: lane_step1<R, 1>(x, e); break;
        case 2: lane_step1<R, 2>(x, e); break;
        case 3: lane_step1<R, 3>(x, e); break;
        default: if constexpr (R > 4) lane_step1<R, 4>(x, e); break;
      }
    }
  }
  float2 last[8];
  int bit = 0;
  if (RAISE) {                             // the last step's gate, before the buffer takes the output
    const AbsorbStep& st = steps[n_steps - 1];
    const float2* G = buf + ((n_steps - 1 - cs) * n_slots + slot) * 16;
    int h = 0;
    for (int i = 0; i < st.nS; ++i) h += (int)bit_of_prefix(pj, st.sq[i]) * st.sw[i];
    bit = st.kpos[0];
    // value n of the new legs with l = lt & 1 at `bit` and t = lt >> 1 at R
    const int n1 = (int)(st.noff[1] >> R & 1u) ? 2 : 1, n2 = 3 - n1;
#pragma unroll
    for (int lt = 0; lt < 4; ++lt) {
      const int n = lt == 1 ? n1 : lt == 2 ? n2 : lt;
#pragma unroll
      for (int k = 0; k < 2; ++k) last[2 * lt + k] = st.nS == 0 ? G[2 * n + k] : G[h + st.nB[n] + st.kB[k]];
    }
  }
  __syncthreads();
  lane_store<R, RAISE, 0>(x, last, bit, buf, out, job0, n_jobs);
}

}  // namespace

// Ranks 4 and 5, those of the per-element parts of chains of depth 5 and 6.  At rank 6 the
// tensor alone would take 128 of a lane's 168 registers (three wavefronts a SIMD); rank 3 and
// below were not tried.
int lane_sweep_rank(const AbsorbStep* st, int n, int r0, bool* raise) {
  if (r0 < 4 || r0 > 5 || n < 1) return 0;
  *raise = false;
  for (int i = 0; i < n; ++i) {
    if (st[i].rA != r0 || st[i].nH != 0) return 0;
    bool in_place = st[i].rC == r0 && st[i].nK == st[i].nN && st[i].nK >= 1 && st[i].nK <= 2;
    for (int k = 0; k < st[i].nK && in_place; ++k)
      in_place = st[i].kpos[k] >= 0 && st[i].kpos[k] < r0 && st[i].koff[1 << k] == (1u << st[i].kpos[k]) &&
                 st[i].noff[1 << k] == st[i].koff[1 << k] && (k == 0 || st[i].kpos[k] > st[i].kpos[0]);
    if (st[i].nK == 2 && st[i].nS != 0) return 0;
    if (in_place) continue;
    // a last step may split its leg in two, one of them the new top position
    const bool split = i == n - 1 && st[i].rC == r0 + 1 && st[i].nK == 1 && st[i].nN == 2 && st[i].kpos[0] >= 0 &&
                       st[i].kpos[0] < r0 && st[i].koff[1] == (1u << st[i].kpos[0]) &&
                       (st[i].noff[1] | st[i].noff[2]) == ((1u << st[i].kpos[0]) | (1u << r0)) &&
                       (st[i].noff[1] & st[i].noff[2]) == 0 && st[i].noff[1] != 0 && st[i].noff[2] != 0 &&
                       st[i].noff[3] == (st[i].noff[1] | st[i].noff[2]);
    if (!split) return 0;
    *raise = true;
  }
  return r0;
}

hipError_t launch_part_lanes(const AbsorbStep* d_steps, int n_steps, int rank, bool raise, GateCtx g, int64_t n_jobs,
                             const int32_t* job_traj, int32_t traj_base, const uint64_t* job_prefix, int NW,
                             const InitArgs& init, float2* out, hipStream_t stream) {
  if (n_jobs <= 0) return hipSuccess;
  const size_t lds = (size_t)64 * kPlRow * sizeof(float2) + 64 * sizeof(int64_t) + (size_t)n_steps * sizeof(int4) +
                     64 * sizeof(int);
  const dim3 grid((unsigned)((n_jobs + 63) / 64));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(64), lds, stream, d_steps, n_steps, g, n_jobs, job_traj, traj_base,
                       job_prefix, NW, init, out);
    return hipGetLastError();
  };
  if (rank == 4) return raise ? go(part_lanes_kernel<4, true>) : go(part_lanes_kernel<4, false>);
  if (rank == 5) return raise ? go(part_lanes_kernel<5, true>) : go(part_lanes_kernel<5, false>);
  return hipErrorInvalidValue;
}

}  // namespace ptsbe
