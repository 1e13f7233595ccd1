// Device helpers of the statevector gate windows (included by the window kernel
// and the ragged-set kernels; everything here is inline): the compact ops' group
// and cluster applications on an LDS tile of 2^NP amplitudes, and the 16-byte
// amplitude-pair tile loads.  Qubit 0 is tile bit 0, so a pair of amplitudes is
// one 16-byte run of the state.
#pragma once

#include <hip/hip_runtime.h>

#include "device_util.h"
#include "internal.h"

namespace ptsbe {
namespace {

constexpr int kSvwThreads = 256;

// LDS layout of a tile: entry l lives at swz(l) = l ^ ((l >> 4) & 15), tile
// bits 4..7 folded into the low four bits (the 8-byte bank slot of a 128-byte
// LDS row).  The 16 lanes of a quarter-wavefront that step along the tile bits
// left free by an op (a gate's other bits, a cluster's columns) then spread over
// more slots: on a 32-bank model this brings cluster accesses from 3.4x to 1.8x
// of conflict-free and two-qubit gates from 1.76x to 1.47x.  A full linear map
// of bits 4..11 gets within 15 % and 6 %, but its index arithmetic costs more
// VALU issue than the conflicts it removes (measured on the window kernel).
// swz is linear, swz(a ^ b) = swz(a) ^ swz(b), so each thread swizzles its own
// part of an index once per op and XORs uniform parts in.
__host__ __device__ inline uint32_t swz(uint32_t l) { return l ^ ((l >> 4) & 15u); }

constexpr int kSvwPlain = -1;   // "precision" of a window without clusters
constexpr int kSvwHyper = -2;   // and of one with gates picked by hyper legs

__device__ inline uint32_t ins0(uint32_t m, int p) {   // zero bit inserted at position p
  const uint32_t lo = (1u << p) - 1u;
  return ((m & ~lo) << 1) | (m & lo);
}

struct SvwArgs {
  int n, n_ops, n_plain, n_cl, cl_first, n_cl_total, G;
  uint32_t live;           // bit mask of the qubits outside the window that tiles are made over
  uint32_t fresh;          // tile positions whose qubits are still |0> on entry
  int P[kFuseMax];
  int64_t n_jobs;
  int32_t traj_base;
  const int32_t* job_traj;   // trajectory of a job; null: traj_base + job
};

typedef __bf16 svw_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 svw_f16x8 __attribute__((ext_vector_type(8)));
template <int PREC> struct SvwSplit;
template <> struct SvwSplit<PTSBE_SPLIT_BF16> {
  typedef __bf16 E;
  typedef svw_bf16x8 V;
  static __device__ floatx4_t mfma(V a, V b, floatx4_t c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
template <> struct SvwSplit<PTSBE_SPLIT_F16> {
  typedef _Float16 E;
  typedef svw_f16x8 V;
  static __device__ floatx4_t mfma(V a, V b, floatx4_t c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};

// Byte address of an LDS tile entry as a lane's part XOR uniform parts (the swizzle is
// linear): positions' bits are deposited with one select and one XOR each.
__device__ inline uint32_t pos_bytes(uint32_t bytes, int i) {   // byte i of `bytes`: a tile position
  return 8u * swz(1u << (bytes >> (8 * i) & 0xffu));
}
__device__ inline float2& tile_at(float2* tile, uint32_t addr) {
  return *reinterpret_cast<float2*>(reinterpret_cast<char*>(tile) + addr);
}

// Addresses of a cluster's entries: lane 16 q + j of wave w, column tile ct takes column
// 64 ct' + 16 w + j (in the order of its column positions: the first four spread over the
// LDS banks), states 4 s + q where it reads (FP32) and 4 q + i where it writes.
template <int NP>
struct ClusterAt {
  uint32_t r, w;            // lane parts: column j and state bits 0, 1 = q (read), 2, 3 = q (written)
  uint32_t s1[4], s4[4];    // states i and 4 i
  uint32_t c[NP - 8];       // column tile bits
  __device__ ClusterAt(uint32_t cpos, uint2 cols) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t j = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) j ^= (lane >> b & 1u) ? pos_bytes(cols.x, b) : 0u;
#pragma unroll
    for (int b = 0; b < 2; ++b) j ^= (wave >> b & 1u) ? pos_bytes(cols.y, b) : 0u;
    uint32_t p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = pos_bytes(cpos, i);
    r = j ^ ((lane & 16u) ? p[0] : 0u) ^ ((lane & 32u) ? p[1] : 0u);
    w = j ^ ((lane & 16u) ? p[2] : 0u) ^ ((lane & 32u) ? p[3] : 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s1[i] = (i & 1 ? p[0] : 0u) ^ (i & 2 ? p[1] : 0u);
      s4[i] = (i & 1 ? p[2] : 0u) ^ (i & 2 ? p[3] : 0u);
    }
#pragma unroll
    for (int b = 0; b < NP - 10; ++b) c[b] = pos_bytes(cols.y, 2 + b);
  }
  __device__ uint32_t tile(int ct) const {       // uniform
    uint32_t a = 0;
#pragma unroll
    for (int b = 0; b < NP - 10; ++b)
      if (ct >> b & 1) a ^= c[b];
    return a;
  }
};

// Split-precision cluster: [Yr; Yi] = [[Ur, -Ui], [Ui, Ur]] [Xr; Xi] with the inner
// index interleaved (k = 2 v + c: state v, c = 0 real / 1 imaginary part), so that
// lane 16 q + j holds states 4q .. 4q+3 of column j (B) or of output row j (A).
// One 16x16x32 MFMA covers the whole inner dimension: per 16 columns, 2 row tiles
// (real and imaginary outputs) x 3 products.  Each wavefront reads and then
// overwrites only its own columns.  Needs blockDim.x == 256 and np >= 10.
template <int PREC, int NP>
__device__ __forceinline__ void apply_cluster_split(const ClusterAt<NP>& at, const float2* __restrict__ U,
                                                    float2* tile) {
  typedef typename SvwSplit<PREC>::E E;
  typedef typename SvwSplit<PREC>::V V;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, q = lane >> 4, j = lane & 15;
  V ah[2], al[2];
  {
    float a[2][8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float2 u = U[j * 16 + 4 * q + i];
      a[0][2 * i] = u.x;  a[0][2 * i + 1] = -u.y;    // real output row:  Ur Xr - Ui Xi
      a[1][2 * i] = u.y;  a[1][2 * i + 1] = u.x;     // imaginary output: Ui Xr + Ur Xi
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const E h = (E)a[rt][i];
        ah[rt][i] = h;
        al[rt][i] = (E)(a[rt][i] - (float)h);
      }
  }
#pragma unroll
  for (int ct = 0; ct < (1 << (NP - 10)); ++ct) {
    const uint32_t pc = at.tile(ct);
    float x[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float2 v = tile_at(tile, at.w ^ (pc ^ at.s1[i]));
      x[2 * i] = v.x;
      x[2 * i + 1] = v.y;
    }
    float scale = 1.f, unscale = 1.f;
    if (PREC == PTSBE_SPLIT_F16) {
      // one power of two per column (its four lanes agree): largest |x| to [2^14, 2^15)
      float m = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(x[i]));
      m = fmaxf(m, __shfl_xor(m, 16));
      m = fmaxf(m, __shfl_xor(m, 32));
      if (m > 0.f) {
        int e;
        (void)frexpf(m, &e);             // m = f 2^e, f in [1/2, 1)
        scale = ldexpf(1.f, 15 - e);
        unscale = ldexpf(1.f, e - 15);
      }
    }
    V bh, bl;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float xs = x[i] * scale;
      const E h = (E)xs;
      bh[i] = h;
      bl[i] = (E)(xs - (float)h);
    }
    floatx4_t acc[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      acc[rt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
      acc[rt] = SvwSplit<PREC>::mfma(ah[rt], bh, acc[rt]);
      acc[rt] = SvwSplit<PREC>::mfma(ah[rt], bl, acc[rt]);
      acc[rt] = SvwSplit<PREC>::mfma(al[rt], bh, acc[rt]);
    }
    // D[4 q + i][j]: output state 4 q + i of column j
#pragma unroll
    for (int i = 0; i < 4; ++i)
      tile_at(tile, at.w ^ (pc ^ at.s1[i])) = make_float2(acc[0][i] * unscale, acc[1][i] * unscale);
  }
  __syncthreads();
}

// FP32 cluster on v_mfma_f32_16x16x4f32 (inner index k < 16 real, >= 16 imaginary
// parts; lane 16 q + j takes states 4 s + q of column j), U in LDS.
template <int NP>
__device__ __forceinline__ void apply_cluster_f32(const ClusterAt<NP>& at, const float2* __restrict__ U, float2* tile) {
  const int lane = threadIdx.x & 63, q = lane >> 4, j = lane & 15;
  float af[2][8];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float2 u = U[j * 16 + 4 * s + q];
    af[0][s] = u.x;  af[0][s + 4] = -u.y;
    af[1][s] = u.y;  af[1][s + 4] = u.x;
  }
#pragma unroll
  for (int ct = 0; ct < (1 << (NP - 10)); ++ct) {
    const uint32_t pc = at.tile(ct);
    float2 x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = tile_at(tile, at.r ^ (pc ^ at.s4[s]));
    floatx4_t acc0 = floatx4_t{0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float b = s < 4 ? x[s].x : x[s - 4].y;
      acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(af[0][s], b, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(af[1][s], b, acc1, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) tile_at(tile, at.w ^ (pc ^ at.s1[i])) = make_float2(acc0[i], acc1[i]);
  }
  __syncthreads();
}

__device__ inline bool czero(float2 v) { return v.x == 0.f && v.y == 0.f; }

// Forms of a staged gate, worked out once per staging: at most one nonzero a row
// (diagonal gates with diagonal Kraus factors, CNOT, Pauli products) costs one product
// per amplitude.  Bits 2n, 2n + 1: the column of row n's nonzero.  A dense one-qubit gate
// whose diagonal or off-diagonal entries are all real or all imaginary (rotations about an
// axis, Hadamard, with Pauli noise and damping) takes half the terms for those: bits 0, 1
// for the diagonal and 2, 3 for the others, kEntry*.
constexpr uint32_t kFormDense = 0x100, kFormDiag = 0x200;
constexpr int kEntryComplex = 0, kEntryReal = 1, kEntryImag = 2;

__device__ inline uint32_t entry_kind(float2 a, float2 b) {
  return a.y == 0.f && b.y == 0.f ? kEntryReal : a.x == 0.f && b.x == 0.f ? kEntryImag : kEntryComplex;
}
__device__ inline uint32_t gate1_form(const float2* G) {
  const bool z00 = czero(G[0]), z01 = czero(G[1]), z10 = czero(G[2]), z11 = czero(G[3]);
  if (!((z00 || z01) && (z10 || z11)))
    return kFormDense | entry_kind(G[0], G[3]) | entry_kind(G[1], G[2]) << 2;
  return (!z00 && !z11) ? kFormDiag : (uint32_t)z00 | ((uint32_t)!z11 << 2);
}
__device__ inline uint32_t gate2_form(const float2* G) {
  uint32_t form = 0;
  bool mono = true, diag = true;
  for (int n = 0; n < 4; ++n) {
    int col = -1;
    for (int k = 0; k < 4; ++k)
      if (!czero(G[4 * n + k])) {
        mono = mono && col < 0;
        col = k;
      }
    diag = diag && (col < 0 || col == n);
    form |= (uint32_t)(col < 0 ? 3 : col) << (2 * n);
  }
  return mono ? (diag ? kFormDiag : form) : kFormDense;
}

// A value that all lanes hold, in scalar registers (a gate entry there leaves the vector
// registers to the amplitudes).
__device__ inline float2 uniform2(float2 v) {
  return make_float2(__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v.x))),
                     __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v.y))));
}

// g a with its roundings spelled out, so that they do not hang on how a kernel is compiled.
__device__ inline float2 gmul(float2 g, float2 a) {
  return make_float2(fmaf(g.x, a.x, -(g.y * a.y)), fmaf(g.y, a.x, g.x * a.y));
}

// gmul and cfma for an entry of known kind: the zero part's terms left out.
template <int KIND>
__device__ __forceinline__ float2 kmul(float2 g, float2 a) {
  if constexpr (KIND == kEntryReal) return make_float2(g.x * a.x, g.x * a.y);
  else if constexpr (KIND == kEntryImag) return make_float2(-(g.y * a.y), g.y * a.x);
  else return gmul(g, a);
}
template <int KIND>
__device__ __forceinline__ float2 kfma(float2 g, float2 a, float2 c) {
  if constexpr (KIND == kEntryReal) return make_float2(fmaf(g.x, a.x, c.x), fmaf(g.x, a.y, c.y));
  else if constexpr (KIND == kEntryImag) return make_float2(fmaf(-g.y, a.y, c.x), fmaf(g.y, a.x, c.y));
  else return cfma(g, a, c);
}

// A dense one-qubit gate on register bit B of x: D and O the kinds of its diagonal and
// off-diagonal entries.
template <int LB, int B, int D, int O>
__device__ __forceinline__ void reg_dense1(float2 (&x)[1 << LB], float2 g00, float2 g01, float2 g10, float2 g11) {
#pragma unroll
  for (int l = 0; l < (1 << LB); ++l)
    if (!(l >> B & 1)) {
      const float2 a0 = x[l], a1 = x[l | 1 << B];
      x[l] = kfma<O>(g01, a1, kmul<D>(g00, a0));
      x[l | 1 << B] = kfma<D>(g11, a1, kmul<O>(g10, a0));
    }
}

// A one-qubit gate on register bit B of x (g: [n][k] row-major in LDS).
template <int LB, int B>
__device__ __forceinline__ void reg_gate1(float2 (&x)[1 << LB], const float2* G, uint32_t form) {
  const float2 g00 = uniform2(G[0]), g01 = uniform2(G[1]), g10 = uniform2(G[2]), g11 = uniform2(G[3]);
  if (form & kFormDense) {
    switch (form & 15u) {
      case kEntryReal | kEntryReal << 2: reg_dense1<LB, B, kEntryReal, kEntryReal>(x, g00, g01, g10, g11); break;
      case kEntryReal | kEntryImag << 2: reg_dense1<LB, B, kEntryReal, kEntryImag>(x, g00, g01, g10, g11); break;
      case kEntryImag | kEntryReal << 2: reg_dense1<LB, B, kEntryImag, kEntryReal>(x, g00, g01, g10, g11); break;
      case kEntryReal: reg_dense1<LB, B, kEntryReal, kEntryComplex>(x, g00, g01, g10, g11); break;
      case kEntryReal << 2: reg_dense1<LB, B, kEntryComplex, kEntryReal>(x, g00, g01, g10, g11); break;
      default: reg_dense1<LB, B, kEntryComplex, kEntryComplex>(x, g00, g01, g10, g11); break;
    }
  } else if (form == kFormDiag) {
#pragma unroll
    for (int l = 0; l < (1 << LB); ++l) x[l] = gmul(l >> B & 1 ? g11 : g00, x[l]);
  } else {
    const bool c0 = form & 1u, c1 = form & 4u;       // rows 0 and 1 take amplitude 1
    const float2 d0 = c0 ? g01 : g00, d1 = c1 ? g11 : g10;
#pragma unroll
    for (int l = 0; l < (1 << LB); ++l)
      if (!(l >> B & 1)) {
        const float2 a0 = x[l], a1 = x[l | 1 << B];
        x[l] = gmul(d0, c0 ? a1 : a0);
        x[l | 1 << B] = gmul(d1, c1 ? a1 : a0);
      }
  }
}

// A two-qubit gate on register bits I (local bit 0) < J (local bit 1) of x.
template <int LB, int I, int J>
__device__ __forceinline__ void reg_gate2(float2 (&x)[1 << LB], const float2* G, uint32_t form) {
  constexpr int o[4] = {0, 1 << I, 1 << J, 1 << I | 1 << J};
  if (form == kFormDense) {
    float2 g[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) g[i] = uniform2(G[i]);
#pragma unroll
    for (int l = 0; l < (1 << LB); ++l)
      if (!(l & o[3])) {
        const float2 a0 = x[l], a1 = x[l | o[1]], a2 = x[l | o[2]], a3 = x[l | o[3]];
#pragma unroll
        for (int n = 0; n < 4; ++n)
          x[l | o[n]] = cfma(g[4 * n + 3], a3, cfma(g[4 * n + 2], a2, cfma(g[4 * n + 1], a1, gmul(g[4 * n], a0))));
        __builtin_amdgcn_sched_barrier(0);   // one quad at a time: eight chains, few registers
      }
  } else if (form == kFormDiag) {
    float2 g[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) g[n] = uniform2(G[5 * n]);
#pragma unroll
    for (int l = 0; l < (1 << LB); ++l)
      if (!(l & o[3]))
#pragma unroll
        for (int n = 0; n < 4; ++n) x[l | o[n]] = gmul(g[n], x[l | o[n]]);
  } else {
    float2 g[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) g[n] = uniform2(G[4 * n + (form >> (2 * n) & 3u)]);
#pragma unroll
    for (int l = 0; l < (1 << LB); ++l)
      if (!(l & o[3])) {
        const float2 a0 = x[l], a1 = x[l | o[1]], a2 = x[l | o[2]], a3 = x[l | o[3]];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          const uint32_t c = form >> (2 * n) & 3u;
          x[l | o[n]] = gmul(g[n], c == 0 ? a0 : c == 1 ? a1 : c == 2 ? a2 : a3);
        }
      }
  }
}

// A gate on register bit B whose matrix g ([n][k]) is the thread's own.
template <int LB, int B>
__device__ __forceinline__ void reg_hyper(float2 (&x)[1 << LB], const float2 (&g)[4]) {
  const float2 zero = make_float2(0.f, 0.f);
#pragma unroll
  for (int l = 0; l < (1 << LB); ++l)
    if (!(l >> B & 1)) {
      const float2 a0 = x[l], a1 = x[l | 1 << B];
      x[l] = cfma(a1, g[1], cfma(a0, g[0], zero));
      x[l | 1 << B] = cfma(a1, g[3], cfma(a0, g[2], zero));
    }
}

// The n gates after a group record (h: its first four dwords) on the tile: 2^(NP - 8)
// amplitudes a thread in registers.  One LDS pass and one barrier for all of them: a pass
// per gate cost 0.5 ms on a 12.9 GB set of states (25 qubits x 48), three times its own
// arithmetic, and a window of 14 gates 12.1 ms where it takes 8.3 now (5.3 ms to read and
// write the states).  group_sv_ops has which gates share a group.
// HYPER: some gates' matrices are picked by bits of the thread's part of the tile position
// or of the tile's own position `base`; such bits are never register bits, so that a thread
// has one matrix for all its amplitudes.
template <int NP, bool HYPER>
__device__ __forceinline__ void apply_group(const uint4 h, const uint4* __restrict__ ops, int n, float2* tile,
                                   const float2* Gs, const uint32_t* forms, uint32_t base) {
  constexpr int LB = NP - 8;
  const uint32_t tid = threadIdx.x;
  uint32_t at_tid = 0;             // this thread's part of the tile position
  if constexpr (HYPER) {
#pragma unroll
    for (int b = 0; b < 8; ++b) at_tid |= (tid >> b & 1u) << ((b < 4 ? h.z : h.w) >> (8 * (b & 3)) & 0xffu);
  }
  uint32_t pt = 0;                 // this thread's part of the address, then the register bits'
#pragma unroll
  for (int b = 0; b < 8; ++b) pt ^= (tid >> b & 1u) ? pos_bytes(b < 4 ? h.z : h.w, b & 3) : 0u;
  uint32_t so[LB];                 // uniform
#pragma unroll
  for (int i = 0; i < LB; ++i) so[i] = pos_bytes(h.y, i);
  float2 x[1 << LB];
#pragma unroll
  for (int l = 0; l < (1 << LB); ++l) {
    uint32_t at = pt;
#pragma unroll
    for (int i = 0; i < LB; ++i)
      if (l >> i & 1) at ^= so[i];
    x[l] = tile_at(tile, at);
  }
  for (int s = 0; s < n; ++s) {
    const uint4 w = ops[2 * s];
    const int slot = (int)w.w;
    const float2* G = Gs + 16 * slot;
    if constexpr (HYPER) {
      if ((w.x & 0xffu) == (uint32_t)kSvOpHyper) {
        const uint32_t c0 = w.y >> 8 & 0xffu, c1 = w.y >> 16 & 0xffu;
        const uint32_t b0 = c0 < 32u ? at_tid >> c0 : base >> (c0 - 32u), b1 = c1 < 32u ? at_tid >> c1 : base >> (c1 - 32u);
        float2 g[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) g[i] = G[4u * ((b0 & 1u) | (b1 & 1u) << 1) + i];
        switch (w.y & 0xffu) {
          case 0: reg_hyper<LB, 0>(x, g); break;
          case 1: reg_hyper<LB, 1>(x, g); break;
          case 2: if constexpr (LB > 2) reg_hyper<LB, 2>(x, g); break;
          default: if constexpr (LB > 3) reg_hyper<LB, 3>(x, g); break;
        }
        continue;
      }
    }
    const uint32_t form = (uint32_t)__builtin_amdgcn_readfirstlane((int)forms[slot]);
    const uint32_t code = (w.x & 0xffu) == (uint32_t)kSvOpGate1 ? (w.y & 0xffu) : 4u + (w.y & 0xffu);
    switch (code) {
      case 0: reg_gate1<LB, 0>(x, G, form); break;
      case 1: reg_gate1<LB, 1>(x, G, form); break;
      case 2: if constexpr (LB > 2) reg_gate1<LB, 2>(x, G, form); break;
      case 3: if constexpr (LB > 3) reg_gate1<LB, 3>(x, G, form); break;
      case 4 + svg_pair(0, 1): reg_gate2<LB, 0, 1>(x, G, form); break;
      case 4 + svg_pair(0, 2): if constexpr (LB > 2) reg_gate2<LB, 0, 2>(x, G, form); break;
      case 4 + svg_pair(0, 3): if constexpr (LB > 3) reg_gate2<LB, 0, 3>(x, G, form); break;
      case 4 + svg_pair(1, 2): if constexpr (LB > 2) reg_gate2<LB, 1, 2>(x, G, form); break;
      case 4 + svg_pair(1, 3): if constexpr (LB > 3) reg_gate2<LB, 1, 3>(x, G, form); break;
      default: if constexpr (LB > 3) reg_gate2<LB, 2, 3>(x, G, form); break;
    }
  }
  asm volatile("" : "+v"(pt));     // the addresses are worked out again, not kept in registers
#pragma unroll
  for (int l = 0; l < (1 << LB); ++l) {
    uint32_t at = pt;
#pragma unroll
    for (int i = 0; i < LB; ++i)
      if (l >> i & 1) at ^= so[i];
    tile_at(tile, at) = x[l];
  }
  __syncthreads();
}

// The window's gates (records [0, n_ops), groups and clusters among them) into Gs, 16
// entries a slot, and their forms; ends with a barrier.
__device__ __forceinline__ void stage_gates(const SvOp* __restrict__ ops, int n_ops, const float2* __restrict__ merged,
                                   float2* Gs, uint32_t* forms) {
  for (int i = threadIdx.x; i < 16 * n_ops; i += kSvwThreads) {
    const SvOp& op = ops[i >> 4];
    const int el = i & 15, d2 = op.kind == kSvOpGate1 ? 4 : 16;
    if ((op.kind != kSvOpGate1 && op.kind != kSvOpGate2 && op.kind != kSvOpHyper) || el >= d2) continue;
    float2 g = merged[(int64_t)op.gate * 16 + op.idx[el]];
    if (op.conj) g.y = -g.y;
    Gs[16 * op.slot + el] = g;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n_ops; i += kSvwThreads) {
    const SvOp& op = ops[i];
    if (op.kind == kSvOpGate1) forms[op.slot] = gate1_form(Gs + 16 * op.slot);
    if (op.kind == kSvOpGate2) forms[op.slot] = gate2_form(Gs + 16 * op.slot);
  }
  __syncthreads();
}

// Global offset of pair slot i of this thread within a tile (pair index
// tid + 256 i = tile bits 1..NP-1; tile bit 0 is qubit 0, the pair's two halves).
template <int NP>
__device__ inline uint32_t pair_hi(const int* P, int i) {
  uint32_t off = 0;
#pragma unroll
  for (int b = 0; b < NP - 9; ++b) off |= (uint32_t)((i >> b) & 1) << P[9 + b];
  return off;
}

// Pair at lane offset lo of the uniform address A: 8 lo fits 32 bits (n <= 30, and lo's
// highest bit P[8] has a window qubit above it), so that the pair's address is a scalar
// base and one 32-bit register for all pairs of the thread.
__device__ inline floatx4_t* pair_at(const float2* A, uint32_t lo) {
  return reinterpret_cast<floatx4_t*>(reinterpret_cast<char*>(const_cast<float2*>(A)) + (size_t)(lo * 8u));
}

// The thread's pairs of one tile (A: the tile's first amplitude) into v.
template <int NP>
__device__ inline void load_pairs(const float2* __restrict__ A, const int* P, uint32_t lo,
                                  floatx4_t (&v)[1 << (NP - 9)]) {
#pragma unroll
  for (int i = 0; i < (1 << (NP - 9)); ++i) v[i] = *pair_at(A + pair_hi<NP>(P, i), lo);
}

// As load_pairs, for a tile whose positions in `fresh` are still |0>: entries with any of
// them set are zero and not read.  Position 0 is fresh in the first window only, where
// every position is and the tile is |0...0>.
template <int NP>
__device__ inline void load_fresh_pairs(const float2* __restrict__ A, const int* P, uint32_t lo, uint32_t fresh,
                                        floatx4_t (&v)[1 << (NP - 9)]) {
  uint32_t e = 2u * threadIdx.x;
  asm volatile("" : "+v"(e));        // the conditions are worked out here, not kept over the tiles
#pragma unroll
  for (int i = 0; i < (1 << (NP - 9)); ++i) {
    v[i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    if (((e + 2u * kSvwThreads * i) & fresh) == 0) {
      if (fresh & 1u) v[i][0] = 1.f;
      else v[i] = *pair_at(A + pair_hi<NP>(P, i), lo);
    }
  }
}

// This thread's pair offset from its own bits (tile bits 1..8 = positions P[1..8]).
__device__ inline uint32_t pair_lo(const int* P) {
  uint32_t lo = 0;
#pragma unroll
  for (int b = 0; b < 8; ++b) lo |= (uint32_t)((threadIdx.x >> b) & 1) << P[b + 1];
  return lo;
}

// The tile's other bits t spread over the positions in `other` (a bit mask).
__device__ inline uint32_t deposit_other(uint32_t t, uint32_t other) {
  uint32_t out = 0, mask = other;
  for (int bit = 0; mask; ++bit, mask &= mask - 1u) out |= ((t >> bit) & 1u) << __builtin_ctz(mask);
  return out;
}

// LDS side of the pair moves: pair index tid + 256 i holds entries e = 2 (tid +
// 256 i) and e + 1, stored at swz(e) and swz(e) ^ 1 (one 16-byte slot, halves
// swapped when swz(e) is odd).  pt2 = swz(2 tid).
__device__ inline void lds_put_pair(floatx4_t* tile4, uint32_t pt2, int i, floatx4_t v) {
  const uint32_t e = pt2 ^ swz(2u * kSvwThreads * (uint32_t)i);
  tile4[e >> 1] = (e & 1u) ? floatx4_t{v[2], v[3], v[0], v[1]} : v;
}
__device__ inline floatx4_t lds_get_pair(const floatx4_t* tile4, uint32_t pt2, int i) {
  const uint32_t e = pt2 ^ swz(2u * kSvwThreads * (uint32_t)i);
  const floatx4_t v = tile4[e >> 1];
  return (e & 1u) ? floatx4_t{v[2], v[3], v[0], v[1]} : v;
}

// Tiles [b0, b1) of a window over the states psi [n_jobs][2^n] (tile t of job j is number
// (j << popc(live)) + t), their trajectories' merged gates and cluster matrices: pairs
// loaded, the groups and clusters applied in LDS, pairs stored.  Where every entry is read
// and clusters are applied the next tile's loads are issued before the current tile's ops;
// windows of plain gates are bound by their products and short of registers.  LDS: the tile, n_plain
// staged gates, n_cl clusters, n_plain forms.  Ends with a barrier.
template <int PREC, int NP, bool FRESH>
__device__ __forceinline__ void window_tiles(const SvwArgs& a, const SvOp* __restrict__ ops,
                                             const float2* __restrict__ merged, const float2* __restrict__ Ucl,
                                             float2* __restrict__ psi, int64_t b0, int64_t b1, floatx4_t* lds) {
  float2* tile = reinterpret_cast<float2*>(lds);
  floatx4_t* tile4 = lds;
  constexpr int PPT = 1 << (NP - 9);     // pairs per thread
  constexpr bool AHEAD = !FRESH && PREC >= 0;
  float2* Gs = tile + (1 << NP);                   // [n_plain][16]
  float2* Us = Gs + 16 * a.n_plain;                // [n_cl][256]
  uint32_t* forms = reinterpret_cast<uint32_t*>(Us + 256 * a.n_cl);   // [n_plain]
  const int tid = threadIdx.x;
  const int tb = __popc(a.live), n = a.n;
  // this thread's pair offset from its own bits (tile bits 1..8 = positions P[1..8])
  const uint32_t lo = pair_lo(a.P), pt2 = swz(2u * tid);
  auto tile_base = [&](int64_t bid) -> uint32_t {   // the tile's other bits, spread over the non-window positions
    return deposit_other((uint32_t)(bid & (((int64_t)1 << tb) - 1)), a.live);
  };
  floatx4_t v[PPT];
  auto load = [&](int64_t bid) {
    const float2* A = psi + ((bid >> tb) << n) + tile_base(bid);
    if (FRESH) load_fresh_pairs<NP>(A, a.P, lo, a.fresh, v);
    else load_pairs<NP>(A, a.P, lo, v);
  };
  auto put = [&]() {
#pragma unroll
    for (int i = 0; i < PPT; ++i) lds_put_pair(tile4, pt2, i, v[i]);
  };
  auto traj_of = [&](int64_t job) -> int64_t {
    return a.job_traj ? (int64_t)__builtin_amdgcn_readfirstlane(a.job_traj[job]) : a.traj_base + job;
  };
  auto stage = [&](int64_t job) {
    for (int i = tid; i < 256 * a.n_cl; i += kSvwThreads)
      Us[i] = Ucl[((int64_t)job * a.n_cl_total + a.cl_first) * 256 + i];
    stage_gates(ops, a.n_ops, merged + traj_of(job) * a.G * 16, Gs, forms);
  };
  load(b0);
  stage(b0 >> tb);
  put();
  for (int64_t bid = b0; bid < b1; ++bid) {
    __syncthreads();   // the tile (and any staging) is complete before the first op
    const bool more = bid + 1 < b1;
    if (AHEAD && more) load(bid + 1);   // in flight during the ops
    for (int s = 0; s < a.n_ops;) {
      // the record's first four dwords as one uniform (scalar-cache) load
      const uint4 w = reinterpret_cast<const uint4*>(ops)[2 * s];
      if ((w.x & 0xffu) == (uint32_t)kSvOpGroup) {
        const int ng = (int)(w.x >> 8 & 0xffu);
        apply_group<NP, PREC == kSvwHyper>(w, reinterpret_cast<const uint4*>(ops) + 2 * (s + 1), ng, tile, Gs, forms,
                                           PREC == kSvwHyper ? tile_base(bid) : 0u);
        s += 1 + ng;
      } else {
        ++s;
        if constexpr (PREC >= 0) {
          const uint4 w2 = reinterpret_cast<const uint4*>(ops)[2 * s - 1];
          const ClusterAt<NP> at(w.y, make_uint2(w2.x, w2.y));
          if constexpr (PREC == PTSBE_C64) apply_cluster_f32<NP>(at, Us + 256 * (int)w.w, tile);
          else apply_cluster_split<PREC, NP>(at, Us + 256 * (int)w.w, tile);
        }
      }
    }
    floatx4_t o[PPT];
#pragma unroll
    for (int i = 0; i < PPT; ++i) o[i] = lds_get_pair(tile4, pt2, i);
    float2* A = psi + ((bid >> tb) << n) + tile_base(bid);
    auto keep = [&]() {
#pragma unroll
      for (int i = 0; i < PPT; ++i) *pair_at(A + pair_hi<NP>(a.P, i), lo) = o[i];
    };
    if (!AHEAD) keep();
    __syncthreads();   // every thread has read its part of the tile
    if (more) {
      if (!AHEAD) load(bid + 1);
      put();
    }
    // with loads ahead the next tile takes this one's place before this one is stored: memory
    // operations finish in order, so a wait for the loads after the stores would wait for
    // them too
    if (AHEAD) keep();
    // the next trajectory's gates
    if (more && (bid + 1) >> tb != bid >> tb && traj_of((bid + 1) >> tb) != traj_of(bid >> tb)) stage((bid + 1) >> tb);
  }
  __syncthreads();
}

}  // namespace
}  // namespace ptsbe
