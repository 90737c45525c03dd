// Device helpers shared by the decode kernels' translation units (gfx950).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "starkv_internal.h"

namespace starkv {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f4 mfma16(h8 a, h8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }
__device__ __forceinline__ uint32_t as_u32(h2 h) { return __builtin_bit_cast(uint32_t, h); }

// A pair of 8-bit or 4-bit codes placed in the low mantissa bits of fp16 1024:
// the fp16 value is 1024 + code exactly.  Subtracting 1024 is exact; the fma
// with (s, z) rounds once.
__device__ __forceinline__ uint32_t deq_pair(uint32_t magic_pair, h2 s, h2 z) {
  h2 c = as_h2(magic_pair) - (h2){(_Float16)1024.0f, (_Float16)1024.0f};
  return as_u32(__builtin_elementwise_fma(c, s, z));
}

// Scores may exceed the shared softmax reference by this much (log2 units)
// before it is raised: probabilities stay below 2^8 in fp16.
constexpr float kLazyMargin = 8.0f;

// value-tile precision variants of the split kernel's p.V' phase
constexpr int kValues8 = 0, kValues4 = 1, kValuesMixed = 2;

__device__ __forceinline__ float wave_max16(float v) {
  v = fmaxf(v, __shfl_xor(v, 16));
  v = fmaxf(v, __shfl_xor(v, 32));
  return v;
}
__device__ __forceinline__ float wave_sum16(float v) {
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}

// ceil(x / k) for 0 <= x < 2^17 + 64 and 1 <= k <= 64, with rk = rcp_up(k),
// the smallest float >= 1/k: the product rounds to the exact quotient's floor
// (x/k is at least 1/64 below the next integer unless it is one, and the
// relative error stays below 2^-22).
__device__ __forceinline__ float rcp_up(int k) {
  float r = __builtin_amdgcn_rcpf((float)k);           // within 1 ulp of 1/k
  const float e = __builtin_fmaf(r, (float)k, -1.0f);  // exact residual
  if (e >= 0.0f) {                                     // step down while still >= 1/k
    const float d = __uint_as_float(__float_as_uint(r) - 1u);
    if (__builtin_fmaf(d, (float)k, -1.0f) >= 0.0f) r = d;
  } else {
    r = __uint_as_float(__float_as_uint(r) + 1u);
  }
  return r;
}
__device__ __forceinline__ int div_up_small(int x, int k, float rk) {
  return (int)((float)(x + k - 1) * rk);
}

// Work plan of one decode step for up to 64 sequences of ragged lengths: the
// split length S = kStepTokens * k is the smallest with at most `cap` work
// items sum_b ceil(L_b / S) (k >= k_lo keeps every sequence at <= 256 splits,
// k <= 64 keeps S <= 8192), and the items are the sequences' splits in order.
// Every wave that calls this gets the same plan.  len: the clamped length held
// by lane b (lanes >= B hold 0).  Returns k; *cnt gets the split count of
// sequence `lane`.
__device__ __forceinline__ int wave_split_plan(int len, int B, int k_lo, int cap, int lane,
                                               int* cnt) {
  const int m = (len + kStepTokens - 1) / kStepTokens;      // steps of sequence `lane`
  const int k = min(k_lo + lane, 64);                       // candidate of this lane
  const float rk = rcp_up(k);
  int items = 0;
  for (int j = 0; j < B; ++j) items += div_up_small(__builtin_amdgcn_readlane(m, j), k, rk);
  const uint64_t ok = __ballot(items <= cap);
  const int ks = ok ? min(k_lo + (int)__builtin_ctzll(ok), 64) : 64;
  *cnt = div_up_small(m, ks, rcp_up(ks));
  return ks;
}

// The work item of a split workgroup: sequence b, its split, the split length S,
// the slot of the item's partials and the sequence's length.  Returns false past
// the last item.  L_in: this lane's loaded context length (of sequence `lane`
// under the work plan, of blockIdx.y otherwise).
struct SplitItem {
  int b, split, S, pitem, L;
};
template <class P>
__device__ __forceinline__ bool split_item(const P& p, int L_in, int w, int lane, SplitItem* it) {
  int L = L_in < 0 ? 0 : (L_in > p.max_ctx ? p.max_ctx : L_in);
  if (p.dyn) {
    int cnt;
    it->S = wave_split_plan(L, p.batch, p.k_lo, p.cap, lane, &cnt) * kStepTokens;
    if (blockIdx.x == 0 && blockIdx.z == 0 && w == 0) {
      // the plan of every sequence for the merge pass: its first item (an
      // exclusive prefix sum of the split counts), split count and length
      int incl = lane < p.batch ? cnt : 0;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
      }
      if (lane < p.batch)
        *reinterpret_cast<int4*>(p.plan + 4 * lane) = make_int4(incl - cnt, cnt, L, 0);
    }
    it->pitem = blockIdx.x;
    // the item's sequence: a scalar walk over the sequences' split counts
    it->b = -1;
    it->split = it->pitem;
    for (int j = 0; j < p.batch; ++j) {
      const int cj = __builtin_amdgcn_readlane(cnt, j);
      if (it->split < cj) { it->b = j; break; }
      it->split -= cj;
    }
    if (it->b < 0) return false;
    it->L = __builtin_amdgcn_readlane(L, it->b);
  } else {
    it->b = blockIdx.y;
    it->split = blockIdx.x;
    it->S = p.split_len;
    it->pitem = it->b * p.n_split + it->split;
    it->L = L;
  }
  return it->split * it->S < it->L;
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ __forceinline__ float load_qf(const uint16_t* q, int idx, int bf16) {
  const uint16_t u = q[idx];
  if (bf16) return __uint_as_float(static_cast<uint32_t>(u) << 16);
  return (float)__builtin_bit_cast(_Float16, u);
}

// A value the compiler cannot fold into instructions as a literal, so that it
// stays in a register (lets v_and_or_b32 take it as an operand).
__device__ __forceinline__ uint32_t opaque_u32(uint32_t v) {
  uint32_t r;
  asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
  return r;
}

// Asynchronous copy of n_bytes (a multiple of 16) from global memory into LDS by
// the whole workgroup, 16 bytes per lane, without passing through registers.
// Completion is tracked by vmcnt.
__device__ __forceinline__ void copy_to_lds(uint8_t* lds, const uint8_t* src, int n_bytes,
                                            int w, int lane) {
  for (int base = w * 1024; base < n_bytes; base += kWaves * 1024) {
    if (base + lane * 16 < n_bytes)
      __builtin_amdgcn_global_load_lds(src + base + lane * 16, lds + base, 16, 0, 0);
  }
}

// Workgroup barrier over LDS traffic only: this wave's LDS operations have
// completed (lgkmcnt(0)), then s_barrier.  The fence of __syncthreads() also
// waits for every global load and LDS copy still in flight (vmcnt(0)); this
// barrier leaves them in flight, and the copies it must cover are waited for
// explicitly (wait_vm) before it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}

// Lane exchanges in the vector registers (__shfl goes through LDS, some 130 cycles).
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                               0xF, 0xF, true));
}
// reductions over the lane's 8, 16 or 32 neighbours (a power-of-two group), to all of them
template <int N, class Op>
__device__ __forceinline__ float reduce_lanes(float v, Op op) {
  v = op(v, dpp<0xB1>(v));                       // quad_perm 1,0,3,2
  v = op(v, dpp<0x4E>(v));                       // quad_perm 2,3,0,1
  v = op(v, dpp<0x141>(v));                      // row_half_mirror
  if (N > 8) v = op(v, dpp<0x140>(v));           // row_mirror
  if (N > 16) v = op(v, __shfl_xor(v, 16));
  return v;
}
// the same over the wave, from the results of its rows of 16 (wave-uniform)
template <class Op>
__device__ __forceinline__ float reduce_wave(float v, Op op) {
  v = reduce_lanes<16>(v, op);
  auto row = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
  const float r = op(op(row(0), row(16)), op(row(32), row(48)));
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(r)));
}
__device__ __forceinline__ float wave_sum(float v) {
  return reduce_wave(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return reduce_wave(v, [](float a, float b) { return fmaxf(a, b); });
}
// v plus the value of lane ^ 16, ^ 32 (all lanes active): the swap of a register with a copy
// of itself leaves the two rows, or halves, in one register each
__device__ __forceinline__ float sum_rows16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_rows32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Raises a kernel's dynamic LDS limit to 160 KiB once per device: `done` holds
// one bit per device index (indices past 63 set it on every launch).
static inline int allow_lds(const void* fn, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  const uint64_t bit = dev < 64 ? 1ull << dev : 0;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return 0;
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e != hipSuccess) return (int)e;
  done.fetch_or(bit, std::memory_order_release);
  return 0;
}

}  // namespace starkv
