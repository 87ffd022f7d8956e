// device_common.hpp -- device-side helpers shared by the gfx950 kernels of
// libentropy: the Philox4x32-10 counter generator and the probe mapping,
// wave64 reductions and MFMA wrappers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace ent {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten S-box rounds over a
// 128-bit counter; the 64-bit key is advanced by the two Weyl constants
// between rounds.
// ---------------------------------------------------------------------------
struct U4 {
  uint32_t x, y, z, w;
};

__device__ __forceinline__ U4 philox10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t lo0 = 0xD2511F53u * c.x;
    const uint32_t hi0 = __umulhi(0xD2511F53u, c.x);
    const uint32_t lo1 = 0xCD9E8D57u * c.z;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z);
    U4 n;
    n.x = hi1 ^ c.y ^ k0;
    n.y = lo1;
    n.z = hi0 ^ c.w ^ k1;
    n.w = lo0;
    c = n;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// Counter layout: (row mod 2^32, block, stream, row >> 32); key = seed.
__device__ __forceinline__ U4 philox_block(uint64_t seed, uint32_t stream, int64_t row,
                                           uint32_t block) {
  U4 c;
  c.x = (uint32_t)((uint64_t)row & 0xffffffffu);
  c.y = block;
  c.z = stream;
  c.w = (uint32_t)((uint64_t)row >> 32);
  return philox10(c, (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32));
}

// 32 Rademacher signs of probes [32*word, 32*word+32) of one row, as a bit
// mask: bit b set means probe 32*word+b is -1.  One Philox block serves 128
// probes: block = probe >> 7, word index (probe >> 5) & 3.
__device__ __forceinline__ uint32_t rademacher_word(uint64_t seed, uint32_t stream, int64_t row,
                                                    int32_t word) {
  const U4 o = philox_block(seed, stream, row, (uint32_t)word >> 2);
  switch (word & 3) {
    case 0: return o.x;
    case 1: return o.y;
    case 2: return o.z;
    default: return o.w;
  }
}

__device__ __forceinline__ double rademacher(uint64_t seed, uint32_t stream, int64_t row,
                                             int64_t probe) {
  const uint32_t w = rademacher_word(seed, stream, row, (int32_t)(probe >> 5));
  return ((w >> (probe & 31)) & 1u) ? -1.0 : 1.0;
}

// Standard Gaussian by Box-Muller on two 53-bit uniforms of one Philox block
// (block = probe >> 1); even probes take the cosine branch, odd the sine.
__device__ __forceinline__ double gaussian(uint64_t seed, uint32_t stream, int64_t row,
                                           int64_t probe) {
  const U4 o = philox_block(seed, stream, row, (uint32_t)((uint64_t)probe >> 1));
  const uint64_t a = ((((uint64_t)o.y) << 32) | o.x) >> 11;
  const uint64_t b = ((((uint64_t)o.w) << 32) | o.z) >> 11;
  const double u1 = ((double)a + 1.0) * 0x1.0p-53;
  const double u2 = (double)b * 0x1.0p-53;
  const double r = sqrt(-2.0 * log(u1));
  const double th = 6.283185307179586476925286766559 * u2;
  return (probe & 1) ? r * sin(th) : r * cos(th);
}

// Structured sketches of the random projection (Section 5.2).  Row sign
// D_jj = -1 iff bit 0 of word x of stream 3's block (row j, block 0); the
// input-sparsity bucket of row j is floor(word y * s / 2^32) of the same
// block; the t-th sampled Hadamard column is word x of stream 4's block
// (row t) modulo N, N = 2^ceil(log2 n).
__device__ __forceinline__ double sketch_sign(uint64_t seed, int64_t j) {
  return (philox_block(seed, 3u, j, 0u).x & 1u) ? -1.0 : 1.0;
}
__device__ __forceinline__ int32_t sketch_bucket(uint64_t seed, int64_t j, int32_t s) {
  return (int32_t)(((uint64_t)philox_block(seed, 3u, j, 0u).y * (uint64_t)s) >> 32);
}
__device__ __forceinline__ int64_t hadamard_order(int64_t n) {
  int64_t N = 1;
  while (N < n) N <<= 1;
  return N;
}
// Entry (j, t) of D H S without the 1/sqrt(s) scale: D_jj (-1)^popcount(j & i_t).
__device__ __forceinline__ double srht_entry(uint64_t seed, int64_t j, int64_t t, int64_t N) {
  const int64_t col = (int64_t)((uint64_t)philox_block(seed, 4u, t, 0u).x % (uint64_t)N);
  return (__popcll((unsigned long long)(j & col)) & 1) ? -sketch_sign(seed, j) : sketch_sign(seed, j);
}

// ---------------------------------------------------------------------------
// wave64 reductions (fixed butterfly order: deterministic).  The exchanges are
// register moves (lane-group swaps between the rows of 16 lanes, DPP rotations
// within one) rather than trips through the LDS crossbar.  The order is that of
// the butterfly xor 32, 16, 8, 4, 2, 1: once the sums repeat every 2 k lanes, a
// rotation by k is the exchange with lane xor k.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// The sum of the two rows of 16 lanes of each half (xor 16), then of the two
// halves (xor 32).
__device__ __forceinline__ double sum_xor16(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return __longlong_as_double(((long long)h[0] << 32) | l[0]) + __longlong_as_double(((long long)h[1] << 32) | l[1]);
}
__device__ __forceinline__ double sum_xor32(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return __longlong_as_double(((long long)h[0] << 32) | l[0]) + __longlong_as_double(((long long)h[1] << 32) | l[1]);
}
// Per column of a 16 x 16 MFMA result: the four lanes l, l + 16, l + 32, l + 48.
__device__ __forceinline__ double column_sum(double v) { return sum_xor32(sum_xor16(v)); }
__device__ __forceinline__ double wave_sum(double v) {
  v = sum_xor16(sum_xor32(v));
  v += dpp_move<0x128>(v);  // row_ror:8
  v += dpp_move<0x124>(v);  // row_ror:4
  v += dpp_move<0x122>(v);  // row_ror:2
  v += dpp_move<0x121>(v);  // row_ror:1
  return v;
}

// ---------------------------------------------------------------------------
// MFMA 16x16x4 for FP64 and FP32.  Operand layout (per lane l of the wave):
//   A: row l%16, k-slot l/16      B: k-slot l/16, column l%16
//   D register r (r = 0..3), column l%16, row:
//     FP32: 4*(l/16) + r      FP64: (l/16) + 4*r
// (measured on gfx950 with a one-wave layout probe against a host product).
// ---------------------------------------------------------------------------
template <typename T>
struct Mfma16;

template <>
struct Mfma16<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int drow(int q, int r) { return q + 4 * r; }
  static __device__ __forceinline__ v4 mma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

template <>
struct Mfma16<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int drow(int q, int r) { return 4 * q + r; }
  static __device__ __forceinline__ v4 mma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// XCD-aware remap of a linear workgroup id: the hardware deals consecutive
// ids round-robin over the 8 XCDs; this gives each XCD a contiguous range of
// logical tiles so that tiles sharing operands share an L2.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
  if ((nb & 7) != 0) return b;
  return (b & 7) * (nb >> 3) + (b >> 3);
}

// ||x||^2 of the previous product from its block triples, on every thread (all
// threads of a block of 256 or 1024 call it; the order of power_reduce_body).
// Called behind the product, so the loads are the only cost.
__device__ __forceinline__ double power_prev_norm(const double *__restrict__ part, int32_t nblk) {
  __shared__ double red[16];
  double a = 0.0;
  if (threadIdx.x < 256)
    for (int i = threadIdx.x; i < nblk; i += 256) a += part[3 * i];
  a = wave_sum(a);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}
__device__ __forceinline__ double power_scale(const PowerPrev &p) {
  if (p.part) return 1.0 / sqrt(power_prev_norm(p.part, p.nblk));
  return p.norm ? 1.0 / sqrt(p.norm[0]) : 1.0;
}

// Tiles of a product with a symmetric R (128 x 128, 256 threads): tile t of the
// lower triangle, row by row (cb <= rb).
constexpr int kSymTile = 128;
__device__ __forceinline__ void sym_tile(int64_t t, int64_t &rb, int64_t &cb) {
  rb = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while (rb * (rb + 1) / 2 > t) --rb;
  while ((rb + 1) * (rb + 2) / 2 <= t) ++rb;
  cb = t - rb * (rb + 1) / 2;
}
// Sums of 16 values a lane over each of a wave's H lane groups (64 / H lanes),
// through LDS in place of 16 sums of six cross-lane steps: sum r is value r / H
// of group r % H, returned on the 4 / H lanes from r * 4 / H on.
template <int H>
__device__ __forceinline__ double sym_sums(const double (&val)[16], double (*buf)[65], int lane) {
#pragma unroll
  for (int i = 0; i < 16; ++i) buf[i][lane] = val[i];
  __builtin_amdgcn_wave_barrier();
  constexpr int LP = 4 / H;  // lanes that share a sum
  const int r = lane / LP, p = lane % LP;
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 16; ++c) s += buf[r / H][(r % H) * (64 / H) + c * LP + p];
  s += dpp_move<0xB1>(s);
  if (LP == 4) s += dpp_move<0x4E>(s);
  __builtin_amdgcn_wave_barrier();
  return s;
}

// Block sums of y^2, xs.y, xs^2 over the rows a block produced (fixed order).
__device__ __forceinline__ void block_power_partials(double yy, double xy, double xx,
                                                     double *part3, int64_t blk) {
  __shared__ double red[3][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  yy = wave_sum(yy);
  xy = wave_sum(xy);
  xx = wave_sum(xx);
  if (lane == 0) {
    red[0][w] = yy;
    red[1][w] = xy;
    red[2][w] = xx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = blockDim.x >> 6;
    double a = 0, b = 0, c = 0;
    for (int i = 0; i < nw; ++i) {
      a += red[0][i];
      b += red[1][i];
      c += red[2][i];
    }
    part3[3 * blk + 0] = a;
    part3[3 * blk + 1] = b;
    part3[3 * blk + 2] = c;
  }
}

// ---------------------------------------------------------------------------
// Persistent batch steps: taking items, waiting for a matrix's previous step,
// publishing a finished tile.  Items are taken from the segment of the XCD
// the workgroup runs on, and every item of a matrix runs on the same XCD, so
// a tile's stores reach the only L2 its consumers read through: publishing
// waits until this workgroup's stores are performed (vmcnt), then one thread
// moves the counter; waiting polls the counter, then invalidates at device
// scope, which drops this CU's L1 (lines that another CU of the XCD has since
// rewritten in L2) and never loses a dirty L2 line.  No L2 write-back is
// needed.  Counters are vector atomics.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int xcc_id() {
  return (int)(__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & (kMaxXcc - 1));  // HW_REG_XCC_ID[3:0]
}

// Next item index of this workgroup, or -1 when its XCD's segment is
// exhausted or a wait has failed.  sh: a __shared__ int of the calling kernel.
// In two parts: sched_reserve (thread 0's value counts) takes the place in the
// queue without waiting for it, sched_item waits and gives it to the workgroup.
// The loops around these begin with a convergent operation and branch on scalar
// values: a loop that began with thread 0's branch would let the compiler send
// the other lanes straight to the barrier behind it.  That it did not is checked
// on the built code (tests/test_kernel_code.py).
__device__ __forceinline__ int sched_reserve(const SchedArgs &s) {
  __builtin_amdgcn_wave_barrier();
  int q = 0;
  if (threadIdx.x == 0) {
    const int seg = s.seg_of_xcc[xcc_id()];
    // the address as a vector value: for one that the compiler knows to be
    // uniform it combines lanes, which waits for the result here
    int v = seg;
    asm("" : "+v"(v));
    if (seg >= 0) q = __hip_atomic_fetch_add(s.head + v, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __builtin_amdgcn_wave_barrier();
  return q;
}
__device__ __forceinline__ int sched_item(const SchedArgs &s, int q, int *sh) {
  __builtin_amdgcn_wave_barrier();
  if (threadIdx.x == 0) {
    int i = -1;
    const int seg = s.seg_of_xcc[xcc_id()];
    const int err = __hip_atomic_load(s.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (seg >= 0) {
      const int end = s.tail && *s.tail == 0 ? s.seg_mid[seg] : s.seg_off[seg + 1];
      if (q < end - s.seg_off[seg] && err == 0) i = s.seg_off[seg] + q;
    }
    *sh = i;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*sh);
}
__device__ __forceinline__ int sched_next(const SchedArgs &s, int *sh) {
  __syncthreads();  // every wave is done with the previous item (and with sh)
  return sched_item(s, sched_reserve(s), sh);
}

// A value of global memory that is the same for every lane, in scalar registers:
// behind stores of the same kernel the compiler loads through vector registers
// and takes every branch and address made from it for divergent.
template <typename T>
__device__ __forceinline__ T uniform_load(const T *p) {
  static_assert(sizeof(T) % 4 == 0, "whole dwords");
  T v = *p;
  int w[sizeof(T) / 4];
  __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
  __builtin_memcpy(&v, w, sizeof(T));
  return v;
}

// Waits until done[b] >= need; false (and *err set) after spin_limit polls.
__device__ __forceinline__ bool sched_wait(const SchedArgs &s, int b, int need, int *sh) {
  if (threadIdx.x == 0) {
    int ok = 1;
    int polls = 0;
    while (__hip_atomic_load(s.done + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
      if (__hip_atomic_load(s.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
          polls++ >= s.spin_limit) {
        __hip_atomic_fetch_or(s.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
    *sh = ok;
  }
  __syncthreads();
  asm volatile("buffer_inv sc1" ::: "memory");  // L1 of this CU (device scope: a group-scope invalidate may keep it)
  return __builtin_amdgcn_readfirstlane(*sh) != 0;
}

// Publishes one finished tile of matrix b.
__device__ __forceinline__ void sched_release(const SchedArgs &s, int b) {
  __builtin_amdgcn_s_waitcnt(0);  // this thread's stores of the tile are performed in L2
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(s.done + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Recurrence of step k of a batch: Chebyshev forward: V_1 = Y_0 - V_0 (g.g in
// slot 0), then V_{k+1} = 2 Y_k - 2 V_k - V_{k-1} written over V_{k-1}; Taylor:
// W_{k+1} = W_k - Y_k into alternating buffers, dots with Y_k; the last step
// writes nothing.  V_0 is the probe block.  Dots: slot k + 1 (Taylor: k), or in
// pairs slots 2k + 1 and 2k + 2 (2k and 2k + 1).
struct StepRule {
  double c1, c2, cw;
  int32_t dot_y, slot, slot_gg, slot_b;
  int vk, vkm1, vout;  // buffer ids: 0 = probe block, 1 = VA, 2 = VB, -1 = none
};
__device__ __forceinline__ StepRule step_rule(int32_t method, int32_t m, int32_t k, int32_t nsteps, bool pair) {
  StepRule r;
  const int out = 1 + (k & 1), prev = 1 + ((k - 1) & 1);
  const int32_t last = (pair ? (nsteps + 1) / 2 : nsteps) - 1;
  if (method == 1) {  // Chebyshev
    r.dot_y = 0;
    r.slot = pair ? 2 * k + 1 : k + 1;
    r.slot_b = pair && 2 * k + 2 <= m ? 2 * k + 2 : -1;
    if (k == 0) {
      r.c1 = 1.0; r.c2 = -1.0; r.cw = 0.0; r.slot_gg = 0;
      r.vk = 0; r.vkm1 = -1;
    } else {
      r.c1 = 2.0; r.c2 = -2.0; r.cw = -1.0; r.slot_gg = -1;
      r.vk = prev; r.vkm1 = k == 1 ? 0 : out;
    }
  } else {  // Taylor
    r.c1 = -1.0; r.c2 = 1.0; r.cw = 0.0;
    r.dot_y = 1; r.slot_gg = -1;
    r.slot = pair ? 2 * k : k;
    r.slot_b = pair && 2 * k + 1 <= m ? 2 * k + 1 : -1;
    r.vk = k == 0 ? 0 : prev;
    r.vkm1 = -1;
  }
  r.vout = k < last ? out : -1;
  return r;
}

// A matrix's dots come in pairs if it equals its transpose.
__device__ __forceinline__ bool batch_pairs(const BatchMat &M) {
  return __builtin_amdgcn_readfirstlane(*(const int32_t *)(M.scal + S_SYM)) == 0;  // one matrix per wave
}

}  // namespace ent
