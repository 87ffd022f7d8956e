// kernels_misc.hip -- probes, power method (Algorithm 4), interval and
// coefficient setup (Lemma 3), trace check, conversions and the final
// reductions of the Hutchinson estimate (Lemma 1, Algorithms 1-2).
#include "device_common.hpp"
#include "kernels.hpp"

namespace ent {

// ---------------------------------------------------------------------------
// Probe blocks
// ---------------------------------------------------------------------------
// One thread per (row, 32-probe word): Rademacher signs from one Philox word.
template <typename T>
__global__ void probe_rademacher_kernel(T *__restrict__ G, uint32_t *__restrict__ signs, int64_t n,
                                        int64_t n_pad, int32_t s, int64_t ldv, uint64_t seed) {
  const int32_t nw = (int32_t)(ldv >> 5);
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_pad * nw) return;
  const int64_t row = t / nw;
  const int32_t word = (int32_t)(t % nw);
  uint32_t bits = 0;
  uint32_t valid = 0;
  if (row < n) {
    bits = rademacher_word(seed, 0u, row, word);
    const int32_t lo = word * 32;
    valid = (s - lo >= 32) ? 0xffffffffu : (s > lo ? ((1u << (s - lo)) - 1u) : 0u);
  }
  if (signs && row < n) signs[row * nw + word] = bits & valid;
  if (G) {
    T *dst = G + row * ldv + (int64_t)word * 32;
#pragma unroll
    for (int b = 0; b < 32; ++b) {
      const bool on = (valid >> b) & 1u;
      dst[b] = on ? (((bits >> b) & 1u) ? T(-1) : T(1)) : T(0);
    }
  }
}

// Sign bits only: one thread per row (grid-stride), each Philox block
// giving four consecutive words of the row, the same bits as
// probe_rademacher_kernel.
__global__ __launch_bounds__(256) void sign_words_kernel(uint32_t *__restrict__ signs, int64_t n, int32_t s,
                                                         int32_t nw, uint64_t seed) {
  for (int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; row < n;
       row += (int64_t)gridDim.x * blockDim.x) {
    uint32_t *dst = signs + row * nw;
    for (int32_t blk = 0; 4 * blk < nw; ++blk) {
      const U4 o = philox_block(seed, 0u, row, (uint32_t)blk);
      const uint32_t w4[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int32_t word = 4 * blk + k;
        if (word >= nw) break;
        const int32_t lo = word * 32;
        const uint32_t valid = (s - lo >= 32) ? 0xffffffffu : (s > lo ? ((1u << (s - lo)) - 1u) : 0u);
        dst[word] = w4[k] & valid;
      }
    }
  }
}

template <typename T>
__global__ void probe_gaussian_kernel(T *__restrict__ G, int64_t n, int64_t n_pad, int32_t s,
                                      int64_t ldv, uint64_t seed) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_pad * ldv) return;
  const int64_t row = t / ldv;
  const int64_t j = t % ldv;
  G[t] = (row < n && j < s) ? (T)gaussian(seed, 0u, row, j) : T(0);
}

template <typename T>
hipError_t launch_probe_gen(T *G, uint32_t *signs, int64_t n, int64_t n_pad, int32_t s,
                            int64_t ldv, uint64_t seed, int32_t dist, hipStream_t st) {
  if (dist == 0) {
    const int64_t tot = n_pad * (ldv >> 5);
    probe_rademacher_kernel<T><<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(G, signs, n, n_pad, s,
                                                                             ldv, seed);
  } else {
    const int64_t tot = n_pad * ldv;
    probe_gaussian_kernel<T><<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(G, n, n_pad, s, ldv, seed);
  }
  return hipGetLastError();
}
template hipError_t launch_probe_gen<double>(double *, uint32_t *, int64_t, int64_t, int32_t,
                                             int64_t, uint64_t, int32_t, hipStream_t);
template hipError_t launch_probe_gen<float>(float *, uint32_t *, int64_t, int64_t, int32_t,
                                            int64_t, uint64_t, int32_t, hipStream_t);

hipError_t launch_sign_gen(uint32_t *signs, int64_t n, int32_t s, int64_t ldv, uint64_t seed,
                           hipStream_t st) {
  if (n < 1 || !signs || ldv % 32 != 0) return hipErrorInvalidValue;
  const int64_t b = (n + 255) / 256;
  sign_words_kernel<<<(unsigned)(b < 8192 ? b : 8192), 256, 0, st>>>(signs, n, s, (int32_t)(ldv >> 5), seed);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Power method
// ---------------------------------------------------------------------------
__global__ void power_start_kernel(double *__restrict__ x, int64_t n, uint64_t seed, int32_t trial) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = rademacher(seed, 1u, i, trial);
}

hipError_t launch_power_start(double *x, int64_t n, uint64_t seed, int32_t trial, hipStream_t st) {
  power_start_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(x, n, seed, trial);
  return hipGetLastError();
}

// Dense y = (R x)/||x_prev||.
// Each wave owns 2 consecutive rows; lanes stride over 16-byte vectors of
// both rows, two vectors in flight per row (FP64 accumulation).
template <typename T>
__device__ __forceinline__ void power_gemv_body(const T *__restrict__ R, int64_t ldr, int64_t n,
                                                const double *__restrict__ x, const PowerPrev &prev,
                                                double *__restrict__ y, double *__restrict__ part3,
                                                int64_t blk) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int VEC = 16 / sizeof(T);
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  const int64_t r0 = (blk * 4 + w) * 2;
  const bool ok0 = r0 < n, ok1 = r0 + 1 < n;
  const T *R0 = R + (ok0 ? r0 : 0) * ldr;
  const T *R1 = R + (ok1 ? r0 + 1 : 0) * ldr;
  double a0 = 0.0, a1 = 0.0, b0 = 0.0, b1 = 0.0;
  const int64_t nvec = n / VEC;
  int64_t v = lane;
  for (; v + 64 < nvec; v += 128) {
    const int64_t k = v * VEC, k2 = (v + 64) * VEC;
    vec_t p0 = {}, p1 = {}, q0 = {}, q1 = {};
    if (ok0) {
      p0 = *(const vec_t *)(R0 + k);
      q0 = *(const vec_t *)(R0 + k2);
    }
    if (ok1) {
      p1 = *(const vec_t *)(R1 + k);
      q1 = *(const vec_t *)(R1 + k2);
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const double xe = x[k + e], xf = x[k2 + e];
      a0 += (double)p0[e] * xe;
      a1 += (double)p1[e] * xe;
      b0 += (double)q0[e] * xf;
      b1 += (double)q1[e] * xf;
    }
  }
  for (; v < nvec; v += 64) {
    const int64_t k = v * VEC;
    vec_t p0 = {}, p1 = {};
    if (ok0) p0 = *(const vec_t *)(R0 + k);
    if (ok1) p1 = *(const vec_t *)(R1 + k);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      a0 += (double)p0[e] * x[k + e];
      a1 += (double)p1[e] * x[k + e];
    }
  }
  for (int64_t k = nvec * VEC + lane; k < n; k += 64) {
    if (ok0) a0 += (double)R0[k] * x[k];
    if (ok1) a1 += (double)R1[k] * x[k];
  }
  const double s0 = wave_sum(a0 + b0), s1 = wave_sum(a1 + b1);
  const double sc = power_scale(prev);
  double yy = 0.0, xy = 0.0, xx = 0.0;
  if (lane == 0) {
    if (ok0) {
      const double yv = sc * s0, xs = sc * x[r0];
      y[r0] = yv;
      yy += yv * yv;
      xy += xs * yv;
      xx += xs * xs;
    }
    if (ok1) {
      const double yv = sc * s1, xs = sc * x[r0 + 1];
      y[r0 + 1] = yv;
      yy += yv * yv;
      xy += xs * yv;
      xx += xs * xs;
    }
  }
  block_power_partials(yy, xy, xx, part3, blk);
}

template <typename T>
__global__ __launch_bounds__(256) void power_gemv_kernel(const T *__restrict__ R, int64_t ldr,
                                                         int64_t n, const double *__restrict__ x,
                                                         PowerPrev prev, double *__restrict__ y,
                                                         double *__restrict__ part3) {
  power_gemv_body<T>(R, ldr, n, x, prev, y, part3, blockIdx.x);
}

// The same product from half of an R that equals its transpose: a workgroup
// reads a 128 x 128 tile on or below the diagonal once and leaves its row sums
// A x_J in part[J][rows of I] and its column sums A^T x_I in part[I][columns of
// J]; power_sym_combine_kernel adds the n / 128 parts of a row in order.
// Consecutive workgroups take consecutive tiles of a row of tiles.  Bound by
// HBM (the combination adds 4 us): n = 8192, FP64 103 -> 50 us a product, FP32
// 48 -> 28; more at power_sym_pays.
template <typename T>
__device__ __forceinline__ void power_sym_body(const T *__restrict__ R, int64_t ldr, int64_t n,
                                               const double *__restrict__ x, double *__restrict__ part, int64_t rb,
                                               int64_t cb, bool cols) {
  constexpr int VEC = 16 / sizeof(T), LPR = kSymTile / VEC, H = 64 / LPR;  // lanes per row, rows at a time
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  __shared__ double buf[4][16][65];
  __shared__ double xr[kSymTile];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int half = lane / LPR, cl = (lane % LPR) * VEC;
  const int64_t c0 = cb * kSymTile + cl, w0 = rb * kSymTile + 32 * w;
  if (tid < kSymTile) xr[tid] = rb * kSymTile + tid < n ? x[rb * kSymTile + tid] : 0.0;
  __syncthreads();
  double xc[VEC], cacc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    xc[e] = c0 + e < n ? x[c0 + e] : 0.0;
    cacc[e] = 0.0;
  }
  // a tile that reaches beyond n reads row n - 1 and column 0 there (x is zero
  // in xr and xc, the row sums are not stored), and a vector across n one by one
  const bool inside = rb * kSymTile + kSymTile <= n && cb * kSymTile + kSymTile <= n;
  const bool whole = c0 + VEC <= n;
#pragma unroll 1
  for (int ch = 0; ch < 2 / H; ++ch) {  // 16 H rows at a time
    const int row0 = 32 * w + ch * 16 * H + half;
    const T *Rr = R + (rb * kSymTile + row0) * ldr + c0;
    double racc[16];
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += 8) {
      vec_t v[8];
      if (inside) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = *(const vec_t *)(Rr + (int64_t)(i0 + i) * H * ldr);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int64_t r = rb * kSymTile + row0 + (i0 + i) * H;
          v[i] = *(const vec_t *)(R + (r < n ? r : n - 1) * ldr + (whole ? c0 : 0));
        }
        if (!whole && c0 < n) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int64_t r = rb * kSymTile + row0 + (i0 + i) * H;
#pragma unroll
            for (int e = 0; e < VEC; ++e)
              if (c0 + e < n) v[i][e] = R[(r < n ? r : n - 1) * ldr + c0 + e];
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const double xv = xr[row0 + (i0 + i) * H];
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          s += (double)v[i][e] * xc[e];
          cacc[e] += (double)v[i][e] * xv;
        }
        racc[i0 + i] = s;
      }
    }
    const double s = sym_sums<H>(racc, buf[w], lane);
    const int64_t r = w0 + ch * 16 * H + lane / (4 / H);
    if (lane % (4 / H) == 0 && r < n) part[cb * n + r] = s;
  }
  if (cols) {
    double(*cs)[kSymTile] = (double(*)[kSymTile])buf;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      double s = cacc[e];
      if (H == 2) s += __shfl_xor(s, 32, 64);
      if (half == 0) cs[w][cl + e] = s;
    }
    __syncthreads();
    if (tid < kSymTile && cb * kSymTile + tid < n)
      part[rb * n + cb * kSymTile + tid] = cs[0][tid] + cs[1][tid] + cs[2][tid] + cs[3][tid];
  }
}

template <typename T>
__global__ __launch_bounds__(256) void power_sym_part_kernel(const T *__restrict__ R, int64_t ldr, int64_t n,
                                                             const double *__restrict__ x,
                                                             double *__restrict__ part) {
  int64_t rb, cb;
  sym_tile(blockIdx.x, rb, cb);
  power_sym_body<T>(R, ldr, n, x, part, rb, cb, rb != cb);
}

// y = sum of the parts (stride rows apart), scaled; 64 rows a workgroup, each
// wave a quarter of the parts.
__device__ __forceinline__ void power_sym_sum(const double *__restrict__ part, int32_t nparts, int64_t stride,
                                              int64_t n, const double *__restrict__ x, const PowerPrev &prev,
                                              double *__restrict__ y, double *__restrict__ part3, int64_t blk) {
  __shared__ double sums[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t r = blk * 64 + lane;
  const int32_t p0 = nparts * w / 4, p1 = nparts * (w + 1) / 4;
  double s = 0.0;
  if (r < n) {
#pragma unroll 8
    for (int32_t p = p0; p < p1; ++p) s += part[p * stride + r];
  }
  sums[w][lane] = s;
  const double sc = power_scale(prev);
  __syncthreads();
  double yy = 0.0, xy = 0.0, xx = 0.0;
  if (w == 0 && r < n) {
    const double yv = sc * (sums[0][lane] + sums[1][lane] + sums[2][lane] + sums[3][lane]), xs = sc * x[r];
    y[r] = yv;
    yy = yv * yv;
    xy = xs * yv;
    xx = xs * xs;
  }
  block_power_partials(yy, xy, xx, part3, blk);
}

__global__ __launch_bounds__(256) void power_sym_combine_kernel(const double *__restrict__ part, int32_t nparts,
                                                                int64_t stride, int64_t n,
                                                                const double *__restrict__ x, PowerPrev prev,
                                                                double *__restrict__ y,
                                                                double *__restrict__ part3) {
  power_sym_sum(part, nparts, stride, n, x, prev, y, part3, blockIdx.x);
}

int32_t power_blocks_sym(int64_t n) { return (int32_t)((n + 63) / 64); }
int64_t power_sym_parts(int64_t n) { return (n + kSymTile - 1) / kSymTile; }

hipError_t launch_power_sym_combine(const double *part, int64_t nparts, int64_t stride, int64_t n, const double *x,
                                    const PowerPrev &prev, double *y, double *part3, int32_t *nblk, hipStream_t st) {
  if (prev.part == part3) return hipErrorInvalidValue;  // read while this product's are written
  *nblk = power_blocks_sym(n);
  power_sym_combine_kernel<<<(unsigned)*nblk, 256, 0, st>>>(part, (int32_t)nparts, stride, n, x, prev, y, part3);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_power_sym(const T *R, int64_t ldr, int64_t n, const double *x, const PowerPrev &prev, double *y,
                            double *part3, double *part, int32_t *nblk, hipStream_t st) {
  const int64_t nb = power_sym_parts(n);
  power_sym_part_kernel<T><<<(unsigned)(nb * (nb + 1) / 2), 256, 0, st>>>(R, ldr, n, x, part);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_power_sym_combine(part, nb, n, n, x, prev, y, part3, nblk, st);
}
template hipError_t launch_power_sym<double>(const double *, int64_t, int64_t, const double *, const PowerPrev &,
                                             double *, double *, double *, int32_t *, hipStream_t);
template hipError_t launch_power_sym<float>(const float *, int64_t, int64_t, const double *, const PowerPrev &,
                                            double *, double *, double *, int32_t *, hipStream_t);

int32_t power_blocks_dense(int64_t n) { return (int32_t)((n + 7) / 8); }
// At most kPowerSelfSum workgroups, so that the next product sums the triples:
// n = 200000, 20.6 entries a row, FP64 24 us in 4096 workgroups and 5.9 for the
// sum, 26 us in 1024 without one; n = 40000 an estimate of 20 products 840 -> 795.
int32_t power_blocks_spmv(int64_t n) {
  const int64_t b = (n + 31) / 32;
  return (int32_t)(b < kPowerSelfSum ? b : kPowerSelfSum);
}
int32_t power_blocks_csr(int64_t n) {
  const int64_t b = (n + 31) / 32;
  return (int32_t)(b < 4096 ? b : 4096);
}

template <typename T>
hipError_t launch_power_gemv(const T *R, int64_t ldr, int64_t n, const double *x,
                             const PowerPrev &prev, double *y, double *part3, int32_t *nblk,
                             hipStream_t st) {
  if (prev.part == part3) return hipErrorInvalidValue;  // read while this product's are written
  const int32_t blocks = power_blocks_dense(n);
  *nblk = blocks;
  power_gemv_kernel<T><<<(unsigned)blocks, 256, 0, st>>>(R, ldr, n, x, prev, y, part3);
  return hipGetLastError();
}
template hipError_t launch_power_gemv<double>(const double *, int64_t, int64_t, const double *,
                                              const PowerPrev &, double *, double *, int32_t *,
                                              hipStream_t);
template hipError_t launch_power_gemv<float>(const float *, int64_t, int64_t, const double *,
                                             const PowerPrev &, double *, double *, int32_t *,
                                             hipStream_t);

// CSR: L lanes per row (L = 1, 2, 4 or 8 by the mean row length), 256 / L
// rows per block per pass, persistent grid-stride over row groups (one
// partial triple per block).
template <typename T, int L>
__global__ __launch_bounds__(256) void power_spmv_kernel(const int64_t *__restrict__ rp,
                                                         const int32_t *__restrict__ ci,
                                                         const T *__restrict__ val, int64_t n,
                                                         const double *__restrict__ x, PowerPrev prev,
                                                         double *__restrict__ y,
                                                         double *__restrict__ part3) {
  constexpr int RPB = 256 / L;  // rows per block per pass
  double sc = 0.0;  // found behind the first rows' products
  const int sub = threadIdx.x % L;
  double yy = 0.0, xy = 0.0, xx = 0.0;
  for (int64_t base = (int64_t)blockIdx.x * RPB; base < n; base += (int64_t)gridDim.x * RPB) {
    const int64_t row = base + threadIdx.x / L;
    double acc = 0.0;
    if (row < n) {
      const int64_t e1 = rp[row + 1];
      for (int64_t e = rp[row] + sub; e < e1; e += L) acc += (double)val[e] * x[ci[e]];
    }
#pragma unroll
    for (int off = L / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (base == (int64_t)blockIdx.x * RPB) sc = power_scale(prev);
    if (row < n && sub == 0) {
      const double yv = sc * acc;
      const double xs = sc * x[row];
      y[row] = yv;
      yy += yv * yv;
      xy += xs * yv;
      xx += xs * xs;
    }
  }
  block_power_partials(yy, xy, xx, part3, blockIdx.x);
}

template <typename T>
hipError_t launch_power_spmv(const int64_t *rp, const int32_t *ci, const T *val, int64_t n,
                             int64_t nnz, const double *x, const PowerPrev &prev, double *y,
                             double *part3, int32_t *nblk, hipStream_t st) {
  if (prev.part == part3) return hipErrorInvalidValue;  // read while this product's are written
  const int32_t blocks = power_blocks_spmv(n);
  *nblk = blocks;
  const double avg = n > 0 ? (double)nnz / (double)n : 0.0;
  if (avg <= 1.5)
    power_spmv_kernel<T, 1><<<(unsigned)blocks, 256, 0, st>>>(rp, ci, val, n, x, prev, y, part3);
  else if (avg <= 3.0)
    power_spmv_kernel<T, 2><<<(unsigned)blocks, 256, 0, st>>>(rp, ci, val, n, x, prev, y, part3);
  else if (avg <= 6.0)
    power_spmv_kernel<T, 4><<<(unsigned)blocks, 256, 0, st>>>(rp, ci, val, n, x, prev, y, part3);
  else
    power_spmv_kernel<T, 8><<<(unsigned)blocks, 256, 0, st>>>(rp, ci, val, n, x, prev, y, part3);
  return hipGetLastError();
}
template hipError_t launch_power_spmv<double>(const int64_t *, const int32_t *, const double *,
                                              int64_t, int64_t, const double *, const PowerPrev &,
                                              double *, double *, int32_t *, hipStream_t);
template hipError_t launch_power_spmv<float>(const int64_t *, const int32_t *, const float *,
                                             int64_t, int64_t, const double *, const PowerPrev &,
                                             double *, double *, int32_t *, hipStream_t);

// Fixed-order sum of the block triples of one product into norm3[0..2].
__device__ __forceinline__ void power_reduce_body(const double *__restrict__ part3, int32_t nblk,
                                                  double *__restrict__ norm3) {
  __shared__ double red[3][4];
  double a = 0.0, b = 0.0, c = 0.0;
  for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
    a += part3[3 * i];
    b += part3[3 * i + 1];
    c += part3[3 * i + 2];
  }
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    red[0][w] = a;
    red[1][w] = b;
    red[2][w] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    norm3[0] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    norm3[1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    norm3[2] = red[2][0] + red[2][1] + red[2][2] + red[2][3];
  }
}

__global__ __launch_bounds__(256) void power_reduce_kernel(const double *__restrict__ part3,
                                                           int32_t nblk, double *__restrict__ norm3) {
  power_reduce_body(part3, nblk, norm3);
}

hipError_t launch_power_reduce(const double *part3, int32_t nblk, double *norm3, hipStream_t st) {
  power_reduce_kernel<<<1, 256, 0, st>>>(part3, nblk, norm3);
  return hipGetLastError();
}

// Rayleigh quotient of a trial from the reduced triple of its final product;
// scal[S_P1] keeps the maximum over trials (trial 0 overwrites).
__device__ __forceinline__ void power_rq_body(double *__restrict__ scal,
                                              const double *__restrict__ norm3, int32_t trial) {
  if (threadIdx.x == 0) {
    const double rq = norm3[1] / norm3[2];
    if (trial == 0 || rq > scal[S_P1]) scal[S_P1] = rq;
  }
}

__global__ void power_rq_kernel(double *__restrict__ scal, const double *__restrict__ norm3,
                                int32_t trial) {
  power_rq_body(scal, norm3, trial);
}

__global__ __launch_bounds__(256) void power_rq_sum_kernel(double *__restrict__ scal,
                                                           const double *__restrict__ part3, int32_t nblk,
                                                           int32_t trial) {
  __shared__ double norm3[3];
  power_reduce_body(part3, nblk, norm3);
  power_rq_body(scal, norm3, trial);  // by the thread that wrote norm3
}

hipError_t launch_power_rq_sum(double *scal, const double *part3, int32_t nblk, int32_t trial, hipStream_t st) {
  power_rq_sum_kernel<<<1, 256, 0, st>>>(scal, part3, nblk, trial);
  return hipGetLastError();
}

hipError_t launch_power_rq(double *scal, const double *norm3, int32_t trial, hipStream_t st) {
  power_rq_kernel<<<1, 64, 0, st>>>(scal, norm3, trial);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Interval [lo, u] and Chebyshev coefficients
// ---------------------------------------------------------------------------
__device__ __forceinline__ void setup_interval_body(double *__restrict__ scal, int32_t method,
                                                    int32_t m, double c, double u_fixed, double lo,
                                                    double norm_div) {
  __shared__ double su;
  if (threadIdx.x == 0) {
    // R / tr R (problem statement, unit trace): every eigenvalue, hence p~1,
    // and every product R v are scaled by 1 / tr R
    double nm = 1.0;
    if (norm_div > 0.0) {
      const double tr = scal[S_TRACE] / norm_div;
      nm = 1.0 / tr;
      if (!(tr > 0.0) || !isfinite(nm)) {
        scal[S_FLAG] = 1.0;
        nm = 1.0;
      }
      scal[S_NORM] = nm;
      if (!(u_fixed > 0.0)) scal[S_P1] *= nm;
    }
    double u;
    if (u_fixed > 0.0) {
      u = u_fixed;
    } else {
      const double p1 = scal[S_P1];
      if (!(p1 > 0.0) || !isfinite(p1)) scal[S_FLAG] = 1.0;
      u = fmin(1.0, c * p1);
    }
    if (!(u > lo)) scal[S_FLAG] = 1.0;
    scal[S_U] = u;
    scal[S_LO] = lo;
    if (method == 0) {  // Taylor: A = R/u, C = I - A
      scal[S_A] = nm / u;
      scal[S_B] = 1.0;
    } else {  // Chebyshev: X = a R - b I maps [lo, u] onto [-1, 1]
      scal[S_A] = nm * 2.0 / (u - lo);
      scal[S_B] = (u + lo) / (u - lo);
    }
    su = u;
  }
  __syncthreads();
  if (method != 1) return;
  const double u = su;
  if (lo == 0.0) {
    for (int w = threadIdx.x; w <= m; w += blockDim.x) {
      // Lemma 3: alpha_0 = (u/2)(ln(u/4)+1), alpha_1 = (u/4)(2 ln(u/4)+3),
      // alpha_w = (-1)^w u / (w^3 - w)
      double a;
      if (w == 0) {
        a = 0.5 * u * (log(0.25 * u) + 1.0);
      } else if (w == 1) {
        a = 0.25 * u * (2.0 * log(0.25 * u) + 3.0);
      } else {
        const double dw = (double)w;
        a = ((w & 1) ? -u : u) / (dw * dw * dw - dw);
      }
      scal[S_ALPHA + w] = a;
    }
    return;
  }
  // Chebyshev projection of x ln x on [lo, u] by an N-point Gauss-Chebyshev
  // rule, N = 1024 (2(m+1) beyond degree 511): independent of m, so the partial
  // sums over the degree are nested.  The function's values at up to kNodes
  // nodes at a time stand in LDS and a wave sums a coefficient, its cosines
  // cos(w th_i) = cos(pi j / 2N), j = w (2i + 1) mod 4N, from a table where N is
  // kNodes (one thread per coefficient and a logarithm and two cosines per node:
  // 518 us at m = 40, now 11).
  constexpr int kNodes = 1024;
  __shared__ double hx[kNodes], table[4 * kNodes];
  const int N = (m + 1) <= 512 ? kNodes : 2 * (m + 1);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if (N == kNodes) {
    for (int j = threadIdx.x; j < 4 * kNodes; j += blockDim.x) table[j] = cospi((double)j / (2.0 * kNodes));
    __syncthreads();
  }
  auto cosine = [&](int64_t j) {
    j %= 4 * (int64_t)N;
    return N == kNodes ? table[j] : cospi((double)j / (2.0 * (double)N));
  };
  for (int base = 0; base < N; base += kNodes) {
    const int nodes = N - base < kNodes ? N - base : kNodes;
    for (int i = threadIdx.x; i < nodes; i += blockDim.x) {
      const double x = 0.5 * (u + lo) + 0.5 * (u - lo) * cosine(2 * (base + i) + 1);
      hx[i] = x > 0.0 ? x * log(x) : 0.0;
    }
    __syncthreads();
    for (int w = wv; w <= m; w += nw) {
      double acc = 0.0;
      for (int i = lane; i < nodes; i += 64) acc += hx[i] * cosine((int64_t)w * (2 * (base + i) + 1));
      acc = wave_sum(acc);
      if (lane == 0) {
        if (base > 0) acc += scal[S_ALPHA + w];
        if (base + kNodes >= N) acc *= (w == 0 ? 1.0 : 2.0) / (double)N;
        scal[S_ALPHA + w] = acc;
      }
    }
    __syncthreads();
  }
}
__global__ __launch_bounds__(1024) void setup_interval_kernel(double *__restrict__ scal, int32_t method, int32_t m,
                                      double c, double u_fixed, double lo, double norm_div) {
  setup_interval_body(scal, method, m, c, u_fixed, lo, norm_div);
}

hipError_t launch_setup_interval(double *scal, int32_t method, int32_t m, double c, double u_fixed,
                                 double lo, hipStream_t st, double norm_div) {
  setup_interval_kernel<<<1, lo == 0.0 ? 256 : 1024, 0, st>>>(scal, method, m, c, u_fixed, lo, norm_div);
  return hipGetLastError();
}

__global__ void set_norm_kernel(double *__restrict__ scal, double norm_div) {
  if (threadIdx.x != 0) return;
  const double tr = scal[S_TRACE] / norm_div;
  const double nm = 1.0 / tr;
  if (!(tr > 0.0) || !isfinite(nm)) {
    scal[S_FLAG] = 1.0;
    scal[S_NORM] = 1.0;
  } else {
    scal[S_NORM] = nm;
  }
}

hipError_t launch_set_norm(double *scal, double norm_div, hipStream_t st) {
  set_norm_kernel<<<1, 64, 0, st>>>(scal, norm_div);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Trace of R (input contract: unit trace)
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void trace_dense_body(const T *__restrict__ R, int64_t ldr, int64_t n,
                                                 double *__restrict__ scal) {
  __shared__ double red[4];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) acc += (double)R[i * ldr + i];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) scal[S_TRACE] = red[0] + red[1] + red[2] + red[3];
}

template <typename T>
__global__ void trace_dense_kernel(const T *__restrict__ R, int64_t ldr, int64_t n,
                                   double *__restrict__ scal) {
  trace_dense_body<T>(R, ldr, n, scal);
}

// The diagonal of a large matrix touches a page per element: with room for the
// partial sums, 256 elements a workgroup (n = 32768: 77 us by one workgroup,
// 6 by 128 and the sum of theirs).
template <typename T>
__global__ __launch_bounds__(256) void trace_part_kernel(const T *__restrict__ R, int64_t ldr, int64_t n,
                                                         double *__restrict__ tmp) {
  __shared__ double red[4];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const double acc = wave_sum(i < n ? (double)R[i * ldr + i] : 0.0);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) tmp[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

template <typename T>
hipError_t launch_trace_dense(const T *R, int64_t ldr, int64_t n, double *scal, hipStream_t st, double *tmp,
                              int64_t room) {
  const int64_t nb = (n + 255) / 256;
  if (nb > 4 && nb <= room) {
    trace_part_kernel<T><<<(unsigned)nb, 256, 0, st>>>(R, ldr, n, tmp);
    trace_dense_kernel<double><<<1, 256, 0, st>>>(tmp, 0, nb, scal);
  } else {
    trace_dense_kernel<T><<<1, 256, 0, st>>>(R, ldr, n, scal);
  }
  return hipGetLastError();
}
template hipError_t launch_trace_dense<double>(const double *, int64_t, int64_t, double *, hipStream_t, double *, int64_t);
template hipError_t launch_trace_dense<float>(const float *, int64_t, int64_t, double *, hipStream_t, double *, int64_t);

// Tile t of the triangle: columns of tiles bj, in each the tiles bi <= bj.
__device__ __forceinline__ void check_tile(int64_t t, int64_t &bi, int64_t &bj) {
  bj = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while (bj * (bj + 1) / 2 > t) --bj;
  while ((bj + 1) * (bj + 2) / 2 <= t) ++bj;
  bi = t - bj * (bj + 1) / 2;
}

// Trace and symmetry in one pass over R (HBM-bound: every element is read
// once).  A workgroup takes a 64 x 64 tile (bi, bj),
// bi <= bj, and its mirror image, both read along rows; the tile is compared
// with the mirror's transpose through LDS (rows padded by one element: no
// bank conflicts down a column).  Diagonal tiles leave their part of the
// trace in tmp[bi].
template <typename T>
__device__ __forceinline__ bool dense_check_tile(const T *__restrict__ R, int64_t ldr, int64_t n, int64_t t,
                                                 T (*tile)[65], double *__restrict__ tmp) {
  int64_t bi, bj;
  check_tile(t, bi, bj);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t r0 = 64 * bi, c0 = 64 * bj;
  T x[16], y[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t r = r0 + 16 * w + i, c = c0 + lane;  // (r, c) of the tile
    x[i] = r < n && c < n ? R[r * ldr + c] : T(0);
    const int64_t rm = c0 + 16 * w + i, cm = r0 + lane;  // of the mirror
    y[i] = rm < n && cm < n ? R[rm * ldr + cm] : T(0);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) tile[16 * w + i][lane] = x[i];
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (!(tile[lane][16 * w + i] == y[i])) bad = true;  // also where either is NaN
  if (tmp && bi == bj && w == 0) {
    const double d = wave_sum((double)tile[lane][lane]);
    if (lane == 0) tmp[bi] = d;
  }
  return __any(bad) != 0;
}

// Sets a flag that many waves may set to the same value, for later kernels: a
// store, where atomics would take turns at its address (12 ns each).
__device__ __forceinline__ void raise_flag(int32_t *p) {
  __hip_atomic_store(p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// An R that rounding has made unequal to its transpose everywhere is read only
// by the workgroups that start before the first mismatch is known; the later ones
// leave their part of the trace (n = 8192 FP64 391 us when every wave set the flag
// by an atomic, 21 now; 4096 FP32 100 and 13; 93 and 13 for an R equal to its
// transpose, with this or without).  The first kCheckFirst workgroups start
// together and need not look.
constexpr unsigned kCheckFirst = 1024;

template <typename T>
__global__ __launch_bounds__(256) void dense_check_kernel(const T *__restrict__ R, int64_t ldr, int64_t n,
                                                          double *__restrict__ tmp, int32_t *__restrict__ asym) {
  __shared__ T tile[64][65];
  if (blockIdx.x >= kCheckFirst && __syncthreads_or(*(volatile int32_t *)asym) != 0) {
    int64_t bi, bj;
    check_tile(blockIdx.x, bi, bj);
    if (bi != bj || threadIdx.x >= 64) return;
    const int64_t r = 64 * bi + threadIdx.x;
    const double d = wave_sum(r < n ? (double)R[r * ldr + r] : 0.0);
    if (threadIdx.x == 0) tmp[bi] = d;
    return;
  }
  if (dense_check_tile<T>(R, ldr, n, blockIdx.x, tile, tmp) && (threadIdx.x & 63) == 0) raise_flag(asym);
}

// Batch: the tiles of matrix blockIdx.y dealt to the workgroups of its row of
// the grid; a mismatch marks the matrix and the batch.
template <typename T>
__global__ __launch_bounds__(256) void batch_check_kernel(const BatchMat *__restrict__ mats, int32_t *tail) {
  __shared__ T tile[64][65];
  const BatchMat &M = mats[blockIdx.y];
  const int64_t nb = (M.n + 63) / 64, nt = nb * (nb + 1) / 2;
  for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
    // a workgroup ends with the first tile that has a mismatch
    if (__syncthreads_or(dense_check_tile<T>((const T *)M.R, M.ldr, M.n, t, tile, nullptr))) {
      if (threadIdx.x == 0) {
        raise_flag((int32_t *)(M.scal + S_SYM));
        raise_flag(tail);
      }
      return;
    }
  }
}

template <typename T>
hipError_t launch_batch_check(const BatchMat *mats, int32_t count, int64_t max_n, int32_t *tail, hipStream_t st) {
  const int64_t nb = (max_n + 63) / 64, nt = nb * (nb + 1) / 2;
  dim3 grid((unsigned)(nt < 128 ? nt : 128), (unsigned)count);
  batch_check_kernel<T><<<grid, 256, 0, st>>>(mats, tail);
  return hipGetLastError();
}
template hipError_t launch_batch_check<double>(const BatchMat *, int32_t, int64_t, int32_t *, hipStream_t);
template hipError_t launch_batch_check<float>(const BatchMat *, int32_t, int64_t, int32_t *, hipStream_t);

__global__ __launch_bounds__(256) void check_finish_kernel(const double *__restrict__ tmp, int32_t cnt,
                                                                 double *__restrict__ scal,
                                                                 int32_t *__restrict__ host_flag) {
  __shared__ double red[4];
  double acc = 0.0;
  for (int i = threadIdx.x; i < cnt; i += 256) acc += tmp[i];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x != 0) return;
  scal[S_TRACE] = red[0] + red[1] + red[2] + red[3];
  if (host_flag) {
    *host_flag = *(const int32_t *)(scal + S_SYM);
    __threadfence_system();
  }
}

hipError_t launch_check_finish(const double *tmp, int32_t cnt, double *scal, int32_t *host_flag, hipStream_t st) {
  check_finish_kernel<<<1, 256, 0, st>>>(tmp, cnt, scal, host_flag);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_dense_check(const T *R, int64_t ldr, int64_t n, double *scal, int32_t *host_flag,
                              hipStream_t st) {
  // tile traces in the scratch tail of the scalar block (4096 doubles)
  const int64_t nb = (n + 63) / 64;
  if (n < 1 || nb > 4096) return hipErrorInvalidValue;
  double *tmp = scal + 4096;
  dense_check_kernel<T><<<(unsigned)(nb * (nb + 1) / 2), 256, 0, st>>>(R, ldr, n, tmp, (int32_t *)(scal + S_SYM));
  return launch_check_finish(tmp, (int32_t)nb, scal, host_flag, st);
}
template hipError_t launch_dense_check<double>(const double *, int64_t, int64_t, double *, int32_t *, hipStream_t);
template hipError_t launch_dense_check<float>(const float *, int64_t, int64_t, double *, int32_t *, hipStream_t);

// CSR: diagonal entries found by a scan of each row, L lanes per row (L by
// the mean row length, as in the power-method product) so that a row's
// column indices are read together; per-block partials are combined by the
// last pass in block order.
template <typename T, int L>
__global__ __launch_bounds__(256) void trace_csr_partial_kernel(const int64_t *__restrict__ rp,
                                                                const int32_t *__restrict__ ci,
                                                                const T *__restrict__ val, int64_t n,
                                                                double *__restrict__ tmp) {
  constexpr int RPB = 256 / L;
  __shared__ double red[4];
  const int sub = threadIdx.x % L;
  double acc = 0.0;
  for (int64_t base = (int64_t)blockIdx.x * RPB; base < n; base += (int64_t)gridDim.x * RPB) {
    const int64_t row = base + threadIdx.x / L;
    if (row < n) {
      const int64_t e1 = rp[row + 1];
      for (int64_t e = rp[row] + sub; e < e1; e += L)
        if (ci[e] == row) acc += (double)val[e];
    }
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) tmp[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ void sum_to_slot_kernel(const double *__restrict__ tmp, int32_t cnt, double *dst) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < cnt; i += 64) acc += tmp[i];
  acc = wave_sum(acc);
  if (threadIdx.x == 0) *dst = acc;
}

template <typename T>
hipError_t launch_trace_csr(const int64_t *rp, const int32_t *ci, const T *val, int64_t n,
                            int64_t nnz, double *scal, hipStream_t st) {
  // scal has room after the coefficient area: use a scratch tail of 1024 doubles
  double *tmp = scal + 4096;
  const int blocks = 1024;
  const double avg = n > 0 ? (double)nnz / (double)n : 0.0;
  if (avg <= 1.5)
    trace_csr_partial_kernel<T, 1><<<blocks, 256, 0, st>>>(rp, ci, val, n, tmp);
  else if (avg <= 3.0)
    trace_csr_partial_kernel<T, 2><<<blocks, 256, 0, st>>>(rp, ci, val, n, tmp);
  else if (avg <= 6.0)
    trace_csr_partial_kernel<T, 4><<<blocks, 256, 0, st>>>(rp, ci, val, n, tmp);
  else
    trace_csr_partial_kernel<T, 8><<<blocks, 256, 0, st>>>(rp, ci, val, n, tmp);
  sum_to_slot_kernel<<<1, 64, 0, st>>>(tmp, blocks, scal + S_TRACE);
  return hipGetLastError();
}
template hipError_t launch_trace_csr<double>(const int64_t *, const int32_t *, const double *,
                                             int64_t, int64_t, double *, hipStream_t);
template hipError_t launch_trace_csr<float>(const int64_t *, const int32_t *, const float *, int64_t,
                                            int64_t, double *, hipStream_t);

// ---------------------------------------------------------------------------
// CSR structure check: row_ptr[0] = 0, non-decreasing, row_ptr[n] = nnz, and
// every column index in [0, n).  Any violation sets flag[0].
// ---------------------------------------------------------------------------
__global__ void validate_csr_kernel(const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                    int64_t n, int64_t nnz, int32_t *__restrict__ flag) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool bad = false;
  for (int64_t i = t0; i <= n; i += stride) {
    const int64_t v = rp[i];
    if (i == 0 && v != 0) bad = true;
    if (i == n && v != nnz) bad = true;
    if (i < n && rp[i + 1] < v) bad = true;
  }
  // column indices, 16 bytes per load when the array allows it (a negative
  // index is a large unsigned one)
  int64_t done = 0;
  if (((uintptr_t)ci & 15) == 0) {
    const int4 *c4 = (const int4 *)ci;
    const int64_t n4 = nnz / 4;
    for (int64_t q = t0; q < n4; q += stride) {
      const int4 v = c4[q];
      if ((int64_t)(uint32_t)v.x >= n || (int64_t)(uint32_t)v.y >= n || (int64_t)(uint32_t)v.z >= n ||
          (int64_t)(uint32_t)v.w >= n)
        bad = true;
    }
    done = n4 * 4;
  }
  for (int64_t e = done + t0; e < nnz; e += stride) {
    const int32_t c = ci[e];
    if (c < 0 || (int64_t)c >= n) bad = true;
  }
  if (bad) atomicOr(flag, 1);
}

hipError_t launch_validate_csr(const int64_t *rp, const int32_t *ci, int64_t n, int64_t nnz,
                               int32_t *flag, hipStream_t st) {
  validate_csr_kernel<<<1024, 256, 0, st>>>(rp, ci, n, nnz, flag);
  return hipGetLastError();
}

// One row per thread: row_ptr's local conditions (rp[0] = 0, rp[n] = nnz,
// 0 <= rp[r] <= rp[r+1] <= nnz) hold for every row exactly when row_ptr is
// valid, and a row's column indices are read only if its range lies in
// [0, nnz), so the entries of a valid structure are each checked once.
//
// With val, also whether R equals its transpose: each off-diagonal entry
// (r, c) needs exactly one entry (c, r) of the same value.  Row c is searched
// from its first entry (short rows: a tridiagonal row has three, adjacent in
// memory to the row's own); its range is checked before it is read, as row_ptr
// is validated in the same pass.  With a row of more than kSymScan entries the
// matrix counts as not symmetric: searched by every other row it would cost n^2
// reads, and looking its own entries up, one after the other in one thread, as
// much time again as all else (star of 200000 vertices: 125 -> 33 ms).
constexpr int64_t kSymScan = 64;

template <typename T>
__global__ __launch_bounds__(256) void validate_csr_rows_kernel(const int64_t *__restrict__ rp,
                                                                const int32_t *__restrict__ ci,
                                                                const T *__restrict__ val, int64_t n,
                                                                int64_t nnz, int32_t *__restrict__ flag) {
  bool bad = false, asym = false;
  int64_t hb = 0;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    const int64_t a = rp[r], b = rp[r + 1];
    if ((r == 0 && a != 0) || (r == n - 1 && b != nnz) || a < 0 || b < a || b > nnz) {
      bad = true;
      continue;
    }
    if (b - a > kSymScan) asym = true;
    for (int64_t e = a; e < b; ++e) {
      const int64_t c = ci[e];
      if (c < 0 || c >= n) {
        bad = true;
      } else {
        const int64_t d = c > r ? c - r : r - c;
        hb = d > hb ? d : hb;
        if (val && d != 0 && !asym) {
          const int64_t a2 = rp[c], b2 = rp[c + 1];
          int found = 0;
          if (a2 >= 0 && b2 <= nnz && b2 - a2 <= kSymScan) {
            for (int64_t f = a2; f < b2; ++f)
              if (ci[f] == r) found += val[f] == val[e] ? 1 : 2;
          }
          asym = found != 1;
        }
      }
    }
  }
  if (bad) atomicOr(flag, 1);
  if (__any(asym) && (threadIdx.x & 63) == 0) atomicOr(flag + 2, 1);
  // n < 2^31 (int32 column indices), so the half-bandwidth fits
  int32_t h = (int32_t)hb;
  for (int off = 32; off > 0; off >>= 1) {
    const int32_t o = __shfl_xor(h, off, 64);
    h = o > h ? o : h;
  }
  if ((threadIdx.x & 63) == 0 && h > 0) atomicMax(flag + 1, h);
}

template <typename T>
hipError_t launch_validate_csr_rows(const int64_t *rp, const int32_t *ci, const T *val, int64_t n, int64_t nnz,
                                    int32_t *flag, hipStream_t st) {
  if (n < 1) return hipErrorInvalidValue;
  const int64_t b = (n + 255) / 256;
  validate_csr_rows_kernel<T><<<(unsigned)(b < 4096 ? b : 4096), 256, 0, st>>>(rp, ci, val, n, nnz, flag);
  return hipGetLastError();
}
template hipError_t launch_validate_csr_rows<double>(const int64_t *, const int32_t *, const double *, int64_t,
                                                     int64_t, int32_t *, hipStream_t);
template hipError_t launch_validate_csr_rows<float>(const int64_t *, const int32_t *, const float *, int64_t,
                                                    int64_t, int32_t *, hipStream_t);

// R = R^T for a validated CSR matrix whose rows ascend strictly in column
// (checked here; other rows count as not symmetric).  Each entry right of the
// diagonal is looked up in its mirror row by bisection (about log2 of the row
// length dependent loads, mostly from L2); the entries left of the diagonal
// are then all mirrors exactly when there are as many of them.  Lanes share a
// row as in the power-method product; a row of more than kWaveRow entries is
// walked by the whole wave (star of 200000 vertices: 26 -> 4 ms).
constexpr int64_t kWaveRow = 512;

template <typename T, int L>
__global__ __launch_bounds__(256) void csr_check_kernel(const int64_t *__restrict__ rp,
                                                        const int32_t *__restrict__ ci,
                                                        const T *__restrict__ val, int64_t n,
                                                        int32_t *__restrict__ asym, int64_t *__restrict__ count) {
  constexpr int RPB = 256 / L;
  const int sub = threadIdx.x % L;
  bool bad = false;
  int64_t net = 0;  // entries right of the diagonal minus entries left of it
  auto entry = [&](int64_t row, int64_t e, int64_t e1) {
    const int64_t c = ci[e];
    if (e + 1 < e1 && ci[e + 1] <= c) bad = true;
    if (c < row) --net;
    if (c <= row) return;
    ++net;
    int64_t lo = rp[c], hi = rp[c + 1];
    const int64_t end = hi;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (ci[mid] < row)
        lo = mid + 1;
      else
        hi = mid;
    }
    if (!(lo < end && ci[lo] == row && val[lo] == val[e])) bad = true;
  };
  for (int64_t base = (int64_t)blockIdx.x * RPB; base < n && !__any(bad); base += (int64_t)gridDim.x * RPB) {
    const int64_t row = base + threadIdx.x / L;
    const int64_t e0 = row < n ? rp[row] : 0, e1 = row < n ? rp[row + 1] : 0;
    const bool whole = e1 - e0 > kWaveRow;
    if (!whole)
      for (int64_t e = e0 + sub; e < e1; e += L) entry(row, e, e1);
    for (unsigned long long m = __ballot(whole && sub == 0); m; m &= m - 1) {
      const int64_t r = base + ((threadIdx.x & ~63u) + __builtin_ctzll(m)) / L;
      const int64_t r1 = rp[r + 1];
      // (to no end once any workgroup has found a mismatch)
      for (int64_t e = rp[r]; e < r1 && !__any(bad) && *(volatile int32_t *)asym == 0; e += 64)
        if (e + (threadIdx.x & 63) < r1) entry(r, e + (threadIdx.x & 63), r1);
    }
  }
  // one addition per workgroup: they meet at one address
  __shared__ int64_t nets[4];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) net += __shfl_xor(net, off, 64);
  if ((threadIdx.x & 63) == 0) nets[threadIdx.x >> 6] = net;
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(asym, 1);
  __syncthreads();
  if (threadIdx.x == 0)
    atomicAdd((unsigned long long *)count, (unsigned long long)(nets[0] + nets[1] + nets[2] + nets[3]));
}

__global__ void publish_flag_kernel(int32_t *__restrict__ flag, const int64_t *__restrict__ count,
                                    int32_t *__restrict__ host_flag) {
  if (threadIdx.x != 0) return;
  int32_t v = *flag;
  if (count && *count != 0) *flag = v = v | 1;
  if (host_flag) {
    *host_flag = v;
    __threadfence_system();
  }
}

hipError_t launch_publish_flag(int32_t *flag, const int64_t *count, int32_t *host_flag, hipStream_t st) {
  publish_flag_kernel<<<1, 64, 0, st>>>(flag, count, host_flag);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_csr_check(const int64_t *rp, const int32_t *ci, const T *val, int64_t n, int32_t *asym,
                            int64_t *count, int32_t *host_flag, hipStream_t st) {
  const int64_t b = (n + 31) / 32;
  csr_check_kernel<T, 8><<<(unsigned)(b < 2048 ? b : 2048), 256, 0, st>>>(rp, ci, val, n, asym, count);
  return launch_publish_flag(asym, count, host_flag, st);
}
template hipError_t launch_csr_check<double>(const int64_t *, const int32_t *, const double *, int64_t, int32_t *,
                                             int64_t *, int32_t *, hipStream_t);
template hipError_t launch_csr_check<float>(const int64_t *, const int32_t *, const float *, int64_t, int32_t *,
                                            int64_t *, int32_t *, hipStream_t);

// ---------------------------------------------------------------------------
// Conversion copies
// ---------------------------------------------------------------------------
template <typename Tin, typename Tout>
__global__ void convert_kernel(const Tin *__restrict__ src, int64_t lds, Tout *__restrict__ dst,
                               int64_t ldd, int64_t rows, int64_t cols) {
  const int64_t r = blockIdx.y;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < ldd;
       c += (int64_t)gridDim.x * blockDim.x)
    dst[r * ldd + c] = (r < rows && c < cols) ? (Tout)src[r * lds + c] : Tout(0);
}

template <typename Tin, typename Tout>
hipError_t launch_convert(const Tin *src, int64_t lds, Tout *dst, int64_t ldd, int64_t rows,
                          int64_t cols, hipStream_t st) {
  dim3 grid((unsigned)((ldd + 255) / 256 < 64 ? (ldd + 255) / 256 : 64), (unsigned)rows);
  convert_kernel<Tin, Tout><<<grid, 256, 0, st>>>(src, lds, dst, ldd, rows, cols);
  return hipGetLastError();
}
template hipError_t launch_convert<double, float>(const double *, int64_t, float *, int64_t, int64_t,
                                                  int64_t, hipStream_t);
template hipError_t launch_convert<float, double>(const float *, int64_t, double *, int64_t, int64_t,
                                                  int64_t, hipStream_t);
template hipError_t launch_convert<double, double>(const double *, int64_t, double *, int64_t,
                                                   int64_t, int64_t, hipStream_t);
template hipError_t launch_convert<float, float>(const float *, int64_t, float *, int64_t, int64_t,
                                                 int64_t, hipStream_t);

// ---------------------------------------------------------------------------
// Hermitian R = B + iC (Section 4): its real form M = [[B, -C], [C, B]]
// (2n x 2n, row-major, leading dimension ldm; columns 2n..ldm-1 are zeroed).
// M [x; y] = [Re(R(x+iy)); Im(R(x+iy))], so the recurrence on M with probes
// [g; 0] is the complex recurrence on R with the real probe g, and
// [g; 0]^T T(M) [g; 0] = g^T Re[T(R)] g.  Every eigenvalue of R appears twice
// in M.  One thread per (row i of R, column j < ldm - n), grid-stride.
// ---------------------------------------------------------------------------
template <typename Tin, typename Tout>
__global__ void realify_kernel(const Tin *__restrict__ Rc, int64_t ldr, int64_t n,
                               Tout *__restrict__ M, int64_t ldm) {
  const int64_t cols = ldm - n;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n * cols;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = t / cols, j = t % cols;
    Tout *top = M + i * ldm, *bot = M + (i + n) * ldm;
    if (j < n) {
      const Tin re = Rc[2 * (i * ldr + j)], im = Rc[2 * (i * ldr + j) + 1];
      top[j] = (Tout)re;
      top[n + j] = (Tout)(-im);
      bot[j] = (Tout)im;
      bot[n + j] = (Tout)re;
    } else {
      // padding columns 2n..ldm-1 of both rows
      top[n + j] = Tout(0);
      bot[n + j] = Tout(0);
    }
  }
}

template <typename Tin, typename Tout>
hipError_t launch_realify(const Tin *Rc, int64_t ldr, int64_t n, Tout *M, int64_t ldm,
                          hipStream_t st) {
  if (ldm < 2 * n || ldr < n) return hipErrorInvalidValue;
  const int64_t tot = n * (ldm - n);
  const int64_t blocks = (tot + 255) / 256 < 65536 ? (tot + 255) / 256 : 65536;
  realify_kernel<Tin, Tout><<<(unsigned)blocks, 256, 0, st>>>(Rc, ldr, n, M, ldm);
  return hipGetLastError();
}
template hipError_t launch_realify<double, double>(const double *, int64_t, int64_t, double *, int64_t,
                                                   hipStream_t);
template hipError_t launch_realify<double, float>(const double *, int64_t, int64_t, float *, int64_t,
                                                  hipStream_t);
template hipError_t launch_realify<float, double>(const float *, int64_t, int64_t, double *, int64_t,
                                                  hipStream_t);
template hipError_t launch_realify<float, float>(const float *, int64_t, int64_t, float *, int64_t,
                                                 hipStream_t);

// ---------------------------------------------------------------------------
// Reductions
// ---------------------------------------------------------------------------
// A sum, X: with the rounding errors of its additions beside it (Knuth's two-sum).
// h_j = -sum alpha_k d_kj cancels to a few per cent of its terms, and a moment from
// dots in pairs is the difference of two sums, one of them doubled: with plain
// sums an FP64 estimate at n = 512, m = 30 (p_i ~ 1/i) came out twice as far from
// its exact value as with one dot per moment (4.0e-15 and 1.7e-15 relative), with
// these as far (3.0e-15 and 3.1e-15 on other inputs), and at n = 8192 half as far
// (2.0e-15 and 4.2e-15).  FP32 and BF16x3 estimates, whose vectors carry the error
// (their values are the same to the last bit), take plain sums.
template <bool X>
struct Sum2 {
  double s = 0.0, c = 0.0;
  __device__ __forceinline__ void add(double x) {
#pragma clang fp contract(off)
    const double t = s + x, z = t - s;
    if (X) c += (s - (t - z)) + (x - z);
    s = t;
  }
  __device__ __forceinline__ void add_product(double a, double b) {
#pragma clang fp contract(off)
    const double p = a * b;
    if (X) c += __builtin_fma(a, b, -p);
    add(p);
  }
  __device__ __forceinline__ double value() const { return X ? s + c : s; }
};

// Tiles [i0, i1) of slot k's sum for probe j.  X and pair: d_k = 2 (sum of slot k)
// - d_{k mod 2} for k >= 2, both sums term by term.
template <bool X>
__device__ __forceinline__ Sum2<X> moment_terms(const double *__restrict__ part, int32_t k, bool pair, int32_t ntile,
                                                int64_t ldv, int64_t j, int32_t i0, int32_t i1) {
  const double *p = part + (int64_t)k * ntile * ldv + j;
  const bool half = X && pair && k >= 2;
  const double *g = part + (int64_t)(half ? k & 1 : k) * ntile * ldv + j;
  const double f = half ? 2.0 : 1.0;
  constexpr int U = 8;  // tiles in flight
  Sum2<X> acc;
  for (int32_t i = i0; i < i1; i += U) {
    double a[U], b[U];
#pragma unroll
    for (int e = 0; e < U; ++e) {
      const int64_t o = (int64_t)(i + e < i1 ? i + e : i0) * ldv;
      a[e] = i + e < i1 ? p[o] : 0.0;
      b[e] = half && i + e < i1 ? g[o] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < U; ++e) {
      acc.add(X ? f * a[e] : a[e]);
      if (X) acc.add(-b[e]);
    }
  }
  return acc;
}

template <bool X>
__device__ __forceinline__ void reduce_moments_body(const double *__restrict__ part, int32_t nslot,
                                                    int32_t ntile, int64_t ldv, int32_t s, bool pair,
                                                    double *__restrict__ d, int64_t t) {
  if (t >= (int64_t)nslot * s) return;
  const int32_t k = (int32_t)(t / s), j = (int32_t)(t % s);
  d[(int64_t)k * s + j] = moment_terms<X>(part, k, pair, ntile, ldv, j, 0, ntile).value();
}

// One estimate's moments: workgroup = (slot, 64 probes); wave w sums the
// tiles of its contiguous sixteenth in order, then the sixteenths are added in
// order (fixed, so repeated runs agree bit for bit).  Bound by latency: the
// workgroups are few (slots x probes / 64), so each takes 16 waves and eight
// loads in flight (n = 200000 CSR, 31 slots: 107 -> 14 us; n = 8192 dense, 51
// slots x 256 probes: 57 -> 13 us; with two-sums and two slots' loads for one 26
// and 19).
constexpr int kReduceWaves = 16;
template <bool X>
__global__ __launch_bounds__(64 * kReduceWaves) void reduce_moments_kernel(const double *__restrict__ part, int32_t nslot,
                                                             int32_t ntile, int64_t ldv, int32_t s, bool pair,
                                                             double *__restrict__ d) {
  __shared__ double q[X ? 2 : 1][kReduceWaves][64];
  const int k = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = blockIdx.y * 64 + lane;
  const int32_t per = (ntile + kReduceWaves - 1) / kReduceWaves;
  const int32_t i0 = w * per, i1 = i0 + per < ntile ? i0 + per : ntile;
  Sum2<X> acc;
  if (j < s) acc = moment_terms<X>(part, k, pair, ntile, ldv, j, i0, i1);
  q[0][w][lane] = acc.s;
  if (X) q[X ? 1 : 0][w][lane] = acc.c;
  __syncthreads();
  if (w == 0 && j < s) {
#pragma unroll
    for (int i = 1; i < kReduceWaves; ++i) {
      acc.add(q[0][i][lane]);
      if (X) acc.c += q[X ? 1 : 0][i][lane];
    }
    d[(int64_t)k * s + j] = acc.value();
  }
}

hipError_t launch_reduce_moments(const double *part, int32_t nslot, int32_t ntile, int64_t ldv,
                                 int32_t s, bool exact, bool pair, double *d, hipStream_t st) {
  if (nslot < 1 || s < 1) return hipSuccess;
  const dim3 grid((unsigned)nslot, (unsigned)((s + 63) / 64));
  if (exact)
    reduce_moments_kernel<true><<<grid, 64 * kReduceWaves, 0, st>>>(part, nslot, ntile, ldv, s, pair, d);
  else
    reduce_moments_kernel<false><<<grid, 64 * kReduceWaves, 0, st>>>(part, nslot, ntile, ldv, s, pair, d);
  return hipGetLastError();
}

// h_j and the mean/standard error.  Chebyshev: h_j = -sum_{k=0}^m alpha_k d_kj
// (Clenshaw schedule: from g^T y_0, g^T y_2 and g^T g, see FINAL_CLENSHAW).
// Taylor: h_j = ln(1/u) + u sum_{k=1}^m e_kj / k  (e_kj = g^T (R/u) C^k g).
//
// Latency-bound (one workgroup, s (m + 1) values): the terms of a probe are
// dealt to up to 16 threads, whose sums are added in order, so that all of its
// loads are in flight at once (m = 50, s = 256: 18 -> 12 us; m = 30, s = 50:
// 12 -> 6 us).
constexpr int kFinalThreads = 1024;

template <bool X>
__device__ __forceinline__ void final_body(double *__restrict__ d, double *__restrict__ scal,
                                           int32_t method, int32_t m, int32_t s,
                                           double *__restrict__ h) {
  __shared__ double red[kFinalThreads / 64], sums[X ? 2 : 1][kFinalThreads];
  __shared__ double smean;
  const int tid = threadIdx.x, nwv = kFinalThreads / 64;
  int sp = 64;  // probes per pass
  while (sp < s && sp < kFinalThreads) sp <<= 1;
  const int tp = kFinalThreads / sp;  // threads per probe (1..16)
  const int jl = tid % sp, q = tid / sp;
  const double u = scal[S_U];
  const double *alpha = scal + S_ALPHA;
  double acc = 0.0;
  for (int jb = 0; jb < s; jb += sp) {
    const int j = jb + jl;
    Sum2<X> v;
    if (j < s) {
      if (method == FINAL_CLENSHAW) {
        // Algorithm 5: g^T f_m g = (alpha_0 g^T g + g^T y_0 - g^T y_2) / 2, with
        // d_k = g^T y_k in slots 0..m (y_2 = 0 for m < 2) and g^T g in slot m+1
        if (q == 0) {
          const double gg = d[(int64_t)(m + 1) * s + j];
          const double y2 = m >= 2 ? d[(int64_t)2 * s + j] : 0.0;
          v.s = -0.5 * (alpha[0] * gg + d[j] - y2);
        }
      } else if (!X && method == FINAL_CHEB_PAIRS) {
        // d_w = 2 (half sum of slot w) - d_{w mod 2}, written back
        const double d0 = d[j], d1 = d[(int64_t)s + j];
        if (q == 0) v.s = -(alpha[0] * d0 + alpha[1] * d1);
        for (int k = 2 + q; k <= m; k += 4 * tp) {
          double r[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = k + e * tp <= m ? d[(int64_t)(k + e * tp) * s + j] : 0.0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int w = k + e * tp;
            if (w > m) break;
            const double dw = 2.0 * r[e] - ((w & 1) ? d1 : d0);
            d[(int64_t)w * s + j] = dw;
            v.s -= alpha[w] * dw;
          }
        }
      } else if (method == 1) {
#pragma unroll 4
        for (int k = q; k <= m; k += tp) v.add_product(-alpha[k], d[(int64_t)k * s + j]);
      } else {
#pragma unroll 4
        for (int k = 1 + q; k <= m; k += tp) v.add(d[(int64_t)k * s + j] / (double)k);
      }
    }
    sums[0][tid] = v.s;
    if (X) sums[X ? 1 : 0][tid] = v.c;
    __syncthreads();
    if (q == 0 && j < s) {
      for (int i = 1; i < tp; ++i) {
        v.add(sums[0][i * sp + jl]);
        if (X) v.c += sums[X ? 1 : 0][i * sp + jl];
      }
      double hj = v.value();
      if (method == 0) hj = log(1.0 / u) + u * hj;
      h[j] = hj;
      acc += hj;
    }
    __syncthreads();
  }
  auto block_sum = [&](double x) {
    x = wave_sum(x);
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = x;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < nwv; ++i) t += red[i];
    return t;
  };
  const double total = block_sum(acc);
  if (tid == 0) smean = total / (double)s;
  __syncthreads();
  const double mean = smean;
  double var = 0.0;
  if (q == 0)
    for (int j = jl; j < s; j += sp) var += (h[j] - mean) * (h[j] - mean);
  const double v2 = block_sum(var);
  if (tid == 0) {
    scal[S_ENT] = mean;
    scal[S_SE] = s > 1 ? sqrt(v2 / ((double)s * (double)(s - 1))) : 0.0;
    if (!isfinite(mean)) scal[S_FLAG] = 1.0;
  }
}

// The results go to pinned host memory with the last stores of the estimate
// (three copies behind it cost 10 to 20 us together).
template <bool X>
__global__ __launch_bounds__(kFinalThreads) void final_kernel(double *__restrict__ d, double *__restrict__ scal, int32_t method,
                             int32_t m, int32_t s, double *__restrict__ h, double *__restrict__ host,
                             int32_t host_moments) {
  final_body<X>(d, scal, method, m, s, h);
  if (!host) return;
  __syncthreads();  // the block's own stores to scal, h and d
  const int head = S_ALPHA + m + 1;
  for (int i = threadIdx.x; i < head; i += kFinalThreads) host[i] = scal[i];
  for (int j = threadIdx.x; j < s; j += kFinalThreads) host[head + j] = h[j];
  if (host_moments) {
    const int64_t cnt = (int64_t)(m + 1) * s;
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < cnt; i += kFinalThreads) host[head + s + i] = d[i];
  }
  __threadfence_system();
}

hipError_t launch_final(double *d, double *scal, bool exact, int32_t method, int32_t m, int32_t s,
                        double *h, hipStream_t st, double *host, bool host_moments) {
  if (exact)
    final_kernel<true><<<1, kFinalThreads, 0, st>>>(d, scal, method, m, s, h, host, host_moments);
  else
    final_kernel<false><<<1, kFinalThreads, 0, st>>>(d, scal, method, m, s, h, host, host_moments);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batches: the same phases over many matrices in one launch each.  Blocks map
// to matrices through the descriptor array (grid.y) or a tile table.
// ---------------------------------------------------------------------------
__global__ void fill_kernel(double *__restrict__ p, int64_t count, double v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_fill(double *p, int64_t count, double v, hipStream_t st) {
  const int64_t blocks = (count + 255) / 256 < 1024 ? (count + 255) / 256 : 1024;
  fill_kernel<<<(unsigned)(blocks > 0 ? blocks : 1), 256, 0, st>>>(p, count, v);
  return hipGetLastError();
}

// Zero bytes [p, p + bytes): 16-byte stores over the aligned bulk, byte
// stores for the head and tail.  Used instead of a memset node so that a
// captured sequence clears its buffers with kernels only.
__global__ void zero_kernel(unsigned char *__restrict__ p, int64_t head, int64_t nvec, int64_t bytes) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  uint4 *v = (uint4 *)(p + head);
  for (int64_t i = tid; i < nvec; i += stride) v[i] = make_uint4(0u, 0u, 0u, 0u);
  const int64_t tail0 = head + 16 * nvec;
  for (int64_t i = tid; i < head; i += stride) p[i] = 0;
  for (int64_t i = tail0 + tid; i < bytes; i += stride) p[i] = 0;
}

__global__ void xcc_probe_kernel(int32_t *ids) {
  if (threadIdx.x == 0) ids[blockIdx.x] = xcc_id();
}

hipError_t launch_xcc_probe(int32_t *ids, int32_t grid, hipStream_t st) {
  xcc_probe_kernel<<<(unsigned)grid, 64, 0, st>>>(ids);
  return hipGetLastError();
}

__global__ void sched_check_kernel(SchedArgs s) {
  const int q = (int)threadIdx.x;
  if (q < s.nseg) {
    const int len = (s.tail && *s.tail == 0 ? s.seg_mid[q] : s.seg_off[q + 1]) - s.seg_off[q];
    if (len > 0 && __hip_atomic_load(s.head + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < len)
      __hip_atomic_fetch_or(s.err, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

hipError_t launch_sched_check(const SchedArgs &s, hipStream_t st) {
  sched_check_kernel<<<1, 64, 0, st>>>(s);
  return hipGetLastError();
}

hipError_t launch_zero(void *p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  const uintptr_t a = (uintptr_t)p;
  int64_t head = (int64_t)((16 - (a & 15)) & 15);
  if ((size_t)head > bytes) head = (int64_t)bytes;
  const int64_t nvec = ((int64_t)bytes - head) / 16;
  const int64_t work = nvec > 0 ? nvec : (int64_t)bytes;
  const int64_t blocks = (work + 255) / 256 < 2048 ? (work + 255) / 256 : 2048;
  zero_kernel<<<(unsigned)(blocks > 0 ? blocks : 1), 256, 0, st>>>((unsigned char *)p, head, nvec,
                                                                   (int64_t)bytes);
  return hipGetLastError();
}

template <typename Tin, typename Tout>
__global__ void batch_convert_kernel(const BatchMat *__restrict__ mats) {
  const BatchMat &M = mats[blockIdx.y];
  const Tin *src = (const Tin *)M.src;
  Tout *dst = (Tout *)M.R;
  const int64_t tot = M.n * M.ldr;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < tot;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / M.ldr, c = t % M.ldr;
    dst[t] = c < M.n ? (Tout)src[r * M.ldsrc + c] : Tout(0);
  }
}

template <typename Tin, typename Tout>
hipError_t launch_batch_convert(const BatchMat *mats, int32_t count, int64_t max_elems,
                                hipStream_t st) {
  const int64_t per = (max_elems + 255) / 256;
  dim3 grid((unsigned)(per < 512 ? per : 512), (unsigned)count);
  batch_convert_kernel<Tin, Tout><<<grid, 256, 0, st>>>(mats);
  return hipGetLastError();
}
template hipError_t launch_batch_convert<double, double>(const BatchMat *, int32_t, int64_t, hipStream_t);
template hipError_t launch_batch_convert<float, float>(const BatchMat *, int32_t, int64_t, hipStream_t);
template hipError_t launch_batch_convert<double, float>(const BatchMat *, int32_t, int64_t, hipStream_t);
template hipError_t launch_batch_convert<float, double>(const BatchMat *, int32_t, int64_t, hipStream_t);

template <typename T>
__global__ void batch_trace_kernel(const BatchMat *__restrict__ mats) {
  const BatchMat &M = mats[blockIdx.x];
  trace_dense_body<T>((const T *)M.R, M.ldr, M.n, M.scal);
}

template <typename T>
hipError_t launch_batch_trace(const BatchMat *mats, int32_t count, hipStream_t st) {
  batch_trace_kernel<T><<<(unsigned)count, 256, 0, st>>>(mats);
  return hipGetLastError();
}
template hipError_t launch_batch_trace<double>(const BatchMat *, int32_t, hipStream_t);
template hipError_t launch_batch_trace<float>(const BatchMat *, int32_t, hipStream_t);

// G of matrix b = its n_pad x ldv region; probes from the matrix's own seed.
template <typename T>
__global__ void batch_probe_kernel(const BatchMat *__restrict__ mats, T *__restrict__ G, int32_t s,
                                   int64_t ldv, int32_t dist) {
  const BatchMat &M = mats[blockIdx.y];
  T *Gb = G + M.voff;
  const int64_t tot = M.n_pad * ldv;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < tot;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = t / ldv, j = t % ldv;
    T v = T(0);
    if (row < M.n && j < s)
      v = (T)(dist == 0 ? rademacher(M.seed, 0u, row, j) : gaussian(M.seed, 0u, row, j));
    Gb[t] = v;
  }
}

template <typename T>
hipError_t launch_batch_probes(const BatchMat *mats, int32_t count, int64_t max_n_pad, T *G,
                               int32_t s, int64_t ldv, int32_t dist, hipStream_t st) {
  const int64_t per = (max_n_pad * ldv + 255) / 256;
  dim3 grid((unsigned)(per < 256 ? per : 256), (unsigned)count);
  batch_probe_kernel<T><<<grid, 256, 0, st>>>(mats, G, s, ldv, dist);
  return hipGetLastError();
}
template hipError_t launch_batch_probes<double>(const BatchMat *, int32_t, int64_t, double *, int32_t,
                                                int64_t, int32_t, hipStream_t);
template hipError_t launch_batch_probes<float>(const BatchMat *, int32_t, int64_t, float *, int32_t,
                                               int64_t, int32_t, hipStream_t);

__global__ void batch_power_start_kernel(const BatchMat *__restrict__ mats, double *__restrict__ x,
                                         int32_t trial) {
  const BatchMat &M = mats[blockIdx.y];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < M.n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[M.xoff + i] = rademacher(M.seed, 1u, i, trial);
}

hipError_t launch_batch_power_start(const BatchMat *mats, int32_t count, int64_t max_n, double *x,
                                    int32_t trial, hipStream_t st) {
  const int64_t per = (max_n + 255) / 256;
  dim3 grid((unsigned)(per < 64 ? per : 64), (unsigned)count);
  batch_power_start_kernel<<<grid, 256, 0, st>>>(mats, x, trial);
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(256) void batch_power_gemv_kernel(const BatchMat *__restrict__ mats,
                                                               const int2 *__restrict__ ptiles,
                                                               const double *x, const double *pprev,
                                                               double *y, double *pout) {
  const int2 t = ptiles[blockIdx.x];
  const BatchMat &M = mats[t.x];
  const PowerPrev prev = {nullptr, pprev ? pprev + M.pboff : nullptr, M.pblk};
  power_gemv_body<T>((const T *)M.R, M.ldr, M.n, x + M.xoff, prev, y + M.xoff, pout + M.pboff, t.y);
}

// The same from half of each matrix that equals its transpose (its answer is on
// the device), the sums in the matrix's V block V: stiles (matrix, tile), tiles
// (matrix, 64 rows).  Of any other matrix the mirror tiles are read too or, with
// rows, it is passed by here and multiplied by rows in the second launch (which is
// faster where stands at its caller): a workgroup per entry of tiles there or, while
// these are few, kRowGroups of them, group g taking every fourth block of 8 rows
// from the g-th on; a combination of 64 rows is the first group's.  Row blocks dealt
// to the workgroups of the first launch, which hold too many registers for it, were
// slower (32 of 1024 FP32 37 + 5 us a product against 4.6 + 24.9).  us a product,
// matrices of up to 2048, first + second launch, one group / four:
//   symmetric   48 FP32 44 + 5.5 / 5.6, 128 FP32 133 + 11.4 / 12.9, 1024 FP32
//               1017 + 69 / 91, 512 FP64 890 + 34 / 44
//   any other   48 FP32 6 + 97 / 85, 128 FP32 15 + 222 / 215, 512 FP32 56 + 842 /
//               834, 48 FP64 5 + 151 / 145, 512 FP64 40 + 1467 / 1457
// where every matrix is read whole 84, 209, 819 and 144, 1439 us.
constexpr int kRowGroups = 4;
constexpr int32_t kRowGroupTiles = 4096;
// Waves per SIMD of the second launch, for its two bodies in one kernel: a wave
// more spills in either type (others: 512 FP64 1467 -> 1538 us, 1024 FP32 1645 ->
// 1996), and without a bound a symmetric batch waits longer (1024 FP32 69 -> 89).
template <typename T>
constexpr int kCombineWaves = sizeof(T) == 4 ? 6 : 7;

// The answers of the symmetry check, sb apart from scal on: a matrix's is read
// beside its descriptor, not behind it (512 others, FP32, passed by: 73 -> 56 us;
// 1024 symmetric FP32 1052 -> 1017).
struct SymFlags {
  const double *scal;
  int64_t sb;
  bool rows;
  __device__ __forceinline__ int32_t of(int32_t b) const {
    return uniform_load((const int32_t *)(scal + b * sb + S_SYM));
  }
};

template <typename T>
__global__ __launch_bounds__(256) void batch_power_sym_kernel(const BatchMat *__restrict__ mats,
                                                              const int2 *__restrict__ stiles, SymFlags flags,
                                                              const double *__restrict__ x, T *V) {
  const int2 t = uniform_load(stiles + blockIdx.x);
  const int32_t differs = flags.of(t.x);
  const BatchMat M = uniform_load(mats + t.x);
  if (differs && flags.rows) return;
  int64_t rb, cb;
  sym_tile(t.y, rb, cb);
  double *part = (double *)(V + M.voff);
  power_sym_body<T>((const T *)M.R, M.ldr, M.n, x + M.xoff, part, rb, cb, !differs && rb != cb);
  if (!differs || rb == cb) return;
  __syncthreads();
  power_sym_body<T>((const T *)M.R, M.ldr, M.n, x + M.xoff, part, cb, rb, false);
}

template <typename T>
__global__ __launch_bounds__(256, kCombineWaves<T>) void batch_power_sym_combine_kernel(
    const BatchMat *__restrict__ mats, const int2 *__restrict__ tiles, SymFlags flags, const double *x,
    const double *pprev, const T *V, double *y, double *pout) {
  const int32_t group = (int32_t)blockIdx.y, groups = (int32_t)gridDim.y;
  const int2 t = uniform_load(tiles + blockIdx.x);
  const int32_t differs = flags.of(t.x);
  const BatchMat M = uniform_load(mats + t.x);
  PowerPrev prev = {nullptr, pprev ? pprev + M.pboff : nullptr, M.pblk};
  if (!differs || !flags.rows) {
    if (group > 0 || (int64_t)t.y * 64 >= M.n) return;
    prev.nblk = (int32_t)((M.n + 63) / 64);
    power_sym_sum((const double *)(V + M.voff), (int32_t)((M.n + kSymTile - 1) / kSymTile), M.n, M.n, x + M.xoff,
                  prev, y + M.xoff, pout + M.pboff, t.y);
  } else {
    for (int blk = t.y * 8 + group; blk < t.y * 8 + 8 && blk < M.pblk; blk += groups) {
      __syncthreads();  // the block before is done with its sums in LDS
      power_gemv_body<T>((const T *)M.R, M.ldr, M.n, x + M.xoff, prev, y + M.xoff, pout + M.pboff, blk);
    }
  }
}

template <typename T>
hipError_t launch_batch_power_sym(const BatchMat *mats, const int2 *stiles, int32_t nstiles, const int2 *tiles,
                                  int32_t ntiles, const double *scal, int64_t sb, bool rows,
                                  const double *x, const double *pprev, T *V, double *y, double *pout, hipStream_t st) {
  if (pprev == pout) return hipErrorInvalidValue;
  const SymFlags flags = {scal, sb, rows};
  const int32_t groups = rows && ntiles <= kRowGroupTiles ? kRowGroups : 1;
  batch_power_sym_kernel<T><<<(unsigned)nstiles, 256, 0, st>>>(mats, stiles, flags, x, V);
  batch_power_sym_combine_kernel<T><<<dim3((unsigned)ntiles, (unsigned)groups), 256, 0, st>>>(mats, tiles, flags, x,
                                                                                              pprev, V, y, pout);
  return hipGetLastError();
}
template hipError_t launch_batch_power_sym<double>(const BatchMat *, const int2 *, int32_t, const int2 *, int32_t,
                                                   const double *, int64_t, bool, const double *, const double *,
                                                   double *, double *, double *, hipStream_t);
template hipError_t launch_batch_power_sym<float>(const BatchMat *, const int2 *, int32_t, const int2 *, int32_t,
                                                  const double *, int64_t, bool, const double *, const double *,
                                                  float *, double *, double *, hipStream_t);

template <typename T>
hipError_t launch_batch_power_gemv(const BatchMat *mats, const int2 *ptiles, int32_t nptiles,
                                   const double *x, const double *pprev, double *y, double *pout,
                                   hipStream_t st) {
  if (pprev == pout) return hipErrorInvalidValue;
  batch_power_gemv_kernel<T><<<(unsigned)nptiles, 256, 0, st>>>(mats, ptiles, x, pprev, y, pout);
  return hipGetLastError();
}
template hipError_t launch_batch_power_gemv<double>(const BatchMat *, const int2 *, int32_t,
                                                    const double *, const double *, double *,
                                                    double *, hipStream_t);
template hipError_t launch_batch_power_gemv<float>(const BatchMat *, const int2 *, int32_t,
                                                   const double *, const double *, double *, double *,
                                                   hipStream_t);

// One block per matrix: its final product's triples and Rayleigh quotient.
__global__ __launch_bounds__(256) void batch_power_rq_kernel(const BatchMat *__restrict__ mats, const double *p,
                                                             int32_t trial, bool half, bool rows) {
  __shared__ double norm3[3];
  const BatchMat &M = mats[blockIdx.x];
  power_reduce_body(p + M.pboff, half && (!rows || batch_pairs(M)) ? (int32_t)((M.n + 63) / 64) : M.pblk, norm3);
  power_rq_body(M.scal, norm3, trial);
}

hipError_t launch_batch_power_rq(const BatchMat *mats, int32_t count, const double *p,
                                 int32_t trial, hipStream_t st, bool half, bool rows) {
  batch_power_rq_kernel<<<(unsigned)count, 256, 0, st>>>(mats, p, trial, half, rows);
  return hipGetLastError();
}

__global__ void batch_setup_kernel(const BatchMat *__restrict__ mats, int32_t method, int32_t m,
                                   double c, double u_fixed, double lo, double norm_div) {
  setup_interval_body(mats[blockIdx.x].scal, method, m, c, u_fixed, lo, norm_div);
}

hipError_t launch_batch_setup(const BatchMat *mats, int32_t count, int32_t method, int32_t m,
                              double c, double u_fixed, double lo, hipStream_t st, double norm_div) {
  batch_setup_kernel<<<(unsigned)count, 256, 0, st>>>(mats, method, m, c, u_fixed, lo, norm_div);
  return hipGetLastError();
}

template <bool X>
__global__ void batch_reduce_kernel(const BatchMat *__restrict__ mats, const double *part, int32_t method,
                                    int32_t nslot, int64_t ldv, int32_t s, double *d) {
  const BatchMat &M = mats[blockIdx.y];
  const bool pair = method == 1 && batch_pairs(M);
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < (int64_t)nslot * s;
       t += (int64_t)gridDim.x * blockDim.x)
    reduce_moments_body<X>(part + M.poff, nslot, M.ntile, ldv, s, pair, d + M.doff, t);
}

hipError_t launch_batch_reduce(const BatchMat *mats, int32_t count, const double *part, bool exact, int32_t method,
                               int32_t nslot, int64_t ldv, int32_t s, double *d, hipStream_t st) {
  const int64_t per = ((int64_t)nslot * s + 255) / 256;
  dim3 grid((unsigned)(per < 64 ? per : 64), (unsigned)count);
  if (exact)
    batch_reduce_kernel<true><<<grid, 256, 0, st>>>(mats, part, method, nslot, ldv, s, d);
  else
    batch_reduce_kernel<false><<<grid, 256, 0, st>>>(mats, part, method, nslot, ldv, s, d);
  return hipGetLastError();
}

template <bool X>
__global__ __launch_bounds__(kFinalThreads) void batch_final_kernel(const BatchMat *__restrict__ mats, double *d,
                                                                    int32_t method, int32_t m, int32_t s,
                                                                    double *h) {
  const BatchMat &M = mats[blockIdx.x];
  const bool halves = !X && method == 1 && batch_pairs(M);
  final_body<X>(d + M.doff, M.scal, halves ? FINAL_CHEB_PAIRS : method, m, s, h + M.hoff);
}

hipError_t launch_batch_final(const BatchMat *mats, int32_t count, double *d, bool exact, int32_t method,
                              int32_t m, int32_t s, double *h, hipStream_t st) {
  if (exact)
    batch_final_kernel<true><<<(unsigned)count, kFinalThreads, 0, st>>>(mats, d, method, m, s, h);
  else
    batch_final_kernel<false><<<(unsigned)count, kFinalThreads, 0, st>>>(mats, d, method, m, s, h);
  return hipGetLastError();
}

}  // namespace ent
