// kernels_rp.hip -- random-projection estimator (Algorithm 3, Section 5):
// sketch R~ = R Pi (Gaussian and Hadamard sketches: product on the existing
// MFMA kernels; input-sparsity sketch: one signed pass over R), Gram matrix
// R~^T R~ in FP64, its eigenvalues by Householder tridiagonalization and
// bisection in one workgroup, singular values sigma = sqrt(lambda), the k
// largest kept and H^ = sum sigma ln(1/sigma).
#include "device_common.hpp"
#include "kernels.hpp"

namespace ent {

// ---------------------------------------------------------------------------
// Sketch Pi, row-major n_pad x ldv: kind 0 entries N(0, 1/s) (Gaussian
// stream 2); kind 1 the subsampled randomized Hadamard transform
// sqrt(N/s) D H S, entries D_jj (-1)^popcount(j & i_t) / sqrt(s).
// ---------------------------------------------------------------------------
template <typename T>
__global__ void sketch_gen_kernel(T *__restrict__ P, int64_t n, int64_t n_pad, int32_t s, int64_t ldv,
                                  uint64_t seed, double scale, int32_t kind) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_pad * ldv) return;
  const int64_t i = t / ldv, j = t % ldv;
  T v = T(0);
  if (i < n && j < s)
    v = (T)(scale * (kind == 1 ? srht_entry(seed, i, j, hadamard_order(n)) : gaussian(seed, 2u, i, j)));
  P[t] = v;
}

template <typename T>
hipError_t launch_sketch_gen(T *P, int64_t n, int64_t n_pad, int32_t s, int64_t ldv, uint64_t seed,
                             int32_t kind, hipStream_t st) {
  const int64_t tot = n_pad * ldv;
  sketch_gen_kernel<T><<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(P, n, n_pad, s, ldv, seed,
                                                                      1.0 / sqrt((double)s), kind);
  return hipGetLastError();
}
template hipError_t launch_sketch_gen<double>(double *, int64_t, int64_t, int32_t, int64_t, uint64_t,
                                              int32_t, hipStream_t);
template hipError_t launch_sketch_gen<float>(float *, int64_t, int64_t, int32_t, int64_t, uint64_t,
                                             int32_t, hipStream_t);

// ---------------------------------------------------------------------------
// Input-sparsity sketch Pi = D S (one entry D_jj per row, in column h(j)).
// R is symmetric, so (R Pi)^T = Pi^T R: row c of Y = (R Pi)^T is the signed
// sum of the rows j of R with h(j) = c.  The rows of each bucket are listed
// in ascending order (count, offsets, fill: one workgroup per bucket), and
// every row of R is then read exactly once: a single pass over R, as the
// construction's input-sparsity running time promises.  Sums are FP64 in
// ascending row order (deterministic).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void cs_count_kernel(uint64_t seed, int64_t n, int32_t s,
                                                       int32_t *__restrict__ cnt) {
  __shared__ int32_t red[4];
  const int32_t c = blockIdx.x;
  int32_t k = 0;
  for (int64_t j = threadIdx.x; j < n; j += blockDim.x) k += sketch_bucket(seed, j, s) == c;
  for (int off = 32; off >= 1; off >>= 1) k += __shfl_xor(k, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = k;
  __syncthreads();
  if (threadIdx.x == 0) cnt[c] = red[0] + red[1] + red[2] + red[3];
}

__global__ void cs_offsets_kernel(const int32_t *__restrict__ cnt, int32_t s, int64_t *__restrict__ off) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  int64_t a = 0;
  for (int32_t c = 0; c < s; ++c) {
    off[c] = a;
    a += cnt[c];
  }
  off[s] = a;
}

__global__ __launch_bounds__(256) void cs_fill_kernel(uint64_t seed, int64_t n, int32_t s,
                                                      const int64_t *__restrict__ off,
                                                      int32_t *__restrict__ rows) {
  __shared__ int32_t wcount[4];
  const int32_t c = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t base = off[c];
  for (int64_t j0 = 0; j0 < n; j0 += blockDim.x) {
    const int64_t j = j0 + threadIdx.x;
    const bool in = j < n && sketch_bucket(seed, j, s) == c;
    const uint64_t mask = __ballot(in);
    const int32_t before = (int32_t)__popcll(mask & ((1ull << lane) - 1ull));
    if (lane == 0) wcount[w] = (int32_t)__popcll(mask);
    __syncthreads();
    int32_t wbase = 0;
    for (int q = 0; q < w; ++q) wbase += wcount[q];
    if (in) rows[base + wbase + before] = (int32_t)j;
    base += wcount[0] + wcount[1] + wcount[2] + wcount[3];
    __syncthreads();
  }
}

// Y[c][col] = sum over the rows j of bucket c of D_jj R[j][col]; workgroup
// (column chunk of 1024, bucket c); thread columns col0 + tid + 256 q.
template <typename T>
__global__ __launch_bounds__(256) void cs_apply_kernel(const T *__restrict__ R, int64_t ldr, int64_t n,
                                                       uint64_t seed, const int64_t *__restrict__ off,
                                                       const int32_t *__restrict__ rows,
                                                       double *__restrict__ Y, int64_t ldy) {
  const int32_t c = blockIdx.y;
  const int64_t col0 = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int64_t r0 = off[c], r1 = off[c + 1];
  int64_t r = r0;
  // four rows at a time: 16 independent loads per thread in flight
  for (; r + 4 <= r1; r += 4) {
    int64_t j[4];
    double d[4];
    T v[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      j[u] = rows[r + u];
      d[u] = sketch_sign(seed, j[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t col = col0 + 256 * q;
        v[u][q] = col < n ? R[j[u] * ldr + col] : T(0);
      }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] += d[u] * (double)v[u][q];
  }
  for (; r < r1; ++r) {
    const int64_t j = rows[r];
    const double d = sketch_sign(seed, j);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t col = col0 + 256 * q;
      if (col < n) acc[q] += d * (double)R[j * ldr + col];
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t col = col0 + 256 * q;
    if (col < ldy) Y[(int64_t)c * ldy + col] = col < n ? acc[q] : 0.0;
  }
}

template <typename T>
hipError_t launch_count_sketch(const T *R, int64_t ldr, int64_t n, int32_t s, uint64_t seed,
                               int32_t *cnt, int64_t *off, int32_t *rows, double *Y, int64_t ldy,
                               hipStream_t st, int phase) {
  if (s < 1 || ldy < n || ldr < n) return hipErrorInvalidValue;
  if (phase == 0) {
    cs_count_kernel<<<(unsigned)s, 256, 0, st>>>(seed, n, s, cnt);
    cs_offsets_kernel<<<1, 64, 0, st>>>(cnt, s, off);
    cs_fill_kernel<<<(unsigned)s, 256, 0, st>>>(seed, n, s, off, rows);
  } else {
    dim3 grid((unsigned)((ldy + 1023) / 1024), (unsigned)s);
    cs_apply_kernel<T><<<grid, 256, 0, st>>>(R, ldr, n, seed, off, rows, Y, ldy);
  }
  return hipGetLastError();
}
template hipError_t launch_count_sketch<double>(const double *, int64_t, int64_t, int32_t, uint64_t,
                                                int32_t *, int64_t *, int32_t *, double *, int64_t,
                                                hipStream_t, int);
template hipError_t launch_count_sketch<float>(const float *, int64_t, int64_t, int32_t, uint64_t,
                                               int32_t *, int64_t *, int32_t *, double *, int64_t,
                                               hipStream_t, int);

// ---------------------------------------------------------------------------
// Gram matrix G = R~^T R~ (s x s, FP64).  R~(i, a) is at X[i*si + a*sa]
// (row-major R~: sa = 1; probe-major: si = 1).
// Workgroup = 64 x 64 block (a0 <= b0) of G over one K range, on the FP64
// matrix cores; the block is stored with its mirror image, and the partials per
// K range are summed in range order by gram_sum_kernel.  Chunks of 32 rows go
// through LDS as doubles, the next chunk's values in registers meanwhile; rows
// of 80 doubles put the four rows of an operand read on disjoint banks.
// Latency-bound (a chunk per round trip): n = 32768, s = 128, FP32 values
// 170 us with 16 x 16 blocks of scalar products, 40 us now.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void gram_partial_kernel(const T *__restrict__ X, int64_t si,
                                                           int64_t sa, int64_t n, int32_t s,
                                                           int64_t rows_per, double *__restrict__ gp) {
  using M = Mfma16<double>;
  constexpr int KC = 32, LD = 80;
  __shared__ double xs[2][KC][LD];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, m16 = lane & 15, kq = lane >> 4;
  // block pair (bi <= bj) of the upper triangle
  int bj = 0, bi = (int)blockIdx.x;
  while (bi > bj) bi -= ++bj;
  const bool diag = bi == bj;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per;
  const int64_t r1 = r0 + rows_per < n ? r0 + rows_per : n;
  // element e of a chunk: consecutive threads take consecutive addresses in
  // either layout
  auto row_of = [&](int e) { return si == 1 ? e % KC : e / 64; };
  auto col_of = [&](int e) { return si == 1 ? e / KC : e % 64; };
  T va[8], vb[8];
  auto load = [&](int64_t base) {
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int e = x * 256 + tid, cc = col_of(e);
      const int64_t i = base + row_of(e);
      const int ca = bi * 64 + cc, cb = bj * 64 + cc;
      va[x] = i < r1 && ca < s ? X[i * si + (int64_t)ca * sa] : T(0);
      vb[x] = !diag && i < r1 && cb < s ? X[i * si + (int64_t)cb * sa] : T(0);
    }
  };
  M::v4 acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = M::v4{0, 0, 0, 0};
  const double(*xb)[LD] = diag ? xs[0] : xs[1];
  load(r0);
  for (int64_t base = r0; base < r1; base += KC) {
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int e = x * 256 + tid, r = row_of(e), cc = col_of(e);
      xs[0][r][cc] = (double)va[x];
      if (!diag) xs[1][r][cc] = (double)vb[x];
    }
    __syncthreads();
    if (base + KC < r1) load(base + KC);
#pragma unroll
    for (int t = 0; t < KC / 4; ++t) {
      const double x = xs[0][4 * t + kq][16 * w + m16];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = M::mma(x, xb[4 * t + kq][16 * c + m16], acc[c]);
    }
    __syncthreads();
  }
  double *out = gp + (int64_t)blockIdx.y * s * s;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int a = bi * 64 + 16 * w + M::drow(kq, r), b = bj * 64 + 16 * c + m16;
      if (a >= s || b >= s) continue;
      out[(int64_t)a * s + b] = acc[c][r];
      if (!diag) out[(int64_t)b * s + a] = acc[c][r];
    }
}

__global__ void gram_sum_kernel(const double *__restrict__ gp, int32_t nsplit, int32_t s,
                                double *__restrict__ G) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= s * s) return;
  double acc = 0.0;
#pragma unroll 16
  for (int k = 0; k < nsplit; ++k) acc += gp[(int64_t)k * s * s + t];
  G[t] = acc;
}

template <typename T>
hipError_t launch_gram(const T *X, int64_t si, int64_t sa, int64_t n, int32_t s, double *scratch,
                       int32_t nsplit, double *G, hipStream_t st) {
  const int64_t rows_per = ((n + nsplit - 1) / nsplit + 63) / 64 * 64;
  const unsigned nb = (unsigned)((s + 63) / 64);
  dim3 grid(nb * (nb + 1) / 2, (unsigned)nsplit);
  gram_partial_kernel<T><<<grid, 256, 0, st>>>(X, si, sa, n, s, rows_per, scratch);
  gram_sum_kernel<<<(unsigned)((s * s + 255) / 256), 256, 0, st>>>(scratch, nsplit, s, G);
  return hipGetLastError();
}
template hipError_t launch_gram<double>(const double *, int64_t, int64_t, int64_t, int32_t, double *,
                                        int32_t, double *, hipStream_t);
template hipError_t launch_gram<float>(const float *, int64_t, int64_t, int64_t, int32_t, double *,
                                       int32_t, double *, hipStream_t);

// ---------------------------------------------------------------------------
// Eigenvalues of a symmetric N x N matrix (N <= 256, even):
//  1. Householder reduction to tridiagonal form T (d on the diagonal, e next
//     to it), one workgroup of 1024 threads: for k = 0..N-3 the reflector
//     H = I - beta v v^T that maps column k below the diagonal onto alpha e_1
//     is applied to the trailing block as A22 -= v w^T + w v^T with
//     p = beta A22 v, w = p - K v, K = (beta/2) v.p (the symmetric rank-2 form
//     of H A22 H; Golub & Van Loan, Section 8.3.1).  The threads that update
//     row k+1 also sum the squares the next step needs.
//  2. each eigenvalue of T by multisection on the Sturm count
//     (sturm_eig_kernel).
// Only eigenvalues are formed.
// ---------------------------------------------------------------------------

// Sum over a group of 8 consecutive lanes, on each of them.
__device__ __forceinline__ double oct_sum(double x) {
  x += dpp_move<0xB1>(x);   // quad_perm: lane ^ 1
  x += dpp_move<0x4E>(x);   // quad_perm: lane ^ 2
  x += dpp_move<0x141>(x);  // row_half_mirror: the other quad
  return x;
}

// N <= 128: the matrix in registers, thread (g, part) holding columns
// 16 q + 2 part, + 1 of rows g + 64 r, so that a step reads only the vectors v
// and p from LDS, each value for two rows, and has two barriers.  A step is a
// serial chain on one compute unit (two sums over 8 lanes, square root,
// division, a sum over the workgroup), so the row that the next step starts
// from is stored as it is, by the threads that own it, and every group of 8
// lanes sums its squares.  s = 128: 237 us (the matrix in LDS, four barriers a
// step, 8-way bank conflicts along its rows, and the eigenvalues in the same
// workgroup: 900; the sum of squares and the masks left to the row's owners: 409).
__global__ __launch_bounds__(512) void tridiag_small_kernel(const double *__restrict__ G, int32_t s, int32_t N,
                                                            double *__restrict__ de) {
  constexpr int NQ = 8, NR = 2, NG = 64;
  __shared__ __attribute__((aligned(16))) double xr[2][128], p[128], red[8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int g = tid >> 3, part = tid & 7;
  typedef double v2 __attribute__((ext_vector_type(2)));
  v2 a[NR][NQ];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int i = g + NG * r, j = 16 * q + 2 * part + c;
        a[r][q][c] = i < s && j < s ? G[(int64_t)i * s + j] : 0.0;
      }
  auto publish = [&](int row, int buf) {
    if (g != (row & (NG - 1))) return;
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (r == row / NG)
#pragma unroll
        for (int q = 0; q < NQ; ++q) *(v2 *)&xr[buf][16 * q + 2 * part] = a[r][q];
  };
  publish(0, 0);
  __syncthreads();
  for (int k = 0; k + 2 < N; ++k) {
    const int i0 = k + 1, buf = k & 1, q0 = i0 >> 4;
    const double x0 = xr[buf][i0];
    if (tid == 0) de[k] = xr[buf][k];
    // x: row k right of i0, zero up to it
    v2 v[NQ];
    double sq = 0.0, acc[NR] = {};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (q < q0) continue;
      v[q] = *(const v2 *)&xr[buf][16 * q + 2 * part];
      if (q == q0)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          if (16 * q + 2 * part + c <= i0) v[q][c] = 0.0;
      sq += v[q][0] * v[q][0] + v[q][1] * v[q][1];
#pragma unroll
      for (int r = 0; r < NR; ++r) acc[r] += a[r][q][0] * v[q][0] + a[r][q][1] * v[q][1];
    }
    double vi[NR], wi[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) vi[r] = g + NG * r > i0 ? xr[buf][g + NG * r] : 0.0;
    const double tail = oct_sum(sq);
    if (tail == 0.0) {  // already tridiagonal in this column (the same in every group)
      if (tid == 0) de[N + k] = x0;
      publish(i0, buf ^ 1);
      __syncthreads();
      continue;
    }
    const double alpha = -copysign(sqrt(tail + x0 * x0), x0);
    const double v0 = x0 - alpha;  // no cancellation: x0 and alpha differ in sign
    const double beta = 2.0 / (tail + v0 * v0);
    // v: x with v0 at i0
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (q == q0)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          if (16 * q + 2 * part + c == i0) {
            v[q][c] = v0;
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[r] += a[r][q][c] * v0;
          }
    double vp = 0.0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int i = g + NG * r;
      if (i == i0) vi[r] = v0;
      const double t = oct_sum(acc[r]);
      wi[r] = i >= i0 ? beta * t : 0.0;
      vp += vi[r] * wi[r];
      if (part == 0) p[i] = wi[r];
    }
    vp = wave_sum(part == 0 ? vp : 0.0);
    if (lane == 0) red[wv] = vp;
    __syncthreads();
    double K = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) K += red[q];
    K *= 0.5 * beta;
    // A22 -= v (p - K v)^T + (p - K v) v^T
#pragma unroll
    for (int r = 0; r < NR; ++r) wi[r] -= K * vi[r];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (q < q0) continue;
      const v2 pj = *(const v2 *)&p[16 * q + 2 * part];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double wj = pj[c] - K * v[q][c];
#pragma unroll
        for (int r = 0; r < NR; ++r) a[r][q][c] -= vi[r] * wj + wi[r] * v[q][c];
      }
    }
    publish(i0, buf ^ 1);
    if (tid == 0) de[N + k] = alpha;
    __syncthreads();
  }
  // rows N - 2 (published last) and N - 1
  if (tid == 0) {
    de[N - 2] = xr[(N - 2) & 1][N - 2];
    de[N + N - 2] = xr[(N - 2) & 1][N - 1];
  }
  publish(N - 1, (N - 1) & 1);
  __syncthreads();
  if (tid == 0) de[N - 1] = xr[(N - 1) & 1][N - 1];
}

// N > 128: the matrix (row-major) stays in memory, overwritten; d and e to its
// first 2N elements at the end.
__global__ __launch_bounds__(1024) void tridiag_large_kernel(double *__restrict__ A, int32_t N) {
  constexpr int NMAX = 256;
  constexpr int TPR = 1024 / NMAX;  // threads per row
  __shared__ double v[NMAX], w[NMAX], d[NMAX], e[NMAX];
  __shared__ double red[16];
  __shared__ double s_tail;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int ld = N;
  // sum over the block in a fixed order, returned to every thread (one
  // barrier; red is next written only after at least one more barrier)
  auto block_sum = [&](double x) -> double {
    x = wave_sum(x);
    if (lane == 0) red[wv] = x;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < 16; ++q) t += red[q];
    return t;
  };
  // sum of squares of row r right of column c0 (all threads)
  auto row_tail = [&](int r, int c0) -> double {
    double sq = 0.0;
    for (int j = c0 + tid; j < N; j += 1024) sq += A[r * ld + j] * A[r * ld + j];
    return block_sum(sq);
  };
  const int rsub = tid / TPR, part = tid % TPR;
  double tail = N > 2 ? row_tail(0, 2) : 0.0;
  for (int k = 0; k + 2 < N; ++k) {
    const int i0 = k + 1;
    // column k below the diagonal is row k right of it (A is symmetric)
    const double x0 = A[k * ld + i0];
    if (tail == 0.0) {  // already tridiagonal in this column
      if (tid == 0) {
        d[k] = A[k * ld + k];
        e[k] = x0;
      }
      __syncthreads();  // every thread has read red from the previous sum
      tail = k + 3 < N ? row_tail(i0, i0 + 2) : 0.0;
      continue;
    }
    const double alpha = -copysign(sqrt(tail + x0 * x0), x0);
    const double v0 = x0 - alpha;  // no cancellation: x0 and alpha differ in sign
    const double beta = 2.0 / (tail + v0 * v0);
    for (int j = i0 + tid; j < N; j += 1024) v[j] = j == i0 ? v0 : A[k * ld + j];
    __syncthreads();
    // p = beta A22 v, kept in w
    const int i = i0 + rsub;
    double acc = 0.0;
    if (i < N)
      for (int j = i0 + part; j < N; j += TPR) acc += A[i * ld + j] * v[j];
#pragma unroll
    for (int off = TPR / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (i < N && part == 0) w[i] = beta * acc;
    __syncthreads();
    const double K = 0.5 * beta * block_sum(tid + i0 < N ? v[tid + i0] * w[tid + i0] : 0.0);
    // A22 -= v (p - K v)^T + (p - K v) v^T; row i0's group also sums the
    // squares of its new entries right of i0 + 1 (the next step's tail)
    double sq = 0.0;
    if (i < N) {
      const double vi = v[i], wi = w[i] - K * v[i];
      for (int j = i0 + part; j < N; j += TPR) {
        const double a_new = A[i * ld + j] - (vi * (w[j] - K * v[j]) + wi * v[j]);
        A[i * ld + j] = a_new;
        if (j >= i0 + 2) sq += a_new * a_new;
      }
    }
    if (rsub == 0) {
#pragma unroll
      for (int off = TPR / 2; off >= 1; off >>= 1) sq += __shfl_xor(sq, off, 64);
      if (part == 0) s_tail = sq;
    }
    if (tid == 0) {
      d[k] = A[k * ld + k];
      e[k] = alpha;
    }
    __syncthreads();
    tail = s_tail;
  }
  if (tid == 0) {
    d[N - 2] = A[(N - 2) * ld + N - 2];
    d[N - 1] = A[(N - 1) * ld + N - 1];
    e[N - 2] = A[(N - 2) * ld + N - 1];
  }
  __syncthreads();
  for (int q = tid; q < N; q += 1024) {
    A[q] = d[q];
    if (q + 1 < N) A[N + q] = e[q];
  }
}

// Eigenvalue blockIdx.x (ascending) of the tridiagonal matrix with diagonal
// de[0, N) and off-diagonal de[N, 2N - 1): from the Gershgorin interval down to
// 2 ulp or 1e-22 ||T||, each iteration counts the eigenvalues below 256 points
// of the interval and keeps the subinterval between the last point with at most
// that many below it and the first with more.  The count is that of the sign
// changes in the leading minors of T - x I, p_r = (d_r - x) p_{r-1} -
// e_{r-1}^2 p_{r-2} (the pivots p_r / p_{r-1} without their divisions, 182 us
// with them at N = 128), on T scaled by a power of two to norm <= 1:
// a pivot below 2^-200 counts as -2^-200.  The pair is scaled, exactly, every
// fourth step, to a larger value in [1/2, 1) whose successor may be 2^-201
// already: four more such pivots leave 2^-1001 (the five before the first scaling
// 2^-1000), a normal double.  At zero the signs, and with them the count of
// every later row, would be lost.  A workgroup
// per eigenvalue fills the chip where one for all of them left it idle:
// s = 128 71 us.
__global__ __launch_bounds__(256) void sturm_eig_kernel(const double *__restrict__ de, int32_t N,
                                                        double *__restrict__ eig) {
  __shared__ double d[256], e2[256], red[2][4];
  __shared__ int first[2][4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, jv = (int)blockIdx.x;
  const double dt = tid < N ? de[tid] : 0.0, er = tid + 1 < N ? de[N + tid] : 0.0;
  double lo = 1.7976931348623157e308, hi = -1.7976931348623157e308;
  if (tid < N) {
    const double r = fabs(tid > 0 ? de[N + tid - 1] : 0.0) + fabs(er);
    lo = dt - r;
    hi = dt + r;
  }
  for (int off = 32; off >= 1; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
  }
  if (lane == 0) {
    red[0][wv] = lo;
    red[1][wv] = hi;
  }
  __syncthreads();
  double a = fmin(fmin(red[0][0], red[0][1]), fmin(red[0][2], red[0][3]));
  double b = fmax(fmax(red[1][0], red[1][1]), fmax(red[1][2], red[1][3]));
  const double big = fmax(fabs(a), fabs(b));
  // (nothing to scale, or to count, in a zero or non-finite matrix)
  const int ex = big > 0.0 && isfinite(big) ? -ilogb(big) - 1 : 0;
  d[tid] = ldexp(dt, ex);
  e2[tid] = ldexp(er, ex) * ldexp(er, ex);
  a = ldexp(a, ex);
  b = ldexp(b, ex);
  const double tnorm = fmax(fabs(a), fabs(b));
  constexpr double kPivot = 0x1p-200;
  __syncthreads();
  for (int it = 0; it < 64; ++it) {
    if (!(b - a > fmax(4.440892098500626e-16 * fmax(fabs(a), fabs(b)), 1e-22 * tnorm))) break;
    const double x = a + (b - a) * (double)(tid + 1) / 257.0;
    unsigned cnt = 0;
    double p2 = 0.0, p1 = 1.0;
    auto minor = [&](int r, double ee) {
      double t = (d[r] - x) * p1 - ee * p2;
      const double least = kPivot * fabs(p1);
      t = fabs(t) < least ? -copysign(least, p1) : t;
      cnt += ((unsigned)__double2hiint(t) ^ (unsigned)__double2hiint(p1)) >> 31;
      p2 = p1;
      p1 = t;
    };
    minor(0, 0.0);
    int r = 1;
    for (; r + 3 < N; r += 4) {
#pragma unroll
      for (int c = 0; c < 4; ++c) minor(r + c, e2[r + c - 1]);
      int e1;
      (void)frexp(fmax(fabs(p1), fabs(p2)), &e1);
      p1 = ldexp(p1, -e1);
      p2 = ldexp(p2, -e1);
    }
    for (; r < N; ++r) minor(r, e2[r - 1]);
    const unsigned long long above = __ballot((int)cnt > jv);
    if (lane == 0) first[it & 1][wv] = above ? wv * 64 + __builtin_ctzll(above) : 256;
    __syncthreads();
    const int *fw = first[it & 1];
    const int f = min(min(fw[0], fw[1]), min(fw[2], fw[3]));
    const double w = b - a, a_old = a;
    if (f > 0) a = a_old + w * (double)f / 257.0;
    if (f < 256) b = a_old + w * (double)(f + 1) / 257.0;
  }
  if (tid == 0) eig[jv] = ldexp(0.5 * (a + b), -ex);
}

// Copy the s x s Gram matrix into an N x N (N even) work matrix.
__global__ void pad_square_kernel(const double *__restrict__ G, int32_t s, double *__restrict__ A,
                                  int32_t N) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < N * N; e += gridDim.x * blockDim.x) {
    const int i = e / N, j = e % N;
    A[e] = (i < s && j < s) ? G[i * s + j] : 0.0;
  }
}

// sigma = sqrt(max(lambda, 0)) in descending order (rank by comparison,
// ties by index), the k largest kept, H^ = sum sigma ln(1/sigma).
__global__ void rp_finish_kernel(const double *__restrict__ eig, int32_t N, int32_t k,
                                 double *__restrict__ sigma, double *__restrict__ scal) {
  __shared__ double si[256], sv[256];
  const int tid = threadIdx.x;
  if (tid < N) si[tid] = eig[tid] > 0.0 ? sqrt(eig[tid]) : 0.0;
  __syncthreads();
  if (tid < N) {
    const double x = si[tid];
    int rank = 0;
    for (int j = 0; j < N; ++j) rank += si[j] > x || (si[j] == x && j < tid);
    sv[rank] = x;
  }
  __syncthreads();
  // S_NORM > 0: singular values of (R / tr R) Pi = those of R Pi / tr R
  const double nm = scal[S_NORM] > 0.0 ? scal[S_NORM] : 1.0;
  const int kept = k < N ? k : N;
  if (tid < kept) {
    const double sg = sv[tid] * nm;
    sigma[tid] = sg;
    si[tid] = sg > 0.0 ? sg * log(1.0 / sg) : 0.0;
  }
  __syncthreads();
  if (tid == 0) {
    double h = 0.0;
    for (int i = 0; i < kept; ++i) h += si[i];
    scal[S_ENT] = h;
    scal[S_SE] = 0.0;
    if (!isfinite(h)) scal[S_FLAG] = 1.0;
  }
}

hipError_t launch_rp_spectrum(const double *G, int32_t s, int32_t k, double *work, double *eig,
                              double *sigma, double *scal, hipStream_t st) {
  const int32_t N = (s + 1) / 2 * 2;
  if (N > 256) return hipErrorInvalidValue;
  if (N <= 128) {
    tridiag_small_kernel<<<1, 512, 0, st>>>(G, s, N, work);
  } else {
    pad_square_kernel<<<64, 256, 0, st>>>(G, s, work, N);
    tridiag_large_kernel<<<1, 1024, 0, st>>>(work, N);
  }
  sturm_eig_kernel<<<(unsigned)N, 256, 0, st>>>(work, N, eig);
  rp_finish_kernel<<<1, 256, 0, st>>>(eig, N, k, sigma, scal);
  return hipGetLastError();
}

}  // namespace ent
