// kernels_dense.hip -- one step of the polynomial recurrence for dense R on
// gfx950 matrix cores (FP64 / FP32 MFMA 16x16x4), with the recurrence update
// and the per-probe dot products fused into the epilogue.
//
//   Y = a * (R V_k)                                  (MFMA, K = n)
//   Z = c1*Y + c2*b*V_k + cw*V_{k-1}  -> V_{k+1}      (epilogue)
//   part[slot][tile][j] = sum_{rows of tile} g_ij * (dot_y ? Y : Z)_ij
//   (pair: V_k in place of g, and Z_ij * (dot_y ? Y : Z)_ij into slot_b)
//
// Chebyshev (Algorithm 2 via the forward three-term recurrence of T_w,
// Section 3 / Appendix B): a = 2/(u-lo), b = (u+lo)/(u-lo); step 0 has
// (c1,c2,cw) = (1,-1,0), later steps (2,-2,-1); dots with Z give
// d_{k+1,j} = g_j^T T_{k+1}(X) g_j.  Taylor (Algorithm 1): a = 1/u, b = 1,
// (c1,c2,cw) = (-1,1,0) so Z = (I - R/u) V_k, dots with Y give
// e_{k,j} = g_j^T (R/u)(I - R/u)^k g_j.
//
// Tiling: a workgroup of 4 waves owns 64*WR rows x BN probe columns; each
// wave owns WR slabs of 16 rows.  K is walked in chunks whose V_k rows and A
// values are loaded straight into LDS three chunks ahead (see
// dense_step_tile).  Row/column padding of the V buffers is zero, so a
// ragged end of K needs no masking of V.
//
// Split-K: when the tile grid is smaller than the chip (n = 4096 with 64
// probes has 64 tiles), each workgroup sums one range of columns into a
// partial block and dense_split_epilogue_kernel adds the partials in split
// order and applies the epilogue, with dot partials per 16 rows.
#include "device_common.hpp"
#include "kernels.hpp"

namespace ent {

// s_waitcnt vmcnt(N) in the gfx9 encoding, expcnt and lgkmcnt left free.
template <int N>
__device__ __forceinline__ void dense_wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt immediate");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// LDS of a tile's stages: two workgroups on a CU; the grouped FP32 batch step
// takes half of it and 16-column chunks, four workgroups on a CU hide each
// other's prologue and epilogue (64 matrices, n <= 2048, 64 probes: 160 us a
// step with 32-column chunks, 136 with 16; n = 1024: 115 and 96; n = 2048, where
// the chunks alone count, 362 and 357; FP64 lacks the registers for it).
constexpr int kChunkLds = 61440, kGroupedLds = 30720;

// Chunk geometry of the dense step: BK columns of R per chunk (32, 16 or 8),
// KPL = BK/4 of them per lane in APL pieces of VEC; one stage holds the chunk's V_k rows (BK x BN,
// shared by the 4 waves) and each wave's A values (WR 16-row slabs x BK); the
// NST stages take at most BUDGET bytes.
template <typename T, int BN, int WR, int BUDGET = kChunkLds>
struct DenseChunk {
  static constexpr int NST = 3;                      // stages (prefetch distance NST - 1)
  static_assert(NST >= 3 && NST <= 4, "the waits cover three or four stages");
  static constexpr int ES = (int)sizeof(T);
  static constexpr int VEC = 16 / ES;                // elements per 16-byte piece
  static constexpr int RB = BN * ES;                 // bytes per V row
  static constexpr int stage_bytes(int bk) { return bk * RB + 64 * WR * bk * ES; }
  static constexpr int BK = (NST * stage_bytes(32) <= BUDGET) ? 32
                          : (NST * stage_bytes(16) <= BUDGET || 2 * ES < 16) ? 16 : 8;
  static constexpr int KPL = BK / 4;                 // k values per lane per chunk
  static constexpr int G = RB / 16;                  // 16-byte groups per V row
  static constexpr int VBYTES = BK * RB;
  static constexpr int NVL = BK * G / 256;           // V pieces per wave (direct loads)
  static constexpr int APL = KPL / VEC;              // A pieces per lane and slab
  static constexpr int NAL = WR * APL;               // A direct loads per wave
  static constexpr int ABYTES = 4 * NAL * 1024;      // A of the 4 waves
  static_assert(KPL % VEC == 0, "a lane's A values must be whole 16-byte pieces");
  static_assert((BK * G) % 256 == 0, "V pieces must split over the 4 waves");
  static_assert(4 * ES <= G, "V rows too short for the swizzle");
  static constexpr int LDS = NST * (VBYTES + ABYTES);  // every stage
  // V row r sits at r * RB bytes, its 16-byte groups XOR-swizzled so that
  // the four 16-lane groups of an MFMA B-operand read (rows t, VEC+t, 2VEC+t,
  // 3VEC+t of a piece, 16 consecutive probes each) fall on disjoint banks
  __device__ static constexpr int swz(int r) { return ((r / VEC) & 3) * ES; }
  // chunk column of MFMA call t in lane group q
  __device__ static constexpr int kcol(int q, int t) { return (t / VEC * 4 + q) * VEC + t % VEC; }
  __device__ static int voff(int r, int col) {
    return r * RB + (((col / VEC) ^ swz(r)) << 4) + (col % VEC) * ES;
  }
};

namespace {
// Column groups whose epilogue operands a batch tile loads together: all of a
// 64-row tile; a 128-row one has no registers left for more than one.
template <int WR>
constexpr int kBatchCols = WR == 1 ? 4 : 1;

// LDS of a tile: its stages and, for a persistent kernel, the two words behind them
// with which its waves agree on the next item.  The kernel's only LDS object: with a
// single one the compiler adds no waits of its own between the direct loads into
// one stage and the reads of another; a second one gives it alias scopes, and every
// chunk's reads then wait for all loads (FP64 persistent batch, 40 symmetric
// matrices of n = 2000: 9.23 -> 7.89 ms a call).  Named as it stands, not by a
// pointer, which changes the schedule of the K loop (n = 8192 FP64 589 -> 603 us a
// step).
constexpr int kHookLds = 2 * sizeof(int);
template <int BYTES>
__shared__ __attribute__((aligned(1024))) unsigned char tile_lds[BYTES];

// What a persistent kernel does inside a tile: ready() once R's first loads are
// out and before anything of the step before is read (false: give up, the tile
// returns false), products_done() before the epilogue.
struct DenseNoHook {
  static constexpr bool on = false;
  __device__ bool ready() { return true; }
  __device__ void products_done() {}
};
struct BatchHook {
  static constexpr bool on = true;
  const SchedArgs &s;
  int b, need;
  int *sh;
  int *next;
  __device__ bool ready() { return sched_wait(s, b, need, sh); }
  __device__ void products_done() { *next = sched_reserve(s); }
};
}  // namespace

// Body of one tile: rows [64*WR*tm, +64*WR) (wave w owns WR 16-row slabs),
// probe columns [BN*tn, +BN), product columns [kbeg, kend) (kbeg a multiple
// of 32; kend a multiple of 32 or >= n).  Shared by the single-matrix kernel
// and the grouped (batched) kernel.  With yout the raw products go to
// yout[row][ldv] (every row of the tile) instead of the epilogue.
//
// Pipeline over chunks of BK columns, three stages deep: the chunk's V_k rows
// and each wave's A values go from global memory straight into LDS (direct
// loads, no registers), two chunks ahead of the MFMAs that read them; every
// wait on them is explicit (vmcnt), one barrier per chunk.  Lane (m, q) of a
// wave loads 16-byte pieces of R[row m] of each of its slabs, piece h at chunk
// column (4 h + q) VEC, so that the four lanes of a row take 64 consecutive
// bytes with each load (pieces of one lane side by side touched every 64 bytes
// twice: n = 5000, 64 probes, FP32 42.1 us a step, now 39.9; n = 8192, bound by
// the products, unchanged), and reads them back from its own 16-byte slots:
// MFMA k-slot q of call t is column kcol(q, t) (the k order inside a chunk is
// permuted consistently for A and B).  A ragged last chunk (n not a multiple of
// BK) reads A into registers at the start, column min(k, n - 1) element by
// element: V_k is zero in rows k >= n, so those products vanish.  RAG false: there
// is none (see dense_step_launch).
template <typename T, int BN, int WR, int EC, int BUDGET = kChunkLds, bool PRE = false, typename H = DenseNoHook,
          bool RAG = true>
__device__ __forceinline__ bool dense_step_tile(const DenseStepArgs &a, int tm, int tn, int64_t kbeg,
                                                int64_t kend, T *yout, H hook = H{}) {
  using M = Mfma16<T>;
  using v4 = typename M::v4;
  using C = DenseChunk<T, BN, WR, BUDGET>;
  constexpr int BM = 64 * WR, BK = C::BK, KPL = C::KPL, VEC = C::VEC;
  constexpr int NSUB = BN / 16;
  constexpr int NVL = C::NVL, NAL = C::NAL, APL = C::APL;
  typedef T vec_t __attribute__((ext_vector_type(VEC)));

  // stage s at tile_lds<BYTES> + s * STAGE: the V_k chunk (VBYTES), then the A values of
  // the 4 waves (ABYTES)
  constexpr int STAGE = C::VBYTES + C::ABYTES, NST = C::NST;
  // the epilogue's per-wave dot sums reuse the stages after the products
  static_assert(C::LDS >= 3 * 4 * BN * 8, "the dot sums fit in the stages");
  constexpr int BYTES = C::LDS + (H::on ? kHookLds : 0);
  double(*red)[4][BN] = (double(*)[4][BN])tile_lds<BYTES>;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t n = a.n, ldv = a.ldv;
  const T *__restrict__ R = (const T *)a.R;
  const T *__restrict__ Vk = (const T *)a.Vk;
  const int64_t col0 = (int64_t)tn * BN;
  const int m16 = lane & 15, kq = lane >> 4;
  const int64_t wrow0 = (int64_t)tm * BM + 16 * WR * w;  // first row of this wave
  // rows beyond n read row n - 1: their products are discarded (zeroed in the
  // epilogue and in yout)
  const T *Arow[WR];
#pragma unroll
  for (int f = 0; f < WR; ++f) {
    const int64_t arow = wrow0 + 16 * f + m16;
    Arow[f] = R + (arow < n ? arow : n - 1) * a.ldr + VEC * kq;
  }
  // V piece q = (i*4 + w)*64 + lane of a chunk: row q / G, swizzled group q % G
  int64_t vsrc[NVL];
#pragma unroll
  for (int i = 0; i < NVL; ++i) {
    const int q = (i * 4 + w) * 64 + lane;
    const int r = q / C::G, gs = q % C::G;
    vsrc[i] = (int64_t)r * ldv + col0 + (int64_t)(gs ^ C::swz(r)) * VEC;
  }

  const int nfull = (int)((kend - kbeg) / BK);
  const bool ragged = RAG && kbeg + (int64_t)nfull * BK < kend;

  using LdsPtr = __attribute__((address_space(3))) void *;
  auto issue_v = [&](int c, unsigned char *st) {
    const T *vb = Vk + (kbeg + (int64_t)c * BK) * ldv;
#pragma unroll
    for (int i = 0; i < NVL; ++i)
      __builtin_amdgcn_global_load_lds((const void *)(vb + vsrc[i]), (LdsPtr)(st + (i * 4 + w) * 1024), 16, 0, 0);
  };
  auto issue_a = [&](int c, unsigned char *st) {
    const int64_t kc = kbeg + (int64_t)c * BK;
#pragma unroll
    for (int f = 0; f < WR; ++f)
#pragma unroll
      for (int h = 0; h < APL; ++h)
        __builtin_amdgcn_global_load_lds((const void *)(Arow[f] + kc + h * 4 * VEC),
                                         (LdsPtr)(st + C::VBYTES + ((w * WR + f) * APL + h) * 1024), 16, 0, 0);
  };

  auto issue = [&](int c, unsigned char *st) {
    issue_v(c, st);
    issue_a(c, st);
  };

  v4 acc[WR][NSUB];
#pragma unroll
  for (int f = 0; f < WR; ++f)
#pragma unroll
    for (int c = 0; c < NSUB; ++c) acc[f][c] = v4{0, 0, 0, 0};

  // operands of one chunk in registers: this lane's A values (APL 16-byte
  // pieces per slab) and B values (KPL x NSUB)
  struct Frag {
    vec_t a[WR][APL];
    T b[KPL][NSUB];
  };
  auto read_frag = [&](Frag &fr, const unsigned char *st) {
#pragma unroll
    for (int f = 0; f < WR; ++f)
#pragma unroll
      for (int h = 0; h < APL; ++h)
        fr.a[f][h] = *(const vec_t *)(st + C::VBYTES + ((w * WR + f) * APL + h) * 1024 + 16 * lane);
#pragma unroll
    for (int t = 0; t < KPL; ++t)
#pragma unroll
      for (int c2 = 0; c2 < NSUB; ++c2) fr.b[t][c2] = *(const T *)(st + C::voff(C::kcol(kq, t), 16 * c2 + m16));
  };
  auto mfma_frag = [&](const Frag &fr) {
#pragma unroll
    for (int t = 0; t < KPL; ++t)
#pragma unroll
      for (int c2 = 0; c2 < NSUB; ++c2)
#pragma unroll
        for (int f = 0; f < WR; ++f) acc[f][c2] = M::mma(fr.a[f][t / VEC][t % VEC], fr.b[t][c2], acc[f][c2]);
  };

  // Chunk j is loaded into stage j % NST at step j - NST (direct loads) and
  // read into registers at step j - 1, after that step's barrier; step j
  // multiplies it.  Step c: wait until this wave's loads of chunk c + 1 have
  // landed and its reads of chunk c have returned, barrier (every wave's part
  // of chunk c + 1 landed; every wave done reading chunk c, whose stage chunk
  // c + NST now takes), issue chunk c + NST, read chunk c + 1, multiply chunk c.
  // A ragged chunk follows as chunk nfull, its A values loaded into registers
  // at the start, its V rows directly when its stage is free (fewer loads than
  // PER: the waits below, which count full chunks only, then wait for more).
  constexpr int PER = NVL + NAL;  // direct loads per wave per chunk
  Frag fx, fy, fr;
  auto load_ragged = [&] {
    const int64_t k0 = kbeg + (int64_t)nfull * BK;
#pragma unroll
    for (int f = 0; f < WR; ++f)
#pragma unroll
      for (int t = 0; t < KPL; ++t) {
        const int64_t k = k0 + C::kcol(kq, t);
        fr.a[f][t / VEC][t % VEC] = (Arow[f] - VEC * kq)[k < n ? k : n - 1];
      }
  };
  // operands of the epilogue, loaded here and not after the products
  const bool use_m1 = (a.cw != 0.0) && a.Vkm1;
  T pk[PRE ? NSUB : 1][WR][4], pm[PRE ? NSUB : 1][WR][4];
  auto load_epilogue = [&] {
#pragma unroll
    for (int c = 0; c < (PRE ? NSUB : 0); ++c)
#pragma unroll
      for (int f = 0; f < WR; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t off = (wrow0 + 16 * f + M::drow(kq, r)) * ldv + col0 + 16 * c + m16;
          pk[c][f][r] = Vk[off];
          pm[c][f][r] = use_m1 ? ((const T *)a.Vkm1)[off] : T(0);
        }
  };
  if constexpr (H::on) {
    // R does not depend on the step before: its loads go out ahead of the wait
    if (ragged) load_ragged();
    for (int c = 0; c < NST; ++c)
      if (c < nfull) issue_a(c, tile_lds<BYTES> + c * STAGE);
    if (!hook.ready()) {
      dense_wait_vm<0>();
      return false;
    }
    load_epilogue();
    for (int c = 0; c < NST; ++c)
      if (c < nfull + (ragged ? 1 : 0)) issue_v(c, tile_lds<BYTES> + c * STAGE);
  } else {
    if (ragged) load_ragged();
    load_epilogue();
    for (int c = 0; c < NST; ++c) {
      if (c < nfull)
        issue(c, tile_lds<BYTES> + c * STAGE);
      else if (c == nfull && ragged)
        issue_v(c, tile_lds<BYTES> + c * STAGE);
    }
  }
  // wait until at most k chunks' loads of this wave are in flight (k < NST)
  auto wait_chunks = [&](int k) {
    if (NST >= 4 && k >= 3)
      dense_wait_vm<(NST >= 4 ? 3 : 0) * PER>();
    else if (k >= 2)
      dense_wait_vm<2 * PER>();
    else if (k >= 1)
      dense_wait_vm<PER>();
    else
      dense_wait_vm<0>();
  };
  // the same for the first chunks behind a hook, of which only the V loads came last
  auto wait_first = [&](int k) {
    if (k >= 2)
      dense_wait_vm<2 * NVL>();
    else if (k >= 1)
      dense_wait_vm<NVL>();
    else
      dense_wait_vm<0>();
  };
  auto step = [&](int c, int s0, Frag &cur, Frag &nxt) {
    // chunks issued after chunk c + 1: c + 2 .. min(c + NST - 1, nfull - 1)
    const int ahead = nfull - 2 - c < NST - 2 ? nfull - 2 - c : NST - 2;
    if (H::on && c == 0)
      wait_first(ahead);
    else
      wait_chunks(ahead);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's reads of chunk c returned
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (c + NST < nfull)
      issue(c + NST, tile_lds<BYTES> + s0 * STAGE);
    else if (c + NST == nfull && ragged)
      issue_v(nfull, tile_lds<BYTES> + s0 * STAGE);
    if (c + 1 < nfull) read_frag(nxt, tile_lds<BYTES> + (s0 == NST - 1 ? 0 : s0 + 1) * STAGE);
    mfma_frag(cur);
  };
  if (nfull > 0) {
    const int ahead = nfull - 1 < NST - 1 ? nfull - 1 : NST - 1;  // chunk 0 landed
    if (H::on)
      wait_first(ahead);
    else
      wait_chunks(ahead);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_frag(fx, tile_lds<BYTES>);
  }
  int c = 0, s0 = 0;
  for (; c + 1 < nfull; c += 2) {
    step(c, s0, fx, fy);
    s0 = s0 == NST - 1 ? 0 : s0 + 1;
    step(c + 1, s0, fy, fx);
    s0 = s0 == NST - 1 ? 0 : s0 + 1;
  }
  if (c < nfull) {
    step(c, s0, fx, fy);
    s0 = s0 == NST - 1 ? 0 : s0 + 1;
  }
  if (ragged) {
    unsigned char *st = tile_lds<BYTES> + s0 * STAGE;
    dense_wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < KPL; ++t)
#pragma unroll
      for (int c2 = 0; c2 < NSUB; ++c2) fr.b[t][c2] = *(const T *)(st + C::voff(C::kcol(kq, t), 16 * c2 + m16));
    mfma_frag(fr);
  }
  __syncthreads();
  if constexpr (H::on) hook.products_done();

  if (yout) {
#pragma unroll
    for (int c = 0; c < NSUB; ++c)
#pragma unroll
      for (int f = 0; f < WR; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t row = wrow0 + 16 * f + M::drow(kq, r);
          yout[row * ldv + col0 + 16 * c + m16] = row < n ? acc[f][c][r] : T(0);
        }
    return true;
  }
  // ---- epilogue ----
  const T ta = (T)a.scal[S_A];
  const T tb = (T)(a.c2 * a.scal[S_B]);
  const T tc1 = (T)a.c1, tcw = (T)a.cw;
  const T *Vkm1 = (const T *)a.Vkm1;
  const T *__restrict__ G = (const T *)a.G;
  T *Vkp1 = (T *)a.Vkp1;
  const bool want_dot = a.slot >= 0;
  const bool want_gg = a.slot_gg >= 0;
  const bool pair = a.pair != 0;
  const bool want_b = pair && a.slot_b >= 0;
  const bool use_cg = a.cg != nullptr;
  const bool use_g = use_cg || (want_dot && !pair);
  const T tcg = use_cg ? (T)a.cg[0] : T(0);
  // The operands of EC column groups are loaded together before any of their
  // results is stored: V_{k+1} may be written over V_{k-1}, so loads left
  // behind a store wait for it, one memory round trip per element (16 in
  // turn at BN = 64; n = 96 in FP64, 20 steps: estimate 502 -> 396 us).
  static_assert(NSUB % EC == 0, "whole batches of column groups");
#pragma unroll
  for (int cb = 0; cb < NSUB; cb += EC) {
    T vk[EC][WR][4], vm[EC][WR][4], gv[EC][WR][4];
#pragma unroll
    for (int e = 0; e < EC; ++e)
#pragma unroll
      for (int f = 0; f < WR; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t off = (wrow0 + 16 * f + M::drow(kq, r)) * ldv + col0 + 16 * (cb + e) + m16;
          vk[e][f][r] = PRE ? pk[PRE ? cb + e : 0][f][r] : Vk[off];
          vm[e][f][r] = PRE ? pm[PRE ? cb + e : 0][f][r] : use_m1 ? Vkm1[off] : T(0);
          gv[e][f][r] = use_g ? G[off] : vk[e][f][r];
        }
#pragma unroll
    for (int e = 0; e < EC; ++e) {
      const int c = cb + e;
      double ds = 0.0, gs = 0.0, bs = 0.0;
#pragma unroll
      for (int f = 0; f < WR; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int64_t row = wrow0 + 16 * f + M::drow(kq, r);
          const T y = row < n ? ta * acc[f][c][r] : T(0);
          T z = tc1 * y + tb * vk[e][f][r];
          if (use_m1) z += tcw * vm[e][f][r];
          if (use_cg) z += tcg * gv[e][f][r];
          if (Vkp1) Vkp1[row * ldv + col0 + 16 * c + m16] = z;
          if (want_dot) {
            const double g = (double)(pair ? vk[e][f][r] : gv[e][f][r]);
            const double q = (double)(a.dot_y ? y : z);
            ds += g * q;
            if (want_gg) gs += g * g;
            if (want_b) bs += (double)z * q;
          }
        }
      ds = column_sum(ds);
      gs = column_sum(gs);
      bs = column_sum(bs);
      if (kq == 0) {
        red[0][w][16 * c + m16] = ds;
        red[1][w][16 * c + m16] = gs;
        red[2][w][16 * c + m16] = bs;
      }
    }
  }
  if (!want_dot) return true;
  __syncthreads();
  for (int col = tid; col < BN; col += 256) {
    const double s = red[0][0][col] + red[0][1][col] + red[0][2][col] + red[0][3][col];
    a.part[((int64_t)a.slot * a.ntile + tm) * ldv + col0 + col] = s;
    if (want_gg) {
      const double g2 = red[1][0][col] + red[1][1][col] + red[1][2][col] + red[1][3][col];
      a.part[((int64_t)a.slot_gg * a.ntile + tm) * ldv + col0 + col] = g2;
    }
    if (want_b) {
      const double b2 = red[2][0][col] + red[2][1][col] + red[2][2][col] + red[2][3][col];
      a.part[((int64_t)a.slot_b * a.ntile + tm) * ldv + col0 + col] = b2;
    }
  }
  return true;
}

template <typename T, int BN, int WR, bool RAG>
__global__ __launch_bounds__(256) void dense_step_kernel(DenseStepArgs a) {
  const int ntn = (int)(a.ldv / BN);
  const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
  dense_step_tile<T, BN, WR, 4, kChunkLds, false, DenseNoHook, RAG>(a, b / ntn, b % ntn, 0, a.n, nullptr);
}

// Split-K product (a kernel of its own, so the fused kernel's code is not
// shaped by this path): tile order row tile fastest within a K-split, so the
// tiles of one split (same V_k rows) are neighbours.
template <typename T, int BN, int WR, bool RAG>
__global__ __launch_bounds__(256) void dense_step_split_kernel(DenseStepArgs a) {
  const int ntn = (int)(a.ldv / BN);
  const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
  const int ntl = a.ntile * ntn;
  const int ks = b / ntl, t = b % ntl;
  const int64_t kbeg = (int64_t)ks * a.kper;
  const int64_t kend = kbeg + a.kper < a.n ? kbeg + a.kper : a.n;
  T *yout = (T *)a.party + (int64_t)ks * (int64_t)a.ntile * 64 * a.ldv;
  dense_step_tile<T, BN, WR, 4, kChunkLds, false, DenseNoHook, RAG>(a, t / ntn, t % ntn, kbeg, kend, yout);
}

// Split-K epilogue: y = a sum_ks party[ks] (split order), z = c1 y + c2 b V_k
// + cw V_{k-1} (+ cg g), V_{k+1} = z, and the per-probe dots over each
// 16-row tile (part is [slot][nptile][ldv]).  Workgroup = (16 rows, 64
// probes); thread = one probe of 4 rows, its loads of every split issued
// together.
template <typename T>
__global__ __launch_bounds__(256) void dense_split_epilogue_kernel(DenseStepArgs a) {
  __shared__ double red[3][4][64];
  const int tp = blockIdx.x, tid = threadIdx.x, pl = tid & 63, rq = tid >> 6;
  const int64_t ldv = a.ldv, col = (int64_t)blockIdx.y * 64 + pl;
  const int64_t pstride = (int64_t)a.ntile * 64 * ldv;
  const T *P = (const T *)a.party;
  const T *Vk = (const T *)a.Vk, *Vkm1 = (const T *)a.Vkm1, *G = (const T *)a.G;
  T *Vkp1 = (T *)a.Vkp1;
  const T ta = (T)a.scal[S_A];
  const T tb = (T)(a.c2 * a.scal[S_B]);
  const T tc1 = (T)a.c1, tcw = (T)a.cw;
  const bool use_m1 = (a.cw != 0.0) && Vkm1;
  const bool want_dot = a.slot >= 0, want_gg = a.slot_gg >= 0;
  const bool pair = a.pair != 0, want_b = pair && a.slot_b >= 0;
  const bool use_cg = a.cg != nullptr;
  const T tcg = use_cg ? (T)a.cg[0] : T(0);
  int64_t off[4];
  T acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    off[i] = ((int64_t)tp * 16 + rq * 4 + i) * ldv + col;
    acc[i] = T(0);
  }
  const bool use_g = use_cg || (want_dot && !pair);
  double ds = 0.0, gs = 0.0, bs = 0.0;
  // operands of every row before the first store (V_{k+1} may overwrite V_{k-1})
  T vk[4], vm[4], gv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    vk[i] = Vk[off[i]];
    vm[i] = use_m1 ? Vkm1[off[i]] : T(0);
    gv[i] = use_g ? G[off[i]] : vk[i];
  }
  // the partials of four splits in flight together: one round trip in place of
  // four (n = 3001, 100 probes, FP32, 5 splits: 7.3 us a step, now 5.0)
  for (int ks = 0; ks < a.ksplit; ks += 4) {
    T pv[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (ks + j < a.ksplit)
#pragma unroll
        for (int i = 0; i < 4; ++i) pv[j][i] = P[(ks + j) * pstride + off[i]];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (ks + j < a.ksplit)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += pv[j][i];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const T y = ta * acc[i];
    T z = tc1 * y + tb * vk[i];
    if (use_m1) z += tcw * vm[i];
    if (use_cg) z += tcg * gv[i];
    if (Vkp1) Vkp1[off[i]] = z;
    if (want_dot) {
      const double g = (double)(pair ? vk[i] : gv[i]);
      const double q = (double)(a.dot_y ? y : z);
      ds += g * q;
      if (want_gg) gs += g * g;
      if (want_b) bs += (double)z * q;
    }
  }
  if (!want_dot) return;
  red[0][rq][pl] = ds;
  red[1][rq][pl] = gs;
  red[2][rq][pl] = bs;
  __syncthreads();
  if (rq == 0) {
    const double s0 = red[0][0][pl] + red[0][1][pl] + red[0][2][pl] + red[0][3][pl];
    a.part[((int64_t)a.slot * a.nptile + tp) * ldv + col] = s0;
    if (want_gg) {
      const double s1 = red[1][0][pl] + red[1][1][pl] + red[1][2][pl] + red[1][3][pl];
      a.part[((int64_t)a.slot_gg * a.nptile + tp) * ldv + col] = s1;
    }
    if (want_b) {
      const double s2 = red[2][0][pl] + red[2][1][pl] + red[2][2][pl] + red[2][3][pl];
      a.part[((int64_t)a.slot_b * a.nptile + tp) * ldv + col] = s2;
    }
  }
}

// ---------------------------------------------------------------------------
// Small problems: one step in one launch of short workgroups.  The tiled kernel
// above walks K chunk by chunk through LDS, a memory latency per chunk, with
// few workgroups when n is small (n = 512, 50 probes: 16), and a second launch
// adds its K-splits.  Here a workgroup owns 16 rows x 16 NS probes and its
// kDirectWaves waves share out K in chunks of 32 columns; a wave loads its
// operands from memory (L2 at these sizes) straight into MFMA order, two
// chunks' loads in flight together, the waves' sums meet in LDS, and the
// epilogue's operands were loaded before the products began.  What is left is
// about three memory latencies per step.  R is read once per probe group and
// V_k once per row tile, from L2; see dense_direct_tiles for where that stops
// paying.
//
// Lane (m, q) of a wave holds R[row m][k0 + VEC (4 h + q) ..] in piece h, so
// the four lanes of a row read 64 contiguous bytes; MFMA k-slot q of call
// (h, e) is column k0 + VEC (4 h + q) + e, for V_k likewise.
// ---------------------------------------------------------------------------
namespace {
constexpr int kDirectWaves = 8;
}  // namespace

template <typename T, int NS>
__global__ __launch_bounds__(64 * kDirectWaves) void dense_direct_kernel(DenseStepArgs a) {
  using M = Mfma16<T>;
  using v4 = typename M::v4;
  constexpr int W = kDirectWaves, VEC = 16 / (int)sizeof(T), KC = 32, H = KC / (4 * VEC);
  constexpr int PAIRS = 4 * NS;               // (register, probe tile) pairs
  constexpr int PPW = (PAIRS + W - 1) / W;    // pairs finished per wave
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  __shared__ T sums[W][NS][4][64];
  __shared__ double red[3][NS][4][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m16 = lane & 15, kq = lane >> 4;
  const int nct = (a.s + 16 * NS - 1) / (16 * NS);
  const int blk = xcd_remap((int)blockIdx.x, (int)gridDim.x);
  const int tp = blk / nct;                   // 16-row tile
  const int64_t col0 = (int64_t)(blk % nct) * 16 * NS;
  const int64_t n = a.n, ldv = a.ldv;
  const T *__restrict__ R = (const T *)a.R;
  const T *__restrict__ Vk = (const T *)a.Vk;
  const T *Vkm1 = (const T *)a.Vkm1;
  const T *__restrict__ G = (const T *)a.G;
  T *Vkp1 = (T *)a.Vkp1;
  const bool use_m1 = (a.cw != 0.0) && Vkm1;
  const bool pair = a.pair != 0, want_gg = a.slot_gg >= 0, want_b = pair && a.slot_b >= 0;
  const bool use_cg = a.cg != nullptr, use_g = use_cg || !pair;
  // epilogue operands of this wave's pairs: (tile c, register r)
  T vk[PPW], vm[PPW], gv[PPW];
#pragma unroll
  for (int i = 0; i < PPW; ++i) {
    const int q = w + W * i;
    if (q < PAIRS) {
      const int64_t off = ((int64_t)tp * 16 + M::drow(kq, q & 3)) * ldv + col0 + 16 * (q >> 2) + m16;
      vk[i] = Vk[off];
      vm[i] = use_m1 ? Vkm1[off] : T(0);
      gv[i] = use_g ? G[off] : vk[i];
    }
  }
  const int64_t arow = (int64_t)tp * 16 + m16;
  const T *__restrict__ Ar = R + (arow < n ? arow : n - 1) * a.ldr;
  const T *__restrict__ Vc = Vk + col0 + m16;
  v4 acc[NS];
#pragma unroll
  for (int c = 0; c < NS; ++c) acc[c] = v4{0, 0, 0, 0};
  struct Chunk {
    vec_t av[H];
    T bv[H][VEC][NS];
  };
  auto load = [&](Chunk &f, int64_t k0) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int64_t k = k0 + VEC * (4 * h + kq);
      if (k + VEC <= n) {
        f.av[h] = *(const vec_t *)(Ar + k);
      } else {
        // V_k is zero in rows >= n, R's padding is not ours to read
#pragma unroll
        for (int e = 0; e < VEC; ++e) f.av[h][e] = k + e < n ? Ar[k + e] : T(0);
      }
#pragma unroll
      for (int e = 0; e < VEC; ++e)
#pragma unroll
        for (int c = 0; c < NS; ++c) f.bv[h][e][c] = Vc[(k + e) * ldv + 16 * c];
    }
  };
  auto mul = [&](const Chunk &f) {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int e = 0; e < VEC; ++e)
#pragma unroll
        for (int c = 0; c < NS; ++c) acc[c] = M::mma(f.av[h][e], f.bv[h][e][c], acc[c]);
  };
  // chunks w, w + W, ... (rows of V_k exist up to n rounded up to 64)
  const int nch = (int)((n + KC - 1) / KC);
  Chunk f0, f1;
  for (int c = w; c < nch; c += 2 * W) {
    load(f0, (int64_t)c * KC);
    const bool two = c + W < nch;
    if (two) load(f1, (int64_t)(c + W) * KC);
    mul(f0);
    if (two) mul(f1);
  }
#pragma unroll
  for (int c = 0; c < NS; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) sums[w][c][r][lane] = acc[c][r];
  __syncthreads();
  const T ta = (T)a.scal[S_A];
  const T tb = (T)(a.c2 * a.scal[S_B]);
  const T tc1 = (T)a.c1, tcw = (T)a.cw;
  const T tcg = use_cg ? (T)a.cg[0] : T(0);
#pragma unroll
  for (int i = 0; i < PPW; ++i) {
    const int q = w + W * i;
    if (q >= PAIRS) break;
    const int r = q & 3, c = q >> 2;
    const int64_t row = (int64_t)tp * 16 + M::drow(kq, r);
    T sum = sums[0][c][r][lane];
#pragma unroll
    for (int x = 1; x < W; ++x) sum += sums[x][c][r][lane];
    const T y = row < n ? ta * sum : T(0);
    T z = tc1 * y + tb * vk[i];
    if (use_m1) z += tcw * vm[i];
    if (use_cg) z += tcg * gv[i];
    if (Vkp1) Vkp1[row * ldv + col0 + 16 * c + m16] = z;
    const double g = (double)(pair ? vk[i] : gv[i]);
    const double dq = (double)(a.dot_y ? y : z);
    double ds = g * dq, gs = g * g, bs = (double)z * dq;
    ds = column_sum(ds);
    gs = column_sum(gs);
    bs = column_sum(bs);
    if (kq == 0) {
      red[0][c][r][m16] = ds;
      red[1][c][r][m16] = gs;
      red[2][c][r][m16] = bs;
    }
  }
  __syncthreads();
  if (tid < 16 * NS * 3) {
    const int k = tid / (16 * NS), col = tid % (16 * NS);
    const int32_t slot = k == 0 ? a.slot : (k == 1 ? a.slot_gg : a.slot_b);
    if (k == 0 || (k == 1 ? want_gg : want_b)) {
      const double(*x)[16] = red[k][col >> 4];
      const int m = col & 15;
      a.part[((int64_t)slot * a.nptile + tp) * ldv + col0 + col] = x[0][m] + x[1][m] + x[2][m] + x[3][m];
    }
  }
}

// ---------------------------------------------------------------------------
// Matrices that fit in the registers of one workgroup (n <= 192): a launch per step or per power product costs more than its work
// (n = 96 in FP64: 3.7 us and 4.2 us a launch, and about 1 us between two).
// The probes are independent, so a workgroup runs the whole recurrence of 16
// of them with no exchange beyond its own barrier, R held in MFMA order in the
// registers of its waves (wave w: rows 16 w .., n padded to 32), V_k in LDS, V_{k-1} and the
// wave's own rows of V_k in registers; one barrier per step.  One workgroup
// likewise runs the whole power method, a few threads to a row.
// ---------------------------------------------------------------------------
template <typename T, int NP>
__global__ __launch_bounds__(4 * NP) void dense_resident_kernel(DenseResidentArgs a) {
  using M = Mfma16<T>;
  using v4 = typename M::v4;
  constexpr int NT = NP / 4;  // k-steps of four columns
  __shared__ T V[2][NP * 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m16 = lane & 15, kq = lane >> 4;
  const int64_t n = a.n, ldv = a.ldv, col = (int64_t)blockIdx.x * 16 + m16;
  const int row0 = 16 * w;
  T ra[NT];
  {
    const int64_t r = row0 + m16;
    const T *Rr = (const T *)a.R + (r < n ? r : 0) * a.ldr;
#pragma unroll
    for (int t = 0; t < NT; ++t) ra[t] = r < n && 4 * t + kq < n ? Rr[4 * t + kq] : T(0);
  }
  const bool clen = a.method == FINAL_CLENSHAW, pair = a.pair != 0;
  T g[4], vk[4], vm[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    g[r] = ((const T *)a.G)[(int64_t)(row0 + M::drow(kq, r)) * ldv + col];
    vk[r] = clen ? T(0) : g[r];
    vm[r] = T(0);
    V[0][(row0 + M::drow(kq, r)) * 16 + m16] = vk[r];
  }
  const double sa = a.scal[S_A], sb = a.scal[S_B];
  const T ta = (T)sa;
  __syncthreads();
  // column sums of a value over the wave's 16 rows, into the wave's tile of a slot
  auto put = [&](int32_t slot, double x) {
    x = column_sum(x);
    if (kq == 0) a.part[((int64_t)slot * (NP / 16) + w) * ldv + col] = x;
  };
  for (int k = 0; k < a.nsteps; ++k) {
    StepRule q{};
    T cg = T(0);
    if (clen) {
      q.c1 = 2.0; q.c2 = -2.0; q.cw = -1.0;  // y_{m+2} = 0 on the first step
      q.slot = a.m - k;
      q.slot_gg = k == 0 ? a.m + 1 : -1;
      q.slot_b = -1;
      cg = (T)a.scal[S_ALPHA + a.m - k];
    } else {
      q = step_rule(a.method, a.m, k, pair ? 2 * a.nsteps : a.nsteps, pair);
    }
    const T *Vb = V[k & 1];
    v4 acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < NT; t += 2) {
      acc0 = M::mma(ra[t], Vb[(4 * t + kq) * 16 + m16], acc0);
      acc1 = M::mma(ra[t + 1], Vb[(4 * t + 4 + kq) * 16 + m16], acc1);
    }
    const T c1 = (T)q.c1, tb = (T)(q.c2 * sb), cw = (T)q.cw;
    double ds = 0.0, gs = 0.0, bs = 0.0;
    T *Vo = V[(k + 1) & 1];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const T y = ta * (acc0[r] + acc1[r]);
      T z = c1 * y + tb * vk[r];
      z += cw * vm[r];
      if (clen) z += cg * g[r];
      const double p = (double)(pair ? vk[r] : g[r]), dq = (double)(q.dot_y ? y : z);
      ds += p * dq;
      gs += p * p;
      bs += (double)z * dq;
      Vo[(row0 + M::drow(kq, r)) * 16 + m16] = z;
      vm[r] = vk[r];
      vk[r] = z;
    }
    put(q.slot, ds);
    if (q.slot_gg >= 0) put(q.slot_gg, gs);
    if (q.slot_b >= 0) put(q.slot_b, bs);
    __syncthreads();
  }
}

template <typename T>
hipError_t launch_dense_resident(const DenseResidentArgs &a, hipStream_t st) {
  if (a.n < 1 || a.n > kDenseResidentMax || a.s < 1 || (a.s + 15) / 16 * 16 > a.ldv ||
      a.nsteps < 1 || (a.pair && a.method == FINAL_CLENSHAW))
    return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((a.s + 15) / 16);
  switch (dense_resident_tiles(a.n)) {
    case 2: dense_resident_kernel<T, 32><<<grid, 128, 0, st>>>(a); break;
    case 4: dense_resident_kernel<T, 64><<<grid, 256, 0, st>>>(a); break;
    case 6: dense_resident_kernel<T, 96><<<grid, 384, 0, st>>>(a); break;
    case 8: dense_resident_kernel<T, 128><<<grid, 512, 0, st>>>(a); break;
    case 10: dense_resident_kernel<T, 160><<<grid, 640, 0, st>>>(a); break;
    default: dense_resident_kernel<T, 192><<<grid, 768, 0, st>>>(a); break;
  }
  return hipGetLastError();
}
template hipError_t launch_dense_resident<double>(const DenseResidentArgs &, hipStream_t);
template hipError_t launch_dense_resident<float>(const DenseResidentArgs &, hipStream_t);

// TPR threads per row of R, columns sub, sub + TPR, ... each.  The iterate of
// product k is scaled by the norm of product k - 1, as in the launches per
// product; the products of a trial follow each other over one barrier.
template <typename T, int NP, int TPR>
__global__ __launch_bounds__(NP * TPR) void power_resident_kernel(const T *__restrict__ R, int64_t ldr, int64_t n,
                                                                  int32_t t, int32_t q, uint64_t seed,
                                                                  double *__restrict__ scal) {
  constexpr int C = NP / TPR, NW = NP * TPR / 64;
  __shared__ double xs[2][NP], red[2][NW], fin[2][NW];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int row = tid / TPR, sub = tid % TPR;
  T r[C];
#pragma unroll
  for (int i = 0; i < C; ++i) r[i] = row < n && sub + TPR * i < n ? R[row * ldr + sub + TPR * i] : T(0);
  for (int32_t trial = 0; trial < q; ++trial) {
    __syncthreads();
    if (sub == 0) xs[0][row] = row < n ? rademacher(seed, 1u, row, trial) : 0.0;
    __syncthreads();
    double sc = 1.0;
    for (int32_t it = 0; it <= t; ++it) {
      const double *x = xs[it & 1];
      double a0 = 0.0, a1 = 0.0;
#pragma unroll
      for (int i = 0; i < C; i += 2) {
        a0 += (double)r[i] * x[sub + TPR * i];
        a1 += (double)r[i + 1] * x[sub + TPR * (i + 1)];
      }
      double s0 = a0 + a1;
#pragma unroll
      for (int off = 1; off < TPR; off <<= 1) s0 += __shfl_xor(s0, off, 64);
      const double yv = sub == 0 ? sc * s0 : 0.0;
      const double yy = wave_sum(yv * yv);
      if (lane == 0) red[it & 1][w] = yy;
      if (sub == 0) xs[(it + 1) & 1][row] = yv;
      if (it == t) {
        const double xv = sub == 0 ? sc * x[row] : 0.0;
        const double xy = wave_sum(xv * yv), xx = wave_sum(xv * xv);
        if (lane == 0) {
          fin[0][w] = xy;
          fin[1][w] = xx;
        }
      }
      __syncthreads();
      double nn = 0.0;
#pragma unroll
      for (int i = 0; i < NW; ++i) nn += red[it & 1][i];
      sc = 1.0 / sqrt(nn);
    }
    if (tid == 0) {
      double xy = 0.0, xx = 0.0;
      for (int i = 0; i < NW; ++i) {
        xy += fin[0][i];
        xx += fin[1][i];
      }
      const double rq = xy / xx;
      if (trial == 0 || rq > scal[S_P1]) scal[S_P1] = rq;
    }
  }
}

template <typename T>
hipError_t launch_power_resident(const T *R, int64_t ldr, int64_t n, int32_t t, int32_t q, uint64_t seed,
                                 double *scal, hipStream_t st) {
  const int64_t np = (n + 63) / 64 * 64;
  if (n < 1 || n > kDenseResidentMax || q < 1 || t < 0) return hipErrorInvalidValue;
  if (np == 64)
    power_resident_kernel<T, 64, 16><<<1, 1024, 0, st>>>(R, ldr, n, t, q, seed, scal);
  else if (np == 128)
    power_resident_kernel<T, 128, 8><<<1, 1024, 0, st>>>(R, ldr, n, t, q, seed, scal);
  else
    power_resident_kernel<T, 192, 4><<<1, 768, 0, st>>>(R, ldr, n, t, q, seed, scal);
  return hipGetLastError();
}
template hipError_t launch_power_resident<double>(const double *, int64_t, int64_t, int32_t, int32_t, uint64_t,
                                                  double *, hipStream_t);
template hipError_t launch_power_resident<float>(const float *, int64_t, int64_t, int32_t, int32_t, uint64_t,
                                                 double *, hipStream_t);

template <typename T>
static hipError_t launch_dense_direct(const DenseStepArgs &a, hipStream_t st) {
  constexpr int VEC = 16 / (int)sizeof(T);
  if (a.slot < 0 || a.s < 1 || a.s > a.ldv || a.nptile != a.ntile * 4 || a.ldr % VEC != 0 ||
      ((uintptr_t)a.R % 16) != 0 || (a.s + 16 * a.direct - 1) / (16 * a.direct) * (16 * a.direct) > a.ldv)
    return hipErrorInvalidValue;
  const unsigned grid = (unsigned)(a.nptile * ((a.s + 16 * a.direct - 1) / (16 * a.direct)));
  switch (a.direct) {
    case 1: dense_direct_kernel<T, 1><<<grid, 64 * kDirectWaves, 0, st>>>(a); break;
    case 2: dense_direct_kernel<T, 2><<<grid, 64 * kDirectWaves, 0, st>>>(a); break;
    case 4: dense_direct_kernel<T, 4><<<grid, 64 * kDirectWaves, 0, st>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// One round of workgroups, as narrow as that allows (narrow ones are the
// quicker: at n = 512, 50 probes, FP64 6.6 us a step with 16 probes each, 7.9
// with 32, 12.3 with 64; past one round a second one costs as much as the
// first: n = 1400, 50 probes 16.7 us with 352 workgroups, 15.6 with 176), and
// up to 4.2e8 elements n^2 s, where the tiled kernel's reuse of R and V_k from
// LDS overtakes.  Both sides, us a step, direct against tiled, FP64 (FP32 alike):
// n = 96, 32 probes 4 / 10; 512, 50: 6.6 / 15.8; 1024, 128: 13.3 / 27.6;
// 1800, 128 (4.1e8): 30.7 / 44.0; 2048, 128 (5.4e8): 35.3 / 31.3; 1400, 256
// (5.0e8): 39.4 / 37.3; 3000, 50 (5.8e8): 42.7 / 36.9.
int32_t dense_direct_tiles(int64_t n, int32_t s) {
  const int64_t rows = (n + 63) / 64 * 4, probes = (s + 15) / 16;
  if ((double)n * (double)n * 16.0 * (double)probes > 4.2e8) return 0;
  for (int32_t ns = 1; ns <= 4; ns *= 2)
    if (rows * ((probes + ns - 1) / ns) <= 256) return ns;
  return 0;
}

// Workgroups run in rounds of one per compute unit, so a split is paid by its
// rounds times its rows (16 more for filling the pipeline and storing the
// partials), and the last of an odd number of rounds, alone on its compute
// unit, an eighth more (n = 8192, 256 probes FP64: 623 us a step in one round,
// 550 in two); each split adds its partials to the epilogue's reads.  Of the
// splits up to the smallest power of two that gives the chip 512 workgroups the
// cheapest one.  Power of two against this rule, us a step, FP32 and FP64:
// n = 2200, 128 probes 31.9 / 24.3 and 51.2 / 36.7 (8 and 7 splits); 2500, 200:
// 47.7 / 42.2 and 80.6 / 73.4 (8, 6); 3001, 100: 38.2 / 33.4 and 63.5 / 56.4
// (8, 5); 4500, 256: 132.8 / 114.0 and 246 / 210 (4, 3); 7000, 100: 139 / 129
// and 254 / 244 (8, 4); 4096, 64 and 8192, 256 stay.
int32_t dense_step_splits(int64_t n, int32_t ntile, int64_t ldv, int32_t bn) {
  const int64_t tiles = (int64_t)ntile * (ldv / bn);
  int32_t most = 1;
  while (tiles * most < 512 && most < 16 && n / (2 * most) >= 256) most *= 2;
  int32_t ks = most;
  int64_t least = INT64_MAX;
  for (int32_t k = most > 1 ? 2 : 1; k <= most; ++k) {
    const int64_t kper = ((n + k - 1) / k + 31) / 32 * 32, rounds = (tiles * k + 255) / 256;
    const int64_t cost = (8 * rounds + rounds % 2) * (kper + 16) + 32 * k;
    if (cost < least) {
      least = cost;
      ks = k;
    }
  }
  return ks;
}

// Step k of a batch's matrix as arguments of the tile body; false: the matrix
// has no step k.
template <typename T>
__device__ __forceinline__ bool batch_dense_args(const BatchPersistArgs &pa, const BatchMat &M, int k,
                                                 DenseStepArgs &a) {
  const bool pair = batch_pairs(M);
  if (pair && k >= (pa.nsteps + 1) / 2) return false;
  const StepRule r = step_rule(pa.method, pa.m, k, pa.nsteps, pair);
  const T *bufs[3] = {(const T *)pa.G + M.voff, (const T *)pa.VA + M.voff, (const T *)pa.VB + M.voff};
  a.R = M.R;
  a.ldr = M.ldr;
  a.n = M.n;
  a.ldv = pa.ldv;
  a.Vk = bufs[r.vk];
  a.Vkm1 = r.vkm1 >= 0 ? bufs[r.vkm1] : nullptr;
  a.Vkp1 = r.vout >= 0 ? (void *)bufs[r.vout] : nullptr;
  a.G = bufs[0];
  a.scal = M.scal;
  a.c1 = r.c1; a.c2 = r.c2; a.cw = r.cw;
  a.dot_y = r.dot_y; a.slot = r.slot; a.slot_gg = r.slot_gg;
  a.pair = pair; a.slot_b = r.slot_b;
  a.part = pa.part + M.poff;
  a.ntile = M.ntile;
  a.bn = 64;
  return true;
}

// Grouped step over a batch: block -> (matrix, row tile) from the tile table
// (x) and 64 probes (y).
template <typename T, int WR>
__global__ __launch_bounds__(256) void batch_dense_step_kernel(BatchPersistArgs pa, int k, const int2 *tiles) {
  constexpr int BUDGET = sizeof(T) == 4 ? kGroupedLds : kChunkLds;
  const int2 tl = tiles[blockIdx.x];
  DenseStepArgs a{};
  if (!batch_dense_args<T>(pa, pa.mats[tl.x], k, a)) return;
  dense_step_tile<T, 64, WR, kBatchCols<WR>, BUDGET>(a, tl.y, (int)blockIdx.y, 0, a.n, nullptr);
}

// Persistent batch steps: each workgroup takes (matrix, row tile, step)
// items in schedule order, waits for the matrix's previous step, runs the
// tile body of the grouped kernel with that step's recurrence, publishes it.
// An item is short (64 rows of n <= 2048: 30 us of products), so what stands
// around its products counted as much again: 6 us for the next item, 4 for the
// first chunk, 3 for a ragged last one, 13 in the epilogue.  The next item is
// reserved before the epilogue, R's first chunks and the ragged chunk's values
// are on their way during the wait, FP32 tiles hold the epilogue's V_k and
// V_{k-1} in registers from the start (FP64 has none left), and the matrix's
// description is in scalar registers.  64 matrices, n <= 2048, 64 probes, FP32:
// 160 -> 127 us a step (two workgroups on a CU; three of 16-column chunks: 193,
// an XCD has 126 tiles a step and they wait for each other).
template <typename T, int WR>
__global__ __launch_bounds__(256, 2) void batch_dense_persistent_kernel(BatchPersistArgs pa) {
  constexpr int LDS = DenseChunk<T, 64, WR>::LDS;
  int *sh = (int *)(tile_lds<LDS + kHookLds> + LDS);
  int next = sched_reserve(pa.sched);
  for (;;) {
    const int i = sched_item(pa.sched, next, sh);
    if (i < 0) return;
    const int4 it = uniform_load(pa.sched.items + i);
    const BatchMat M = uniform_load(pa.mats + it.x);
    DenseStepArgs a{};
    if (!batch_dense_args<T>(pa, M, it.z, a)) {  // nor has the matrix any later step
      next = sched_reserve(pa.sched);
      __syncthreads();  // every wave has read sh[0]
      continue;
    }
    a.ldv = 64;
    BatchHook hook{pa.sched, it.x, it.z * M.ntile, sh + 1, &next};
    if (!dense_step_tile<T, 64, WR, kBatchCols<WR>, kChunkLds, sizeof(T) == 4 && WR == 1, BatchHook>(a, it.y, 0, 0, a.n, nullptr,
                                                                                                           hook))
      return;
    sched_release(pa.sched, it.x);
  }
}

template <typename T>
hipError_t launch_batch_dense_persistent(const BatchPersistArgs &pa, int32_t wr, int32_t grid,
                                         hipStream_t st) {
  if (pa.ldv != 64 || grid < 1) return hipErrorInvalidValue;
  if (wr == 1)
    batch_dense_persistent_kernel<T, 1><<<(unsigned)grid, 256, 0, st>>>(pa);
  else if (wr == 2)
    batch_dense_persistent_kernel<T, 2><<<(unsigned)grid, 256, 0, st>>>(pa);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}
template hipError_t launch_batch_dense_persistent<double>(const BatchPersistArgs &, int32_t, int32_t, hipStream_t);
template hipError_t launch_batch_dense_persistent<float>(const BatchPersistArgs &, int32_t, int32_t, hipStream_t);

// Resident workgroups of the persistent step kernels (CUs x occupancy).
int32_t batch_persistent_grid(int32_t precision, int32_t wr, int64_t ldv) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  hipError_t e = hipErrorInvalidValue;
  if (precision == 0)
    e = wr == 2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, batch_dense_persistent_kernel<double, 2>, 256, 0)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, batch_dense_persistent_kernel<double, 1>, 256, 0);
  else if (precision == 1)
    e = wr == 2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, batch_dense_persistent_kernel<float, 2>, 256, 0)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, batch_dense_persistent_kernel<float, 1>, 256, 0);
  else
    return bf16x3_persistent_grid(ldv);
  if (e != hipSuccess) return 0;
  return cus * (per > 0 ? per : 1);
}

template <typename T>
hipError_t launch_dense_split_epilogue(const DenseStepArgs &a, hipStream_t st) {
  if (a.ksplit < 2 || !a.party || a.nptile != a.ntile * 4) return hipErrorInvalidValue;
  dense_split_epilogue_kernel<T><<<dim3((unsigned)a.nptile, (unsigned)(a.ldv / 64)), 256, 0, st>>>(a);
  return hipGetLastError();
}
template hipError_t launch_dense_split_epilogue<double>(const DenseStepArgs &, hipStream_t);
template hipError_t launch_dense_split_epilogue<float>(const DenseStepArgs &, hipStream_t);

// FP64 with n a multiple of the chunk: the instance without a ragged one, whose
// branches in every step cost 1 to 2% (n = 8192, 256 probes 594.7 us a step with
// them, 585.5 without; 4096, 64 46.4 / 45.4; 2200, 128 31.5 / 30.8).  FP32 gains
// nothing by it (8192, 256 304 / 306).
template <typename T, int BN, bool RAG>
static void dense_step_launch_as(const DenseStepArgs &a, unsigned grid, hipStream_t st) {
  if (a.ksplit > 1)
    dense_step_split_kernel<T, BN, 1, RAG><<<grid, 256, 0, st>>>(a);
  else
    dense_step_kernel<T, BN, 1, RAG><<<grid, 256, 0, st>>>(a);
}
template <typename T, int BN>
static void dense_step_launch(const DenseStepArgs &a, unsigned grid, hipStream_t st) {
  if (sizeof(T) == 8 && a.n % DenseChunk<T, BN, 1>::BK == 0)
    dense_step_launch_as<T, BN, sizeof(T) != 8>(a, grid, st);
  else
    dense_step_launch_as<T, BN, true>(a, grid, st);
}

template <typename T>
hipError_t launch_dense_step(const DenseStepArgs &a, hipStream_t st, bool epilogue) {
  if (a.direct > 0) return launch_dense_direct<T>(a, st);
  const int ntn = (int)(a.ldv / a.bn);
  if (a.ksplit > 1 && (!a.party || a.kper % 32 != 0 || (int64_t)a.ksplit * a.kper < a.n ||
                       a.nptile != a.ntile * 4))
    return hipErrorInvalidValue;
  const unsigned grid = (unsigned)(a.ntile * ntn * (a.ksplit > 1 ? a.ksplit : 1));
  switch (a.bn) {
    case 64: dense_step_launch<T, 64>(a, grid, st); break;
    case 128: dense_step_launch<T, 128>(a, grid, st); break;
    case 256: dense_step_launch<T, 256>(a, grid, st); break;
    default: return hipErrorInvalidValue;
  }
  if (a.ksplit > 1 && epilogue) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_dense_split_epilogue<T>(a, st);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_dense_step(const BatchPersistArgs &pa, int32_t k, const int2 *tiles, int32_t ntiles,
                                   int32_t wr, hipStream_t st) {
  if (pa.ldv % 64 != 0 || ntiles < 1) return hipErrorInvalidValue;
  const dim3 grid((unsigned)ntiles, (unsigned)(pa.ldv / 64));
  if (wr == 1)
    batch_dense_step_kernel<T, 1><<<grid, 256, 0, st>>>(pa, k, tiles);
  else if (wr == 2)
    batch_dense_step_kernel<T, 2><<<grid, 256, 0, st>>>(pa, k, tiles);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}
template hipError_t launch_batch_dense_step<double>(const BatchPersistArgs &, int32_t, const int2 *, int32_t, int32_t,
                                                     hipStream_t);
template hipError_t launch_batch_dense_step<float>(const BatchPersistArgs &, int32_t, const int2 *, int32_t, int32_t,
                                                    hipStream_t);
template hipError_t launch_dense_step<double>(const DenseStepArgs &, hipStream_t, bool);
template hipError_t launch_dense_step<float>(const DenseStepArgs &, hipStream_t, bool);

}  // namespace ent
