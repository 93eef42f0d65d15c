// Latent write for new tokens: z = x L (Sec. III-A write
// side; per-group L_g of Sec. III-C; whole-projection L_v of Sec. III-D),
// accumulated in fp32, rounded to nearest-even into the paged pool.
//
// Output column space of one token: [0, R_Kp + r_v)
//   c <  R_K          key column c           -> page key part (chunk-major)
//   R_K <= c < R_Kp   key-row padding         -> written as zero
//   c >= R_Kp         value column c - R_Kp   -> page value part, tile-major
#include <algorithm>

#include "device.h"
#include "internal.h"

namespace dckv {
namespace {

// Chunk-major key part: column c of slot s at (c/32)*2048 + s*32 + c%32.
__device__ __forceinline__ int64_t key_elem(int s, int c) {
  return int64_t(c >> 5) * (32 * DCKV_PAGE_TOKENS) + s * 32 + (c & 31);
}

// Tile-major value part (from the value base): column j of slot s at
// (j/16)*1024 + (s/32)*512 + (j%16)*32 + s%32.
__device__ __forceinline__ int64_t value_elem(int s, int j) {
  return int64_t(j >> 4) * (16 * DCKV_PAGE_TOKENS) + (s >> 5) * 512 + (j & 15) * 32 + (s & 31);
}

constexpr int kTileTok = 64;
constexpr int kTileCol = 64;
constexpr int kTileK = 16;

// Portable VALU kernel (where m is a multiple of neither 64, bf16, nor 16,
// fp32): 64 tokens x 64 columns per 256-thread block, 4x4 outputs a thread.
template <typename T>
__global__ __launch_bounds__(256) void append_valu(const T* __restrict__ x, const T* __restrict__ Lk,
                                                   const T* __restrict__ Lv,
                                                   const int64_t* __restrict__ slot,
                                                   T* __restrict__ pool, int n_tok, int m, int RK,
                                                   int RKp, int rv, int64_t page_elems,
                                                   int64_t value_base, int64_t num_pages) {
  __shared__ float xs[kTileK][kTileTok + 4];
  __shared__ float ls[kTileK][kTileCol + 4];
  const int tid = threadIdx.x;
  const int tx = tid % 16, ty = tid / 16;
  const int tok0 = blockIdx.y * kTileTok;
  const int col0 = blockIdx.x * kTileCol;
  const int ncols = RKp + rv;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  for (int k0 = 0; k0 < m; k0 += kTileK) {
    for (int e = tid; e < kTileTok * kTileK; e += 256) {
      const int tt = e / kTileK, kk = e % kTileK;
      const int tok = tok0 + tt, k = k0 + kk;
      xs[kk][tt] = (tok < n_tok && k < m) ? to_f32(x[int64_t(tok) * m + k]) : 0.f;
    }
    for (int e = tid; e < kTileK * kTileCol; e += 256) {
      const int cc = e / kTileK, kk = e % kTileK;
      const int c = col0 + cc, k = k0 + kk;
      float v = 0.f;
      if (k < m) {
        if (c < RK)
          v = to_f32(Lk[int64_t(c) * m + k]);
        else if (c >= RKp && c < ncols)
          v = to_f32(Lv[int64_t(c - RKp) * m + k]);
      }
      ls[kk][cc] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < kTileK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = xs[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = ls[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }

  const int64_t slot_end = num_pages * DCKV_PAGE_TOKENS;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int tok = tok0 + ty * 4 + i;
    if (tok >= n_tok) continue;
    const int64_t sl = slot[tok];
    if (sl < 0 || sl >= slot_end) continue;
    T* pg = pool + (sl / DCKV_PAGE_TOKENS) * page_elems;
    const int s = int(sl % DCKV_PAGE_TOKENS);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = col0 + tx * 4 + j;
      if (c >= ncols) continue;
      if (c < RK)
        pg[key_elem(s, c)] = from_f32<T>(acc[i][j]);
      else if (c < RKp)
        pg[key_elem(s, c)] = from_f32<T>(0.f);
      else
        pg[value_base + value_elem(s, c - RKp)] = from_f32<T>(acc[i][j]);
    }
  }
}

// bf16 MFMA kernel (m a multiple of 64).  Output C[token][column] =
// sum_k x[token][k] * LT[column][k]: both operands are contiguous in k.
// Work-group tile BM tokens x BN columns.  k advances in stages of 64.  A
// stage (both tiles, BM + BN rows x 128 B) is copied from global memory
// straight into LDS by the loads' LDS path (no registers, no LDS store
// instructions): one wave instruction moves 8 rows x 128 B, whole cache
// lines, to 1 KB of LDS in lane order, and the lane -> 16-byte piece map is
// xor-swizzled by the row (LDS piece p of row r holds global piece p ^ (r %
// 8)) so that the 16 rows an MFMA operand load touches fall in distinct
// banks.  NB stage buffers: the loads run NB - 1 stages ahead, and one barrier
// a stage (after the wave's own loads of that stage and its LDS reads of the
// stage before have completed) both publishes the stage and frees the buffer
// the next loads refill.  Eight waves, two a SIMD (one wave alone cannot keep
// the matrix pipe busy across the per-stage barrier), as WR x WC positions of
// 16 TM tokens x 16 TN columns times KH parts of a stage's k: with KH = 2 the
// two waves of a position take 32 k each, which halves the operands read from
// LDS for a product, and exchange halves of their sums at the end (each sum
// lower part + upper part).
// Work-group ids that are equal mod 8 run on one XCD; the id -> tile map gives
// each XCD a run of consecutive tiles, numbered in bands of eight token tiles
// with the token tiles of one column tile adjacent, so that the XCD's
// work-groups share few token and column tiles in its L2 (numbered column tile
// by column tile instead, 4093 tokens x 4096 columns took 336 us for 233 on
// 128 x 64 tiles).  Rows past the token count or the column space are clamped
// to valid rows and their results discarded, so no load leaves its matrix.
// Bound by the compute unit's own pipes: a 64-wide stage of 128 x 256 takes
// 1370 cycles with few work-groups on the chip, its products 1024, its operand
// reads and stage writes in LDS 1400, its loads' addresses 768; with every
// compute unit busy 4093 x 4096 x 4096 takes 143 us (0.96 PFLOP/s).
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kBK = 64;                   // k a stage (one 128-byte line a row)
constexpr int kThreads = 512;
constexpr int kBand = 8;                  // token tiles of a band
constexpr int kComputeUnits = 256;        // MI355X

// 16 bytes a lane from global memory to LDS, in lane order from p on.
__device__ __forceinline__ void load_lds16(const bf16* g, unsigned char* p) {
  __builtin_amdgcn_global_load_lds(g, p, 16, 0, 0);
}

// id -> (token tile, column tile)
__device__ __forceinline__ void append_tile_of(int id, int n_tok_tiles, int n_col_tiles, int& tt,
                                               int& ct) {
  const int n_tiles = n_tok_tiles * n_col_tiles;
  const int xcd = id & 7, per = n_tiles >> 3, extra = n_tiles & 7;
  const int lin = xcd * per + min(xcd, extra) + (id >> 3);
  const int band = lin / (kBand * n_col_tiles), t0 = band * kBand;
  const int in = lin - t0 * n_col_tiles, bt = min(kBand, n_tok_tiles - t0);
  ct = in / bt;
  tt = t0 + in - ct * bt;
}

template <int WR, int WC, int KH, int TM, int TN, int NB>
__global__ __launch_bounds__(kThreads, 1) void append_mfma(
    const bf16* __restrict__ x, const bf16* __restrict__ LkT, const bf16* __restrict__ LvT,
    const int64_t* __restrict__ slot, bf16* __restrict__ pool, int n_tok, int m, int RK, int RKp,
    int rv, int64_t page_elems, int64_t value_base, int64_t num_pages, int n_tok_tiles,
    int n_col_tiles) {
  static_assert(WR * WC * KH == 8, "eight waves");
  constexpr int BM = 16 * TM * WR, BN = 16 * TN * WC;
  constexpr int BUF = (BM + BN) * kBK * 2;             // one stage
  constexpr int LPW = (BM + BN) / 64;                  // 8-row loads a wave a stage
  static_assert((BM + BN) % 64 == 0 && BM % 8 == 0, "whole 8-row blocks a wave");
  static_assert(KH == 1 || 8 * (TM * TN / 2) * 1024 <= NB * BUF, "the exchange fits the stage buffers");
  extern __shared__ __align__(1024) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int ncols = RKp + rv;
  int tt, ct;
  append_tile_of(blockIdx.x, n_tok_tiles, n_col_tiles, tt, ct);
  const int tok0 = tt * BM, col0 = ct * BN;
  const int pos = w % (WR * WC), kh = w / (WR * WC);
  const int wm = 16 * TM * (pos % WR);                 // this wave's first token
  const int wn = 16 * TN * (pos / WR);                 // and column

  // loads: wave w fills 8-row blocks LPW w .. of a stage (the x blocks, then
  // the L blocks); lane: row lane / 8 of its block, LDS piece lane % 8, which
  // holds global piece (lane % 8) ^ (row % 8)
  const int lrow = lane >> 3, gpiece = (lane & 7) ^ lrow;
  const bf16* gsrc[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int blk = LPW * w + j;
    const bf16* r;
    if (blk < BM / 8) {
      const int t = min(tok0 + 8 * blk + lrow, n_tok - 1);
      r = x + int64_t(t) * m;
    } else {
      const int c = col0 + 8 * (blk - BM / 8) + lrow;
      if (c < RK)
        r = LkT + int64_t(c) * m;
      else if (c < RKp)
        r = LkT;                                // padding column: written as zero below
      else
        r = LvT + int64_t(min(c - RKp, rv - 1)) * m;
    }
    gsrc[j] = r + 8 * gpiece;
  }
  const int nst = m / kBK;
  auto issue = [&](int st, unsigned char* buf, int j) {   // past the end: re-read the last stage
    load_lds16(gsrc[j] + min(st, nst - 1) * kBK, buf + (LPW * w + j) * 1024);
  };

  floatx4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};

  // A stage is P phases of 32 k a wave; the operands of a phase are read while
  // the products of the phase before run (two register sets).
  constexpr int P = 2 / KH;
  u32x4_t a[2][TM], b[2][TN];
  auto read = [&](int set, int ph, unsigned char* buf) {
    const int kp = 4 * (KH == 2 ? kh : ph) + lq;      // this lane's 16-byte k piece
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int row = wn + 16 * j + lr;
      b[set][j] = *reinterpret_cast<const u32x4_t*>(buf + BM * 128 + row * 128 + 16 * (kp ^ (row & 7)));
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = wm + 16 * i + lr;
      a[set][i] = *reinterpret_cast<const u32x4_t*>(buf + row * 128 + 16 * (kp ^ (row & 7)));
    }
  };
  // the products of a phase, with loads j0 .. j1 - 1 of stage st into buf
  // between them: eight waves' loads issued together keep the address unit
  // busy (16 cycles a load) for as long as a phase's products take, and a
  // wave's products wait behind its loads
  auto multiply = [&](int set, int st, unsigned char* buf, int j0, int j1) {
    constexpr int N = TM * TN;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int i = q / TN, j = q % TN;
#pragma unroll
      for (int l = j0; l < j1; ++l)
        if ((l - j0) * N / (j1 - j0) == q) {
          __builtin_amdgcn_sched_barrier(0);
          issue(st, buf, l);
          __builtin_amdgcn_sched_barrier(0);
        }
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[set][i]),
                                                          __builtin_bit_cast(bf16x8_t, b[set][j]),
                                                          acc[i][j], 0, 0, 0);
    }
  };
  // stage st lies in cur, the next one in nxt; set: the register set that
  // holds the operands of st's first phase.  With two phases the loads that
  // refill a buffer are spread over the second phase of its stage and the
  // first of the next.
  constexpr int J1 = P == 1 ? LPW : (LPW + 1) / 2;
  auto stage = [&](int st, int set, unsigned char* prv, unsigned char* cur, unsigned char* nxt) {
    if constexpr (P == 2) {
      read((set + 1) & 1, 1, cur);
      __builtin_amdgcn_sched_barrier(0);
      multiply(set & 1, st - 1 + NB, prv, J1, LPW);
    }
    // wait until this wave's loads of the next stage (the oldest of the NB - 1
    // in flight) and its LDS reads of this one are done, then meet the other
    // waves: the next stage is whole and cur is free.  The asm is a compiler
    // barrier too, so no LDS access moves across it.
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(LPW * (NB - 2)) : "memory");
    read((set + P) & 1, 0, nxt);
    __builtin_amdgcn_sched_barrier(0);
    multiply((set + P - 1) & 1, st + NB, cur, 0, J1);
  };
  // the last buffer's second half is issued by stage 0's first phase
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int j = 0; j < (u == NB - 1 ? J1 : LPW); ++j) issue(u, smem + u * BUF, j);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(LPW * (NB - 2) + J1) : "memory");
  read(0, 0, smem);
  constexpr int U = P == 1 && NB % 2 ? 2 * NB : NB;    // stages a loop body: buffers and sets repeat
  if (nst % U == 0) {
    for (int st0 = 0; st0 < nst; st0 += U) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        stage(st0 + u, P == 1 ? u & 1 : 0, smem + ((u + NB - 1) % NB) * BUF, smem + (u % NB) * BUF,
              smem + ((u + 1) % NB) * BUF);
    }
  } else {
    for (int st0 = 0; st0 < nst; st0 += U) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (st0 + u < nst)
          stage(st0 + u, P == 1 ? u & 1 : 0, smem + ((u + NB - 1) % NB) * BUF,
                smem + (u % NB) * BUF, smem + ((u + 1) % NB) * BUF);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);                      // the re-reads past the end have landed

  // stores: lane holds tokens 4*lq + v of each token tile, column lr of each column tile
  const int64_t slot_end = num_pages * DCKV_PAGE_TOKENS;
  auto store = [&](int i) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int t = tok0 + wm + 16 * i + 4 * lq + v;
      if (t >= n_tok) continue;
      const int64_t sl = slot[t];
      if (sl < 0 || sl >= slot_end) continue;
      bf16* pg = pool + (sl / DCKV_PAGE_TOKENS) * page_elems;
      const int sp = int(sl % DCKV_PAGE_TOKENS);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int c = col0 + wn + 16 * j + lr;
        if (c >= ncols) continue;
        const float val = acc[i][j][v];
        if (c < RK)
          pg[key_elem(sp, c)] = static_cast<bf16>(val);
        else if (c < RKp)
          pg[key_elem(sp, c)] = static_cast<bf16>(0.f);
        else
          pg[value_base + value_elem(sp, c - RKp)] = static_cast<bf16>(val);
      }
    }
  };
  if constexpr (KH == 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i) store(i);
  } else {
    // the lower k half keeps the upper token tiles, the upper k half the
    // lower ones (lane-private slots, same order everywhere)
    constexpr int H = TM / 2;
    floatx4_t* ex = reinterpret_cast<floatx4_t*>(smem) + lane;   // [2][positions][H * TN][64]
    auto send = [&](int i0) {
#pragma unroll
      for (int i = 0; i < H; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) ex[((kh * WR * WC + pos) * H * TN + i * TN + j) * 64] = acc[i0 + i][j];
    };
    auto finish = [&](int i0) {
#pragma unroll
      for (int i = 0; i < H; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i0 + i][j] += ex[(((1 - kh) * WR * WC + pos) * H * TN + i * TN + j) * 64];
        store(i0 + i);
      }
    };
    __syncthreads();                                     // stage buffers no longer read
    if (kh == 0) send(H);
    else send(0);
    __syncthreads();
    if (kh == 0) finish(0);
    else finish(H);
  }
}

template <int WR, int WC, int KH, int TM, int TN, int NB>
hipError_t launch_append_mfma(const dckv_plan& p, const void* x, int32_t n_tok, const void* Lk,
                              const void* Lv, const int64_t* slot, void* pool, int64_t num_pages,
                              hipStream_t stream) {
  constexpr int BM = 16 * TM * WR, BN = 16 * TN * WC;
  constexpr int lds = NB * (BM + BN) * kBK * 2;
  const int ncols = p.RKp + p.rv;
  const int n_tok_tiles = (n_tok + BM - 1) / BM, n_col_tiles = (ncols + BN - 1) / BN;
  auto kern = append_mfma<WR, WC, KH, TM, TN, NB>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(n_tok_tiles * n_col_tiles), dim3(kThreads), lds, stream,
                     static_cast<const bf16*>(x), static_cast<const bf16*>(Lk),
                     static_cast<const bf16*>(Lv), slot, static_cast<bf16*>(pool), n_tok, p.m,
                     p.RK, p.RKp, p.rv, p.page_elems, p.value_base, num_pages, n_tok_tiles, n_col_tiles);
  return hipGetLastError();
}

// Few tokens (a decode step's, at most 16 NT): bound by reading L once.  One
// work-group a 16-column tile of L for all tokens, its eight waves splitting
// k; a wave keeps U 16-byte loads of L (32 U k of its 16 rows) in flight, for U
// = 16 a whole 128 KB tile over the work-group at m = 4096, and takes the token
// operands (read by every work-group, so from L2) all (NT = 1) or half of them
// (NT = 2) ahead.  The waves' sums are added in wave order through LDS.  8
// tokens, m = 4096, 4096 columns: 11 us (3.0 TB/s; 19 us on 128 x 64 tiles).
template <int NT, int U>
__global__ __launch_bounds__(kThreads, 1) void append_few(
    const bf16* __restrict__ x, const bf16* __restrict__ LkT, const bf16* __restrict__ LvT,
    const int64_t* __restrict__ slot, bf16* __restrict__ pool, int n_tok, int m, int RK, int RKp,
    int rv, int64_t page_elems, int64_t value_base, int64_t num_pages) {
  constexpr int SB = U / NT;                           // steps of a token batch
  __shared__ floatx4_t red[8][NT][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int ncols = RKp + rv, col0 = 16 * blockIdx.x;
  const int nst = m >> 5;                              // 32-k steps
  const int s0 = w * nst / 8, s1 = (w + 1) * nst / 8;
  const int c = col0 + lr;
  const bf16* lrow = c < RK ? LkT + int64_t(c) * m
                   : c < RKp ? LkT                     // padding column: written as zero below
                             : LvT + int64_t(min(c - RKp, rv - 1)) * m;
  const bf16* xrow[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) xrow[t] = x + int64_t(min(16 * t + lr, n_tok - 1)) * m;
  floatx4_t acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  auto at = [&](int st) { return 32 * min(st, s1 - 1) + 8 * lq; };    // past the share: its last step again
  u32x4_t lv[U], xv[2][SB][NT];
  auto xload = [&](int set, int st) {
#pragma unroll
    for (int k = 0; k < SB; ++k)
#pragma unroll
      for (int t = 0; t < NT; ++t) xv[set][k][t] = *reinterpret_cast<const u32x4_t*>(xrow[t] + at(st + k));
  };
  for (int st = s0; st < s1; st += U) {
#pragma unroll
    for (int k = 0; k < U; ++k) lv[k] = *reinterpret_cast<const u32x4_t*>(lrow + at(st + k));
    xload(0, st);
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      if (b + 1 < NT) xload((b + 1) & 1, st + (b + 1) * SB);
#pragma unroll
      for (int k = 0; k < SB; ++k)
        if (st + b * SB + k < s1) {
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8_t, lv[b * SB + k]),
                __builtin_bit_cast(bf16x8_t, xv[b & 1][k][t]), acc[t], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) red[w][t][lane] = acc[t];
  __syncthreads();
  // element e: token 16 (e / 256) + (e / 4) % 16, column 4 (e / 64) % 4 + e % 4
  const float* rf = reinterpret_cast<const float*>(red);
  const int64_t slot_end = num_pages * DCKV_PAGE_TOKENS;
  for (int e = tid; e < 256 * NT; e += kThreads) {
    float val = rf[e];
#pragma unroll
    for (int k = 1; k < 8; ++k) val += rf[k * 256 * NT + e];
    const int ln = (e >> 2) & 63, tok = 16 * (e >> 8) + (ln & 15);
    const int cc = col0 + 4 * (ln >> 4) + (e & 3);
    if (tok >= n_tok || cc >= ncols) continue;
    const int64_t sl = slot[tok];
    if (sl < 0 || sl >= slot_end) continue;
    bf16* pg = pool + (sl / DCKV_PAGE_TOKENS) * page_elems;
    const int sp = int(sl % DCKV_PAGE_TOKENS);
    if (cc < RKp)
      pg[key_elem(sp, cc)] = static_cast<bf16>(cc < RK ? val : 0.f);
    else
      pg[value_base + value_elem(sp, cc - RKp)] = static_cast<bf16>(val);
  }
}

template <int NT, int U>
hipError_t launch_append_few(const dckv_plan& p, const void* x, int32_t n_tok, const void* Lk,
                             const void* Lv, const int64_t* slot, void* pool, int64_t num_pages,
                             hipStream_t stream) {
  const int ncols = p.RKp + p.rv;
  hipLaunchKernelGGL((append_few<NT, U>), dim3((ncols + 15) / 16), dim3(kThreads), 0, stream,
                     static_cast<const bf16*>(x), static_cast<const bf16*>(Lk),
                     static_cast<const bf16*>(Lv), slot, static_cast<bf16*>(pool), n_tok, p.m,
                     p.RK, p.RKp, p.rv, p.page_elems, p.value_base, num_pages);
  return hipGetLastError();
}

// U: a wave's share of the 32-k steps, as a power of two up to 16.  Loads past
// the share cost their issue: 32 tokens, 4096 columns take 4.2 us at m = 512
// with U = 2 (13.2 with 16; 9.3 on 128 x 64 tiles), 5.5 at m = 1024 with 4
// (13.4; 11.2), 8.0 at m = 2048 with 8 (13.3; 14.8).
template <int NT>
hipError_t launch_append_few(const dckv_plan& p, const void* x, int32_t n_tok, const void* Lk,
                             const void* Lv, const int64_t* slot, void* pool, int64_t num_pages,
                             hipStream_t stream) {
  const int steps = (p.m / 32 + 7) / 8;
  if (steps <= 2) return launch_append_few<NT, 2>(p, x, n_tok, Lk, Lv, slot, pool, num_pages, stream);
  if (steps <= 4) return launch_append_few<NT, 4>(p, x, n_tok, Lk, Lv, slot, pool, num_pages, stream);
  if (steps <= 8) return launch_append_few<NT, 8>(p, x, n_tok, Lk, Lv, slot, pool, num_pages, stream);
  return launch_append_few<NT, 16>(p, x, n_tok, Lk, Lv, slot, pool, num_pages, stream);
}

// fp32 latents on the fp32 matrix instruction (m a multiple of 16): fp32
// products and sums.  A 32-token x 32-column tile a work-group, its four waves
// splitting k (a small layer has few tiles: 256 tokens x 256 columns make 64,
// each a chain of m / 64 load steps a wave); a wave takes 16-byte pieces of 16
// k of 32 + 32 rows, four steps of them in flight, element e of a piece
// feeding the e-th of four 16x16x4 products (any order of k serves both
// operands).  The waves' sums are added in wave order through LDS.  256 tokens
// x 512 x 256: 8 us against 70 us on append_valu.
__global__ __launch_bounds__(256) void append_f32(const float* __restrict__ x,
                                                  const float* __restrict__ Lk,
                                                  const float* __restrict__ Lv,
                                                  const int64_t* __restrict__ slot,
                                                  float* __restrict__ pool, int n_tok, int m, int RK,
                                                  int RKp, int rv, int64_t page_elems,
                                                  int64_t value_base, int64_t num_pages) {
  constexpr int U = 4;                                 // load steps in flight
  __shared__ floatx4_t red[4][4][64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  const int ncols = RKp + rv, col0 = 32 * blockIdx.y, tok0 = 32 * blockIdx.x;
  const int nst = m >> 4, s0 = w * nst / 4, s1 = (w + 1) * nst / 4;
  const float* src[4];                                 // two token tiles, two column tiles
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    src[i] = x + int64_t(min(tok0 + 16 * i + lr, n_tok - 1)) * m + 4 * lq;
    const int c = col0 + 16 * i + lr;
    src[2 + i] = (c < RK ? Lk + int64_t(c) * m
                  : c < RKp ? Lk                       // padding column: written as zero below
                            : Lv + int64_t(min(c - RKp, rv - 1)) * m) + 4 * lq;
  }
  floatx4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  floatx4_t v[U][4];
  const int last = max(s1, 1) - 1;                     // past the share: its last step again
  auto load = [&](int k, int st) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[k][i] = *reinterpret_cast<const floatx4_t*>(src[i] + 16 * min(st, last));
  };
#pragma unroll
  for (int k = 0; k < U; ++k) load(k, s0 + k);
  for (int st = s0; st < s1; st += U) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (st + k < s1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[k][i][e], v[k][2 + j][e], acc[i][j], 0, 0, 0);
      }
      load(k, st + k + U);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) red[w][2 * i + j][lane] = acc[i][j];
  __syncthreads();
  // wave w finishes tile (w / 2, w % 2): tokens 4 lq + v, column lr
  floatx4_t t = red[0][w][lane];
#pragma unroll
  for (int k = 1; k < 4; ++k) t += red[k][w][lane];
  const int c = col0 + 16 * (w & 1) + lr;
  if (c >= ncols) return;
  const int64_t slot_end = num_pages * DCKV_PAGE_TOKENS;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int tok = tok0 + 16 * (w >> 1) + 4 * lq + q;
    if (tok >= n_tok) continue;
    const int64_t sl = slot[tok];
    if (sl < 0 || sl >= slot_end) continue;
    float* pg = pool + (sl / DCKV_PAGE_TOKENS) * page_elems;
    const int sp = int(sl % DCKV_PAGE_TOKENS);
    if (c < RKp)
      pg[key_elem(sp, c)] = c < RK ? t[q] : 0.f;
    else
      pg[value_base + value_elem(sp, c - RKp)] = t[q];
  }
}

template <typename T>
hipError_t launch_append_t(const dckv_plan& p, const void* x, int32_t n_tok, const void* Lk,
                           const void* Lv, const int64_t* slot, void* pool, int64_t num_pages,
                           hipStream_t stream) {
  const int ncols = p.RKp + p.rv;
  dim3 grid((ncols + kTileCol - 1) / kTileCol, (n_tok + kTileTok - 1) / kTileTok);
  hipLaunchKernelGGL(append_valu<T>, grid, dim3(256), 0, stream, static_cast<const T*>(x),
                     static_cast<const T*>(Lk), static_cast<const T*>(Lv), slot,
                     static_cast<T*>(pool), n_tok, p.m, p.RK, p.RKp, p.rv, p.page_elems,
                     p.value_base, num_pages);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_append(const dckv_plan& p, const void* x, int32_t n_tok, const void* L_keys,
                         const void* L_value, const int64_t* slot, void* pool, int64_t num_pages,
                         hipStream_t stream) {
  if (p.dtype == DCKV_F32 && p.m % 16 == 0) {
    const int ncols = p.RKp + p.rv;
    hipLaunchKernelGGL(append_f32, dim3((n_tok + 31) / 32, (ncols + 31) / 32), dim3(256), 0, stream,
                       static_cast<const float*>(x), static_cast<const float*>(L_keys),
                       static_cast<const float*>(L_value), slot, static_cast<float*>(pool), n_tok,
                       p.m, p.RK, p.RKp, p.rv, p.page_elems, p.value_base, num_pages);
    return hipGetLastError();
  }
  if (p.dtype == DCKV_F32)
    return launch_append_t<float>(p, x, n_tok, L_keys, L_value, slot, pool, num_pages, stream);
  if (p.m % kBK == 0) {
    // up to 32 tokens: L is read once whatever the tile, and sixteen columns a
    // work-group spread it over most compute units (m = 4096, 4096 columns: 8
    // tokens 11.2 us against 14.4 on 64 x 64 tiles and 18.9 on 128 x 64, 32
    // tokens 15.7 / 16.4 / 19.6; 64 tokens, whose token operands every
    // work-group would read from L2: 24.1 / 18.9 / 21.2)
    if (n_tok <= 16)
      return launch_append_few<1>(p, x, n_tok, L_keys, L_value, slot, pool, num_pages, stream);
    if (n_tok <= 32)
      return launch_append_few<2>(p, x, n_tok, L_keys, L_value, slot, pool, num_pages, stream);
    // Tiles: the size whose rounds over the compute units cost least.  A round
    // of full tiles at m = 4096 takes about 15 us (64 x 64), 23 (128 x 64), 33
    // (128 x 128) and 55 (128 x 256), the costs below without the launch; a
    // larger tile reads fewer bytes a product, a smaller one leaves fewer
    // compute units idle.  Measured, 4096 columns, us for the four sizes: 256
    // tokens 17.7 / 23.6 / 31.6 / 53.5; 512: 30.0 / 27.0 / 34.6 / 55.6; 1024:
    // 57.6 / 52.5 / 43.0 / 61.0; 1536: 83.3 / 75.4 / 74.3 / 65.4; 4093: 243 /
    // 237 / 167 / 143.
    const int64_t ncols = p.RKp + p.rv;
    auto cost = [&](int bm, int bn, int64_t round) {
      const int64_t tiles = ((n_tok + bm - 1) / bm) * ((ncols + bn - 1) / bn);
      return (tiles + kComputeUnits - 1) / kComputeUnits * round;
    };
    const int64_t c0 = cost(64, 64, 12), c1 = cost(128, 64, 20), c2 = cost(128, 128, 30),
                  c3 = cost(128, 256, 52);
    const int64_t least = std::min(std::min(c0, c1), std::min(c2, c3));
    if (c0 == least)
      return launch_append_mfma<2, 2, 2, 2, 2, 4>(p, x, n_tok, L_keys, L_value, slot, pool, num_pages, stream);
    if (c1 == least)
      return launch_append_mfma<4, 1, 2, 2, 4, 4>(p, x, n_tok, L_keys, L_value, slot, pool, num_pages, stream);
    if (c2 == least)
      return launch_append_mfma<2, 2, 2, 4, 4, 4>(p, x, n_tok, L_keys, L_value, slot, pool, num_pages, stream);
    return launch_append_mfma<2, 4, 1, 4, 4, 3>(p, x, n_tok, L_keys, L_value, slot, pool, num_pages, stream);
  }
  return launch_append_t<bf16>(p, x, n_tok, L_keys, L_value, slot, pool, num_pages, stream);
}

}  // namespace dckv
