// Offline contractions of the compression pipeline.
//
// gram: G = A~^T A~ for A [rows, cols] (row-major, one sample a row), with
// A~ = A - 1 mu^T (column means) when centring is asked for.  It feeds the
// CKA head similarity (Sec. III-A: CKA compares centred representations;
// Sec. III-C: S[i][j] between the heads' activations) and the calibration
// Gram X^T X of the value refinement (Sec. III-D).  The products run on the
// bf16 matrix instruction with fp32 accumulators and lose nothing to it:
// plain bf16 samples are its operands as they are (gram_bf16), and an fp32
// value (a sample, or a sample less its column's mean) is taken as the exact
// sum of three bf16 parts (gram_split).
//
// head_similarity: S[i][j] = ||G_ij||_F^2 / (||G_ii||_F ||G_jj||_F) over the
// d_h x d_h blocks of a centred Gram, which is linear CKA (Sec. III-A).
#include <cmath>
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace dckv {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kMeanRows = 256;            // rows a column-sum work-group
constexpr int kMeanBlocks = 64;           // row blocks whose sums a tile adds up by itself

// Column sums of rows [rb * kMeanRows, ...) for 64 columns a work-group:
// thread t sums columns 4 (t % 16) .. +3 of rows t / 16, t / 16 + 16, ...,
// all its loads in flight, and the sixteen row groups are added in order.
template <typename T>
__global__ __launch_bounds__(256) void colsum_partial(const T* __restrict__ A, int64_t rows,
                                                      int cols, float* __restrict__ part) {
  constexpr int RG = 16, N = kMeanRows / RG;
  __shared__ floatx4 red[256];
  const int tid = threadIdx.x, rg = tid >> 4;
  const int c = blockIdx.x * 64 + 4 * (tid & 15);                // cols is a multiple of 8
  const int64_t r0 = int64_t(blockIdx.y) * kMeanRows;
  const int n = int(rows < r0 + kMeanRows ? rows - r0 : kMeanRows);
  const T* src = A + r0 * cols + (c < cols ? c : 0);
  uint32_t v[N][sizeof(T)];                                      // four values: 16 or 8 bytes
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const uint32_t* p = reinterpret_cast<const uint32_t*>(src + int64_t(min(rg + RG * k, n - 1)) * cols);
#pragma unroll
    for (int j = 0; j < int(sizeof(T)); ++j) v[k][j] = p[j];
  }
  floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < N; ++k) {
    floatx4 f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      f[j] = sizeof(T) == 4 ? __uint_as_float(v[k][j % sizeof(T)])
                            : __uint_as_float((j & 1) ? v[k][j >> 1] & 0xFFFF0000u : v[k][j >> 1] << 16);
    if (rg + RG * k < n) s += f;
  }
  red[tid] = s;
  __syncthreads();
  if (tid < 16 && c < cols) {
    for (int g = 1; g < RG; ++g) s += red[g * 16 + tid];
    *reinterpret_cast<floatx4*>(part + int64_t(blockIdx.y) * cols + c) = s;
  }
}

// mu[c] = (sum of the partial sums in row-block order) / rows.
__device__ __forceinline__ float column_mean(const float* __restrict__ part, int nblk, int64_t rows,
                                             int cols, int c) {
  float s = 0.f;
  int b = 0;
  for (; b + 8 <= nblk; b += 8) {                                // eight loads in flight
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = part[int64_t(b + k) * cols + c];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += v[k];
  }
  for (; b < nblk; ++b) s += part[int64_t(b) * cols + c];
  return s / float(rows);
}
__global__ __launch_bounds__(256) void colmean_finish(const float* __restrict__ part, int nblk,
                                                      int64_t rows, int cols,
                                                      float* __restrict__ mu) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c < cols) mu[c] = column_mean(part, nblk, rows, cols, c);
}

// ---------------------------------------------------------------------------
// Tiles.  One work-group of eight waves computes one TS x TS tile (ti <= tj)
// of G, TS = 64 NS columns, and writes it twice, as is and mirrored, so G is
// exactly symmetric.  A wave owns the rows 64 s + 32 wi .. +31 and columns
// 64 s + 32 wj .. +31 of every 64-wide slab s (2 NS x 2 NS products of
// 16 x 16); the two waves of a position (kh = 0, 1: they share a SIMD) split
// the work of a stage and their sums are added at the end.
//
// The contraction runs over the rows of A, so an operand's eight k of one
// column lie in eight rows: a stage is staged in LDS as it lies in memory and
// read through the transposing LDS load, where sixteen lanes take four rows
// of sixteen columns and each gets one column's four values.  Lane group lq
// takes rows 4 lq .. +3 and 16 + 4 lq .. +3 of a 32-row step (any order of k
// serves, as both operands use the same one): with 128-byte rows whose
// 32-byte pieces are xor-swizzled by (row / 2) % 4, the eight rows that half
// a wave reads at once fall in distinct banks.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef short short8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t* lds_short4;

constexpr int kGramThreads = 512;
constexpr int kGramNB = 3;                // stage buffers of gram_bf16
constexpr int kGramSuper = 6;             // tiles a side of a super-block

// Work-group id -> tile.  The tiles are numbered super-block after
// super-block (6 x 6 tiles of the upper triangle) and each XCD (ids equal mod
// 8) takes one run of consecutive numbers, so that the work-groups of an XCD
// read few different column panels and share them in its L2.
__device__ __forceinline__ void gram_tile_of(int id, int n_tiles, int nt, int& ti, int& tj) {
  const int xcd = id & 7, per = n_tiles >> 3, extra = n_tiles & 7;
  int lin = xcd * per + min(xcd, extra) + (id >> 3);
  const int nb = (nt + kGramSuper - 1) / kGramSuper;
  ti = tj = 0;
  for (int bi = 0; bi < nb; ++bi) {
    const int r0 = bi * kGramSuper, nr = min(kGramSuper, nt - r0);
    const int tri = nr * (nr + 1) / 2;
    if (lin < tri) {
      int i = 0;
      while (lin >= nr - i) {
        lin -= nr - i;
        ++i;
      }
      ti = r0 + i;
      tj = ti + lin;
      return;
    }
    lin -= tri;
    const int right = nt - r0 - nr;         // columns of the super-blocks to the right
    if (lin < nr * right) {
      int c0 = r0 + nr;
      while (lin >= nr * min(kGramSuper, nt - c0)) {
        lin -= nr * min(kGramSuper, nt - c0);
        c0 += kGramSuper;
      }
      ti = r0 + lin % nr;
      tj = c0 + lin / nr;
      return;
    }
    lin -= nr * right;
  }
}

__device__ __forceinline__ floatx4 mfma_bf16(short8_t a, short8_t b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 16 bytes a lane from global memory to LDS, in lane order from p on.
__device__ __forceinline__ void load_lds16(const bf16* g, unsigned char* p) {
  __builtin_amdgcn_global_load_lds(g, p, 16, 0, 0);
}

// One operand fragment (16 columns x 32 rows): p addresses this lane's piece
// of rows 0..15, rows 16..31 lie 2048 bytes on.
__device__ __forceinline__ short8_t read_frag(unsigned char* p) {
  const short4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p));
  const short4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p + 2048));
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// The same loads for a kernel whose stages come by the loads' LDS path: the
// compiler puts a wait for every load in flight before a transposing LDS
// load of its own (it cannot tell which buffer the load writes), so these
// are written out, each block waiting for its own results.
__device__ __forceinline__ uint32_t lds_address(unsigned char* p) {
  return uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)(p)));
}
__device__ __forceinline__ void read_slab(short8_t (&f)[2], uint32_t p0, uint32_t p1) {
  short4_t t0 = {}, t1 = {}, t2 = {}, t3 = {};
#ifdef __HIP_DEVICE_COMPILE__                      // the host pass knows no vector registers
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:2048\n\t"
      "ds_read_b64_tr_b16 %2, %5\n\tds_read_b64_tr_b16 %3, %5 offset:2048\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
      : "v"(p0), "v"(p1)
      : "memory");
#endif
  f[0] = __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7);
  f[1] = __builtin_shufflevector(t2, t3, 0, 1, 2, 3, 4, 5, 6, 7);
}
template <int NS>
__device__ __forceinline__ void read_rows(short8_t (&f)[2 * NS], uint32_t p0, uint32_t p1) {
  if constexpr (NS == 3) {
    short4_t t0 = {}, t1 = {}, t2 = {}, t3 = {}, t4 = {}, t5 = {}, t6 = {}, t7 = {}, t8 = {}, t9 = {},
             ta = {}, tb = {};
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile(
        "ds_read_b64_tr_b16 %0, %12\n\tds_read_b64_tr_b16 %1, %12 offset:2048\n\t"
        "ds_read_b64_tr_b16 %2, %13\n\tds_read_b64_tr_b16 %3, %13 offset:2048\n\t"
        "ds_read_b64_tr_b16 %4, %12 offset:8192\n\tds_read_b64_tr_b16 %5, %12 offset:10240\n\t"
        "ds_read_b64_tr_b16 %6, %13 offset:8192\n\tds_read_b64_tr_b16 %7, %13 offset:10240\n\t"
        "ds_read_b64_tr_b16 %8, %12 offset:16384\n\tds_read_b64_tr_b16 %9, %12 offset:18432\n\t"
        "ds_read_b64_tr_b16 %10, %13 offset:16384\n\tds_read_b64_tr_b16 %11, %13 offset:18432\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3), "=&v"(t4), "=&v"(t5), "=&v"(t6), "=&v"(t7),
          "=&v"(t8), "=&v"(t9), "=&v"(ta), "=&v"(tb)
        : "v"(p0), "v"(p1)
        : "memory");
#endif
    f[0] = __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7);
    f[1] = __builtin_shufflevector(t2, t3, 0, 1, 2, 3, 4, 5, 6, 7);
    f[2] = __builtin_shufflevector(t4, t5, 0, 1, 2, 3, 4, 5, 6, 7);
    f[3] = __builtin_shufflevector(t6, t7, 0, 1, 2, 3, 4, 5, 6, 7);
    f[4] = __builtin_shufflevector(t8, t9, 0, 1, 2, 3, 4, 5, 6, 7);
    f[5] = __builtin_shufflevector(ta, tb, 0, 1, 2, 3, 4, 5, 6, 7);
  } else {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      short8_t t[2];
      read_slab(t, p0 + s * 8192, p1 + s * 8192);
      f[2 * s] = t[0];
      f[2 * s + 1] = t[1];
    }
  }
}

// The end of a tile: the two waves of a position exchange halves of their
// sums through LDS (kh = 0 keeps the upper row fragments, kh = 1 the lower),
// add them and write the tile and its mirror.  A diagonal tile writes its
// upper triangle and the mirror of it.  Returns whether this thread wrote an
// element that is not finite.
template <int NS>
__device__ __forceinline__ bool gram_write(floatx4 (&acc)[2 * NS][2 * NS], unsigned char* smem,
                                           float* __restrict__ G, int cols, int i0, int j0, int wi,
                                           int wj, int kh, int pos, int lane) {
  constexpr int F = 2 * NS;
  bool odd = false;
  const int lr = lane & 15, lq = lane >> 4;
  floatx4* ex = reinterpret_cast<floatx4*>(smem) + lane;         // [8][NS * F][64]
  const bool diag = i0 == j0;
  auto send = [&](int x0, int slot) {
#pragma unroll
    for (int x = 0; x < NS; ++x)
#pragma unroll
      for (int y = 0; y < F; ++y) ex[((slot * NS + x) * F + y) * 64] = acc[x0 + x][y];
  };
  auto finish = [&](int x0, int slot) {
#pragma unroll
    for (int x = 0; x < NS; ++x) {
      const int i = i0 + 64 * ((x0 + x) >> 1) + 32 * wi + 16 * ((x0 + x) & 1) + 4 * lq;
#pragma unroll
      for (int y = 0; y < F; ++y) {
        const int j = j0 + 64 * (y >> 1) + 32 * wj + 16 * (y & 1) + lr;
        floatx4 t = acc[x0 + x][y] + ex[((slot * NS + x) * F + y) * 64];
        if (i >= cols || j >= cols) continue;                    // cols is a multiple of 8
#pragma unroll
        for (int v = 0; v < 4; ++v) odd |= !(fabsf(t[v]) < INFINITY);
        if (!diag) {
          *reinterpret_cast<floatx4*>(G + int64_t(j) * cols + i) = t;
#pragma unroll
          for (int v = 0; v < 4; ++v) G[int64_t(i + v) * cols + j] = t[v];
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (i + v <= j) {
              G[int64_t(j) * cols + i + v] = t[v];
              G[int64_t(i + v) * cols + j] = t[v];
            }
        }
      }
    }
  };
  __syncthreads();                                               // stages no longer read
  if (kh == 0) send(NS, pos);
  else send(0, 4 + pos);
  __syncthreads();
  if (kh == 0) finish(0, 4 + pos);
  else finish(NS, pos);
  return odd;
}

// bf16 samples, no centring: the samples are the operands, every product is
// exact.  A stage is 64 rows (kh takes 32 of them) copied from global memory
// straight into LDS, three buffers, the loads two stages ahead, one barrier a
// stage.  Bound by the matrix pipe and, at 96 x 96 a wave, two thirds as much
// by LDS reads: 8192 x 4096 samples (253 tiles of 192) take 140 us, 1.1
// PFLOP/s of issued products, against 1370 us on the fp32 matrix instruction.
template <int NS>
__global__ __launch_bounds__(kGramThreads, 1) void gram_bf16(const bf16* __restrict__ A,
                                                            int64_t rows, int cols,
                                                            float* __restrict__ G, int nt,
                                                            int n_tiles) {
  constexpr int F = 2 * NS, OP = NS * 8192, BUF = 2 * OP;        // bytes an operand, a stage
  extern __shared__ __align__(1024) unsigned char smem[];        // [kGramNB][2][NS][64][128]
  int ti, tj;
  gram_tile_of(blockIdx.x, n_tiles, nt, ti, tj);
  const int i0 = ti * 64 * NS, j0 = tj * 64 * NS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pos = w & 3, kh = w >> 2, wi = pos >> 1, wj = pos & 1;
  const int lq = lane >> 4, li = lane & 15;

  // loads: wave w fills rows 8 w .. +7 of every (operand, slab); lane: row
  // lane / 8 of them, 16-byte LDS piece lane % 8, which holds global piece
  // (lane % 8) ^ (row & 6)
  const int lrow = 8 * w + (lane >> 3), gp = (lane & 7) ^ ((lane >> 3) & 6);
  uint32_t goff[2 * NS];
#pragma unroll
  for (int f = 0; f < 2 * NS; ++f) {
    const int c = (f < NS ? i0 + 64 * f : j0 + 64 * (f - NS)) + 8 * gp;
    goff[f] = uint32_t(lrow) * uint32_t(cols) + uint32_t(min(c, cols - 8));
  }
  const int nst = int(rows >> 6);                                // whole stages
  const int rest = int(rows & 63);
  auto issue = [&](int st, unsigned char* buf) {                 // past the end: the last stage again
    const bf16* base = A + int64_t(min(st, nst - 1)) * 64 * cols;
#pragma unroll
    for (int f = 0; f < 2 * NS; ++f) load_lds16(base + goff[f], buf + f * 8192 + w * 1024);
  };

  floatx4 acc[F][F];
#pragma unroll
  for (int x = 0; x < F; ++x)
#pragma unroll
    for (int y = 0; y < F; ++y) acc[x][y] = floatx4{0.f, 0.f, 0.f, 0.f};
  int oi[2], oj[2];                                              // this lane's fragment offsets
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int sw = 2 * (lq & 1) + (li >> 3);
    const int at = kh * 4096 + (4 * lq + (li >> 2)) * 128 + 8 * (li & 3);
    oi[e] = at + 32 * ((2 * wi + e) ^ sw);
    oj[e] = OP + at + 32 * ((2 * wj + e) ^ sw);
  }
  auto products = [&](unsigned char* cur) {
    const uint32_t base = lds_address(cur);
    short8_t a[F], b[2];
    read_rows<NS>(a, base + oi[0], base + oi[1]);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      read_slab(b, base + oj[0] + s * 8192, base + oj[1] + s * 8192);
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int x = 0; x < F; ++x) acc[x][2 * s + y] = mfma_bf16(a[x], b[y], acc[x][2 * s + y]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (nst > 0) {
#pragma unroll
    for (int u = 0; u < kGramNB - 1; ++u) issue(u, smem + u * BUF);
    for (int st0 = 0; st0 < nst; st0 += kGramNB) {
#pragma unroll
      for (int u = 0; u < kGramNB; ++u)
        if (st0 + u < nst) {
          // this wave's loads of the stage and its LDS reads of the one
          // before are done, then all waves': the stage is whole and the
          // buffer that the next loads fill is free
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(2 * NS * (kGramNB - 2)) : "memory");
          issue(st0 + u + kGramNB - 1, smem + ((u + kGramNB - 1) % kGramNB) * BUF);
          products(smem + u * BUF);
        }
    }
    __builtin_amdgcn_s_waitcnt(0);                               // the re-reads past the end have landed
  }
  if (rest) {                                                    // the last rows, zero past the end
    __syncthreads();
    const bf16* base = A + int64_t(nst) * 64 * cols;
#pragma unroll
    for (int f = 0; f < 2 * NS; ++f) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (lrow < rest) v = *reinterpret_cast<const u32x4*>(base + goff[f]);
      *reinterpret_cast<u32x4*>(smem + f * 8192 + w * 1024 + lane * 16) = v;
    }
    __syncthreads();
    products(smem);
  }
  gram_write<NS>(acc, smem, G, cols, i0, j0, wi, wj, kh, pos, lane);
}

// Any samples: d = a - mu in fp32, taken as the exact sum of three bf16 parts
// (hi: the upper 16 bits of d; mid: the rest rounded to bf16; lo: what is
// left, at most 8 significant bits).  Six of the nine products of parts are
// summed; the three left out are below 2^-22 of the full one.  kh = 0 takes
// hi hi, hi mid and mid hi, kh = 1 mid mid, hi lo and lo hi: the small ones
// have accumulators of their own, since added to the large sums they can stay
// below half a unit of their last place and be lost, step after step, where
// they all have one sign (bf16 samples less one mean).  A stage is 32 rows:
// raw loads a stage ahead in registers, split and written to the other of two
// LDS buffers beside the products of the current one.  mu: null (no
// centring), the means (nblk 0), or nblk row blocks' column sums, of which
// every work-group takes the means of its own columns.
// FEW, for at most 32 rows (one stage): all nine products, kh = 0 taking hi hi
// alone (at most 16 significant bits a product) and kh = 1 the other eight, so
// that the one rounding of a large sum is the last addition's, as in a single
// fp32 product.  With few terms the three products left out would show: 2-norm
// error of one row 4.0e-8 with six products, 2.5e-8 on the fp32 matrix
// instruction and here; of 8 rows 4.7e-8 / 5.3e-8 / 2.8e-8.
// Bound by the matrix pipe (six products) with the splitting beside it: 2048 x
// 4096 fp32 samples, centred, 205 us against 395 us on the fp32 matrix
// instruction, error against float64 4.9e-7 against 7.5e-7 (2-norm; bf16
// samples, centred: 4.9e-7 against 7.9e-7).
__device__ __forceinline__ void split_pair(float d0, float d1, uint32_t& h, uint32_t& m, uint32_t& l) {
  const uint32_t u0 = __float_as_uint(d0), u1 = __float_as_uint(d1);
  h = (u0 >> 16) | (u1 & 0xFFFF0000u);
  const float r0 = d0 - __uint_as_float(u0 & 0xFFFF0000u), r1 = d1 - __uint_as_float(u1 & 0xFFFF0000u);
  const bf16 m0 = static_cast<bf16>(r0), m1 = static_cast<bf16>(r1);
  m = uint32_t(__builtin_bit_cast(uint16_t, m0)) | (uint32_t(__builtin_bit_cast(uint16_t, m1)) << 16);
  const float s0 = r0 - __uint_as_float(m << 16), s1 = r1 - __uint_as_float(m & 0xFFFF0000u);
  l = (__float_as_uint(s0) >> 16) | (__float_as_uint(s1) & 0xFFFF0000u);
}

// The class of d as bf16: 0, +-1, +-inf or NaN.
__device__ __forceinline__ uint32_t class_of(float d) {
  const uint32_t u = __float_as_uint(d), m = u & 0x7FFFFFFFu;
  if (m > 0x7F800000u) return 0x7FC0u;
  return (u >> 16 & 0x8000u) | (m == 0 ? 0u : m < 0x7F800000u ? 0x3F80u : 0x7F80u);
}

// Infinities do not survive the split (inf has NaN for a rest, and inf times a
// part that is 0 is NaN).  A tile that holds an element that is not finite
// walks its samples once more and takes each as its class: 0, +-1 for a finite
// value, +-inf, NaN.  Sums of products of classes are infinite or NaN where
// those of the values are, and those elements are written again; where they
// are finite the samples are too, and what was written is a sum that left
// fp32's range.  One product a term: whatever the samples hold, less than the
// walk before took.  Everything is worked out anew from the thread's number
// (which the compiler is kept from recognising), so that none of it stays live
// through the walk before: sharing its offsets cost that one up to 4 % (1387 x
// 2048 bf16 samples, centred, 83.2 -> 86.7 us).
template <typename T, int NS>
__device__ __forceinline__ void gram_classes(const T* __restrict__ A, int64_t rows, int cols,
                                             unsigned char* smem, float* __restrict__ G, int i0, int j0) {
  constexpr int F = 2 * NS, OP = NS * 4096, BUF = 6 * OP, NQ = sizeof(T) / 2;
  const float* smu = reinterpret_cast<const float*>(smem + 2 * BUF);
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, w = tid >> 6, pos = w & 3, wi = pos >> 1, wj = pos & 1;
  const int lq = lane >> 4, li = lane & 15;
  const int crow = (tid & 255) >> 3, cpiece = tid & 7, nst = int((rows + 31) >> 5);
  floatx4 acc[F][F];
#pragma unroll
  for (int x = 0; x < F; ++x)
#pragma unroll
    for (int y = 0; y < F; ++y) acc[x][y] = floatx4{0.f, 0.f, 0.f, 0.f};
  int oi[2], oj[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int sw = 2 * (lq & 1) + (li >> 3);
    const int at = (4 * lq + (li >> 2)) * 128 + 8 * (li & 3);
    oi[e] = at + 32 * ((2 * wi + e) ^ sw);
    oj[e] = OP + at + 32 * ((2 * wj + e) ^ sw);
  }
  for (int st = 0; st < nst; ++st) {
    __syncthreads();                                             // the stage before has been read
    const int64_t r = int64_t(st) * 32 + crow;
    const T* row = A + min(r, rows - 1) * cols;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const int f = 2 * q + (w >> 2);
      const int c0 = (f < NS ? i0 + 64 * f : j0 + 64 * (f - NS)) + 8 * cpiece;
      u32x4 v[NQ], c;
#pragma unroll
      for (int k = 0; k < NQ; ++k) v[k] = reinterpret_cast<const u32x4*>(row + min(c0, cols - 8))[k];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float d0, d1;
        if constexpr (NQ == 2) {
          d0 = __uint_as_float(v[k >> 1][2 * (k & 1)]);
          d1 = __uint_as_float(v[k >> 1][2 * (k & 1) + 1]);
        } else {
          d0 = __uint_as_float(v[0][k] << 16);
          d1 = __uint_as_float(v[0][k] & 0xFFFF0000u);
        }
        d0 -= smu[64 * f + 8 * cpiece + 2 * k];
        d1 -= smu[64 * f + 8 * cpiece + 2 * k + 1];
        c[k] = r < rows ? class_of(d0) | class_of(d1) << 16 : 0u;
      }
      *reinterpret_cast<u32x4*>(smem + f * 4096 + crow * 128 + 16 * (cpiece ^ (crow & 6))) = c;
    }
    __syncthreads();
    if (w < 4) {
      short8_t a[F];
#pragma unroll
      for (int x = 0; x < F; ++x) a[x] = read_frag(smem + oi[x & 1] + (x >> 1) * 4096);
#pragma unroll
      for (int y = 0; y < F; ++y) {
        const short8_t b = read_frag(smem + oj[y & 1] + (y >> 1) * 4096);
#pragma unroll
        for (int x = 0; x < F; ++x) acc[x][y] = mfma_bf16(a[x], b, acc[x][y]);
      }
    }
  }
  if (w >= 4) return;
#pragma unroll
  for (int x = 0; x < F; ++x)
#pragma unroll
    for (int y = 0; y < F; ++y) {
      const int i = i0 + 64 * (x >> 1) + 32 * wi + 16 * (x & 1) + 4 * lq;
      const int j = j0 + 64 * (y >> 1) + 32 * wj + 16 * (y & 1) + li;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (i < cols && j < cols && (i0 != j0 || i + v <= j) && !(fabsf(acc[x][y][v]) < INFINITY)) {
          G[int64_t(j) * cols + i + v] = acc[x][y][v];
          G[int64_t(i + v) * cols + j] = acc[x][y][v];
        }
    }
}

template <typename T, int NS, bool FEW = false>
__global__ __launch_bounds__(kGramThreads, 1) void gram_split(const T* __restrict__ A, int64_t rows,
                                                             int cols, const float* __restrict__ mu,
                                                             int nblk, float* __restrict__ G, int nt,
                                                             int n_tiles) {
  constexpr int F = 2 * NS, OP = NS * 4096, PL = 2 * OP, BUF = 3 * PL;   // operand, plane, stage
  constexpr int NQ = sizeof(T) / 2;                              // 16-byte loads a chunk of 8 columns
  extern __shared__ __align__(1024) unsigned char smem[];        // [2][3][2][NS][32][128], then mu
  float* smu = reinterpret_cast<float*>(smem + 2 * BUF);         // [2][64 NS]
  int ti, tj;
  gram_tile_of(blockIdx.x, n_tiles, nt, ti, tj);
  const int i0 = ti * 64 * NS, j0 = tj * 64 * NS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pos = w & 3, kh = w >> 2, wi = pos >> 1, wj = pos & 1;
  const int lq = lane >> 4, li = lane & 15;

  for (int e = tid; e < 128 * NS; e += kGramThreads) {
    const int c = e < 64 * NS ? i0 + e : j0 + e - 64 * NS;
    smu[e] = !mu || c >= cols ? 0.f : nblk ? column_mean(mu, nblk, rows, cols, c) : mu[c];
  }
  // chunk q of this thread: (operand, slab) 2 q + w / 4, row and 16-byte
  // piece (8 columns) fixed
  const int crow = (tid & 255) >> 3, cpiece = tid & 7;
  uint32_t goff[NS];
  int moff[NS], soff[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) {
    const int f = 2 * q + (w >> 2);
    const int c = (f < NS ? i0 + 64 * f : j0 + 64 * (f - NS)) + 8 * cpiece;
    goff[q] = uint32_t(sizeof(T)) * uint32_t(min(c, cols - 8));
    moff[q] = 64 * f + 8 * cpiece;
    soff[q] = f * 4096 + crow * 128 + 16 * (cpiece ^ (crow & 6));
  }
  const int nst = int((rows + 31) >> 5);
  u32x4 raw[NS][NQ];
  auto load = [&](int st) {                                      // clamped: every load is in bounds
    const int64_t r = min(int64_t(st) * 32 + crow, rows - 1);
    const char* base = reinterpret_cast<const char*>(A + r * cols);
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
      for (int k = 0; k < NQ; ++k) raw[q][k] = *reinterpret_cast<const u32x4*>(base + goff[q] + 16 * k);
  };
  auto convert = [&](int st, unsigned char* buf) {               // zeros past the last row
    const bool live = int64_t(st) * 32 + crow < rows;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const floatx4 m0 = *reinterpret_cast<const floatx4*>(smu + moff[q]);
      const floatx4 m1 = *reinterpret_cast<const floatx4*>(smu + moff[q] + 4);
      u32x4 h, m, l;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float d0, d1;
        if constexpr (NQ == 2) {
          d0 = __uint_as_float(raw[q][k >> 1][2 * (k & 1)]);
          d1 = __uint_as_float(raw[q][k >> 1][2 * (k & 1) + 1]);
        } else {
          d0 = __uint_as_float(raw[q][0][k] << 16);
          d1 = __uint_as_float(raw[q][0][k] & 0xFFFF0000u);
        }
        d0 -= k < 2 ? m0[2 * k] : m1[2 * k - 4];
        d1 -= k < 2 ? m0[2 * k + 1] : m1[2 * k - 3];
        uint32_t ph, pm, pl;
        split_pair(live ? d0 : 0.f, live ? d1 : 0.f, ph, pm, pl);
        h[k] = ph;
        m[k] = pm;
        l[k] = pl;
      }
      *reinterpret_cast<u32x4*>(buf + soff[q]) = h;
      *reinterpret_cast<u32x4*>(buf + PL + soff[q]) = m;
      *reinterpret_cast<u32x4*>(buf + 2 * PL + soff[q]) = l;
    }
  };

  floatx4 acc[F][F];
#pragma unroll
  for (int x = 0; x < F; ++x)
#pragma unroll
    for (int y = 0; y < F; ++y) acc[x][y] = floatx4{0.f, 0.f, 0.f, 0.f};
  int oi[2], oj[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int sw = 2 * (lq & 1) + (li >> 3);
    const int at = (4 * lq + (li >> 2)) * 128 + 8 * (li & 3);
    oi[e] = at + 32 * ((2 * wi + e) ^ sw);
    oj[e] = OP + at + 32 * ((2 * wj + e) ^ sw);
  }
  // sums of hi p and p hi for part p (plane offset P), and with HH of hi hi
  auto cross = [&](unsigned char* cur, auto plane, auto hh) {
    constexpr int P = decltype(plane)::value;
    short8_t ah[F], ap[F];
#pragma unroll
    for (int x = 0; x < F; ++x) {
      ah[x] = read_frag(cur + oi[x & 1] + (x >> 1) * 4096);
      ap[x] = read_frag(cur + P + oi[x & 1] + (x >> 1) * 4096);
    }
#pragma unroll
    for (int y = 0; y < F; ++y) {
      const short8_t bh = read_frag(cur + oj[y & 1] + (y >> 1) * 4096);
      const short8_t bp = read_frag(cur + P + oj[y & 1] + (y >> 1) * 4096);
#pragma unroll
      for (int x = 0; x < F; ++x) acc[x][y] = mfma_bf16(ah[x], bp, acc[x][y]);
#pragma unroll
      for (int x = 0; x < F; ++x) acc[x][y] = mfma_bf16(ap[x], bh, acc[x][y]);
      if constexpr (decltype(hh)::value) {
#pragma unroll
        for (int x = 0; x < F; ++x) acc[x][y] = mfma_bf16(ah[x], bh, acc[x][y]);
      }
      // three slabs: no operand is read far ahead (registers)
      if (NS == 3 && (decltype(hh)::value || (y & 1))) __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto mid_mid = [&](unsigned char* cur) {
    short8_t am[F];
#pragma unroll
    for (int x = 0; x < F; ++x) am[x] = read_frag(cur + PL + oi[x & 1] + (x >> 1) * 4096);
#pragma unroll
    for (int y = 0; y < F; ++y) {
      const short8_t bm = read_frag(cur + PL + oj[y & 1] + (y >> 1) * 4096);
#pragma unroll
      for (int x = 0; x < F; ++x) acc[x][y] = mfma_bf16(am[x], bm, acc[x][y]);
    }
    if (NS == 3) __builtin_amdgcn_sched_barrier(0);
  };
  // the products of part p of one operand and part q of the other
  auto part_part = [&](int p, int q) {
    short8_t a[F];
#pragma unroll
    for (int x = 0; x < F; ++x) a[x] = read_frag(smem + p * PL + oi[x & 1] + (x >> 1) * 4096);
#pragma unroll
    for (int y = 0; y < F; ++y) {
      const short8_t b = read_frag(smem + q * PL + oj[y & 1] + (y >> 1) * 4096);
#pragma unroll
      for (int x = 0; x < F; ++x) acc[x][y] = mfma_bf16(a[x], b, acc[x][y]);
    }
  };
  load(0);
  __syncthreads();                                               // the means
  convert(0, smem);
  __syncthreads();
  if constexpr (FEW) {
    if (kh == 0) {
      part_part(0, 0);
    } else {
#pragma unroll
      for (int s = 4; s >= 1; --s)                               // small products first
#pragma unroll
        for (int p = max(0, s - 2); p <= min(2, s); ++p) part_part(p, s - p);
    }
  } else {
    // the two waves of a SIMD take the stage in opposite order, so one splits
    // while the other multiplies
    if (NS < 3 || kh == 0) load(1);
    if (kh == 0) {
      for (int st = 0; st < nst; ++st) {
        convert(st + 1, smem + ((st + 1) & 1) * BUF);
        load(st + 2);
        if (NS == 3) __builtin_amdgcn_sched_barrier(0);
        cross(smem + (st & 1) * BUF, std::integral_constant<int, PL>{}, std::true_type{});
        __syncthreads();
      }
    } else {
      for (int st = 0; st < nst; ++st) {
        cross(smem + (st & 1) * BUF, std::integral_constant<int, 2 * PL>{}, std::false_type{});
        if (NS == 3) load(st + 1);             // later than need be: registers
        mid_mid(smem + (st & 1) * BUF);
        __builtin_amdgcn_sched_barrier(0);     // not among the products (2 slabs: 84 -> 78 us at 1387 x 2048 bf16)
        convert(st + 1, smem + ((st + 1) & 1) * BUF);
        if (NS < 3) load(st + 2);
        __syncthreads();
      }
    }
  }
  if (!__syncthreads_or(gram_write<NS>(acc, smem, G, cols, i0, j0, wi, wj, kh, pos, lane))) return;
  gram_classes<T, NS>(A, rows, cols, smem, G, i0, j0);
}

// F[i][j] = F[j][i] = ||G_ij||_F^2 (i <= j), one work-group a block, fixed-order
// sums; F is written into S's memory and turned into S by head_sim_finish.
// VEC (d a multiple of 4, G 16-byte aligned): 32 threads a row of the block, 16-byte loads, eight
// rows in flight; else one value at a time.
template <bool VEC>
__global__ __launch_bounds__(256) void head_sim_blocks(const float* __restrict__ G, int h, int d,
                                                       float* __restrict__ F) {
  const int i = blockIdx.x, j = blockIdx.y;
  if (i > j) return;
  const int n = h * d, tid = threadIdx.x;
  __shared__ float red[256];
  float f = 0.f;
  if constexpr (VEC) {
    const int c0 = 4 * (tid & 31);
    const float* base = G + int64_t(i) * d * n + int64_t(j) * d;
    for (int c = c0; c < d; c += 128)
      for (int r0 = tid >> 5; r0 < d; r0 += 64) {
        floatx4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          v[k] = *reinterpret_cast<const floatx4*>(base + int64_t(min(r0 + 8 * k, d - 1)) * n + c);
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (r0 + 8 * k < d) {
#pragma unroll
            for (int e = 0; e < 4; ++e) f = fmaf(v[k][e], v[k][e], f);
          }
      }
  } else {
    for (int e = tid; e < d * d; e += 256) {
      const float g = G[int64_t(i * d + e / d) * n + j * d + e % d];
      f = fmaf(g, g, f);
    }
  }
  red[tid] = f;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  if (tid == 0) {
    F[i * h + j] = red[0];
    F[j * h + i] = red[0];
  }
}

// S[i][j] = F[i][j] / (sqrt(F[i][i]) sqrt(F[j][j])) in place: one work-group
// reads every F it needs before any thread writes.
__global__ __launch_bounds__(1024) void head_sim_finish(float* __restrict__ S, int h) {
  const int tid = threadIdx.x, nn = h * h;
  float v[4], di[4], dj[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int e = tid + 1024 * k;
    v[k] = di[k] = dj[k] = 0.f;
    if (e < nn) {
      v[k] = S[e];
      di[k] = S[(e / h) * h + e / h];
      dj[k] = S[(e % h) * h + e % h];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int e = tid + 1024 * k;
    if (e < nn) {
      const float den = sqrtf(di[k]) * sqrtf(dj[k]);
      S[e] = den > 0.f ? v[k] / den : 0.f;
    }
  }
}

constexpr int kComputeUnits = 256;        // MI355X

template <typename K, typename... Args>
hipError_t launch_gram_kernel(K kern, size_t lds, int n_tiles, hipStream_t stream, Args... args) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(unsigned(n_tiles)), dim3(kGramThreads), lds, stream, args...);
  return hipGetLastError();
}

template <int NS, bool FEW = false>
hipError_t launch_tiles(const void* A, int32_t dtype, int64_t rows, int32_t cols, const float* mu,
                        int nblk, float* G, hipStream_t stream) {
  const int nt = (cols + 64 * NS - 1) / (64 * NS), n_tiles = nt * (nt + 1) / 2;
  // gram_write's exchange takes 16 NS^2 KB, no more than either kernel's stages
  constexpr size_t lds_bf16 = size_t(kGramNB) * 2 * NS * 8192;
  constexpr size_t lds_split = size_t(2) * 6 * NS * 4096 + 512 * NS;
  static_assert(16 * 1024 * NS * NS <= lds_bf16 && 16 * 1024 * NS * NS <= lds_split, "the exchange fits");
  if (dtype == DCKV_BF16 && !mu)
    return launch_gram_kernel(gram_bf16<NS>, lds_bf16, n_tiles, stream, static_cast<const bf16*>(A),
                              rows, int(cols), G, nt, n_tiles);
  if (dtype == DCKV_BF16)
    return launch_gram_kernel(gram_split<bf16, NS, FEW>, lds_split, n_tiles, stream,
                              static_cast<const bf16*>(A), rows, int(cols), mu, nblk, G, nt, n_tiles);
  return launch_gram_kernel(gram_split<float, NS, FEW>, lds_split, n_tiles, stream,
                            static_cast<const float*>(A), rows, int(cols), mu, nblk, G, nt, n_tiles);
}

}  // namespace

size_t gram_workspace_bytes(int64_t rows, int32_t cols) {
  const int64_t nblk = (rows + kMeanRows - 1) / kMeanRows;
  return size_t((nblk + 1) * cols) * sizeof(float);
}

hipError_t launch_gram(const void* A, int32_t dtype, int64_t rows, int32_t cols, bool center,
                       float* G, void* workspace, hipStream_t stream) {
  const float* mu = nullptr;
  int sums = 0;                              // row blocks of column sums that mu holds (0: means)
  if (center) {
    float* part = static_cast<float*>(workspace);
    const int nblk = int((rows + kMeanRows - 1) / kMeanRows);
    const dim3 g1((cols + 63) / 64, nblk);
    if (dtype == DCKV_BF16)
      hipLaunchKernelGGL(colsum_partial<bf16>, g1, dim3(256), 0, stream,
                         static_cast<const bf16*>(A), rows, cols, part);
    else
      hipLaunchKernelGGL(colsum_partial<float>, g1, dim3(256), 0, stream,
                         static_cast<const float*>(A), rows, cols, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    mu = part;
    sums = nblk;
    if (nblk > kMeanBlocks) {
      float* m = part + int64_t(nblk) * cols;
      hipLaunchKernelGGL(colmean_finish, dim3((cols + 255) / 256), dim3(256), 0, stream, part, nblk,
                         rows, cols, m);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
      mu = m;
      sums = 0;
    }
  }
  // one stage of rows: every product (precision; bf16 samples that are not
  // centred are exact as they are)
  if (rows <= 32 && (mu || dtype == DCKV_F32))
    return launch_tiles<1, true>(A, dtype, rows, cols, mu, sums, G, stream);
  // Tile size: the one whose most loaded compute unit has the least work
  // (one work-group a compute unit), a tile of NS slabs a side costing NS^2
  // products and NS of staging
  int best = 1;
  int64_t best_cost = -1;
  for (int ns = 3; ns >= 1; --ns) {
    const int64_t nt = (cols + 64 * ns - 1) / (64 * ns), tiles = nt * (nt + 1) / 2;
    const int64_t cost = (tiles + kComputeUnits - 1) / kComputeUnits * (ns * ns + ns);
    if (best_cost < 0 || cost < best_cost) {
      best = ns;
      best_cost = cost;
    }
  }
  if (best == 3) return launch_tiles<3>(A, dtype, rows, cols, mu, sums, G, stream);
  if (best == 2) return launch_tiles<2>(A, dtype, rows, cols, mu, sums, G, stream);
  return launch_tiles<1>(A, dtype, rows, cols, mu, sums, G, stream);
}

hipError_t launch_head_similarity(const float* G, int32_t h, int32_t d, float* S,
                                  hipStream_t stream) {
  // 16-byte loads where every row of a block starts on 16 bytes; G itself need
  // only be aligned to its elements
  if (d % 4 == 0 && aligned(G, 16))
    hipLaunchKernelGGL(head_sim_blocks<true>, dim3(h, h), dim3(256), 0, stream, G, h, d, S);
  else
    hipLaunchKernelGGL(head_sim_blocks<false>, dim3(h, h), dim3(256), 0, stream, G, h, d, S);
  hipLaunchKernelGGL(head_sim_finish, dim3(1), dim3(1024), 0, stream, S, h);
  return hipGetLastError();
}

}  // namespace dckv
