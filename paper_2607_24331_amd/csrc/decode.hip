// Decode attention over the compressed cache without rebuilding keys or
// values (read side of Sec. III-A, x W ~ z R):
//   fold   q~_h = q_h R_{g,h}^T * log2(e)/sqrt(d_h)   (Sec. III-C group factor)
//   split  per (sequence, head, context split): scores s_t = q~_h . z_{g,t},
//          online softmax in base 2, acc = sum_t p_t z_{v,t} in value-latent
//          space (Sec. III-D shared value latent)
//   merge  fixed ascending-split log-sum-exp merge, then o_h = (acc / l)
//          R_v[:, kv(h) block] (one up-projection per head)
#include <algorithm>
#include <vector>
#include <cmath>

#include "device.h"
#include "internal.h"

namespace dckv {
namespace {

constexpr int kThreads = 256;
constexpr int kTargetWorkgroups = 256;    // MI355X compute units
constexpr int32_t kValuSplitTokens = 1024;
constexpr int kAccPerThread = DCKV_MAX_VALUE_RANK / kThreads;

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---------------------------------------------------------------- fold
template <typename T>
__global__ __launch_bounds__(kThreads) void fold_kernel(const float* __restrict__ q,
                                                        const T* __restrict__ Rk,
                                                        float* __restrict__ qt, HeadTables tb,
                                                        float scale) {
  const int h = blockIdx.x, b = blockIdx.y;
  const int dh = tb.head_dim;
  __shared__ float qs[DCKV_MAX_HEAD_DIM];
  for (int d = threadIdx.x; d < dh; d += kThreads) qs[d] = q[(int64_t(b) * tb.n_q_heads + h) * dh + d];
  __syncthreads();
  const int r = tb.rank_of_q[h];
  const T* base = Rk + tb.roff_of_q[h] + tb.rcol_of_q[h];
  const int stride = tb.rstride_of_q[h];
  float* dst = qt + int64_t(b) * tb.qlen + tb.qoff[h];
  for (int j = threadIdx.x; j < r; j += kThreads) {
    const T* row = base + int64_t(j) * stride;
    float acc = 0.f;
    for (int d = 0; d < dh; ++d) acc = fmaf(qs[d], to_f32(row[d]), acc);
    dst[j] = acc * scale;
  }
}

// ------------------------------------------------- split (portable VALU)
// Eight (or, for fp32, twice four) consecutive latents as floats.
template <typename T>
__device__ __forceinline__ void load8(const T* p, float (&v)[8]) {
  if constexpr (sizeof(T) == 4) {
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
    const uint4 a = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] = __uint_as_float(w[j] << 16);
      v[2 * j + 1] = __uint_as_float(w[j] & 0xFFFF0000u);
    }
  }
}

// One 256-thread block per (split, query head, query row): query row
// bq = b * Q + i is query i of sequence b, which sees the first
// T_b - Q + i + 1 cache positions (causal inside the chunk of Q).  Scores:
// four threads (one of each wave) a token, each taking eight columns of every
// 32-column key chunk that meets the group's columns (columns outside it are
// left out, whatever they hold).  Softmax: every wave reduces the page's
// scores by itself.  Values: each thread owns value columns tid, tid + 256,
// ..., and where r_v <= 128 one token half of column tid % 128, the halves
// added at the end.  Latency-bound on the small layers it serves: 8 heads x 64
// over 256 tokens take 6 us in four splits (36 us as one split of scalar
// loads).
template <typename T>
__global__ __launch_bounds__(kThreads) void split_valu(
    const float* __restrict__ qt, const T* __restrict__ pool, int64_t num_pages,
    const int32_t* __restrict__ page_table, int max_pages, const int32_t* __restrict__ seq_lens,
    int max_context, int split_tokens, int n_split, int rv, int64_t page_elems,
    int64_t value_base, float* __restrict__ part_ml, float* __restrict__ part_acc, HeadTables tb) {
  const int split = blockIdx.x, h = blockIdx.y, bq = blockIdx.z;
  const int b = bq / tb.n_queries, qi = bq % tb.n_queries;
  const int tid = threadIdx.x;
  __shared__ float qs[DCKV_MAX_GROUP_RANK + 64];       // folded query from its first chunk's column on
  __shared__ float part[4][DCKV_PAGE_TOKENS];
  __shared__ float ps[DCKV_PAGE_TOKENS];
  __shared__ float half_acc[128];

  int T_b = seq_lens[b];
  T_b = T_b < 0 ? 0 : (T_b > max_context ? max_context : T_b);
  const int T_q = max(0, T_b - tb.n_queries + qi + 1);   // positions this query sees
  const int t0 = split * split_tokens;
  const int t1 = min(t0 + split_tokens, T_q);
  const int r = tb.rank_of_q[h];
  const int koff = tb.koff_of_q[h];
  const int lead = koff & 31, c_lo = koff >> 5;          // columns before the group's in its first chunk
  const int nch = ((koff + r - 1) >> 5) - c_lo + 1;
  for (int j = tid; j < 32 * nch; j += kThreads)
    qs[j] = j >= lead && j < lead + r ? qt[int64_t(bq) * tb.qlen + tb.qoff[h] + j - lead] : 0.f;
  __syncthreads();

  float acc[kAccPerThread];
#pragma unroll
  for (int i = 0; i < kAccPerThread; ++i) acc[i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const int slot = tid & (DCKV_PAGE_TOKENS - 1), quarter = tid >> 6;
  const bool halves = rv <= 128;

  for (int tok = t0; tok < t1; tok += DCKV_PAGE_TOKENS) {
    const int n = min(DCKV_PAGE_TOKENS, t1 - tok);
    const int page = page_table[int64_t(b) * max_pages + tok / DCKV_PAGE_TOKENS];
    const bool valid = page >= 0 && page < num_pages;
    const T* pg = pool + (valid ? int64_t(page) * page_elems : 0);
    float sp = 0.f;
    if (valid && slot < n) {
      // chunk-major keys: column c of this slot at (c/32)*2048 + slot*32 + c%32
      const T* kslot = pg + int64_t(c_lo) * 2048 + slot * 32 + 8 * quarter;
#pragma unroll 4
      for (int c = 0; c < nch; ++c) {
        float v[8];
        load8(kslot + c * 2048, v);
        const int j0 = 32 * c + 8 * quarter;
        const bool inside = j0 >= lead && j0 + 8 <= lead + r;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bool in = inside || (j0 + j >= lead && j0 + j < lead + r);
          sp = fmaf(qs[j0 + j], in ? v[j] : 0.f, sp);
        }
      }
    }
    part[quarter][slot] = sp;
    __syncthreads();
    // every wave: the page's scores, one a lane, and their maximum
    const float s = (valid && slot < n) ? (part[0][slot] + part[1][slot]) + (part[2][slot] + part[3][slot])
                                        : -INFINITY;
    float cmax = s;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, o));
    const float m_new = fmaxf(m_run, cmax);
    if (m_new == -INFINITY) {          // uniform: no valid token so far
      __syncthreads();                 // part is rewritten next page
      continue;
    }
    const float alpha = exp2f(m_run - m_new);
    const float p = s == -INFINITY ? 0.f : exp2f(s - m_new);
    float csum = p;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) csum += __shfl_xor(csum, o);
    if (quarter == 0) ps[slot] = p;
    __syncthreads();
    l_run = l_run * alpha + csum;
    // tile-major values: column j of slot t at (j/16)*1024 + (t/32)*512 + (j%16)*32 + t%32
    auto column = [&](int j, int h0, int h1, float a) {
      const T* vcol = pg + value_base + int64_t(j >> 4) * 1024 + (j & 15) * 32;
      for (int hf = h0; hf < h1; ++hf) {
        if (n >= 32 * hf + 32) {
          float v[4][8];
#pragma unroll
          for (int k = 0; k < 4; ++k) load8(vcol + hf * 512 + 8 * k, v[k]);
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 8; ++e) a = fmaf(ps[32 * hf + 8 * k + e], v[k][e], a);
        } else {
          for (int t = 32 * hf; t < n; ++t) a = fmaf(ps[t], to_f32(vcol[hf * 512 + (t & 31)]), a);
        }
      }
      return a;
    };
    if (halves) {
      const int j = tid & 127, hf = tid >> 7;
      acc[0] *= alpha;
      if (valid && j < rv) acc[0] = column(j, hf, hf + 1, acc[0]);
    } else {
#pragma unroll
      for (int i = 0; i < kAccPerThread; ++i) {
        const int j = tid + i * kThreads;
        if (j < rv) {
          acc[i] *= alpha;
          if (valid) acc[i] = column(j, 0, 2, acc[i]);
        }
      }
    }
    m_run = m_new;
    __syncthreads();                   // part and ps are rewritten next page
  }

  const int64_t row = (int64_t(bq) * tb.n_q_heads + h) * n_split + split;
  if (tid == 0) {
    part_ml[row * 2 + 0] = m_run;
    part_ml[row * 2 + 1] = l_run;
  }
  if (halves) {
    if (tid >= 128) half_acc[tid - 128] = acc[0];
    __syncthreads();
    if (tid < rv) part_acc[row * rv + tid] = acc[0] + half_acc[tid];
    return;
  }
#pragma unroll
  for (int i = 0; i < kAccPerThread; ++i) {
    const int j = tid + i * kThreads;
    if (j < rv) part_acc[row * rv + j] = acc[i];
  }
}

// ------------------------------------------------------ merge + up-project
// The up-projection's ranks are dealt to 256 / ceil64(d_h) thread groups whose
// sums are added in group order.
template <typename T>
__global__ __launch_bounds__(kThreads) void merge_upproject(
    const float* __restrict__ part_ml, const float* __restrict__ part_acc,
    const T* __restrict__ Rv, float* __restrict__ out, int n_split, int rv, HeadTables tb) {
  const int h = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x;
  const int dh = tb.head_dim;
  const int n = tb.n_kv_heads * dh;
  const int kv = h / tb.q_per_kv;
  __shared__ float ash[DCKV_MAX_VALUE_RANK];
  __shared__ float red[kThreads];
  const int64_t row0 = (int64_t(b) * tb.n_q_heads + h) * n_split;
  float M = -INFINITY;
  for (int s = 0; s < n_split; ++s) M = fmaxf(M, part_ml[(row0 + s) * 2]);
  float* o = out + (int64_t(b) * tb.n_q_heads + h) * dh;
  if (M == -INFINITY) {
    for (int d = tid; d < dh; d += kThreads) o[d] = 0.f;
    return;
  }
  float L = 0.f;
  for (int s = 0; s < n_split; ++s) L += exp2f(part_ml[(row0 + s) * 2] - M) * part_ml[(row0 + s) * 2 + 1];
  const float inv = 1.f / L;
  for (int j = tid; j < rv; j += kThreads) {
    float a = 0.f;
    for (int s = 0; s < n_split; ++s) {
      const float w = exp2f(part_ml[(row0 + s) * 2] - M);
      a = fmaf(w, part_acc[(row0 + s) * rv + j], a);
    }
    ash[j] = a * inv;
  }
  __syncthreads();
  const int width = (dh + 63) & ~63, groups = kThreads / width;      // d_h <= 256: at least one
  const int d = tid % width, g = tid / width;
  float acc = 0.f;
  if (d < dh && g < groups) {
    const T* col = Rv + int64_t(kv) * dh + d;
#pragma unroll 8
    for (int j = g; j < rv; j += groups) acc = fmaf(ash[j], to_f32(col[int64_t(j) * n]), acc);
  }
  red[tid] = acc;
  __syncthreads();
  if (tid < dh) {
    for (int k = 1; k < groups; ++k) acc += red[k * width + tid];
    o[tid] = acc;
  }
}

template <typename T>
hipError_t launch_decode_t(const dckv_plan& p, const DecodeShape& sh, const float* q,
                           const void* pool, int64_t num_pages, const int32_t* page_table,
                           int32_t max_pages, const int32_t* seq_lens, const void* R_keys,
                           const void* R_value, float* out, void* workspace, hipStream_t stream) {
  char* ws = static_cast<char*>(workspace);
  float* qt = reinterpret_cast<float*>(ws + sh.off_qt);
  float* ml = reinterpret_cast<float*>(ws + sh.off_ml);
  float* acc = reinterpret_cast<float*>(ws + sh.off_acc);
  const float scale = kLog2e / std::sqrt(float(p.dh));
  const int rows = sh.batch * p.Q;               // query rows (sequence, query)
  hipLaunchKernelGGL(fold_kernel<T>, dim3(p.Hq, rows), dim3(kThreads), 0, stream, q,
                     static_cast<const T*>(R_keys), qt, p.tables, scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (p.prof_before && p.prof_after)   // events stamped by the kernel's own dispatch
    hipExtLaunchKernelGGL(split_valu<T>, dim3(sh.n_split, p.Hq, rows), dim3(kThreads), 0u,
                          stream, p.prof_before, p.prof_after, 0u, qt, static_cast<const T*>(pool),
                          num_pages, page_table, max_pages, seq_lens, sh.max_context,
                          sh.split_tokens, sh.n_split, p.rv, p.page_elems, p.value_base, ml, acc,
                          p.tables);
  else
    hipLaunchKernelGGL(split_valu<T>, dim3(sh.n_split, p.Hq, rows), dim3(kThreads), 0, stream,
                       qt, static_cast<const T*>(pool), num_pages, page_table, max_pages, seq_lens,
                       sh.max_context, sh.split_tokens, sh.n_split, p.rv, p.page_elems,
                       p.value_base, ml, acc, p.tables);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(merge_upproject<T>, dim3(p.Hq, rows), dim3(kThreads), 0, stream, ml, acc,
                     static_cast<const T*>(R_value), out, sh.n_split, p.rv, p.tables);
  return hipGetLastError();
}

}  // namespace

// Two-pass shape.  Score work-groups of eight pages, so that ragged batches
// balance over the compute units.  Value work-groups (sequence, chunk, rank
// group): the tiles a group and the chunk count are chosen so that the
// work-groups fill whole rounds of the compute units, with fewer chunks
// (fewer partials) on ties; split_tokens / 64, when given, is the chunk
// length.  One row slice: waves take pages of the chunk, a group of 4, 6 or
// 8 tiles; the estimate is rounds x (pages a wave x (tiles + head tiles, the
// weight loads counted at half a tile each) + a fixed cost of 4).  Several
// slices: the eight waves walk the chunk's pages together, 2 or 1 tiles a
// wave (1 only beyond 8 row tiles); the estimate, in sixteenths of a page
// of one tile a wave, is rounds x (pages x (16 tiles + 8 + row tiles) + 64):
// a page's weights staged and a barrier cost about half a tile, each row
// tile a sixteenth more.
static DecodeShape pass_shape(const dckv_plan& p, int32_t batch, int32_t max_context) {
  DecodeShape s{};
  s.batch = batch;
  s.max_context = max_context;
  s.pass = true;
  const int64_t npm = std::max<int64_t>(1, (int64_t(max_context) + DCKV_PAGE_TOKENS - 1) / DCKV_PAGE_TOKENS);
  s.npm = int32_t(npm);
  s.unit_pages = kUnitPages;
  s.units_per_seq = int32_t((npm + s.unit_pages - 1) / s.unit_pages);
  const int64_t cap = pass_max_chunk_pages(p);
  const int64_t B = std::max<int32_t>(batch, 1);
  const int32_t RT = p.pass.n_slices * p.pass.nt;
  const bool shared = p.pass.n_slices > 1;
  std::vector<int32_t> options;
  if (!shared) options = {8, 6, 4};
  else if (RT <= 8) options = {2, 1};
  else options = {1};
  int64_t best_cost = -1;
  for (int32_t rgt : options) {
    const int64_t tiles = shared ? int64_t(kSharedWaves) * rgt : rgt;   // value tiles a work-group
    const int64_t nrg = (p.pass.mt_v + tiles - 1) / tiles;
    auto consider = [&](int64_t cp) {
      const int64_t nc = (npm + cp - 1) / cp;
      const int64_t rounds = (B * nc * nrg + kTargetWorkgroups - 1) / kTargetWorkgroups;
      const int64_t cost = shared ? rounds * (cp * (16 * rgt + 8 + RT) + 64)
                                  : rounds * ((cp + 7) / 8 * (rgt + p.pass.nt) + 4);
      if (best_cost < 0 || cost < best_cost || (cost == best_cost && nc < s.n_chunks)) {
        best_cost = cost;
        s.rgt = rgt;
        s.n_rgroups = int32_t(nrg);
        s.chunk_pages = int32_t(cp);
        s.n_chunks = int32_t(nc);
      }
    };
    if (p.split_tokens > 0) {
      consider(std::min<int64_t>(cap, std::max<int64_t>(1, p.split_tokens / DCKV_PAGE_TOKENS)));
    } else {
      // from the fewest chunks the cap allows to about two work-groups a
      // compute unit (at least the first candidate)
      const int64_t lo = (npm + cap - 1) / cap;
      const int64_t hi = std::min(npm, std::max(lo, std::max<int64_t>(1, 2 * kTargetWorkgroups / (B * nrg)) + 1));
      for (int64_t nc = lo; nc <= hi; ++nc) consider((npm + nc - 1) / nc);
    }
  }
  s.split_tokens = s.chunk_pages * DCKV_PAGE_TOKENS;
  s.n_split = s.n_chunks;
  const size_t ns = 16 * size_t(RT);          // row slots
  s.off_qt = 0;
  s.off_p = align_up(size_t(batch) * p.pass.n_slices * p.pass.max_pairs * 2048, 256);
  s.off_ml = s.off_p + align_up(size_t(batch) * npm * RT * 2560, 256);   // weights and records
  const size_t rows = size_t(batch) * s.n_chunks;
  s.off_acc = s.off_ml + align_up(rows * 2 * ns * sizeof(float), 256);
  s.off_opart = s.off_acc + align_up(rows * ns * size_t(p.rv) * sizeof(float), 256);
  s.bytes = s.off_opart + align_up(size_t(batch) * p.Q * p.Hq * p.rv * sizeof(float), 256);
  return s;
}

// Workspace of the single-pass and the portable kernels whose splits leave
// `rows` rows of partials.
static void lay_out(const dckv_plan& p, DecodeShape& s, size_t rows) {
  const size_t nh = s.mfma ? 16 * size_t(p.mfma.nt) : 1;
  s.off_qt = 0;
  s.off_ml = s.mfma   // hi/lo query blocks of 2 KB per (sequence, slice, chunk)
                 ? align_up(size_t(s.batch) * p.mfma.n_slices * p.mfma.max_pairs * 2048, 256)
                 : align_up(size_t(s.batch) * p.Q * p.qlen * sizeof(float), 256);
  s.off_acc = s.off_ml + align_up(rows * 2 * nh * sizeof(float), 256);
  s.off_opart = s.off_acc + align_up(rows * nh * size_t(p.rv) * sizeof(float), 256);
  s.bytes = s.off_opart;
  if (s.mfma) s.bytes += align_up(size_t(s.batch) * p.Q * p.Hq * p.rv * sizeof(float), 256);
}

static size_t sched_bytes(int64_t units, int32_t batch) {
  return align_up(size_t(units) * sizeof(SchedUnit) + size_t(batch) * sizeof(SchedSeq), 256);
}

DecodeShape decode_shape(const dckv_plan& p, int32_t batch, int32_t max_context, bool plain) {
  // The two-pass kernels when asked for, when the single-pass kernel does not
  // apply, or when it would cut the rows into several slices (a value rank
  // beyond what one slice's accumulators hold), each slice reading the whole
  // value part again, and the batch holds enough pages to give every wave of
  // the chip one.  Otherwise the single-pass kernel: measured on the one-query
  // layers it is as fast or faster, the two passes each paying a work-group
  // prologue and a tail.
  if (p.pass_ok) {
    const int64_t npm = (int64_t(max_context) + DCKV_PAGE_TOKENS - 1) / DCKV_PAGE_TOKENS;
    const bool many_pages = int64_t(batch) * npm >= int64_t(8) * kTargetWorkgroups;
    if (p.decode_passes == 2 || !p.mfma_ok || (many_pages && p.mfma.n_slices > 1))
      return pass_shape(p, batch, max_context);
  }
  DecodeShape s{};
  s.batch = batch;
  s.max_context = max_context;
  s.mfma = p.mfma_ok;
  int64_t L = p.split_tokens;
  // Two value slices where a compute unit's share is at most three pages: a
  // split's partials (value rank x rows fp32, whatever its length) are then
  // most of the traffic beside the latents, and twice the splits' length
  // halves them, the keys, which both halves read, coming the second time
  // from their XCD's L2.  Measured, 8 sequences, one slice / two, us: value
  // rank 2048: 512 tokens 46.8 / 41.7, 2048: 67.2 / 59.6, 4096: 89.9 / 86.3,
  // 6144: 111.5 / 108.9, 8192: 133.0 / 132.7, 16384: 216 / 223; 1536: 39.2 /
  // 35.8, 53.4 / 47.7, 70.1 / 64.9, 84.1 / 83.2, 98.1 / 99.6, 153 / 163.
  if (s.mfma && L == 0 && p.mfma2_ok && !plain) {
    const int64_t npm = (int64_t(max_context) + DCKV_PAGE_TOKENS - 1) / DCKV_PAGE_TOKENS;
    s.halves = int64_t(batch) * npm * p.mfma.n_slices <= 3 * kTargetWorkgroups;
  }
  const int vs = s.halves ? 2 : 1;
  if (L == 0) {
    if (s.mfma) {
      // about one work-group per compute unit over the whole batch, at most
      // the split kernel's page-list capacity
      const int64_t tokens = int64_t(batch) * max_context * p.mfma.n_slices * vs;
      L = (tokens + kTargetWorkgroups - 1) / kTargetWorkgroups;
      L = std::max<int64_t>(DCKV_PAGE_TOKENS, (L + DCKV_PAGE_TOKENS - 1) / DCKV_PAGE_TOKENS * DCKV_PAGE_TOKENS);
      L = std::min<int64_t>(L, mfma_max_split_tokens());
    } else {
      // kValuSplitTokens, less while that leaves compute units without a block
      const int64_t work = int64_t(batch) * p.Q * p.Hq * max_context;
      L = (work + kTargetWorkgroups - 1) / kTargetWorkgroups;
      L = std::max<int64_t>(DCKV_PAGE_TOKENS, (L + DCKV_PAGE_TOKENS - 1) / DCKV_PAGE_TOKENS * DCKV_PAGE_TOKENS);
      L = std::min<int64_t>(L, kValuSplitTokens);
    }
  }
  if (s.mfma && L > mfma_max_split_tokens()) s.mfma = false;   // an explicit split beyond the cap
  s.split_tokens = int32_t(L);
  s.n_split = max_context > 0 ? int32_t((max_context + L - 1) / L) : 1;
  lay_out(p, s, size_t(batch) * s.n_split * (s.mfma ? p.mfma.n_slices : p.Q * p.Hq));
  if (s.mfma) {
    const int64_t units = int64_t(batch) * s.n_split;
    s.n_units = int32_t((units + 7) / 8 * 8);
    s.merge_ranks = mfma_merge_ranks(p, batch);
    s.n_rchunks = (p.rv + s.merge_ranks - 1) / s.merge_ranks;
    // Balanced splits: several sequences, no split size asked for, and a head
    // size whose fold kernel cuts them.  Never more splits than the fixed cut
    // has (their partials share its workspace), and a whole number of rounds
    // over the compute units where that leaves one a sequence and none longer
    // than the split kernel's page list.  Fixed splits are sized by
    // max_context: 64 sequences of 1024 to 8192 tokens leave a third of the
    // compute units without work (split kernel 370 us, balanced 292).  The
    // line does not lie at a batch: the host does not know the lengths, and
    // whole calls on a 32/8-head layer over lengths of an eighth to the whole
    // of 131072 / batch tokens go 74.3 -> 72.6 us at 4 sequences, 81.3 -> 73.0
    // at 16, 90.3 -> 80.1 at 64.  One sequence is cut evenly as it is.
    if (!plain && p.split_tokens == 0 && batch >= 2 && batch <= kSchedMaxBatch && units <= kSchedMaxUnits &&
        (p.dh == 64 || p.dh == 128)) {
      const int64_t npm = (int64_t(max_context) + DCKV_PAGE_TOKENS - 1) / DCKV_PAGE_TOKENS;
      const int64_t cap = mfma_max_split_tokens() / DCKV_PAGE_TOKENS;
      const int64_t target = std::max<int64_t>(1, kTargetWorkgroups / (p.mfma.n_slices * vs));
      int64_t U = units;
      const int64_t whole = U / target * target;
      if (whole >= batch && int64_t(batch) * ((npm + cap - 1) / cap) <= whole) U = whole;
      // The fixed cut itself, which needs no record, where every sequence has
      // at least this many pages: all its splits less a page each (no cut into
      // as many splits is shorter), or five eighths of them where a sequence
      // has 24 splits or more.  The call is bound by memory, so that compute
      // units without a split cost nothing while enough others have one in
      // every XCD; with fewer splits a sequence the short ones' missing splits
      // are the same XCDs'.  32/8-head layer, lengths from the given part of
      // 131072 / batch tokens on, fixed / balanced, us: 4 sequences 0.4: 81.7 /
      // 80.1, 0.5: 82.3 / 82.9, 0.7: 85.7 / 87.4; 8: 0.5: 82.4 / 81.1, 0.6:
      // 83.7 / 84.8, 0.8: 87.4 / 88.6; 16: 0.6: 90.0 / 86.5, 0.8: 94.2 / 92.8.
      const int64_t Lp = L / DCKV_PAGE_TOKENS;
      int64_t least = s.n_split * (Lp - 1) + 1;
      if (s.n_split >= 24) least = std::min(least, (5 * s.n_split * Lp + 7) / 8);
      s.fixed_pages = U == units ? int32_t(least) : INT32_MAX;
      s.n_sched = int32_t(U);
      s.n_units = int32_t((U + 7) / 8 * 8);
      s.off_sched = s.bytes;
      s.sched_bytes = sched_bytes(U, batch);
      s.bytes += s.sched_bytes;
    }
  }
  return s;
}

// A buffer of this size serves every call of at most that many sequences and
// tokens.  Where the library chooses the split size, a shorter context may
// leave more splits (longer splits come in whole pages), so the size is not
// the call's own but that of a bound on the rows of partials: splits that were
// lengthened to make about kTargetWorkgroups of them are at most that many and
// one more a row of the batch, and never more than a page each; those at the
// longest split length grow with the context.
size_t decode_workspace_bytes(const dckv_plan& p, int32_t batch, int32_t max_context) {
  const DecodeShape s = decode_shape(p, batch, max_context);
  if (p.split_tokens > 0 || (s.pass && (p.decode_passes == 2 || !p.mfma_ok))) return s.bytes;
  DecodeShape t{};
  t.batch = batch;
  t.mfma = p.mfma_ok;
  const int64_t per_seq = p.mfma_ok ? p.mfma.n_slices : int64_t(p.Q) * p.Hq;
  const int64_t longest = (p.mfma_ok ? mfma_max_split_tokens() : kValuSplitTokens) / DCKV_PAGE_TOKENS;
  const int64_t npm = std::max<int64_t>(1, (int64_t(max_context) + DCKV_PAGE_TOKENS - 1) / DCKV_PAGE_TOKENS);
  const int64_t rows = std::max(batch * per_seq * ((npm + longest - 1) / longest),
                                std::min(kTargetWorkgroups + batch * per_seq, batch * per_seq * npm));
  lay_out(p, t, size_t(rows));
  if (t.mfma) t.bytes += sched_bytes(kSchedMaxUnits, std::min(batch, kSchedMaxBatch));
  return std::max(s.bytes, t.bytes);
}

hipError_t launch_decode(const dckv_plan& p, const DecodeShape& shape, const float* q,
                         const void* pool, int64_t num_pages, const int32_t* page_table,
                         int32_t max_pages, const int32_t* seq_lens, const void* R_keys,
                         const void* R_value, float* out, void* workspace, hipStream_t stream) {
  if (shape.pass)
    return launch_decode_pass(p, shape, q, pool, num_pages, page_table, max_pages, seq_lens, R_keys,
                              R_value, out, workspace, stream);
  if (shape.mfma)
    return launch_decode_mfma(p, shape, q, pool, num_pages, page_table, max_pages, seq_lens, R_keys,
                              R_value, out, workspace, stream);
  if (p.dtype == DCKV_F32)
    return launch_decode_t<float>(p, shape, q, pool, num_pages, page_table, max_pages, seq_lens,
                                  R_keys, R_value, out, workspace, stream);
  return launch_decode_t<bf16>(p, shape, q, pool, num_pages, page_table, max_pages, seq_lens, R_keys,
                               R_value, out, workspace, stream);
}

}  // namespace dckv
