// Decoder kernels of the rollout decode step and the prompt prefill (gfx950).
//
// Per layer, over the rows of a batch (occupied slots in decode, prompt
// tokens in prefill):
//   q|k|v GEMM with RoPE and the paged KV append in its epilogue (a short bf16
//   prefill chunk: split-K partials and k_qkv_epilogue)
//   paged GQA attention over ragged contexts (split-context + combine)
//   gemm(o, W_o)   -> residual add + RMSNorm -> x
//   gemm(x, W_gu) with SwiGLU in its epilogue -> a
//   gemm(a, W_d)   -> residual add + RMSNorm of the next layer (or final) -> x
// then the LM head gemm and the Gumbel-max sampler.  The layers of a bf16
// prefill are in prefill_kernels.hip, its tile GEMM in gemm_tile.h.
//
// GEMMs take both operands with K contiguous and run on the bf16 MFMA
// (v_mfma_f32_16x16x32_bf16), fp32 models' on the fp32 one
// (v_mfma_f32_16x16x4_f32), with fp32 accumulation; split-K partials go to a
// workspace and are summed in split order by the consumer, so results do not
// depend on scheduling.
#include <mutex>

#include "gemm_tile.h"
#include "sara_internal.h"

#include <math.h>
#include <string.h>

#include <algorithm>

namespace sara {

// ---------------------------------------------------------------------------
// block reductions (fixed tree order -> deterministic)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
// place of feature k of row i in the GEMM inputs that both dtypes' kernels
// write (prefill, and the q|k|v input of a decode step): fragment-major in bf16
// models, row-major in fp32 ones
template <typename T>
__device__ __forceinline__ size_t x_index(int64_t i, int64_t k, int64_t K) {
  return sizeof(T) == 2 ? (size_t)tiled_index(i, k, K) : (size_t)(i * K + k);
}
// 8 consecutive stored values (16-byte aligned) as fp32, and back
__device__ __forceinline__ void load8(const float* p, float (&e)[8]) {
  const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
#pragma unroll
  for (int q = 0; q < 4; ++q) { e[q] = a[q]; e[q + 4] = b[q]; }
}
__device__ __forceinline__ void load8(const uint16_t* p, float (&e)[8]) {
  const u32x4 a = *(const u32x4*)p;
#pragma unroll
  for (int q = 0; q < 4; ++q) { e[2 * q] = __uint_as_float(a[q] << 16); e[2 * q + 1] = __uint_as_float(a[q] & 0xFFFF0000u); }
}
__device__ __forceinline__ void store8(float* p, float a, float b, float c, float d, float e, float f, float g, float h) {
  *(f32x4*)p = f32x4{a, b, c, d};
  *(f32x4*)(p + 4) = f32x4{e, f, g, h};
}
__device__ __forceinline__ void store8(uint16_t* p, float a, float b, float c, float d, float e, float f, float g, float h) {
  *(u32x4*)p = u32x4{pack_bf16(a, b), pack_bf16(c, d), pack_bf16(e, f), pack_bf16(g, h)};
}
// sum over a 256-thread block; every thread gets the result
__device__ float block_sum256(float v, float* red) {
  v = wave_sum(v);
  int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float r = (red[0] + red[1]) + (red[2] + red[3]);
  return r;
}

// ---------------------------------------------------------------------------
// Gumbel-max sampling helpers
// ---------------------------------------------------------------------------
// score_v = fp32(logit_v / T) + fp32(-log(-log u_v)), u_v = ((w >> 8) + 1/2) 2^-24
// from word v % 4 of Philox(rid, gen, v / 4, 0); the token is the lowest id
// of the maximal score.
__device__ __forceinline__ void better(float& bs, int& bi, float s, int i) {
  if (s > bs || (s == bs && i < bi)) { bs = s; bi = i; }
}
// The noise as the sampler defines it: fp64 logs, rounded to fp32.
__device__ __forceinline__ float gumbel_exact(uint32_t w) {
  const double u = ((double)(w >> 8) + 0.5) * 0x1p-24;
  return (float)(-log(-log(u)));
}
// fp32 estimate of gumbel_exact on the hardware log2 (v_log_f32): -ln(u) for
// u < 1/2 (u exact in fp32), and -log1p(-d) with d = 1 - u (exact in fp32)
// otherwise, through log1p(x) = ln(1 + x) x / ((1 + x) - 1) (Goldberg), then
// -ln of the result.  Its distance to gumbel_exact is below kGumbelFastErr
// for every one of the 2^24 inputs (sara_gumbel_fast_max_error measures it
// exhaustively).
constexpr float kGumbelFastErr = 2e-5f;
__device__ __forceinline__ float ln_hw(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945309f; }
__device__ __forceinline__ float gumbel_fast(uint32_t w) {
  const uint32_t m = w >> 8;
  float t;
  if (m < (1u << 23)) {
    t = -ln_hw(((float)m + 0.5f) * 0x1p-24f);
  } else {
    const float dl = (((float)((1u << 24) - m) - 0.5f) * 0x1p-24f);
    const float y = 1.0f - dl;
    t = (y == 1.0f) ? dl : ln_hw(y) * (dl * __builtin_amdgcn_rcpf(y - 1.0f));
  }
  return -ln_hw(t);
}
// Upper bound of gumbel_exact without a logarithm: -log(-log u) <= -ln(1 - u)
// (as -ln u >= 1 - u), and log2 x >= exponent + mantissa fraction of x, which is
// x's bit pattern read as a fixed-point number.  Above the noise by at most
// 0.11 for u > 0.9 (where most winners lie), with 1e-4 of slack for every
// rounding on the way.
__device__ __forceinline__ float gumbel_upper(uint32_t w) {
  const float x = (float)(~w >> 8) + 0.5f;   // (1 - u) 2^24
  return fmaf((float)(int)__float_as_uint(x), -8.26295829e-8f, 104.665224f + 1e-4f);   // -ln2 2^-23, 151 ln2
}
// fp32(logit / T); UNIT: T = 1, where the division is exact and skipped.
template <bool UNIT>
__device__ __forceinline__ float temper(float x, float temp) { return UNIT ? x : __fdiv_rn(x, temp); }
// Lower bound on every exact score that can still be maximal, given the
// largest fast score smax: each fast score is within
// kGumbelFastErr + 2^-22 |score| of its exact value (the noise error plus
// the two fp32 roundings of the sum), so candidates lie within twice that
// of smax (with slack for |score| near |smax|).
__device__ __forceinline__ float gumbel_candidate_floor(float smax) {
  if (smax == INFINITY) return smax;   // only infinite scores can win
  return smax - 2.0f * kGumbelFastErr - (fabsf(smax) + 1.0f) * 0x1p-20f;
}

// ---------------------------------------------------------------------------
// embedding gather + first RMSNorm (decode and prefill rows)
// ---------------------------------------------------------------------------
// sum of v over a 256-thread block (buf: 4 ints; ends with a barrier)
__device__ __forceinline__ int block_count256(int v, int* buf) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) buf[threadIdx.x >> 6] = v;
  __syncthreads();
  const int r = (buf[0] + buf[1]) + (buf[2] + buf[3]);
  __syncthreads();
  return r;
}

// Decode rows + embedding gather + first RMSNorm in one launch: row i of the
// batch is occupied slot active[i]; the device row count goes to rows_M.  A
// row costs three dependent loads: its slot, the slot's count and input token,
// the embedding row; a thread takes 8 features at a time and keeps them in
// registers between the sum of squares and the norm.  The last block lists the
// decode attention's items meanwhile.
template <typename T>
__global__ __launch_bounds__(256) void k_decode_embed(const Ctl* __restrict__ ctl,
    const ActiveRow* __restrict__ active, const int32_t* __restrict__ slot_gen, const int32_t* __restrict__ slot_tok,
    int k, RowDesc* __restrict__ rows, int32_t* __restrict__ rows_M, int do_embed, const T* __restrict__ embed,
    const float* __restrict__ w, int d, float eps, float* __restrict__ h, T* __restrict__ x,
    int U, int PB, int SB, const float2* __restrict__ rope, int half, float2* __restrict__ row_rope,
    AttnItem* __restrict__ items, int32_t* __restrict__ n_items, int spg, const PromptPlace* __restrict__ places,
    int hkv, int rows_per_item, int resident, int V) {
  __shared__ float red[4];
  __shared__ int scan[4];
  const int M = ctl->done ? 0 : ctl->M;
  if (blockIdx.x == 0 && threadIdx.x == 0) *rows_M = M;
  if (items != nullptr && blockIdx.x == gridDim.x - 1) {
    // The decode attention's work list for this step (the same for every
    // layer): the context splits of spg pages of every row.  256 rows at a
    // time, thread t lists one at the prefix sum of the earlier ones' counts.
    // As long as all items are resident at once (items x hkv <= resident), each
    // row has its own, row-major.  Beyond that K and V traffic counts, not
    // latency, and rows of one prompt share the items of the splits that lie
    // wholly in its prompt pages, up to rows_per_item rows each, in prompt
    // order; the splits and so the results are the same.
    int done = 0;
    bool shared = M > 256;
    for (int base = 0; base < M; base += 256) {
      const int j = base + (int)threadIdx.x;
      AttnItem it{};
      int first = 0, ns = 0, lead = 0;      // own splits [first, ns), shared splits [0, lead) that it lists
      auto row_item = [&](int i) {
        const ActiveRow a = active[i];
        it.i = i;
        it.n = 1;
        it.kv0 = a.uid * PB;
        it.kv1 = U * PB + a.slot * SB;
        it.pl = a.plen;                     // context P + g exceeds the P - 1 prompt positions
        it.vcnt = slot_gen[a.slot] + 1;
        const int nch = ((it.pl + 15) >> 4) + ((it.vcnt + 15) >> 4);
        ns = (nch + spg - 1) / spg;
      };
      if (!shared) {
        if (j < M) row_item(j);
        // M <= 256: the whole batch's item count
        const int all = block_count256(ns, scan);
        shared = all * hkv > resident;
      }
      int members = 1;
      if (shared) {
        ns = 0;
        if (j < M) {
          const PromptPlace p = places[j];
          row_item(p.row);
          const int at = p.rank % rows_per_item;
          members = min(rows_per_item, p.n - ((int)p.rank - at));
          if (members > 1) {
            first = ((it.pl + 15) >> 4) / spg;
            if (at == 0) lead = first;
          }
        }
      }
      int incl = ns - first + lead;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if ((int)(threadIdx.x & 63) >= o) incl += v;
      }
      if ((threadIdx.x & 63) == 63) scan[threadIdx.x >> 6] = incl;
      __syncthreads();
      int at = done + incl - (ns - first + lead), total = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q < (int)(threadIdx.x >> 6)) at += scan[q];
        total += scan[q];
      }
      AttnItem sh = it;
      sh.i = j;
      sh.n = members;
      for (int cc = 0; cc < lead; ++cc) {
        sh.c = cc;
        items[at++] = sh;
      }
      for (int cc = first; cc < ns; ++cc) {
        it.c = cc;
        items[at++] = it;
      }
      done += total;
      __syncthreads();   // scan[] is reused by the next rows
    }
    if (threadIdx.x == 0) *n_items = done;
  }
  constexpr int VPT = 2;                    // 8-feature groups a thread takes: d <= 4096 in registers
  for (int i = blockIdx.x; i < M; i += gridDim.x) {
    const ActiveRow a = active[i];
    const int g = slot_gen[a.slot], tok = slot_tok[a.slot];
    RowDesc r;
    r.tok = tok;
    r.pos = a.plen + g;
    r.plen = a.plen;
    r.slot = a.slot;
    r.rid = a.uid * k + a.j;
    r.gen = g;
    r.uid = a.uid;
    r.kv0 = a.uid * PB;
    r.kv1 = U * PB + a.slot * SB;
    if (threadIdx.x == 0) rows[i] = r;
    // rotation angles of this row's position, read by every layer's q|k|v kernel
    for (int e = threadIdx.x; e < half; e += 256) row_rope[(size_t)i * half + e] = rope[(size_t)r.pos * half + e];
    if (!do_embed) continue;
    // a row whose logits were all NaN has no best id and carries INT_MAX
    const T* er = embed + (size_t)min((uint32_t)tok, (uint32_t)V - 1u) * d;
    float* hr = h + (size_t)i * d;
    float v[VPT][8];
    float ss = 0.f;
    // groups past VPT (fp32 models wider than 4096) are read again below
    for (int u = 0, c = 8 * (int)threadIdx.x; c < d; ++u, c += 2048) {
      float e[8];
      load8(er + c, e);
#pragma unroll
      for (int q = 0; q < 8; ++q) ss += e[q] * e[q];
#pragma unroll
      for (int t = 0; t < VPT; ++t)
        if (u == t)
#pragma unroll
          for (int q = 0; q < 8; ++q) v[t][q] = e[q];
    }
    float tot = block_sum256(ss, red);
    float inv = 1.0f / sqrtf(tot / (float)d + eps);
    for (int u = 0, c = 8 * (int)threadIdx.x; c < d; ++u, c += 2048) {
      float e[8];
      if (u >= VPT) load8(er + c, e);
#pragma unroll
      for (int t = 0; t < VPT; ++t)
        if (u == t)
#pragma unroll
          for (int q = 0; q < 8; ++q) e[q] = v[t][q];
      *(f32x4*)(hr + c) = f32x4{e[0], e[1], e[2], e[3]};
      *(f32x4*)(hr + c + 4) = f32x4{e[4], e[5], e[6], e[7]};
      const f32x4 w0 = *(const f32x4*)(w + c), w1 = *(const f32x4*)(w + c + 4);
      store8(x + x_index<T>(i, c, d), e[0] * inv * w0[0], e[1] * inv * w0[1], e[2] * inv * w0[2], e[3] * inv * w0[3],
             e[4] * inv * w1[0], e[5] * inv * w1[1], e[6] * inv * w1[2], e[7] * inv * w1[3]);
    }
    __syncthreads();   // red[] is reused by the next row
  }
}

// Prefill rows of the chunk [r0, r0 + n): global prompt-token row r maps to
// prompt u (pre[u] <= r < pre[u+1]) and token t = r - pre[u].
__global__ __launch_bounds__(256) void k_prefill_rows(const int32_t* __restrict__ pre, int U,
    int r0, int n, const int32_t* __restrict__ tok, const int32_t* __restrict__ off,
    RowDesc* __restrict__ rows, int32_t* __restrict__ rows_M, int PB) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *rows_M = n;
  if (i >= n) return;
  int r = r0 + i;
  int lo = 0, hi = U;  // largest u with pre[u] <= r
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (pre[mid] <= r) lo = mid; else hi = mid;
  }
  int u = lo, t = r - pre[u];
  RowDesc d;
  d.tok = tok[off[u] + t];
  d.pos = t;
  d.plen = off[u + 1] - off[u] - 1;
  d.slot = -1;
  d.rid = -1;
  d.gen = -1;
  d.uid = u;
  d.kv0 = u * PB;
  d.kv1 = -1;
  rows[i] = d;
}

__global__ __launch_bounds__(256) void k_embed_norm(const int32_t* __restrict__ M_ptr,
    const RowDesc* __restrict__ rows, const float* __restrict__ embed, const float* __restrict__ w,
    int d, float eps, float* __restrict__ h, float* __restrict__ x) {
  __shared__ float red[4];
  int i = blockIdx.x;
  if (i >= *M_ptr) return;
  int t = rows[i].tok;
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += 256) {
    float v = embed[(size_t)t * d + c];
    h[(size_t)i * d + c] = v;
    ss += v * v;
  }
  float tot = block_sum256(ss, red);
  float inv = 1.0f / sqrtf(tot / (float)d + eps);
  for (int c = threadIdx.x; c < d; c += 256)
    x[(size_t)i * d + c] = h[(size_t)i * d + c] * inv * w[c];
}

// ---------------------------------------------------------------------------
// GEMM: out[s][m][n] = sum_{k in split s} X[m][k] * W[n][k]
// ---------------------------------------------------------------------------
// Gumbel-max sampling over this block's vocabulary rows, straight from the
// LM-head accumulators (no logits round trip through memory).  Lane (row,
// grp) holds, for activation tile t and weight tile nt, the logits of
// vocabulary ids v = n0 + 16 nt + 4 grp + q (q < 4) of decode row
// m_base + 16 t + row: exactly the four ids one Philox call keys.
//  1. upper bounds of all scores (gumbel_upper: a handful of instructions an
//     id, no logarithm), the fast score (fp32 noise, gumbel_fast) of each lane's
//     best bound, and the block maximum of those per row;
//  2. exact scores (fp64 noise, gumbel_exact) for the candidates whose bound
//     reaches gumbel_candidate_floor(max): the block's exact winner is always
//     among them, so the result equals an exact evaluation of every id;
//  3. exact (score, id) maximum per row to sa.best / sa.idx [vocabulary block][ld].
// LDS: the X staging buffer, free after the k loop.  151936 ids, 32 rows: 88 us with
// the GEMM against 95 with a logarithm an id and exact scores place by place;
// 32768 ids, 512 rows: 119 against 174.
// Exact score of vocabulary id 4 b + q of decode rollout (rid, gen), given
// the tempered logit a = fp32(logit / T).  Out of line: it is called for a
// handful of candidates per row and block, and keeps the fp64 logs out of
// the unrolled epilogue.
__device__ __attribute__((noinline)) float exact_score(float a, uint32_t rid, uint32_t gen, uint32_t b, int q,
                                                       uint32_t k0, uint32_t k1) {
  const U32x4 w = philox4x32_10(rid, gen, b, 0u, k0, k1);
  const uint32_t wq = q == 0 ? w.x : q == 1 ? w.y : q == 2 ? w.z : w.w;
  return __fadd_rn(a, gumbel_exact(wq));
}

// One round of the sampling epilogue over activation tiles T0 .. T0 + TC - 1
// (compile-time tile indices, so the accumulators stay in registers).  wave:
// this wave's quarter of the ids, tid: the thread among the four waves that
// share the rows, xs: their LDS, chunk: the vocabulary block.  Every wave of the
// thread block takes part in the same rounds.
template <int NT, int MT, int TC, int T0, bool UNIT>
__device__ __forceinline__ void sample_round(const f32x4 (&acc)[NT][MT], int M, int m_base, int N, int n0,
    const SampleArgs& sa, float temp, uint32_t k0, uint32_t k1, void* xs, int wave, int tid, int chunk) {
  static_assert(NT * TC <= 8, "one bit a (tile, id) place of a lane");
  const int lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;
  float* red_max = (float*)xs;                          // [4][TC][16]
  float* red_s = red_max + 4 * TC * 16;                 // [4][TC][16]
  int* red_i = (int*)(red_s + 4 * TC * 16);             // [4][TC][16]
  // (rid, gen, slot) of the decode rows of this round's tiles
  int s_rid[TC], s_gen[TC], s_slot[TC];
#pragma unroll
  for (int tt = 0; tt < TC; ++tt) {
    const RowDesc r = sa.rows[min(m_base + 16 * (T0 + tt) + row, M - 1)];
    s_rid[tt] = r.rid; s_gen[tt] = r.gen; s_slot[tt] = r.slot;
  }
  __syncthreads();                                      // LDS: the k loop or the previous round is done
  float f[NT][TC][4];                                   // upper bounds of the scores
#pragma unroll
  for (int tt = 0; tt < TC; ++tt) {
    float lub = -INFINITY, la = -INFINITY;               // the lane's best bound, its logit
    uint32_t lw = 0u;                                    // and its noise word
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int v0 = n0 + 16 * nt + 4 * grp;
      const U32x4 w = philox4x32_10((uint32_t)s_rid[tt], (uint32_t)s_gen[tt], (uint32_t)(v0 >> 2), 0u, k0, k1);
      const uint32_t wd[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = temper<UNIT>(acc[nt][T0 + tt][q], temp);
        f[nt][tt][q] = (v0 + q < N) ? a + gumbel_upper(wd[q]) : __builtin_nanf("");
        if (f[nt][tt][q] > lub) { lub = f[nt][tt][q]; la = a; lw = wd[q]; }
      }
    }
    float lmax = __fadd_rn(la, gumbel_fast(lw));
    lmax = fmaxf(lmax, __shfl_xor(lmax, 16, 64));
    lmax = fmaxf(lmax, __shfl_xor(lmax, 32, 64));
    if (grp == 0) red_max[(wave * TC + tt) * 16 + row] = lmax;
  }
  // optional copy of the logits (parity runs)
  if (sa.logits) {
#pragma unroll
    for (int tt = 0; tt < TC; ++tt) {
      const int m = m_base + 16 * (T0 + tt) + row;
      if (m >= M) continue;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int v = n0 + 16 * nt + 4 * grp + q;
          if (v < N) sa.logits[(size_t)s_slot[tt] * N + v] = acc[nt][T0 + tt][q];
        }
    }
  }
  __syncthreads();
  // candidates of this lane over the round's tiles, one bit each
  uint32_t cand = 0u;
  float bs[TC];
  int bi[TC];
#pragma unroll
  for (int tt = 0; tt < TC; ++tt) {
    const float* rm = red_max + tt * 16 + row;
    const float bmax = fmaxf(fmaxf(rm[0], rm[TC * 16]), fmaxf(rm[2 * TC * 16], rm[3 * TC * 16]));
    const float floor_ = gumbel_candidate_floor(bmax);
    bs[tt] = -INFINITY;
    bi[tt] = 0x7FFFFFFF;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (f[nt][tt][q] >= floor_) cand |= 1u << ((tt * NT + nt) * 4 + q);
  }
  // Exact scores, every lane its own next candidate at once: a row has one or
  // two per block, so the wave goes through the fp64 logarithms once or twice a
  // round, not once for each (tile, id) place that holds a candidate.
  while (__any(cand != 0u)) {
    if (cand != 0u) {
      const int bit = __ffs((int)cand) - 1;
      cand &= cand - 1u;
      const int tt_ = bit / (4 * NT), nt_ = (bit >> 2) % NT, q_ = bit & 3;
      float a = 0.f;
      uint32_t rid = 0u, gen = 0u;
#pragma unroll
      for (int tt = 0; tt < TC; ++tt) {
        if (tt_ == tt) { rid = (uint32_t)s_rid[tt]; gen = (uint32_t)s_gen[tt]; }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (bit == (tt * NT + nt) * 4 + q) a = acc[nt][T0 + tt][q];
      }
      const int v0 = n0 + 16 * nt_ + 4 * grp;
      const float s = exact_score(temper<UNIT>(a, temp), rid, gen, (uint32_t)(v0 >> 2), q_, k0, k1);
#pragma unroll
      for (int tt = 0; tt < TC; ++tt)
        if (tt_ == tt) better(bs[tt], bi[tt], s, v0 + q_);
    }
  }
#pragma unroll
  for (int tt = 0; tt < TC; ++tt) {
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float s2 = __shfl_xor(bs[tt], o, 64);
      const int i2 = __shfl_xor(bi[tt], o, 64);
      better(bs[tt], bi[tt], s2, i2);
    }
    if (grp == 0) { red_s[(wave * TC + tt) * 16 + row] = bs[tt]; red_i[(wave * TC + tt) * 16 + row] = bi[tt]; }
  }
  __syncthreads();
  if (tid < TC * 16) {
    const int tt = tid >> 4, r = tid & 15, m = m_base + 16 * (T0 + tt) + r;
    if (m < M) {
      float bs = -INFINITY;
      int bi = 0x7FFFFFFF;
#pragma unroll
      for (int w = 0; w < 4; ++w) better(bs, bi, red_s[(w * TC + tt) * 16 + r], red_i[(w * TC + tt) * 16 + r]);
      sa.best[(size_t)chunk * sa.ld + m] = bs;
      sa.idx[(size_t)chunk * sa.ld + m] = bi;
    }
  }
}

template <int NT, int MT>
__device__ __forceinline__ void sample_epilogue(const f32x4 (&acc)[NT][MT], int M, int m_base, int N, int n0,
    const SampleArgs& sa, uint16_t* __restrict__ xs) {
  // activation tiles per round: a divisor of MT
  constexpr int TC = MT % 4 == 0 ? 4 : (MT % 2 == 0 ? 2 : 1);
  const CtlParams* cp = sa.cp;
  const float temp = cp->temperature;
  uint32_t k0, k1;
  sampler_key(cp->seed, cp->step, k0, k1);
#define SARA_SR(r, U) \
  if constexpr (MT > (r) * TC) \
    sample_round<NT, MT, TC, (r) * TC, U>(acc, M, m_base, N, n0, sa, temp, k0, k1, xs, threadIdx.x >> 6, threadIdx.x, \
                                          blockIdx.x);
  if (temp == 1.0f) {
    SARA_SR(0, true) SARA_SR(1, true) SARA_SR(2, true) SARA_SR(3, true)
    SARA_SR(4, true) SARA_SR(5, true) SARA_SR(6, true) SARA_SR(7, true)
  } else {
    SARA_SR(0, false) SARA_SR(1, false) SARA_SR(2, false) SARA_SR(3, false)
    SARA_SR(4, false) SARA_SR(5, false) SARA_SR(6, false) SARA_SR(7, false)
  }
#undef SARA_SR
}

// One m-block of MT 16-row tiles.  Block = 4 waves; wave w owns weight rows
// [n0, n0 + 16*NT) and all 16*MT activation rows.  The k loop is a 4-slot
// software pipeline: stage s loads the X chunk (block-cooperative) and the
// wave's W chunk for k chunk s into register slot s % 4, three stages ahead
// of its use; at its turn the X chunk goes to one of two LDS buffers and the
// MFMAs read X from LDS and W from registers.  The loop has no peeled
// prologue (its first trip only loads), so the wait counts the compiler
// derives at the loop header are exact and three stages stay in flight.
//
// EPI = 0: fp32 partial sums to out[split][m][n].
// EPI = 1: SwiGLU epilogue (one split only): the weight rows are interleaved
//          per 16-row tile as gate (even tiles) and up (odd tiles) of the same
//          16 features; out receives bf16 silu(g) * u as [m][N/2].
// XT: X (and the SwiGLU output) is fragment-major (tiled_index), as the
// prefill writes it, else row-major.  A decode batch stays row-major: with few
// live rows a fragment-major row is spread over 16 times as many cache lines
// (gate|up 13.0 -> 13.5 us, LM head 95 -> 104 us at 32 rows).
// EPI = 2: Gumbel-max sampling epilogue of the LM head (one split only), see
//          sample_epilogue; out is unused.
// EPI = 3: fp32 logits of the LM head to sa.logits[slot][N] (one split only), for
//          the nucleus sampler; out is unused.
template <int NT, int MT, int KC, int EPI, bool XT>
__device__ __forceinline__ void gemm_mblock(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
    void* __restrict__ out, int M, int m_base, int N, int K, int kps, int64_t split_stride,
    uint16_t* __restrict__ xs, const SampleArgs& sa) {
  constexpr int MR = 16 * MT;
  constexpr int PITCH = KC + 8;                 // halves: rows shift by 4 banks, conflict-free b128 reads
  constexpr int C8 = KC / 8;                    // uint4 per X row per chunk
  constexpr int XU = (MR * C8 + 255) / 256;     // uint4 per thread per X chunk
  constexpr int CPK = KC / 32;                  // 16x16x32 MFMA k steps per chunk
  constexpr int BUF = MR * PITCH;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;
  const int n0 = (blockIdx.x * 4 + wave) * 16 * NT;
  const int k_begin = blockIdx.y * kps;
  const int k_end = min(K, k_begin + kps);
  const int nchunks = (k_end - k_begin) / KC;
  // W is in the wtiled_index layout: chunk = one 64-wide k block, whose
  // N / 16 tiles are 1024 elements apart.
  // Element offsets are 32-bit: N * K < 2^31 for every supported shape.
  static_assert(KC == 64, "a chunk is one k block of the weight layout");
  const int wchunk = (N / 16) * 1024;
  int woff[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    woff[nt] = (k_begin / 64) * wchunk + min(n0 / 16 + nt, N / 16 - 1) * 1024 + lane * 8;
  int xoff[XU], xdst[XU];
#pragma unroll
  for (int q = 0; q < XU; ++q) {
    // threads past the tile repeat its last element (same value, same place)
    int u = min((int)threadIdx.x + 256 * q, MR * C8 - 1);
    int rr = u / C8, c8 = u % C8;
    // 8 consecutive k of a row are one 16-byte run in either layout
    const int m = min(m_base + rr, M - 1);
    xoff[q] = XT ? (int)tiled_index(m, k_begin + 8 * c8, K) : m * K + 8 * c8 + k_begin;
    xdst[q] = rr * PITCH + 8 * c8;
  }
  // the four pipeline slots are distinct variables (not an indexed array),
  // so that they live in registers
  struct Stage { u32x4 x[XU]; u32x4 w[NT][CPK]; };
  Stage s0, s1, s2, s3;
  f32x4 acc[NT][MT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[nt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int last = max(nchunks - 1, 0);
  // loads are unconditional (clamped into [0, last]); surplus loads are unused
  auto load = [&](Stage& st, int chunk) {
    const int ch = max(min(chunk, last), 0);
#pragma unroll
    for (int q = 0; q < XU; ++q) st.x[q] = *(const u32x4*)(X + xoff[q] + ch * (XT ? 1024 : KC));
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int cc = 0; cc < CPK; ++cc) st.w[nt][cc] = *(const u32x4*)(W + woff[nt] + ch * wchunk + 512 * cc);
  };
  auto consume = [&](Stage& st, int buf, int ch) {
    // buffer `buf` was last read two chunks ago, before the previous barrier
#pragma unroll
    for (int q = 0; q < XU; ++q) *(u32x4*)&xs[buf * BUF + xdst[q]] = st.x[q];
    __syncthreads();
    if (ch < nchunks) {
      // rows past M read a clamped (valid) X row; their results are never stored
#pragma unroll
      for (int t = 0; t < MT; ++t) {
#pragma unroll
        for (int cc = 0; cc < CPK; ++cc) {
          u32x4 xv = *(const u32x4*)&xs[buf * BUF + (16 * t + row) * PITCH + 8 * grp + 32 * cc];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[nt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, st.w[nt][cc]), __builtin_bit_cast(bf16x8, xv), acc[nt][t], 0, 0, 0);
        }
      }
    }
  };
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): nothing of an earlier m-block is still pending
  int base0 = -4;
  asm volatile("" : "+s"(base0));       // opaque start: the first (load-only) trip stays in the loop
  for (int base = base0; base < nchunks; base += 4) {
    load(s3, base + 3);
    if (base >= 0) consume(s0, 0, base);
    load(s0, base + 4);
    if (base >= 0) consume(s1, 1, base + 1);
    load(s1, base + 5);
    if (base >= 0) consume(s2, 0, base + 2);
    load(s2, base + 6);
    if (base >= 0) consume(s3, 1, base + 3);
  }
  if constexpr (EPI == 2) {
    sample_epilogue<NT, MT>(acc, M, m_base, N, n0, sa, xs);
  } else if constexpr (EPI == 3) {
    // a caller's buffer may be 4-byte aligned only
    const bool wide = (reinterpret_cast<uintptr_t>(sa.logits) & 15) == 0;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int m = m_base + 16 * t + row;
      if (m >= M) continue;
      float* o = sa.logits + (size_t)sa.rows[m].slot * N + n0 + 4 * grp;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        if (n0 + 16 * nt >= N) continue;
        if (wide) {
          *(f32x4*)(o + 16 * nt) = acc[nt][t];
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) o[16 * nt + q] = acc[nt][t][q];
        }
      }
    }
  } else if (EPI == 0) {
    float* o = (float*)out + (size_t)blockIdx.y * split_stride;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if (n0 + 16 * nt >= N) continue;
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        int m = m_base + 16 * t + row;
        if (m < M) *(f32x4*)(o + (size_t)m * N + n0 + 16 * nt + 4 * grp) = acc[nt][t];
      }
    }
  } else {
    // tile pair (gate, up) = (nt 0, nt 1) of this wave: features (n0/32)*16 + 4*grp + q
    uint16_t* o = (uint16_t*)out;
    const int F = N / 2;
    const int f0 = (n0 / 32) * 16 + 4 * grp;
    if (n0 < N) {
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        int m = m_base + 16 * t + row;
        if (m < M) {
          const f32x4 r = silu_mul(acc[0][t], acc[NT - 1][t]);
          *(uint2*)(o + (XT ? (size_t)tiled_index(m, f0, F) : (size_t)m * F + f0)) =
              make_uint2(pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3]));
        }
      }
    }
  }
}

// bf16 MFMA GEMM over tiled weights.  The live row count M is read on the
// device; each m-block of up to 16*MTMAX rows runs the instance with just
// enough 16-row tiles (ceil(rows / 16)), so small batches spend no MFMA,
// LDS or X traffic on empty tiles.  Launches have one z block per m-block of
// the row capacity; z blocks past the live rows exit after reading M.
// PF: 0 decode, 1 prefill (fragment-major X), 2 as 0 for the decode
// attention-output projection (a label in profiles, so that every decode
// weight matrix has a class).
template <int NT, int MTMAX, int KC, int EPI, int PF>
__global__ __launch_bounds__(256, 2) void k_gemm_bf16_lds(const uint16_t* __restrict__ X,
    const uint16_t* __restrict__ W, void* __restrict__ out, const int32_t* __restrict__ M_ptr,
    int N, int K, int kps, int64_t split_stride, SampleArgs sa) {
  __shared__ __attribute__((aligned(16))) uint16_t xs[2 * 16 * MTMAX * (KC + 8)];
  const int M = *M_ptr;
  for (int m_base = blockIdx.z * 16 * MTMAX; m_base < M; m_base += gridDim.z * 16 * MTMAX) {
    const int mt = min(MTMAX, (M - m_base + 15) >> 4);
#define SARA_MB(c) \
    if constexpr (MTMAX >= c) { \
      if (mt == c) gemm_mblock<NT, c, KC, EPI, PF == 1>(X, W, out, M, m_base, N, K, kps, split_stride, xs, sa); \
    }
    SARA_MB(1) SARA_MB(2) SARA_MB(3) SARA_MB(4) SARA_MB(5) SARA_MB(6) SARA_MB(7) SARA_MB(8)
#undef SARA_MB
    __syncthreads();   // the LDS tiles are reused by the next m-block
  }
}

// Row-major [n_tiles*16][K] bf16 -> the GEMM weight layout (wtiled_index)
// of a dst_tiles-tile matrix; source tile j lands in destination tile
// j * tile_mul + tile_add, which builds the gate/up-interleaved matrix in place.
__global__ void k_tile_weights(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, int n_tiles,
                               int K, int tile_mul, int tile_add, int dst_tiles) {
  const int64_t per_tile = (int64_t)16 * K;
  const int64_t total = per_tile * n_tiles;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int64_t r = e / K, k = e - r * K;
    const int64_t j = r >> 4;
    const int64_t drow = (j * tile_mul + tile_add) * 16 + (r & 15);
    dst[wtiled_index(drow, k, dst_tiles)] = src[e];
  }
}

// Rotation-pair order of the bf16 q|k|v weight rows: within each head, the
// 16-row tile j holds natural dims 8j..8j+7 (tile rows 0-7) and
// HD/2 + 8j..HD/2 + 8j + 7 (tile rows 8-15), so both members of every
// rotate-half pair (d, d + HD/2) land in one tile and in MFMA output lanes
// l and l ^ 32.  Returns the stored row (output column) of dim d of head h.
__host__ __device__ __forceinline__ int qkv_pair_col(int h, int d, int HD) {
  const int half = HD / 2;
  const int e = d < half ? d : d - half;
  return h * HD + 16 * (e >> 3) + (e & 7) + (d < half ? 0 : 8);
}

// Row-major [n_rows][K] bf16 rows of heads head_off, head_off + 1, .. (HD
// rows each, natural dim order) -> the GEMM weight layout of a
// dst_tiles-tile matrix, rows in rotation-pair order.
__global__ void k_tile_weights_pairs(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, int n_rows,
                                     int K, int head_off, int HD, int dst_tiles) {
  const int64_t total = (int64_t)n_rows * K;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int64_t r = e / K, k = e - r * K;
    const int drow = qkv_pair_col(head_off + (int)(r / HD), (int)(r % HD), HD);
    dst[wtiled_index(drow, k, dst_tiles)] = src[e];
  }
}

// fp32 GEMM on v_mfma_f32_16x16x4_f32 (fp32 products and sums) for the fp32
// models: out[m][n] = sum_k X[m][k] W[n][k], K a multiple of 64, N of 16.
// Block = 16 MT rows x 2 weight tiles of 16 rows; its 4 waves take a quarter of
// K each, every lane loading 4 consecutive k of a row at a time (the k order
// inside the MFMA is the same for X and W, so it is moot), D steps of 16 k in
// flight, and meet in LDS in wave order.  Small batches are latency bound: the
// loads wait for nothing (not even the live row count), K is not split over
// blocks, and the epilogues replace passes of their own:
// EPI 0: out[m][n], tiles 2b and 2b + 1.
// EPI 1: SwiGLU; tile b of the gate rows and of the up rows (N = 2 ffn), out[m][ffn].
// EPI 2: q|k|v; tiles b and b + half / 16 of a head: rotate-half RoPE of q and k,
//        q to qbuf, k and v to the row's KV page.
// 32 rows of 256 -> 2048: 5 us, where 16 x 16 tiles on the vector unit with a
// barrier every 32 k took 10.
struct F32Epi {
  const RowDesc* rows;
  const float2* rope;
  float *qbuf, *kc, *vc;
  int hq, hkv, hd, layer;
  int64_t n_blocks;
};
template <int MT, int EPI>
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ X, const float* __restrict__ W,
    float* __restrict__ out, const int32_t* __restrict__ M_ptr, int M_cap, int N, int K, F32Epi ep) {
  constexpr int D = 4;                                  // steps of 16 k in flight
  __shared__ f32x4 red[4][2][MT][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;
  const int m0 = blockIdx.y * 16 * MT, ntl = N >> 4;
  int t0, t1;                                           // the block's two weight tiles
  if (EPI == 0) {
    t0 = 2 * blockIdx.x;
    t1 = min(t0 + 1, ntl - 1);
  } else if (EPI == 1) {
    t0 = blockIdx.x;
    t1 = t0 + (ntl >> 1);
  } else {
    const int ht = ep.hd >> 5;                          // tiles in half a head
    t0 = (blockIdx.x / ht) * 2 * ht + blockIdx.x % ht;
    t1 = t0 + ht;
  }
  const int kq = K >> 2, steps = kq >> 4;
  const float* w0 = W + (size_t)(16 * t0 + row) * K + wave * kq + 4 * grp;
  const float* w1 = W + (size_t)(16 * t1 + row) * K + wave * kq + 4 * grp;
  const float* xp[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t)   // rows past the live ones are computed and dropped
    xp[t] = X + (size_t)min(m0 + 16 * t + row, M_cap - 1) * K + wave * kq + 4 * grp;
  struct Stage { f32x4 a, b, x[MT]; };
  Stage st[D];
  auto load = [&](Stage& s, int j) {
    const int o = 16 * min(j, steps - 1);
    s.a = *(const f32x4*)(w0 + o);
    s.b = *(const f32x4*)(w1 + o);
#pragma unroll
    for (int t = 0; t < MT; ++t) s.x[t] = *(const f32x4*)(xp[t] + o);
  };
#pragma unroll
  for (int j = 0; j < D; ++j) load(st[j], j);
  const int M = *M_ptr;
  if (m0 >= M) return;
  f32x4 acc[2][MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[0][t] = acc[1][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int base = 0; base < steps; base += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      if (base + j < steps) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            acc[0][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(st[j].a[q], st[j].x[t][q], acc[0][t], 0, 0, 0);
            acc[1][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(st[j].b[q], st[j].x[t][q], acc[1][t], 0, 0, 0);
          }
      }
      if (base + D < steps) load(st[j], base + D + j);
    }
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    red[wave][0][t][lane] = acc[0][t];
    red[wave][1][t][lane] = acc[1][t];
  }
  __syncthreads();
  // wave w finishes (weight tile, row tile) pairs: lane (row, grp) holds row m, columns 4 grp ..+3
  if (EPI == 0) {
    for (int e = wave; e < 2 * MT; e += 4) {
      const int i = e & 1, t = e >> 1, m = m0 + 16 * t + row;
      const f32x4 v = ((red[0][i][t][lane] + red[1][i][t][lane]) + red[2][i][t][lane]) + red[3][i][t][lane];
      if (m < M) *(f32x4*)(out + (size_t)m * N + 16 * (i ? t1 : t0) + 4 * grp) = v;
    }
    return;
  }
  for (int t = wave; t < MT; t += 4) {
    const int m = m0 + 16 * t + row;
    const f32x4 a = ((red[0][0][t][lane] + red[1][0][t][lane]) + red[2][0][t][lane]) + red[3][0][t][lane];
    const f32x4 b = ((red[0][1][t][lane] + red[1][1][t][lane]) + red[2][1][t][lane]) + red[3][1][t][lane];
    if (m >= M) continue;
    if (EPI == 1) {
      f32x4 r;
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] = a[q] / (1.0f + expf(-a[q])) * b[q];
      *(f32x4*)(out + (size_t)m * (N >> 1) + 16 * t0 + 4 * grp) = r;
    } else {
      const int hd = ep.hd, half = hd >> 1, h = 16 * t0 / hd, c = 16 * t0 % hd + 4 * grp;
      const RowDesc r = ep.rows[m];
      // page of the row's own position
      const int rel = r.pos - r.plen;
      const size_t pg = (size_t)ep.layer * ep.n_blocks + (rel < 0 ? r.kv0 + (r.pos >> 4) : r.kv1 + (rel >> 4));
      const int tok = (rel < 0 ? r.pos : rel) & 15;
      if (h < ep.hq + ep.hkv) {
        f32x4 ra, rb;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float2 cs = ep.rope[(size_t)r.pos * half + c + q];
          ra[q] = a[q] * cs.x - b[q] * cs.y;
          rb[q] = b[q] * cs.x + a[q] * cs.y;
        }
        float* dst = h < ep.hq ? ep.qbuf + ((size_t)m * ep.hq + h) * hd
                               : ep.kc + ((pg * ep.hkv + (h - ep.hq)) * kBlockTok + tok) * hd;
        *(f32x4*)(dst + c) = ra;
        *(f32x4*)(dst + c + half) = rb;
      } else {
        float* vp = ep.vc + (pg * ep.hkv + (h - ep.hq - ep.hkv)) * (size_t)hd * kBlockTok + tok;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          vp[(size_t)(c + q) * kBlockTok] = a[q];
          vp[(size_t)(c + half + q) * kBlockTok] = b[q];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// epilogues
// ---------------------------------------------------------------------------
// Sum of the split-K partials of one element in a fixed order (four running
// sums over splits s = 0,4,8.. / 1,5,.. / 2,6,.. / 3,7,.. combined as
// (a0 + a1) + (a2 + a3)): deterministic, with the loads issued together.
__device__ __forceinline__ float split_sum(const float* ws, int splits, int64_t stride, size_t idx) {
  float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
  int s = 0;
  for (; s + 4 <= splits; s += 4) {
    a0 += ws[(size_t)s * stride + idx];
    a1 += ws[(size_t)(s + 1) * stride + idx];
    a2 += ws[(size_t)(s + 2) * stride + idx];
    a3 += ws[(size_t)(s + 3) * stride + idx];
  }
  if (s < splits) a0 += ws[(size_t)s * stride + idx];
  if (s + 1 < splits) a1 += ws[(size_t)(s + 1) * stride + idx];
  if (s + 2 < splits) a2 += ws[(size_t)(s + 2) * stride + idx];
  return (a0 + a1) + (a2 + a3);
}

// Loads that only some threads or iterations need are written as
// unconditional loads from a clamped, always valid address whose value is
// then multiplied by a 0/1 mask (finite data, so x * 0 = 0 exactly).  A load
// under a condition, or one whose value is only used under a condition,
// becomes a branch that waits for the load before going on, which would
// serialise the memory round trips.
__device__ __forceinline__ float mask01(bool keep) { return keep ? 1.0f : 0.0f; }

// Split-K sum of the fused q|k|v output of a short prefill chunk (columns in
// rotation-pair order, see qkv_pair_col), rotate-half RoPE on q and k, q -> bf16
// buffer, k and v -> the row's prompt page.  V pages are stored transposed,
// [hd][16 tokens] per (page, KV head), so that the PV product reads
// consecutive tokens of one dimension per lane.
__global__ __launch_bounds__(256) void k_qkv_epilogue(const int32_t* __restrict__ M_ptr,
    const RowDesc* __restrict__ rows, const float* __restrict__ ws, int splits, int64_t stride,
    const float2* __restrict__ rope, int hq, int hkv, int hd, int layer, int64_t n_blocks,
    uint16_t* __restrict__ qbuf, uint16_t* __restrict__ kc, uint16_t* __restrict__ vc) {
  const int half = hd >> 1, nh = hq + 2 * hkv, N = nh * hd;
  const int M = *M_ptr;
  for (int item = blockIdx.x; item < M * nh; item += gridDim.x) {
    const int i = item / nh, h = item - i * nh, c = threadIdx.x;
    const RowDesc r = rows[i];
    float a = split_sum(ws, splits, stride, (size_t)i * N + qkv_pair_col(h, c, hd));
    float b = split_sum(ws, splits, stride, (size_t)i * N + qkv_pair_col(h, c + half, hd));
    const size_t pg = (size_t)layer * n_blocks + r.kv0 + (r.pos >> 4);
    const int tok = r.pos & 15;
    if (h < hq + hkv) {
      float2 cs = rope[(size_t)r.pos * half + c];
      uint16_t* dst = h < hq ? qbuf + ((size_t)i * hq + h) * hd : kc + ((pg * hkv + (h - hq)) * kBlockTok + tok) * hd;
      dst[c] = f32_to_bf16(a * cs.x - b * cs.y);
      dst[c + half] = f32_to_bf16(b * cs.x + a * cs.y);
    } else {
      uint16_t* vp = vc + (pg * hkv + (h - hq - hkv)) * (size_t)hd * kBlockTok + tok;
      vp[(size_t)c * kBlockTok] = f32_to_bf16(a);
      vp[(size_t)(c + half) * kBlockTok] = f32_to_bf16(b);
    }
  }
}

// h += split-K sum; x = RMSNorm(h) * w  (stored in the model dtype).
// One 1024-thread block per row.
template <typename T>
__global__ __launch_bounds__(1024) void k_residual_norm(const int32_t* __restrict__ M_ptr,
    const float* __restrict__ ws, int splits, int64_t stride, int d, float* __restrict__ h,
    const float* __restrict__ w, float eps, T* __restrict__ x) {
  __shared__ float red[16];
  const int M = *M_ptr;
  for (int i = blockIdx.x; i < M; i += gridDim.x) {
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += 1024) {
    size_t idx = (size_t)i * d + c;
    float v = h[idx] + split_sum(ws, splits, stride, idx);
    h[idx] = v;
    ss += v * v;
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int q = 0; q < 16; q += 4) tot += (red[q] + red[q + 1]) + (red[q + 2] + red[q + 3]);
  float inv = 1.0f / sqrtf(tot / (float)d + eps);
  for (int c = threadIdx.x; c < d; c += 1024) {
    size_t idx = (size_t)i * d + c;
    st_f32(x, x_index<T>(i, c, d), h[idx] * inv * w[c]);
  }
  __syncthreads();   // red[] is reused by the next row
  }
}

// Same operation for rows of d <= 256 * VPT features and at most
// kMaxSplitsDec splits: one 256-thread block per row, every thread owns VPT
// features (c = threadIdx.x + 256 v) and keeps them in registers; the split
// partials are summed in the order of split_sum with every load in flight at
// once.
template <typename T, int VPT>
__global__ __launch_bounds__(256) void k_residual_norm_v(const int32_t* __restrict__ M_ptr,
    const float* __restrict__ ws, int splits, int64_t stride, int d, float* __restrict__ h,
    const float* __restrict__ w, float eps, T* __restrict__ x) {
  __shared__ float red[4];
  const int M = *M_ptr;
  for (int i = blockIdx.x; i < M; i += gridDim.x) {
    const size_t rb = (size_t)i * d;
    float a0[VPT], a1[VPT], a2[VPT], a3[VPT], hv[VPT];
    // unconditional loads from clamped indices, masked (see mask01)
    float wv[VPT];
#pragma unroll
    for (int v = 0; v < VPT; ++v) {
      const int c = min((int)threadIdx.x + 256 * v, d - 1);
      a0[v] = a1[v] = a2[v] = a3[v] = 0.f;
      hv[v] = h[rb + c] * mask01((int)threadIdx.x + 256 * v < d);
      wv[v] = w[c];
    }
    float pv[kMaxSplitsDec][VPT];
#pragma unroll
    for (int s = 0; s < kMaxSplitsDec; ++s)
#pragma unroll
      for (int v = 0; v < VPT; ++v) {
        const int c = min((int)threadIdx.x + 256 * v, d - 1);
        pv[s][v] = ws[(size_t)min(s, splits - 1) * stride + rb + c] *
                   mask01(s < splits && (int)threadIdx.x + 256 * v < d);
      }
#pragma unroll
    for (int s = 0; s < kMaxSplitsDec; s += 4)
#pragma unroll
      for (int v = 0; v < VPT; ++v) {
        a0[v] += pv[s][v];
        a1[v] += pv[s + 1][v];
        a2[v] += pv[s + 2][v];
        a3[v] += pv[s + 3][v];
      }
    float ss = 0.f;
#pragma unroll
    for (int v = 0; v < VPT; ++v) {
      const int c = threadIdx.x + 256 * v;
      const float val = hv[v] + ((a0[v] + a1[v]) + (a2[v] + a3[v]));
      hv[v] = val;
      if (c < d) {
        h[rb + c] = val;
        ss += val * val;
      }
    }
    const float tot = block_sum256(ss, red);
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int v = 0; v < VPT; ++v) {
      const int c = threadIdx.x + 256 * v;
      if (c < d) st_f32(x, x_index<T>(i, c, d), hv[v] * inv * wv[v]);
    }
    __syncthreads();   // red[] is reused by the next row
  }
}

// bf16 decode variant of the residual norm: one row per block, one float4
// of the row per thread (blockDim = d/4 rounded up to whole waves).  The
// residual, the norm weight and the row's split-K partials of that float4
// (only the splits the GEMM wrote) are loaded at once, summed in split order
// into four interleaved accumulators, and the row's sum of squares is
// reduced over the block's waves in wave order; x receives four bf16 per
// thread in one 8-byte store (row-major, or fragment-major for the q|k|v
// kernel, where four consecutive k of a row are contiguous).
__global__ __launch_bounds__(1024) void k_residual_norm_f4(const int32_t* __restrict__ M_ptr,
    const float* __restrict__ ws, int splits, int64_t stride, int d, float* __restrict__ h,
    const float* __restrict__ w, float eps, uint16_t* __restrict__ x, int x_tiled) {
  __shared__ float red[16];
  const int M = *M_ptr;
  const int nq = d >> 2, q = threadIdx.x, lane = q & 63, wave = q >> 6;
  const int nw = (blockDim.x + 63) >> 6;
  const bool on = q < nq;
  const int qc = on ? q : nq - 1;
  for (int i = blockIdx.x; i < M; i += gridDim.x) {
    const size_t rb = (size_t)i * d;
    const float4 hv = ((const float4*)(h + rb))[qc];
    const float4 wv = ((const float4*)w)[qc];
    float4 p[kMaxSplitsDec];
#pragma unroll
    for (int sp = 0; sp < kMaxSplitsDec; ++sp)
      p[sp] = (sp < splits) ? ((const float4*)(ws + (size_t)sp * stride + rb))[qc] : make_float4(0.f, 0.f, 0.f, 0.f);
    float4 a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int sp = 0; sp < kMaxSplitsDec; ++sp) {
      a[sp & 3].x += p[sp].x; a[sp & 3].y += p[sp].y; a[sp & 3].z += p[sp].z; a[sp & 3].w += p[sp].w;
    }
    float4 v;
    v.x = hv.x + ((a[0].x + a[1].x) + (a[2].x + a[3].x));
    v.y = hv.y + ((a[0].y + a[1].y) + (a[2].y + a[3].y));
    v.z = hv.z + ((a[0].z + a[1].z) + (a[2].z + a[3].z));
    v.w = hv.w + ((a[0].w + a[1].w) + (a[2].w + a[3].w));
    float ss = 0.f;
    if (on) {
      ((float4*)(h + rb))[q] = v;
      ss = (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
    }
    ss = wave_sum(ss);
    if (lane == 0) red[wave] = ss;
    __syncthreads();
    float tot = 0.f;
    for (int k = 0; k < nw; ++k) tot += red[k];
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
    if (on) {
      const uint32_t lo = (uint32_t)f32_to_bf16(v.x * inv * wv.x) | ((uint32_t)f32_to_bf16(v.y * inv * wv.y) << 16);
      const uint32_t hi = (uint32_t)f32_to_bf16(v.z * inv * wv.z) | ((uint32_t)f32_to_bf16(v.w * inv * wv.w) << 16);
      const size_t o = x_tiled ? (size_t)tiled_index(i, 4 * q, d) : rb + 4 * q;
      *(uint2*)(x + o) = make_uint2(lo, hi);
    }
    __syncthreads();   // red[] is reused by the next row
  }
}

// ---------------------------------------------------------------------------
// paged GQA attention
// ---------------------------------------------------------------------------
// fp32 models.  Block (row i, KV head g, context split c) attends the G query
// heads of KV head g over positions [c*SPLIT, min(ctx, (c+1)*SPLIT)) of the row's
// sequence with an online softmax, tiles of 64 tokens staged in LDS.  A context
// of at most one split (n_splits == 1) writes its output; otherwise the
// unnormalised output, running max and sum go to a partial buffer that the
// combine kernel merges across splits.  Positions below plen live in the
// prompt's shared pages (kv0 + e), later ones in the row's private pages (kv1 +
// e).
template <int HD>
__global__ __launch_bounds__(256) void k_attention(const int32_t* __restrict__ M_ptr,
    const RowDesc* __restrict__ rows, const float* __restrict__ qbuf, const float* __restrict__ kc,
    const float* __restrict__ vc, int layer, int64_t n_blocks, int hq, int hkv, int n_splits, float scale,
    float* __restrict__ part, float* __restrict__ out) {
  __shared__ float q_s[kMaxGroup][HD];
  __shared__ float k_s[kAttnTile][HD + 1];
  __shared__ float v_s[HD][kAttnTile + 1];
  __shared__ float p_s[kMaxGroup][kAttnTile];
  __shared__ float m_s[kMaxGroup], l_s[kMaxGroup], al_s[kMaxGroup];
  const int i = blockIdx.x, g = blockIdx.y, c = blockIdx.z;
  if (i >= *M_ptr) return;
  const RowDesc r = rows[i];
  const int ctx = r.pos + 1;
  const int t0 = c * kAttnSplit;
  if (t0 >= ctx) return;
  const int t1 = min(ctx, t0 + kAttnSplit);
  const int G = hq / hkv;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  constexpr int DPT = HD / 64;  // dims per thread in the PV product
  // (page, offset) of position pos as the offset of its 16-token page slice plus the token
  auto page_of = [&](int pos, int& tok) {
    const int rel = pos - r.plen;
    tok = (rel < 0 ? pos : rel) & 15;
    const size_t b = (size_t)layer * n_blocks + (rel < 0 ? r.kv0 + (pos >> 4) : r.kv1 + (rel >> 4));
    return (b * hkv + g) * (size_t)(kBlockTok * HD);
  };
  for (int e = tid; e < G * HD; e += 256) {
    int gh = e / HD, dd = e - gh * HD;
    q_s[gh][dd] = qbuf[((size_t)i * hq + g * G + gh) * HD + dd];
  }
  if (tid < kMaxGroup) { m_s[tid] = -INFINITY; l_s[tid] = 0.f; }
  float o[2][DPT];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < DPT; ++b) o[a][b] = 0.f;
  __syncthreads();
  for (int ts = t0; ts < t1; ts += kAttnTile) {
    const int n = min(kAttnTile, t1 - ts);
    {
      // K: thread (token tid / 4, a quarter of its dims); V: thread (token lane,
      // every fourth dim); tokens past the tile repeat its last
      constexpr int KQ = HD / 16, VQ = HD / 4;
      int tok;
      const float* kp = kc + page_of(min(ts + (tid >> 2), t1 - 1), tok) + (tid & 3) * (HD / 4);
      kp += tok * HD;
      f32x4 kv[KQ];
#pragma unroll
      for (int e = 0; e < KQ; ++e) kv[e] = *(const f32x4*)(kp + 4 * e);
      const size_t vpg = page_of(min(ts + lane, t1 - 1), tok);
      const float* vp = vc + vpg + tok;
      float vv[VQ];
#pragma unroll
      for (int e = 0; e < VQ; ++e) vv[e] = vp[(wave + 4 * e) * kBlockTok];
#pragma unroll
      for (int e = 0; e < KQ; ++e)
#pragma unroll
        for (int q = 0; q < 4; ++q) k_s[tid >> 2][(tid & 3) * (HD / 4) + 4 * e + q] = kv[e][q];
#pragma unroll
      for (int e = 0; e < VQ; ++e) v_s[wave + 4 * e][lane] = vv[e];
    }
    __syncthreads();
    // scores and online softmax update: thread (token lane), heads wave and wave + 4
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      int gh = wave + 4 * a;
      if (gh < G) {
        float sc = -INFINITY;
        if (lane < n) {
          float acc = 0.f;
#pragma unroll 8
          for (int dd = 0; dd < HD; ++dd) acc = fmaf(q_s[gh][dd], k_s[lane][dd], acc);
          sc = acc * scale;
        }
        float mt = wave_max(sc);
        float mo = m_s[gh];
        float mn = fmaxf(mo, mt);
        float pv = (lane < n) ? expf(sc - mn) : 0.f;
        float sum = wave_sum(pv);
        p_s[gh][lane] = pv;
        if (lane == 0) {
          float al = expf(mo - mn);
          al_s[gh] = al;
          l_s[gh] = l_s[gh] * al + sum;
          m_s[gh] = mn;
        }
      }
    }
    __syncthreads();
    // o = o * alpha + P V ; thread (dims lane, lane + 64, heads wave, wave + 4)
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      int gh = wave + 4 * a;
      if (gh < G) {
        float al = al_s[gh];
#pragma unroll
        for (int b = 0; b < DPT; ++b) o[a][b] *= al;
        for (int tk = 0; tk < n; ++tk) {
          float pv = p_s[gh][tk];
#pragma unroll
          for (int b = 0; b < DPT; ++b) o[a][b] = fmaf(pv, v_s[lane + 64 * b][tk], o[a][b]);
        }
      }
    }
    __syncthreads();
  }
  // partial layout: [row][g][split][gh][HD + 2]  (o..., m, l)
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    int gh = wave + 4 * a;
    if (gh < G) {
      if (n_splits == 1) {
        float* dst = out + ((size_t)i * hq + g * G + gh) * HD;
#pragma unroll
        for (int b = 0; b < DPT; ++b) dst[lane + 64 * b] = o[a][b] / l_s[gh];
        continue;
      }
      float* dst = part + ((((size_t)i * hkv + g) * n_splits + c) * kMaxGroup + gh) * (HD + 2);
#pragma unroll
      for (int b = 0; b < DPT; ++b) dst[lane + 64 * b] = o[a][b];
      if (lane == 0) { dst[HD] = m_s[gh]; dst[HD + 1] = l_s[gh]; }
    }
  }
}

// Fused q|k|v projection of the decode rows with the rotary / KV-append
// epilogue (bf16 weights in rotation-pair order, see qkv_pair_col).  Block = NT
// 16-row weight tiles; its 4 waves take a quarter of K each and stream
// their weight fragments and the activation fragments of up to 16*MT rows
// through a D-stage register pipeline (the waves share no k range, so the
// activations need no LDS staging).  The wave partial sums meet in LDS and
// are added in wave order (deterministic).  Wave t % 4 then finishes
// activation tile t: rotate-half RoPE on q and k heads (the two members of
// a rotation pair sit in lanes l and l ^ 32), q to qbuf as bf16, k and v to
// the row's newest KV page (the attention kernel reads them from there).
template <int HD, int MT, int D, int KS, int NT>
__device__ __forceinline__ void qkv_rope_mblock(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
    int M, int m_base, int K, f32x4 (*red)[8][64], const RowDesc* __restrict__ rows,
    const float2* __restrict__ row_rope, int hq, int hkv, int layer, int64_t n_blocks,
    uint16_t* __restrict__ qbuf, uint16_t* __restrict__ kc, uint16_t* __restrict__ vc) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;
  const int tile0 = blockIdx.x * NT;
  // KS = K / 128 32-wide k steps per wave; D divides KS, so the pipeline
  // issues D - 1 surplus (clamped, cache-hit) loads at most, none when D = KS
  static_assert(KS % D == 0, "pipeline depth must divide the k steps");
  const int ks0 = wave * KS;
  // W in the wtiled_index layout: k step j of this wave sits in k block
  // (ks0 + j) / 2 (KS is even, so ks0 starts a block)
  const int wblock = ((hq + 2 * hkv) * HD / 16) * 1024;
  const int woff = (ks0 / 2) * wblock + tile0 * 1024 + lane * 8;
  // activation fragments: X is fragment-major (tiled_index layout, as the
  // weights), so each fragment load of a wave is one contiguous 1 KiB read;
  // lanes of rows past M read rows of the last tile whose results are dropped
  int xoff[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) xoff[t] = ((m_base / 16 + t) * (K >> 5) + ks0) * 512 + lane * 8;
  // Epilogue inputs of the tiles this wave finishes (t = wave + 4 * tt),
  // loaded before the k loop so that their latency hides behind it:
  // the row's newest-token KV slot and the rotation angles of its position.
  constexpr int TT = (MT + 3) / 4;
  constexpr int half = HD / 2;
  const bool second = grp >= 2;
  // rotation index of the lane's first dim in weight tile tile0 + n
  const auto rot = [&](int n) { return 8 * (((tile0 + n) * 16 % HD) >> 4) + 4 * (grp & 1); };
  size_t pg_e[TT];
  int on_e[TT];
  float2 cs_e[TT][NT][4];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    const int m = min(m_base + 16 * (wave + 4 * tt) + row, M - 1);
    const RowDesc r = rows[m];
    const int rel = r.pos - r.plen;                 // private position of the newest token
    pg_e[tt] = (size_t)layer * n_blocks + r.kv1 + (rel >> 4);
    on_e[tt] = rel & 15;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int q = 0; q < 4; ++q) cs_e[tt][n][q] = row_rope[(size_t)m * half + rot(n) + q];
  }
  struct Stage { u32x4 w[NT]; u32x4 x[MT]; };
  Stage st[D];
  f32x4 acc[NT][MT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int last = KS - 1;
  auto load = [&](Stage& sg, int step) {
    const int kk = max(min(step, last), 0);
#pragma unroll
    for (int n = 0; n < NT; ++n)
      sg.w[n] = *(const u32x4*)(W + woff + n * 1024 + (kk >> 1) * wblock + (kk & 1) * 512);
#pragma unroll
    for (int t = 0; t < MT; ++t) sg.x[t] = *(const u32x4*)(X + xoff[t] + kk * 512);
  };
  auto consume = [&](Stage& sg, int step) {
    if (step < KS) {
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n)
          acc[n][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, sg.w[n]),
                                                              __builtin_bit_cast(bf16x8, sg.x[t]), acc[n][t], 0, 0, 0);
    }
  };
  if constexpr (D == KS) {
    // every k step in flight at once: exactly KS loads, then the MFMAs
#pragma unroll
    for (int j = 0; j < KS; ++j) load(st[j], j);
#pragma unroll
    for (int j = 0; j < KS; ++j) consume(st[j], j);
  } else {
    int base0 = -D;
    asm volatile("" : "+s"(base0));     // opaque start: the first (load-only) trip stays in the loop
    for (int base = base0; base < KS; base += D) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        load(st[(j + D - 1) % D], base + j + D - 1);
        if (base >= 0) consume(st[j], base + j);
      }
    }
  }
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int h = (tile0 + n) * 16 / HD;
    const int nd = (second ? half : 0) + rot(n);      // natural dim of the lane's first value
#pragma unroll
    for (int t = 0; t < MT; ++t) red[wave][t][lane] = acc[n][t];
    __syncthreads();
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int t = wave + 4 * tt;
      if (t >= MT) break;
      f32x4 v = red[0][t][lane];
      v += red[1][t][lane];
      v += red[2][t][lane];
      v += red[3][t][lane];
      f32x4 pv;
#pragma unroll
      for (int q = 0; q < 4; ++q) pv[q] = __shfl_xor(v[q], 32, 64);
      const int m = m_base + 16 * t + row;
      if (m >= M) continue;
      float o[4];
      if (h < hq + hkv) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float2 c = cs_e[tt][n][q];
          o[q] = second ? (v[q] * c.x + pv[q] * c.y) : (v[q] * c.x - pv[q] * c.y);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = v[q];
      }
      const uint32_t p01 = (uint32_t)f32_to_bf16(o[0]) | ((uint32_t)f32_to_bf16(o[1]) << 16);
      const uint32_t p23 = (uint32_t)f32_to_bf16(o[2]) | ((uint32_t)f32_to_bf16(o[3]) << 16);
      const size_t pg = pg_e[tt];
      const int on = on_e[tt];
      if (h < hq) {
        *(uint2*)(qbuf + ((size_t)m * hq + h) * HD + nd) = make_uint2(p01, p23);
      } else if (h < hq + hkv) {
        *(uint2*)(kc + ((pg * hkv + (h - hq)) * kBlockTok + on) * HD + nd) = make_uint2(p01, p23);
      } else {
        uint16_t* vp = vc + (pg * hkv + (h - hq - hkv)) * (size_t)HD * kBlockTok + on;
        vp[(size_t)(nd + 0) * kBlockTok] = (uint16_t)(p01 & 0xFFFF);
        vp[(size_t)(nd + 1) * kBlockTok] = (uint16_t)(p01 >> 16);
        vp[(size_t)(nd + 2) * kBlockTok] = (uint16_t)(p23 & 0xFFFF);
        vp[(size_t)(nd + 3) * kBlockTok] = (uint16_t)(p23 >> 16);
      }
    }
    __syncthreads();   // red is reused by the next weight tile or m-block
  }
}

// Live row count read on the device.  Grid: x = one block per NT weight tiles,
// z = one block per 128 rows of the capacity.  The live 16-row activation
// tiles are shared out in contiguous runs over the first min(gridDim.z,
// zspread) z blocks (at most 8 tiles per block), so that a small batch keeps
// several blocks per weight tile busy instead of one; zspread is chosen on
// the host so that the whole grid's working blocks stay resident at once.
// Every tile's arithmetic is the same whichever block computes it.
// NT: 2 in the many-row loop, where the activation tiles read from L2 once per
// weight tile are the bound (512 rows, d 2048, 2560 outputs: 27.5 us at one
// weight tile a block, 22.6 at two), else 1 (few rows: twice the blocks).
// KS = d_model / 128, one of 4, 8, 12, 16, 24, 32 (checked by sara_init).
template <int HD, int KS, int NT>
__global__ __launch_bounds__(256) void k_qkv_rope(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
    const int32_t* __restrict__ M_ptr, int K, const RowDesc* __restrict__ rows,
    const float2* __restrict__ row_rope, int hq, int hkv, int layer, int64_t n_blocks,
    uint16_t* __restrict__ qbuf, uint16_t* __restrict__ kc, uint16_t* __restrict__ vc, int zspread) {
  __shared__ f32x4 red[4][8][64];
  const int M = *M_ptr;
  const int ntl = (M + 15) >> 4;
  const int zs = max(1, min((int)gridDim.z, zspread));
  const int tpz = min(8, (ntl + zs - 1) / zs);      // tiles per z block
  for (int m_base = blockIdx.z * tpz * 16; m_base < M; m_base += gridDim.z * tpz * 16) {
    const int mt = min(tpz, (M - m_base + 15) >> 4);
    // depth for up to 32 rows: every k step in flight below 16 k steps, half
    // of them from 16 on (the 16-step instance then fits two blocks per CU);
    // a half and a quarter of that for more rows
#define SARA_QR(MT_, D_) \
    if (mt == MT_) qkv_rope_mblock<HD, MT_, D_, KS, NT>(X, W, M, m_base, K, red, rows, row_rope, hq, hkv, layer, \
                                                        n_blocks, qbuf, kc, vc);
    // (two weight tiles: 4 and 2 steps, their registers hold no more)
    constexpr int D1 = NT > 1 ? 4 : (KS < 16 ? KS : KS / 2), D3 = NT > 1 ? 4 : D1 / 2, D5 = NT > 1 ? 2 : D1 / 4;
    SARA_QR(1, D1) SARA_QR(2, D1) SARA_QR(3, D3) SARA_QR(4, D3)
    SARA_QR(5, D5) SARA_QR(6, D5) SARA_QR(7, D5) SARA_QR(8, D5)
#undef SARA_QR
  }
}

// Decode attention (bf16, MFMA) over the KV pages, q read from qbuf (the
// q|k|v kernel has already rotated q and appended this position's k and v).
// Work item = (entry e of the step's work list, KV head g): entry e names a
// row and one of its context splits of kDecPages pages; wave w owns pages
// w and w + 4 of the split, all K and V loads issued before any compute, so
// a split costs one HBM round trip.  The entry carries the row's two KV
// extents (kv0 + e: shared prompt pages, kv1 + e: private pages), so the
// page loads wait on that one load only, and a block's next entry is loaded
// while it computes; the grid is the number of blocks that are resident at
// once, so up to that many items all run in one round.  Per wave, its two
// pages (32 tokens) at once:
//   S^T = K q^T  (v_mfma_f32_16x16x32_bf16; G <= 8 query heads a row, 16
//                 columns; lane (token l%16, k-group l/16) of K meets column l%16
//                 of q over the same HD/4 dims, so the k order inside the MFMA is moot)
//   softmax per column in base 2 over the 4 lanes holding its 32 scores.  The
//                 maximum is kept as the base-2 value that was subtracted, so
//                 that merging waves and splits adds no rounding of its own: at
//                 scores near 100 weights scaled anew from the raw maxima were
//                 8e-7 off on average, these are 2e-8
//   O^T = V^T P^T (the score registers already have the B-operand layout, four
//                 tokens of each page a lane, and transposed V pages give the A
//                 operand; P enters as a bf16 hi + lo pair, so the product
//                 keeps fp32 accuracy without a bf16 rounding point)
// An entry of n > 1 rows (at most 16 / G) is a split of whole prompt pages that
// the rows share: G columns each; a column's arithmetic is the same wherever it
// stands.  The 4 waves' (max, sum, O) merge in LDS, four consecutive dims of a
// column a thread, its four weights computed once.  A row with a single split
// writes its normalised output to `out` ([row][hq][HD], bf16); other rows leave
// a partial per split for k_attn_combine.
// With many rows it is bound by the vector unit, with few by its load round
// trips.  512 rows of 16 heads at contexts near 660: 37 us, where masks, two
// softmax steps and natural exponentials per merged element took 59 (and 61
// with the prompts' rows sharing items); 32 rows at contexts near 3,800: 14.4
// against 21.9 us; 32 rows near 350: 6.3 against 6.8.
template <int HD>
__global__ __launch_bounds__(256, 2) void k_attn_dec(const AttnItem* __restrict__ items,
    const int32_t* __restrict__ n_items, const PromptPlace* __restrict__ places, int cap,
    const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc,
    int layer, int64_t n_blocks, int hq, int hkv, int n_splits, float scale,
    const uint16_t* __restrict__ qb, float* __restrict__ part, uint16_t* __restrict__ out) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  constexpr int DPL = HD / 4, NCC = HD / 32, NT = HD / 16, SPG = kDecPages;
  static_assert(kDecPpw == 2, "a wave takes two pages of a split");
  constexpr int PITCH = HD + 4;
  constexpr int TPC = HD / 4, CPP = 256 / TPC;              // merge: threads per column, columns per pass
  __shared__ float m_w[4][16], l_w[4][16];
  __shared__ __attribute__((aligned(16))) float o_w[4][16][PITCH];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;
  const int G = hq / hkv;
  const int cr = row / G, chd = row - cr * G;               // this column's row within the item, and head
  const float sl2 = scale * 1.4426950408889634f;
  // the list length and the first entry are loaded together (the entry index
  // stays below the list's capacity); every later entry an item ahead
  const int n = *n_items;
  int item = blockIdx.x;
  if (item >= cap * hkv) return;
  int4 e0 = *(const int4*)&items[item / hkv].i, e1 = *(const int4*)&items[item / hkv].pl;
  while (item < n * hkv) {
    const int next = item + gridDim.x, ni = min(next / hkv, cap - 1);
    const int4 f0 = *(const int4*)&items[ni].i, f1 = *(const int4*)&items[ni].pl;
    const int c = e0.y, g = item % hkv, nr = e1.z;
    // row r of the item (a single row's item names it directly)
    auto row_of = [&](int r) { return nr == 1 ? e0.x : (int)places[e0.x + r].row; };
    // q operand: independent of anything but the entry, loaded first
    const bool on = cr < nr;
    uint4 qv[NCC];
    {
      const uint4* qp = (const uint4*)(qb + ((size_t)row_of(on ? cr : 0) * hq + g * G + chd) * HD + DPL * grp);
#pragma unroll
      for (int cc = 0; cc < NCC; ++cc) qv[cc] = qp[cc];
    }
    const int kv0 = e0.z, kv1 = e0.w;
    const int pl = e1.x;                                   // prompt positions attended
    const int pc = (pl + 15) >> 4;                         // prompt pages
    const int vcnt = e1.y;                                 // private positions (>= 1)
    const int nch = pc + ((vcnt + 15) >> 4);
    const int ch0 = c * SPG;
    const int ch1 = min(nch, ch0 + SPG);
    struct Pg { u32x4 k[NCC]; u32x2 v[NT]; int n; };
    Pg pg[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int ch = ch0 + wave + 4 * p;
      const int cv = (ch < ch1) ? ch : ch0;                // pages past the split re-read its first
      int m;
      if (cv < pc) m = min(16, pl - 16 * cv);
      else m = min(16, vcnt - 16 * (cv - pc));
      pg[p].n = (ch < ch1) ? m : 0;
      const int blk = (cv < pc) ? kv0 + cv : kv1 + (cv - pc);
      const size_t pgi = ((size_t)layer * n_blocks + blk) * hkv + g;
      const u32x4* kp = (const u32x4*)(kc + (pgi * kBlockTok + row) * HD + DPL * grp);
#pragma unroll
      for (int cc = 0; cc < NCC; ++cc) pg[p].k[cc] = kp[cc];
      const uint16_t* vp = vc + pgi * (size_t)HD * kBlockTok + 4 * grp;
#pragma unroll
      for (int t = 0; t < NT; ++t) pg[p].v[t] = *(const u32x2*)(vp + (size_t)(16 * t + row) * kBlockTok);
    }
    if (!on) {
#pragma unroll
      for (int cc = 0; cc < NCC; ++cc) qv[cc] = make_uint4(0, 0, 0, 0);
    }
    float mx = -INFINITY, ls = 0.f;
    f32x4 o[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (pg[0].n > 0) {
      f32x4 sc[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        sc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cc = 0; cc < NCC; ++cc)
          sc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pg[p].k[cc]),
                                                          __builtin_bit_cast(bf16x8, qv[cc]), sc[p], 0, 0, 0);
      }
      // lane holds tokens 4*grp + q (q < 4) of both pages, column `row`; tokens
      // beyond a page's valid ones may hold stale bits: their scores count
      // nothing and their V is zeroed
      if (pg[0].n + pg[1].n < 32) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int left = pg[p].n - 4 * grp;               // valid tokens of this lane's four
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (q >= left) sc[p][q] = -INFINITY;
          const uint32_t v0 = (left > 0 ? 0xFFFFu : 0u) | (left > 1 ? 0xFFFF0000u : 0u);
          const uint32_t v1 = (left > 2 ? 0xFFFFu : 0u) | (left > 3 ? 0xFFFF0000u : 0u);
#pragma unroll
          for (int t = 0; t < NT; ++t) { pg[p].v[t].x &= v0; pg[p].v[t].y &= v1; }
        }
      }
#pragma unroll
      for (int p = 0; p < 2; ++p)
        mx = fmaxf(mx, fmaxf(fmaxf(sc[p][0], sc[p][1]), fmaxf(sc[p][2], sc[p][3])));
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      mx *= sl2;
      u32x4 ph, plo;
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[p][q], sl2, -mx));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[p][q + 1], sl2, -mx));
          ls += p0 + p1;
          const uint32_t hi = pack_bf16(p0, p1);
          ph[2 * p + (q >> 1)] = hi;
          plo[2 * p + (q >> 1)] = pack_bf16(p0 - __uint_as_float(hi << 16), p1 - __uint_as_float(hi & 0xFFFF0000u));
        }
      ls += __shfl_xor(ls, 16, 64);
      ls += __shfl_xor(ls, 32, 64);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const u32x4 vw = {pg[0].v[t].x, pg[0].v[t].y, pg[1].v[t].x, pg[1].v[t].y};
        const bf16x8 vf = __builtin_bit_cast(bf16x8, vw);
        o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, ph), o[t], 0, 0, 0);
        o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, plo), o[t], 0, 0, 0);
      }
    }
    // merge the 4 waves: lane (row, grp) holds dims 16 t + 4 grp ..+3 of column row
    const int cols = nr * G;
    if (grp == 0) { m_w[wave][row] = mx; l_w[wave][row] = ls; }
    if (row < cols) {
#pragma unroll
      for (int t = 0; t < NT; ++t) *(f32x4*)&o_w[wave][row][16 * t + 4 * grp] = o[t];
    }
    __syncthreads();
    const bool single = nch <= SPG;
    for (int col = (int)threadIdx.x / TPC; col < cols; col += CPP) {
      const int rr = col / G, head = col - rr * G, i = row_of(rr), d4 = 4 * ((int)threadIdx.x % TPC);
      const float m = fmaxf(fmaxf(m_w[0][col], m_w[1][col]), fmaxf(m_w[2][col], m_w[3][col]));
      f32x4 num = {0.f, 0.f, 0.f, 0.f};
      float den = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float wt = __builtin_amdgcn_exp2f(m_w[w][col] - m);   // 0 for a wave without pages
        num += wt * *(const f32x4*)&o_w[w][col][d4];
        den += wt * l_w[w][col];
      }
      if (single) {
        *(uint2*)(out + ((size_t)i * hq + g * G + head) * HD + d4) =
            make_uint2(pack_bf16(num[0] / den, num[1] / den), pack_bf16(num[2] / den, num[3] / den));
      } else {
        float* dst = part + ((((size_t)i * hkv + g) * n_splits + c) * kMaxGroup + head) * (HD + 2);
        *(float2*)(dst + d4) = make_float2(num[0], num[1]);
        *(float2*)(dst + d4 + 2) = make_float2(num[2], num[3]);
        if (d4 == 0) *(float2*)(dst + HD) = make_float2(m, den);
      }
    }
    __syncthreads();   // LDS is reused by the next item
    item = next;
    e0 = f0;
    e1 = f1;
  }
}

// merge the context splits of every (row, query head) into o (model dtype)
// skip_single: rows with one split were written by the attention kernel.
// One pass over the splits, eight at a time with all their loads in flight,
// rescaling the running (max, numerator, denominator) as it goes.  Maxima are
// natural in the fp32 attention's partials, base 2 in the bf16 one's.
template <typename T, int HD>
__global__ __launch_bounds__(HD) void k_attn_combine(const int32_t* __restrict__ M_ptr,
    const RowDesc* __restrict__ rows, const float* __restrict__ part, int hq, int hkv,
    int n_splits, int paged_splits, int skip_single, T* __restrict__ out) {
  // paged_splits: pages per context split of the paged (bf16) attention
  // kernels, 0 for the fp32 attention's token splits
  const auto weight = [](float x) { return sizeof(T) == 2 ? __builtin_amdgcn_exp2f(x) : expf(x); };
  const int M = *M_ptr;
  for (int item = blockIdx.x; item < M * hq; item += gridDim.x) {
    const int i = item / hq, h = item - i * hq;
    const int G = hq / hkv, g = h / G, gh = h - g * G;
    const RowDesc r = rows[i];
    const int ctx = r.pos + 1;
    int ns;
    if (paged_splits) {
      const int pl = min(ctx, r.plen);
      const int nch = ((pl + 15) >> 4) + ((ctx - pl + 15) >> 4);
      ns = (nch + paged_splits - 1) / paged_splits;
    } else {
      ns = (ctx + kAttnSplit - 1) / kAttnSplit;
    }
    if (skip_single && ns == 1) continue;
    const float* base = part + (((size_t)i * hkv + g) * n_splits * kMaxGroup + gh) * (HD + 2);
    const size_t sstride = (size_t)kMaxGroup * (HD + 2);
    float mx = -INFINITY, num = 0.f, den = 0.f;
    for (int c0 = 0; c0 < ns; c0 += 8) {
      float pm[8], pl_[8], po[8];
      float mk[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        // unconditional loads from a clamped split index (see mask01): the
        // surplus entries repeat split ns - 1 of this chunk, which leaves the
        // maximum unchanged, and their weight is masked to zero
        const float* p = base + (size_t)min(c0 + q, ns - 1) * sstride;
        pm[q] = p[HD];
        pl_[q] = p[HD + 1];
        po[q] = p[threadIdx.x];
        mk[q] = mask01(c0 + q < ns);
      }
      float m2 = mx;
#pragma unroll
      for (int q = 0; q < 8; ++q) m2 = fmaxf(m2, pm[q]);
      const float sc = (mx == -INFINITY) ? 0.f : weight(mx - m2);
      num *= sc;
      den *= sc;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float wgt = ((pm[q] == -INFINITY) ? 0.f : weight(pm[q] - m2)) * mk[q];
        num += wgt * po[q];
        den += wgt * pl_[q];
      }
      mx = m2;
    }
    st_f32(out, ((size_t)i * hq + h) * HD + threadIdx.x, num / den);
  }
}

// ---------------------------------------------------------------------------
// sampler: Gumbel-max over the vocabulary with Philox4x32-10 noise
// ---------------------------------------------------------------------------
// (score definition and helpers: see "Gumbel-max sampling helpers")

// top-p helpers: order-preserving key of z (larger z, larger key) and the
// integer weight of z under the row maximum (see the top-p sampler below)
__device__ __forceinline__ uint32_t zkey(float z) {
  uint32_t u = __float_as_uint(z);
  if ((u & 0x7FFFFFFFu) == 0u) u = 0u;   // -0 and +0 are one value
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ uint64_t nucleus_weight(float z, float zmax) {
  // 0 <= w <= 2^44 (NaN: 0), so w + 2^52 holds the whole number in its low bits
  const double w = fmax(floor(ldexp(exp((double)z - (double)zmax), 44)), 0.0);
  return (uint64_t)__double_as_longlong(w + 4503599627370496.0) & 0xFFFFFFFFFFFFFull;
}

// Gumbel-max over vocabulary chunk c of nch of row i: the chunk's exact best
// (score, id) to best / bidx [row][nch].  Each thread bounds the scores of Q
// quads of ids (the four words of one Philox call) at a time, by gumbel_upper,
// and keeps the bounds in registers; each wave then re-scores exactly the ids
// whose bound reaches the floor under its best fast score (the exact winner is
// always among them, as in the fused LM-head sampler), so Philox runs once per
// id, logarithms once per thread, and the waves meet only at the end.  Bound by
// Philox's integer multiplies: 64 rows x 151936 ids 22.6 us against 44.6 with two
// passes of Philox and noise over every id (128 rows 38.6 against 79).  thr:
// top-p only, ids whose key reaches the row's threshold.
template <int Q>
__global__ __launch_bounds__(256) void k_sample_partial(const int32_t* __restrict__ M_ptr, int M,
    const int32_t* __restrict__ rid_arr, const int32_t* __restrict__ pos_arr,
    const RowDesc* __restrict__ rows, const float* __restrict__ logits, int V, int by_slot,
    const uint32_t* __restrict__ thr, const CtlParams* __restrict__ cpd, uint64_t seed, int32_t step,
    float temp, int nch, float* __restrict__ best, int32_t* __restrict__ bidx) {
  __shared__ float sb[4];
  __shared__ int si[4];
  // persistent over (row, vocabulary chunk) items of the live rows
  if (M_ptr) M = *M_ptr;
  if (cpd) { seed = cpd->seed; step = cpd->step; temp = cpd->temperature; }
  uint32_t k0, k1;
  sampler_key(seed, step, k0, k1);
  const int nblk = (V + 3) >> 2, per = (nblk + nch - 1) / nch;
  for (int item = blockIdx.x; item < M * nch; item += gridDim.x) {
    const int i = item / nch, c = item - i * nch;
    const uint32_t rid = rows ? rows[i].rid : rid_arr[i];
    const uint32_t gen = rows ? rows[i].gen : pos_arr[i];
    const int b0 = min(nblk, c * per), b1 = min(nblk, b0 + per);
    const float* lg = logits + (size_t)(by_slot ? rows[i].slot : i) * V;
    const bool wide = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(lg) & 15) == 0;
    const uint32_t kth = thr ? thr[i] : 0u;
    float bs = -INFINITY;
    int bi = 0x7FFFFFFF;
    float smax = -INFINITY;                              // the wave's best fast score so far
    for (int base = b0; base < b1; base += 256 * Q) {
      f32x4 z[Q];
#pragma unroll
      for (int e = 0; e < Q; ++e) {
        const int b = base + 256 * e + (int)threadIdx.x;
        if (wide) {
          z[e] = ((const f32x4*)lg)[min(b, nblk - 1)];
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) z[e][q] = lg[min(4 * b + q, V - 1)];
        }
      }
      if (temp != 1.0f) {                                // one branch around all divisions
#pragma unroll
        for (int e = 0; e < Q; ++e)
#pragma unroll
          for (int q = 0; q < 4; ++q) z[e][q] = __fdiv_rn(z[e][q], temp);
      }
      f32x4 f[Q];                                        // score bounds, NaN for ids that take no part
      float lub = -INFINITY, lz = -INFINITY;             // the lane's best bound, its z
      uint32_t lw = 0u;                                  // and its noise word
#pragma unroll
      for (int e = 0; e < Q; ++e) {
        const int b = base + 256 * e + (int)threadIdx.x;
        bool in[4], any = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          in[q] = b < b1 && 4 * b + q < V && zkey(z[e][q]) >= kth;
          any |= in[q];
          f[e][q] = __builtin_nanf("");
        }
        if (!any) continue;
        const U32x4 w = philox4x32_10(rid, gen, (uint32_t)b, 0u, k0, k1);
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (in[q]) {
            f[e][q] = z[e][q] + gumbel_upper(ws[q]);
            if (f[e][q] > lub) { lub = f[e][q]; lz = z[e][q]; lw = ws[q]; }
          }
      }
      smax = fmaxf(smax, wave_max(__fadd_rn(lz, gumbel_fast(lw))));
      const float floor_ = gumbel_candidate_floor(smax);
#pragma unroll
      for (int e = 0; e < Q; ++e)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (f[e][q] >= floor_) {
            const int b = base + 256 * e + (int)threadIdx.x;
            better(bs, bi, exact_score(z[e][q], rid, gen, (uint32_t)b, q, k0, k1), 4 * b + q);
          }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float s2 = __shfl_xor(bs, o, 64);
      const int i2 = __shfl_xor(bi, o, 64);
      better(bs, bi, s2, i2);
    }
    if ((threadIdx.x & 63) == 0) { sb[threadIdx.x >> 6] = bs; si[threadIdx.x >> 6] = bi; }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
      for (int w = 1; w < 4; ++w) better(bs, bi, sb[w], si[w]);
      best[(size_t)i * nch + c] = bs;
      bidx[(size_t)i * nch + c] = bi;
    }
    __syncthreads();   // sb/si are reused by the next item
  }
}
// quads a thread takes at once, by the chunk's length: 1 or 2 cover the chunks of
// small vocabularies or few rows, else 5 (10 leave two waves a SIMD)
template <typename F>
static void with_sample_quads(int V, int nch, F launch) {
  const int per = ((V + 3) / 4 + nch - 1) / nch;
  if (per <= 256) launch(k_sample_partial<1>);
  else if (per <= 512) launch(k_sample_partial<2>);
  else launch(k_sample_partial<5>);
}

// ---------------------------------------------------------------------------
// top-p (nucleus) sampler, top_p < 1 (nucleus sampling, Holtzman et al.),
// over each row's fp32 logits.  Mass is counted in integer weights
// q_v = floor(exp(z_v - z_max) * 2^44), z_v = fp32(logit_v / T), so the cut
// is an exact integer decision whatever the order of the sums: the nucleus
// is {v : z_v >= z*}, with z* the largest z whose upper set holds weight
// >= t = ceil(top_p * Q), Q the total weight; every id tied with the cut is
// kept.  z* comes from a radix descent over the order-preserving bits of z
// (digits of 11, 11 and 10 bits), each digit in two launches:
//   k_topp_hist  (row, chunk) blocks: histogram of the weights of the keys
//                that match the bits decided so far, by the next digit
//                (2048 bins per chunk, integer LDS atomics: exact)
//   k_topp_pick  one block per row: sums the chunk histograms in chunk order
//                and picks the one bin where the weight of the keys above it
//                and in it first reaches t (after the first digit, with the
//                weight above the current range carried per row)
// after k_topp_max has taken the chunk maxima of z.  The Gumbel-max over the
// nucleus is then k_sample_partial with z*'s key as a threshold.
// ---------------------------------------------------------------------------
constexpr int kTopPThreads = 1024;
constexpr int kTopPWaves = kTopPThreads / 64;
static_assert(kTopPBins == 2 * kTopPThreads, "two histogram bins per pick thread");

// z = fp32(logit / T); dividing by 1 is exact, so it is skipped
__device__ __forceinline__ float zval(const float* lg, int v, float temp) {
  return (temp == 1.0f) ? lg[v] : __fdiv_rn(lg[v], temp);
}

// Vocabulary chunks per row in the top-p passes: enough (row, chunk) blocks to
// fill the GPU, and no more, since every chunk writes and every pick reads a
// 16 KiB histogram (128 rows x 151936 ids: a pick 6.0 us at 8 chunks, 9 at 16,
// the histogram passes alike).
__device__ __forceinline__ int topp_chunks(int M) { return max(1, min(kTopPChunks, 1024 / max(M, 1))); }
// Chunk c: [c*per, min(V, (c+1)*per)) with per a multiple of 4, so a chunk of a
// row whose length V is a multiple of 4 starts 16-byte aligned.
__device__ __forceinline__ int topp_chunk_len(int V, int nch) { return (((V + nch - 1) / nch) + 3) & ~3; }

// Calls f(z, true) for every id of [v0, v1) of the row lg, z = fp32(lg[v] / T),
// on all lanes of a wave together (f(z, false) where a lane has no id).  A row
// that starts 16-byte aligned and whose length is divisible by 4 is read as
// float4, kTopPLoads loads of a thread at a time and the next ones in flight
// while these are used; any other row one float at a time.
constexpr int kTopPLoads = 4;
template <typename F>
__device__ __forceinline__ void topp_visit(const float* __restrict__ lg, int V, int v0, int v1, float temp, F f) {
  const int tid = threadIdx.x;
  if ((V & 3) == 0 && (reinterpret_cast<uintptr_t>(lg) & 15) == 0) {
    const float4* l4 = reinterpret_cast<const float4*>(lg);
    const int q1 = v1 >> 2;
    constexpr int kStep = 256 * kTopPLoads;
    const auto load = [&](float4 (&x)[kTopPLoads], int base) {
#pragma unroll
      for (int u = 0; u < kTopPLoads; ++u) {
        const int qq = base + u * 256 + tid;
        if (qq < q1) x[u] = l4[qq];
      }
    };
    const auto use = [&](float4 (&x)[kTopPLoads], int base) {
      // one branch around all divisions: a choice for each value computes the
      // division (11 instructions) and throws it away
      if (temp != 1.0f) {
#pragma unroll
        for (int u = 0; u < kTopPLoads; ++u)
          x[u] = make_float4(__fdiv_rn(x[u].x, temp), __fdiv_rn(x[u].y, temp), __fdiv_rn(x[u].z, temp),
                             __fdiv_rn(x[u].w, temp));
      }
#pragma unroll
      for (int u = 0; u < kTopPLoads; ++u) {
        if (base + u * 256 >= q1) break;   // uniform
        const bool ok = base + u * 256 + tid < q1;
        f(x[u].x, ok);
        f(x[u].y, ok);
        f(x[u].z, ok);
        f(x[u].w, ok);
      }
    };
    float4 x[kTopPLoads] = {}, y[kTopPLoads] = {};
    int base = v0 >> 2;
    load(x, base);
    for (; base < q1; base += 2 * kStep) {
      load(y, base + kStep);
      use(x, base);
      load(x, base + 2 * kStep);
      use(y, base + kStep);
    }
  } else {
    for (int v = v0; v < v1; v += 256) {
      const bool ok = v + tid < v1;
      f(ok ? zval(lg, v + tid, temp) : 0.0f, ok);
    }
  }
}

__global__ __launch_bounds__(256) void k_topp_max(const int32_t* __restrict__ M_ptr, int M,
    const RowDesc* __restrict__ rows, const float* __restrict__ logits, int V, int by_slot,
    const CtlParams* __restrict__ cpd, float temp, float* __restrict__ pmax) {
  __shared__ float red[4];
  if (cpd) temp = cpd->temperature;
  if (M_ptr) M = *M_ptr;
  const int nch = topp_chunks(M), per = topp_chunk_len(V, nch);
  for (int item = blockIdx.x; item < M * nch; item += gridDim.x) {
    const int i = item / nch, c = item - i * nch;
    const float* lg = logits + (size_t)(by_slot ? rows[i].slot : i) * V;
    const int v0 = min(V, c * per), v1 = min(V, v0 + per);
    float zm = -INFINITY;
    topp_visit(lg, V, v0, v1, temp, [&](float z, bool ok) { zm = ok ? fmaxf(zm, z) : zm; });
    zm = wave_max(zm);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = zm;
    __syncthreads();
    if (threadIdx.x == 0) pmax[item] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();   // red is reused by the next item
  }
}

__device__ __forceinline__ float row_zmax(const float* __restrict__ pmax, int i, int nch) {
  float zm = pmax[(size_t)i * nch];
  for (int c = 1; c < nch; ++c) zm = fmaxf(zm, pmax[(size_t)i * nch + c]);
  return zm;
}

// digit d of the descent: bits 31..21 (d = 0), 20..10 (d = 1), 9..0 (d = 2)
__host__ __device__ constexpr int digit_shift(int d) { return d == 0 ? 21 : (d == 1 ? 10 : 0); }

// Histogram pass of digit D.  The first is bound by the fp64 exponential of each
// id (about 30 instructions of 4 cycles a wave); the others by reading the
// logits and their histograms, since few ids match the bits decided so far: a
// wave queues those in LDS and takes the exponential of 64 at once, where one
// match in the wave would cost as much as 64.  128 rows x 151936 ids 38 / 26 /
// 22 us (k_topp_max, which only reads, 14.7), 35 us on average for the three with
// an exponential for each wave that holds a match and a discarded division.
template <int D>
__global__ __launch_bounds__(256) void k_topp_hist(const int32_t* __restrict__ M_ptr, int M,
    const RowDesc* __restrict__ rows, const float* __restrict__ logits, int V, int by_slot,
    const CtlParams* __restrict__ cpd, float temp, const float* __restrict__ pmax,
    const uint32_t* __restrict__ prefix, unsigned long long* __restrict__ hist) {
  __shared__ unsigned long long h[kTopPBins];
  __shared__ float queue[4][128];
  float* const wq = queue[threadIdx.x >> 6];
  if (cpd) temp = cpd->temperature;
  if (M_ptr) M = *M_ptr;
  const int nch = topp_chunks(M), per = topp_chunk_len(V, nch);
  constexpr int sh = digit_shift(D);
  constexpr int nbins = (D == 2) ? 1024 : kTopPBins;
  constexpr uint32_t dmask = nbins - 1;
  constexpr int hi = (D == 1) ? 21 : 10;   // the bits decided before digit D (D > 0)
  const int lane = threadIdx.x & 63;
  for (int item = blockIdx.x; item < M * nch; item += gridDim.x) {
    const int i = item / nch, c = item - i * nch;
    const float* lg = logits + (size_t)(by_slot ? rows[i].slot : i) * V;
    const int v0 = min(V, c * per), v1 = min(V, v0 + per);
    const float zm = row_zmax(pmax, i, nch);
    const uint32_t pre = (D > 0) ? prefix[i] : 0u;
    for (int b = threadIdx.x; b < nbins; b += 256) h[b] = 0ull;
    __syncthreads();
    const auto add = [&](float z) {
      const uint64_t q = nucleus_weight(z, zm);
      if (q) atomicAdd(&h[(zkey(z) >> sh) & dmask], (unsigned long long)q);
    };
    if (D == 0) {
      topp_visit(lg, V, v0, v1, temp, [&](float z, bool ok) { if (ok) add(z); });
    } else {
      int put = 0, got = 0;
      topp_visit(lg, V, v0, v1, temp, [&](float z, bool ok) {
        const bool hit = ok && (zkey(z) >> hi) == (pre >> hi);
        const unsigned long long hits = __ballot(hit);
        if (hits == 0ull) return;
        if (hit) wq[(put + __popcll(hits & ((1ull << lane) - 1ull))) & 127] = z;
        put += __popcll(hits);
        if (put - got >= 64) {
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          add(wq[(got + lane) & 127]);
          got += 64;
        }
      });
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (lane < put - got) add(wq[(got + lane) & 127]);
    }
    __syncthreads();
    unsigned long long* out = hist + (size_t)item * kTopPBins;
    for (int b = threadIdx.x; b < nbins; b += 256) out[b] = h[b];
    __syncthreads();   // h is cleared for the next item
  }
}

static auto topp_hist_kernel(int d) { return d == 0 ? k_topp_hist<0> : (d == 1 ? k_topp_hist<1> : k_topp_hist<2>); }

// Per-row state of the descent: prefix (z*'s key bits decided so far; after
// digit 2, z*'s key), above (weight of keys above the current range), target.
__global__ __launch_bounds__(kTopPThreads) void k_topp_pick(const int32_t* __restrict__ M_ptr, int M,
    const CtlParams* __restrict__ cpd, float top_p, int d, const unsigned long long* __restrict__ hist,
    uint32_t* __restrict__ prefix, unsigned long long* __restrict__ above_arr,
    unsigned long long* __restrict__ target_arr) {
  __shared__ unsigned long long wsum[kTopPWaves];
  __shared__ unsigned long long sel_above, target;
  __shared__ uint32_t sel_digit;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (cpd) top_p = cpd->top_p;
  if (M_ptr) M = *M_ptr;
  const int nch = topp_chunks(M);
  const int sh = digit_shift(d);
  for (int i = blockIdx.x; i < M; i += gridDim.x) {
    // the chunk histograms, summed in chunk order
    const ulonglong2* hr = (const ulonglong2*)(hist + (size_t)i * nch * kTopPBins) + tid;
    unsigned long long h0 = 0ull, h1 = 0ull;
    if (d < 2 || tid < 512) {                 // the last digit has 1024 bins
      for (int c = 0; c < nch; c += 8) {      // 8 loads in flight
        ulonglong2 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = hr[(size_t)min(c + u, nch - 1) * kTopPThreads];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (c + u < nch) { h0 += x[u].x; h1 += x[u].y; }
      }
    }
    unsigned long long above = 0ull;
    uint32_t pre = 0u;
    if (d == 0) {
      // the first digit's histograms cover every weight: Q and the target
      unsigned long long tot = h0 + h1;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) tot += __shfl_xor(tot, o, 64);
      if (lane == 0) wsum[wave] = tot;
      __syncthreads();
      if (tid == 0) {
        unsigned long long Q = 0ull;
        for (int w = 0; w < kTopPWaves; ++w) Q += wsum[w];
        target = (unsigned long long)ceil((double)top_p * (double)Q);
      }
    } else {
      if (tid == 0) target = target_arr[i];
      above = above_arr[i];
      pre = prefix[i];
    }
    // suffix sums of the histogram: thread t owns bins 2t and 2t+1
    unsigned long long incl = h0 + h1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long y = __shfl_down(incl, o, 64);
      if (lane + o < 64) incl += y;
    }
    __syncthreads();
    if (lane == 0) wsum[wave] = incl;
    __syncthreads();
    unsigned long long excl = incl - (h0 + h1);
    for (int w = wave + 1; w < kTopPWaves; ++w) excl += wsum[w];
    // the one bin where the upper-set weight first reaches the target
    const unsigned long long t = target;
    const unsigned long long a1 = above + excl, a0 = a1 + h1;
    if (a1 < t && a1 + h1 >= t) { sel_digit = 2 * tid + 1; sel_above = a1; }
    if (a0 < t && a0 + h0 >= t) { sel_digit = 2 * tid; sel_above = a0; }
    __syncthreads();
    if (tid == 0) {
      prefix[i] = pre | (sel_digit << sh);
      above_arr[i] = sel_above;
      if (d == 0) target_arr[i] = t;
    }
    __syncthreads();   // wsum, target and the selection are rewritten for the next row
  }
}

__device__ __forceinline__ bool forced_eos_fires(uint64_t seed, int32_t step, int rid, int gen,
                                                 uint32_t thr) {
  if (thr == 0u) return false;
  uint32_t k0, k1;
  sampler_key(seed, step, k0, k1);
  U32x4 w = philox4x32_10((uint32_t)rid, (uint32_t)gen, 0u, 1u, k0, k1);
  return w.x < thr;
}

// Final token of each decode row: the best of the row's nchunks partial
// (score, id) winners (chunk c of row i at [c * cstride + i * rstride]),
// forced EOS, teacher forcing, forced length, reward
// hash chain, termination and the per-slot finish flag.  One block per row
// (persistent over the live rows); the (score desc, id asc) order is total,
// so the reduction order does not matter.
__global__ __launch_bounds__(256) void k_sample_final(const Ctl* __restrict__ ctl,
    const RowDesc* __restrict__ rows, const float* __restrict__ best,
    const int32_t* __restrict__ bidx, int nchunks, int cstride, int rstride, const int32_t* __restrict__ forced,
    const int32_t* const* __restrict__ forced_at, const int32_t* __restrict__ flen, int model_free,
    const CtlParams* __restrict__ cpp,
    const double* __restrict__ p, int32_t* __restrict__ out_tok, int32_t* __restrict__ samp_tok,
    int32_t* __restrict__ slot_gen, int32_t* __restrict__ slot_tok, uint64_t* __restrict__ slot_hash,
    int32_t* __restrict__ fin, int32_t* __restrict__ r_len, int32_t* __restrict__ r_reward) {
  __shared__ float sb[256];
  __shared__ int si[256];
  if (forced_at) forced = *forced_at;                      // captured loop: the table of the running sara_run
  const int M = ctl->done ? 0 : ctl->M;
  for (int i = blockIdx.x; i < M; i += gridDim.x) {
    float bs = -INFINITY;
    int bi = 0x7FFFFFFF;
    if (!model_free)
      for (int c = threadIdx.x; c < nchunks; c += 256)
        better(bs, bi, best[(size_t)c * cstride + (size_t)i * rstride], bidx[(size_t)c * cstride + (size_t)i * rstride]);
    sb[threadIdx.x] = bs;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (threadIdx.x < o) {
        float s2 = sb[threadIdx.x];
        int i2 = si[threadIdx.x];
        better(s2, i2, sb[threadIdx.x + o], si[threadIdx.x + o]);
        sb[threadIdx.x] = s2;
        si[threadIdx.x] = i2;
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      const CtlParams cp = *cpp;
      const int32_t* fl = cp.has_flen ? flen : nullptr;
      const RowDesc r = rows[i];
      const int rid = r.rid, gen = r.gen, s = r.slot;
      int samp;
      if (model_free) {
        samp = forced[(size_t)rid * cp.max_new + gen];
      } else {
        samp = si[0];
        if (cp.eos >= 0 && forced_eos_fires(cp.seed, cp.step, rid, gen, cp.forced_eos)) samp = cp.eos;
      }
      int tok = forced ? forced[(size_t)rid * cp.max_new + gen] : samp;
      bool done = false;
      if (fl && gen + 1 == fl[rid]) {
        if (cp.eos >= 0) tok = cp.eos;
        done = true;
      }
      if (cp.eos >= 0 && tok == cp.eos) done = true;
      if (gen + 1 == cp.max_new) done = true;
      out_tok[(size_t)rid * cp.max_new + gen] = tok;
      samp_tok[(size_t)rid * cp.max_new + gen] = samp;
      uint64_t hsh = mix64(slot_hash[s] ^ (uint64_t)(uint32_t)(tok + 1));
      slot_hash[s] = hsh;
      slot_gen[s] = gen + 1;
      slot_tok[s] = tok;
      if (done) {
        r_len[rid] = gen + 1;
        double u = (double)(hsh >> 11) * 0x1p-53;
        r_reward[rid] = (u < p[r.uid]) ? 1 : 0;
        fin[s] = 1;
      }
    }
    __syncthreads();   // sb/si are reused by the next row
  }
}

// stand-alone sampler for given logits: the best of a row's chunk winners, one
// wave per row
__global__ __launch_bounds__(256) void k_sample_rows_final(int n_rows, const int32_t* __restrict__ rid,
    const int32_t* __restrict__ pos, const float* __restrict__ best,
    const int32_t* __restrict__ bidx, int nch, uint64_t seed, int32_t step, int eos, uint32_t feos,
    int32_t* __restrict__ tok) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n_rows) return;
  const int r = rid[i], g = pos[i];
  float bs = -INFINITY;
  int bi = 0x7FFFFFFF;
  for (int c = lane; c < nch; c += 64) better(bs, bi, best[(size_t)i * nch + c], bidx[(size_t)i * nch + c]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float s2 = __shfl_xor(bs, o, 64);
    const int i2 = __shfl_xor(bi, o, 64);
    better(bs, bi, s2, i2);
  }
  if (lane != 0) return;
  if (eos >= 0 && forced_eos_fires(seed, step, r, g, feos)) bi = eos;
  tok[i] = bi;
}

__global__ void k_copy_logits(const Ctl* __restrict__ ctl, const RowDesc* __restrict__ rows,
                              const float* __restrict__ ws, int V, float* __restrict__ dst) {
  int M = ctl->done ? 0 : ctl->M;
  int i = blockIdx.y;
  if (i >= M) return;
  int s = rows[i].slot;
  for (int v = blockIdx.x * 256 + threadIdx.x; v < V; v += gridDim.x * 256)
    dst[(size_t)s * V + v] = ws[(size_t)i * V + v];
}


// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
// K splits of a decode GEMM into fp32 partials: until 64-row weight blocks reach
// one block per CU (the live rows are few and known only on the device), as an
// even division of the k chunks (the last split of an uneven one runs alone):
// the largest count in [6, kMaxSplitsDec] with >= 4 chunks per split, else the
// occupancy target.  Consumers sum at most kMaxSplitsDec partials in one batch
// of loads.  Returns the K range of a split.
static int decode_split_k(const sara_ctx* c, int M_cap, int N, int K) {
  const int tiles_n = (N + 63) / 64, chunks = K / 64;
  const int want = (tiles_n >= 256) ? 1 : (256 + tiles_n - 1) / tiles_n;
  int splits = std::min(want, std::max(1, chunks / 4));
  for (int s = kMaxSplitsDec; s >= 6; --s)
    if (s <= want && chunks % s == 0 && chunks / s >= 4) { splits = s; break; }
  splits = std::max(1, std::min(splits, kMaxSplitsDec));
  const int kps = ((chunks + splits - 1) / splits) * 64;
  return (int64_t)((K + kps - 1) / kps) * M_cap * N > c->ws_floats ? K : kps;
}

// bf16 GEMM of a short prefill chunk into fp32 partials ws[split][M][N]
int gemm_bf16(sara_ctx* c, const void* X, const void* W, const int32_t* M_ptr, int M, int N, int K, int& splits_out) {
  const int64_t stride = (int64_t)M * N;
  // weight rows per block: 128 (two 16-row tiles per wave) for long K, 64
  // otherwise; split K until the grid has about one block per CU (each split
  // keeps >= 4 k chunks): wide GEMMs need no split, narrow ones trade fp32
  // partial traffic for occupancy
  constexpr int MT = 8;
  const bool two = K >= 4096;
  const int rows_per_block = two ? 128 : 64;
  const int tiles_n = (N + rows_per_block - 1) / rows_per_block, zb = (M + 16 * MT - 1) / (16 * MT);
  const int64_t blocks = (int64_t)tiles_n * zb;
  const int want = (blocks >= 256) ? 1 : (int)((256 + blocks - 1) / blocks);
  const int chunks = K / 64;
  int splits = std::max(1, std::min(want, std::max(1, chunks / 4)));
  int kps = ((chunks + splits - 1) / splits) * 64;
  splits = (K + kps - 1) / kps;
  if ((int64_t)splits * stride > c->ws_floats) { splits = 1; kps = K; }
  const dim3 grid(tiles_n, splits, zb);
#define SARA_GEMM(NT_)                                                                                            \
  launch_k(c, c->stream, (k_gemm_bf16_lds<NT_, MT, 64, 0, 1>), grid, dim3(256), 0, (const uint16_t*)X,            \
           (const uint16_t*)W, (void*)c->ws, M_ptr, N, K, kps, stride, SampleArgs{})
  if (two) SARA_GEMM(2);
  else SARA_GEMM(1);
#undef SARA_GEMM
  splits_out = splits;
  return SARA_OK;
}

// bf16 GEMM of a decode step into fp32 partials ws[split][M_cap][N]; returns
// the splits.  One z block per m-block of the capacity; the live row count is
// read on the device, and z blocks past it exit at once (blocks are dispatched
// z-major, so the live m-blocks start first).
static int gemm_decode(sara_ctx* c, const void* X, const void* W, const int32_t* M_ptr, int M_cap, int N, int K,
                       bool oproj) {
  const int64_t stride = (int64_t)M_cap * N;
  const int kps = decode_split_k(c, M_cap, N, K), splits = (K + kps - 1) / kps;
  // down on tiles (512 rows of 11008 -> 2048: 40 us against 49); the o
  // projection's splits are too short for them (8 steps: 19 us against 17)
  if (c->tile_rows && !oproj) {
    GemmTileArgs a{};
    a.M_ptr = M_ptr;
    a.out = c->ws;
    a.split_stride = stride;
    a.steps = kps / 32;
    gemm_tile<0>(c, X, W, M_cap, N, K, a);
    return splits;
  }
  const dim3 grid((N + 63) / 64, splits, (M_cap + 127) / 128);
#define SARA_GEMM(PF_)                                                                                            \
  launch_k(c, c->stream, (k_gemm_bf16_lds<1, 8, 64, 0, PF_>), grid, dim3(256), 0, (const uint16_t*)X,             \
           (const uint16_t*)W, (void*)c->ws, M_ptr, N, K, kps, stride, SampleArgs{})
  if (oproj) SARA_GEMM(2);
  else SARA_GEMM(0);
#undef SARA_GEMM
  return splits;
}

// fp32 GEMM into out (see k_gemm_f32).  Four row tiles a block in a prefill,
// two in decode, where few rows are live and the row count is known on the
// device only.
template <int EPI>
static void gemm_f32(sara_ctx* c, const void* X, const void* W, float* out, const int32_t* M_ptr, int M_cap, int N,
                     int K, int layer = 0) {
  const F32Epi ep{c->rows, c->rope, (float*)c->qbuf, (float*)c->kc, (float*)c->vc, c->hq, c->hkv, c->hd, layer,
                  c->n_blocks};
  const int bx = EPI == 0 ? (N / 16 + 1) / 2 : N / 32;
  if (c->in_prefill)
    launch_k(c, c->stream, (k_gemm_f32<4, EPI>), dim3(bx, (M_cap + 63) / 64), dim3(256), 0, (const float*)X,
             (const float*)W, out, M_ptr, M_cap, N, K, ep);
  else
    launch_k(c, c->stream, (k_gemm_f32<2, EPI>), dim3(bx, (M_cap + 31) / 32), dim3(256), 0, (const float*)X,
             (const float*)W, out, M_ptr, M_cap, N, K, ep);
}

#define PROF_B(c) do { if ((c)->prof_active) prof_begin(c); } while (0)
#define PROF_E(c, cls, N, K) do { if ((c)->prof_active) prof_end((c), (cls), (N), (K)); } while (0)

// gate|up GEMM with the SwiGLU epilogue (bf16 models; W_gu rows interleaved
// per 16-row tile at init), writing a = silu(g) * u to c->xa, fragment-major [m][ffn]
// (prefill; row-major in decode)
void gemm_swiglu(sara_ctx* c, const void* X, const void* W, const int32_t* M_ptr, int M_cap) {
  constexpr int MT = 8;
  const int N = 2 * c->ffn, K = c->d;
  if (!c->in_prefill && c->tile_rows) {
    GemmTileArgs a{};
    a.M_ptr = M_ptr;
    a.steps = K / 32;
    a.xa = (uint16_t*)c->xa;
    gemm_tile<1>(c, X, W, M_cap, N, K, a);
    return;
  }
  dim3 grid((N + 127) / 128, 1, (M_cap + 16 * MT - 1) / (16 * MT));
  if (c->in_prefill)
    launch_k(c, c->stream, (k_gemm_bf16_lds<2, MT, 64, 1, 1>), grid, dim3(256), 0, (const uint16_t*)X,
                       (const uint16_t*)W, (void*)c->xa, M_ptr, N, K, K, (int64_t)0, SampleArgs{});
  else
    launch_k(c, c->stream, (k_gemm_bf16_lds<2, MT, 64, 1, 0>), grid, dim3(256), 0, (const uint16_t*)X,
                       (const uint16_t*)W, (void*)c->xa, M_ptr, N, K, K, (int64_t)0, SampleArgs{});
}

// z blocks over which the q|k|v kernel shares out a small batch's 16-row
// tiles: as many per weight tile as keep every working block resident at
// once (blocks per CU x CUs / weight tiles), computed once per context
template <typename F>
static int qkv_spread(sara_ctx* c, F kernel) {
  if (c->qkv_spread == 0) {
    int per_cu = 0, dev = 0, n_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      per_cu = 1, n_cu = 256;
    c->qkv_spread = std::max(1, std::max(1, per_cu) * std::max(1, n_cu) / std::max(1, c->nqkv / 16));
  }
  return c->qkv_spread;
}

// blocks of the decode attention that are resident at once (every item of a
// list that short runs in one round), computed once per context
static int attn_resident(sara_ctx* c) {
  if (c->attn_dec_grid == 0) {
    int per_cu = 0, dev = 0, n_cu = 0;
    const hipError_t e = c->hd == 128 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_attn_dec<128>, 256, 0)
                                      : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_attn_dec<64>, 256, 0);
    if (e != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      per_cu = 2, n_cu = 256;
    c->attn_dec_grid = std::max(1, per_cu) * std::max(1, n_cu);
  }
  return c->attn_dec_grid;
}

// h += split-K sum of ws; x = RMSNorm(h) * w (fp32 models, bf16 prefill)
template <typename T>
static void residual_norm(sara_ctx* c, const int32_t* M_ptr, int M_cap, int sp, const float* w) {
  const int d = c->d, vpt = (d + 255) / 256;
  const dim3 grid(std::min(M_cap, 1024));
  const int64_t stride = (int64_t)M_cap * d;
  T* x = (T*)c->x;
#define SARA_RN(V) launch_k(c, c->stream, (k_residual_norm_v<T, V>), grid, dim3(256), 0, M_ptr, c->ws, \
                                      sp, stride, d, c->h, w, c->md.rms_eps, x)
  switch (sp <= kMaxSplitsDec ? vpt : 0) {
    case 1: SARA_RN(1); break;
    case 2: SARA_RN(2); break;
    case 3: SARA_RN(3); break;
    case 4: SARA_RN(4); break;
    case 5: case 6: SARA_RN(6); break;
    case 7: case 8: SARA_RN(8); break;
    default:
      launch_k(c, c->stream, k_residual_norm<T>, dim3(std::min(M_cap, 256)), dim3(1024), 0, M_ptr,
                         c->ws, sp, stride, d, c->h, w, c->md.rms_eps, x);
  }
#undef SARA_RN
}
void residual_norm_bf16(sara_ctx* c, const int32_t* M_ptr, int M_cap, int sp, const float* w) {
  residual_norm<uint16_t>(c, M_ptr, M_cap, sp, w);
}
// the same for the rows of a bf16 decode step (d <= 4096, at most
// kMaxSplitsDec splits)
static void residual_norm_decode(sara_ctx* c, const int32_t* M_ptr, int M_cap, int sp, const float* w, int x_tiled) {
  launch_k(c, c->stream, k_residual_norm_f4, dim3(std::min(M_cap, 1024)), dim3((c->d / 4 + 63) / 64 * 64), 0, M_ptr,
           c->ws, sp, (int64_t)M_cap * c->d, c->d, c->h, w, c->md.rms_eps, (uint16_t*)c->x, x_tiled);
}

void launch_qkv_epilogue_bf16(sara_ctx* c, const int32_t* M_ptr, int M, int sp, int layer) {
  launch_k(c, c->stream, k_qkv_epilogue, dim3(2048), dim3(c->hd / 2), 0, M_ptr, c->rows, c->ws, sp,
           (int64_t)M * c->nqkv, c->rope, c->hq, c->hkv, c->hd, layer, c->n_blocks, (uint16_t*)c->qbuf,
           (uint16_t*)c->kc, (uint16_t*)c->vc);
}

// bf16 decode: the live rows of a step through every layer
template <int HD>
static void decode_layers_bf16(sara_ctx* c, const int32_t* M_ptr, int M_cap) {
  hipStream_t st = c->stream;
  const int d = c->d;
  uint16_t* x = (uint16_t*)c->x;
  // many rows: the tile GEMMs' inputs fragment-major (a row-major stride of a
  // power of two sends a fragment's 16 rows to few channels: gate|up of 512
  // rows of d 2048 57 us against 44)
  const int xt = c->tile_rows ? 1 : 0;
  for (int l = 0; l < c->L; ++l) {
    int sp = 1;
    // q|k|v projection with the RoPE / KV-append epilogue, the paged
    // attention, then the merge of rows with several context splits
    PROF_B(c);
#define SARA_QKV_N(KS_, NT_) \
    launch_k(c, st, (k_qkv_rope<HD, KS_, NT_>), dim3(c->nqkv / (16 * NT_), 1, (M_cap + 127) / 128), dim3(256), 0, \
             (const uint16_t*)x, (const uint16_t*)c->w_qkv[l], M_ptr, d, c->rows, c->row_rope, c->hq, c->hkv, l, \
             c->n_blocks, (uint16_t*)c->qbuf, (uint16_t*)c->kc, (uint16_t*)c->vc, \
             NT_ * qkv_spread(c, k_qkv_rope<HD, KS_, 1>))
#define SARA_QKV(KS_) \
    if (c->tile_rows) SARA_QKV_N(KS_, 2); \
    else SARA_QKV_N(KS_, 1)
    switch (d / 128) {
      case 4: SARA_QKV(4); break;
      case 8: SARA_QKV(8); break;
      case 12: SARA_QKV(12); break;
      case 16: SARA_QKV(16); break;
      case 24: SARA_QKV(24); break;
      default: SARA_QKV(32); break;
    }
#undef SARA_QKV
#undef SARA_QKV_N
    PROF_E(c, kPQkvRope, c->nqkv, d);
    PROF_B(c);
    const int cap = M_cap * c->dec_splits_max;
    const int dg = (int)std::min<int64_t>((int64_t)cap * c->hkv, attn_resident(c));
    launch_k(c, st, (k_attn_dec<HD>), dim3(dg), dim3(256), 0, (const AttnItem*)c->attn_items,
             (const int32_t*)c->attn_nitems, (const PromptPlace*)c->places, cap, (const uint16_t*)c->kc, (const uint16_t*)c->vc, l, c->n_blocks,
             c->hq, c->hkv, c->dec_splits_max, 1.0f / sqrtf((float)HD), (const uint16_t*)c->qbuf, c->attn_part, x);
    PROF_E(c, kPAttn, 0, 0);
    PROF_B(c);
    // blocks of two waves: 1024 leave a CU 8 waves (512 rows of 16 heads: 14.0 us,
    // 10.5 with 4096, 8.9 with base-2 weights), but exit sooner where a few rows need no more
    launch_k(c, st, (k_attn_combine<uint16_t, HD>), dim3(c->tile_rows ? 4096 : 1024), dim3(HD), 0, M_ptr, c->rows, c->attn_part, c->hq,
             c->hkv, c->dec_splits_max, kDecPages, 1, x);
    PROF_E(c, kPCombine, 0, 0);
    PROF_B(c);
    sp = gemm_decode(c, x, c->w_o[l], M_ptr, M_cap, d, c->qdim, true);
    PROF_E(c, kPGemmO1, d, c->qdim);
    PROF_B(c);
    residual_norm_decode(c, M_ptr, M_cap, sp, c->norms + (size_t)(2 * l + 1) * d, xt);
    PROF_E(c, kPResNorm, d, 0);
    PROF_B(c);
    gemm_swiglu(c, x, c->w_gu[l], M_ptr, M_cap);
    PROF_E(c, kPGemmGU, 2 * c->ffn, d);
    PROF_B(c);
    sp = gemm_decode(c, c->xa, c->w_d[l], M_ptr, M_cap, d, c->ffn, false);
    PROF_E(c, kPGemmN1, d, c->ffn);
    PROF_B(c);
    // the next layer's norm (its q|k|v kernel reads fragment-major rows) or the
    // final one, in the order its reader takes: the tile LM head fragment-major,
    // the few-row ones (the only form that writes logits for top-p) row-major
    residual_norm_decode(c, M_ptr, M_cap, sp, c->norms + (size_t)(2 * l + 2) * d, l + 1 < c->L ? 1 : xt && !c->topp);
    PROF_E(c, kPResNorm, d, 0);
  }
}

// fp32 models: the rows of a decode step or a prefill chunk through every
// layer.  A prefill ends with the K and V of the last layer: nothing reads
// what follows.
template <int HD>
static void layers_f32(sara_ctx* c, const int32_t* M_ptr, int M_cap) {
  hipStream_t st = c->stream;
  const int d = c->d;
  float* x = (float*)c->x;
  for (int l = 0; l < c->L; ++l) {
    PROF_B(c);
    gemm_f32<2>(c, x, c->w_qkv[l], nullptr, M_ptr, M_cap, c->nqkv, d, l);
    PROF_E(c, kPQkvRope, c->nqkv, d);
    if (c->in_prefill && l + 1 == c->L) break;
    PROF_B(c);
    launch_k(c, st, (k_attention<HD>), dim3(M_cap, c->hkv, c->attn_splits_max), dim3(256), 0, M_ptr, c->rows,
             (const float*)c->qbuf, (const float*)c->kc, (const float*)c->vc, l, c->n_blocks, c->hq, c->hkv,
             c->attn_splits_max, 1.0f / sqrtf((float)HD), c->attn_part, x);
    PROF_E(c, kPAttn, 0, 0);
    if (c->attn_splits_max > 1) {
      PROF_B(c);
      launch_k(c, st, (k_attn_combine<float, HD>), dim3(1024), dim3(HD), 0, M_ptr, c->rows, c->attn_part, c->hq, c->hkv,
               c->attn_splits_max, 0, 0, x);
      PROF_E(c, kPCombine, 0, 0);
    }
    PROF_B(c);
    gemm_f32<0>(c, x, c->w_o[l], c->ws, M_ptr, M_cap, d, c->qdim);
    PROF_E(c, kPGemmN1, d, c->qdim);
    PROF_B(c);
    residual_norm<float>(c, M_ptr, M_cap, 1, c->norms + (size_t)(2 * l + 1) * d);
    PROF_E(c, kPResNorm, d, 0);
    PROF_B(c);
    gemm_f32<1>(c, x, c->w_gu[l], (float*)c->xa, M_ptr, M_cap, 2 * c->ffn, d);
    PROF_E(c, kPGemmGU, 2 * c->ffn, d);
    PROF_B(c);
    gemm_f32<0>(c, c->xa, c->w_d[l], c->ws, M_ptr, M_cap, d, c->ffn);
    PROF_E(c, kPGemmN1, d, c->ffn);
    PROF_B(c);
    residual_norm<float>(c, M_ptr, M_cap, 1, c->norms + (size_t)(2 * l + 2) * d);   // the next layer's, or the final one
    PROF_E(c, kPResNorm, d, 0);
  }
}

static void run_layers(sara_ctx* c, const int32_t* M_ptr, int M_cap) {
  if (c->md.dtype == SARA_BF16) {
    if (c->hd == 128) decode_layers_bf16<128>(c, M_ptr, M_cap);
    else decode_layers_bf16<64>(c, M_ptr, M_cap);
  } else {
    if (c->hd == 128) layers_f32<128>(c, M_ptr, M_cap);
    else layers_f32<64>(c, M_ptr, M_cap);
  }
}

int launch_prefill(sara_ctx* c) {
  hipStream_t st = c->stream;
  c->in_prefill = true;
  // prefix sums of (P - 1): prompt-token rows of the pool, chunked
  std::vector<int64_t> pre(c->U + 1, 0);
  for (int u = 0; u < c->U; ++u) pre[u + 1] = pre[u] + (c->h_off[u + 1] - c->h_off[u] - 1);
  int64_t rows_total = pre[c->U];
  int chunk = 0;
  for (int64_t r0 = 0; r0 < rows_total; r0 += c->prefill_rows, ++chunk) {
    int n = (int)((rows_total - r0 < c->prefill_rows) ? rows_total - r0 : c->prefill_rows);
    launch_k(c, st, k_prefill_rows, dim3((n + 255) / 256), dim3(256), 0, c->pre, c->U, (int)r0,
                       n, c->tok, c->off, c->rows, c->rows_M, c->PB);
    if (c->md.dtype == SARA_BF16) {
      prefill_layers_bf16(c, c->rows_M, n, chunk);
    } else {
      launch_k(c, st, k_embed_norm, dim3(n), dim3(256), 0, c->rows_M, c->rows,
                         (const float*)c->embed, c->norms, c->d, c->md.rms_eps, c->h, (float*)c->x);
      run_layers(c, c->rows_M, n);
    }
  }
  c->in_prefill = false;
  return SARA_OK;
}

// Gumbel-max of the live rows over the ids whose key reaches thr (all without
// it): winners [row][kSampleChunks]
static void launch_sample_decode(sara_ctx* c, hipStream_t st, const float* lg, int by_slot, const uint32_t* thr) {
  with_sample_quads(c->V, kSampleChunks, [&](auto kernel) {
    launch_k(c, st, kernel, dim3(std::min(c->S * kSampleChunks, 2048)), dim3(256), 0, (const int32_t*)c->rows_M, 0,
             (const int32_t*)nullptr, (const int32_t*)nullptr, (const RowDesc*)c->rows, lg, c->V, by_slot, thr,
             (const CtlParams*)c->cp_dev, (uint64_t)0, 0, 1.0f, kSampleChunks, c->samp_best, c->samp_idx);
  });
}

// Top-p passes over the live rows' logits (lg: [slot][V] when by_slot, else
// [row][V]) -> z*'s key per row, then the Gumbel-max over the nucleus by
// k_sample_partial with that threshold: winners [row][kSampleChunks].
static void launch_topp_decode(sara_ctx* c, hipStream_t st, const float* lg, int by_slot) {
  const int S = c->S;
  const CtlParams* cp = (const CtlParams*)c->cp_dev;
  const int32_t* Mp = c->rows_M;
  const RowDesc* rw = c->rows;
  const int g = std::min(S * kTopPChunks, 2048);
  PROF_B(c);
  launch_k(c, st, k_topp_max, dim3(g), dim3(256), 0, Mp, 0, rw, lg, c->V, by_slot, cp, 1.0f, c->topp_max);
  PROF_E(c, kPToppMax, c->V, 0);
  for (int d = 0; d < 3; ++d) {
    PROF_B(c);
    launch_k(c, st, topp_hist_kernel(d), dim3(g), dim3(256), 0, Mp, 0, rw, lg, c->V, by_slot, cp, 1.0f,
             (const float*)c->topp_max, (const uint32_t*)c->topp_thr, c->topp_hist);
    PROF_E(c, kPToppHist, c->V, 0);
    PROF_B(c);
    launch_k(c, st, k_topp_pick, dim3(std::min(S, 1024)), dim3(kTopPThreads), 0, Mp, 0, cp, 1.0f, d,
             (const unsigned long long*)c->topp_hist, c->topp_thr, c->topp_above, c->topp_target);
    PROF_E(c, kPToppSel, 0, 0);
  }
  PROF_B(c);
  launch_sample_decode(c, st, lg, by_slot, (const uint32_t*)c->topp_thr);
  PROF_E(c, kPSampleP, c->V, 0);
}

int launch_decode(sara_ctx* c, const int32_t* forced, const int32_t* const* forced_at, float* logits, int model_free) {
  hipStream_t st = c->stream;
  const int S = c->S;
  PROF_B(c);
  const int eg = std::min(S, 512);
#define SARA_EMBED(T_, items_)                                                                                    \
  launch_k(c, st, k_decode_embed<T_>, dim3(eg), dim3(256), 0, c->ctl, (const ActiveRow*)c->active, c->slot_gen,      \
           c->slot_tok, c->k, c->rows, c->rows_M, model_free ? 0 : 1, (const T_*)c->embed, c->norms, c->d,           \
           c->md.rms_eps, c->h, (T_*)c->x, c->U, c->PB, c->SB, c->rope, c->hd / 2, c->row_rope, items_, c->attn_nitems, \
           kDecPages, (const PromptPlace*)c->places, c->hkv, 16 / c->G, attn_resident(c), c->V)
  if (c->md.dtype == SARA_BF16) SARA_EMBED(uint16_t, model_free ? (AttnItem*)nullptr : c->attn_items);
  else SARA_EMBED(float, (AttnItem*)nullptr);
#undef SARA_EMBED
  PROF_E(c, kPEmbed, c->d, 0);
  int nchunks = kSampleChunks;
  if (!model_free) {
    if (c->md.dtype == SARA_BF16) {
      run_layers(c, c->rows_M, S);
      const int nb = (c->V + 127) / 128;
      const dim3 lm_grid(nb, 1, (S + 127) / 128);
      if (c->topp) {
        // top-p < 1: the GEMM writes the logits ([slot][V]) and the nucleus
        // sampler draws from them (drawing in the epilogue as well, only to be
        // replaced: 233 against 104 us at 128 rows)
        float* lg_out = logits ? logits : c->topp_logits;
        PROF_B(c);
        launch_k(c, st, (k_gemm_bf16_lds<2, 8, 64, 3, 0>), lm_grid, dim3(256), 0, (const uint16_t*)c->x,
                 (const uint16_t*)c->lm_head, (void*)nullptr, c->rows_M, c->V, c->d, c->d, (int64_t)0,
                 SampleArgs{c->rows, (const CtlParams*)c->cp_dev, lg_out, nullptr, nullptr, S});
        PROF_E(c, kPGemmLM, c->V, c->d);
        launch_topp_decode(c, st, lg_out, 1);
      } else {
        // LM head with the Gumbel-max sampling epilogue: per (row, 128-id block)
        // exact winners, reduced by k_sample_final
        const SampleArgs sa{c->rows, (const CtlParams*)c->cp_dev, logits, c->samp_best, c->samp_idx, S};
        nchunks = nb;
        PROF_B(c);
        if (c->tile_rows) {
          nchunks = (c->V + 255) / 256;
          GemmTileArgs a{};
          a.M_ptr = c->rows_M;
          a.steps = c->d / 32;
          a.sample = sa;
          gemm_tile<5>(c, c->x, c->lm_head, S, c->V, c->d, a);
        } else
        launch_k(c, st, (k_gemm_bf16_lds<2, 8, 64, 2, 0>), lm_grid, dim3(256), 0, (const uint16_t*)c->x,
                 (const uint16_t*)c->lm_head, (void*)nullptr, c->rows_M, c->V, c->d, c->d, (int64_t)0,
                 sa);
        PROF_E(c, kPGemmLM, c->V, c->d);
      }
    } else {
      run_layers(c, c->rows_M, S);
      PROF_B(c);
      gemm_f32<0>(c, c->x, c->lm_head, c->ws, c->rows_M, S, c->V, c->d);   // logits [M][V]
      PROF_E(c, kPGemmLM, c->V, c->d);
      if (c->topp) {
        launch_topp_decode(c, st, c->ws, 0);
      } else {
        PROF_B(c);
        launch_sample_decode(c, st, c->ws, 0, nullptr);
        PROF_E(c, kPSampleP, c->V, 0);
      }
      if (logits) {
        PROF_B(c);
        launch_k(c, st, k_copy_logits, dim3(64, S), dim3(256), 0, c->ctl, c->rows, c->ws, c->V,
                           logits);
        PROF_E(c, kPCopy, c->V, 0);
      }
    }
  }
  PROF_B(c);
  // chunk winners: [row][kSampleChunks] from k_sample_partial (also after
  // the top-p passes), [chunk][S] from the fused LM head
  const bool fused = !model_free && c->md.dtype == SARA_BF16 && !c->topp;
  launch_k(c, st, k_sample_final, dim3(std::min(S, 1024)), dim3(256), 0, c->ctl, c->rows,
                     c->samp_best, c->samp_idx, nchunks, fused ? S : 1, fused ? 1 : nchunks, forced, forced_at, c->flen,
                     model_free,
                     (const CtlParams*)c->cp_dev, c->p, c->out_tok, c->samp_tok, c->slot_gen, c->slot_tok, c->slot_hash, c->fin,
                     c->r_len, c->r_reward);
  PROF_E(c, kPSampleF, 0, 0);
  return SARA_OK;
}

// Buffers of the stand-alone sampler: per-row chunk winners and, for top-p <
// 1, the descent's chunk maxima, histograms and per-row state.  Every kernel
// below writes a buffer before reading it, so the contents left by an earlier
// call never matter.
struct SampleBufs {
  float* best;
  int32_t* bidx;
  float* pmax;
  unsigned long long* hist;
  unsigned long long* state;   // per row: above, target
  uint32_t* thr;
};

// Vocabulary chunks per row of the stand-alone sampler: kSampleChunks, more
// for a few rows (one row: up to 128 blocks of 1024 ids or more, where 16
// blocks took 27 us for 151936 ids).  rows * chunks never exceeds
// max(1024, rows * kSampleChunks).
static int sample_chunks(int n_rows, int V) {
  const int fill = std::min(128, 1024 / std::max(1, n_rows));
  return std::max(kSampleChunks, std::min(fill, (V + 1023) / 1024));
}

static void enqueue_sample_rows(const SampleBufs& b, const float* logits, int n_rows, int V, const int32_t* rid,
                                const int32_t* pos, uint64_t seed, int step, float temp, float top_p, int eos,
                                uint32_t feos, int32_t* tok, hipStream_t st) {
  const int32_t* none = nullptr;
  const RowDesc* no_rows = nullptr;
  const CtlParams* no_cp = nullptr;
  const bool topp = top_p < 1.0f;
  if (topp) {
    const int g = std::min(n_rows * kTopPChunks, 2048);
    hipLaunchKernelGGL(k_topp_max, dim3(g), dim3(256), 0, st, none, n_rows, no_rows, logits, V, 0, no_cp, temp, b.pmax);
    for (int d = 0; d < 3; ++d) {
      hipLaunchKernelGGL(topp_hist_kernel(d), dim3(g), dim3(256), 0, st, none, n_rows, no_rows, logits, V, 0, no_cp,
                         temp, (const float*)b.pmax, (const uint32_t*)b.thr, b.hist);
      hipLaunchKernelGGL(k_topp_pick, dim3(std::min(n_rows, 1024)), dim3(kTopPThreads), 0, st, none, n_rows, no_cp,
                         top_p, d, (const unsigned long long*)b.hist, b.thr, b.state, b.state + n_rows);
    }
  }
  const int nch = sample_chunks(n_rows, V);
  const uint32_t* thr = topp ? b.thr : nullptr;
  const dim3 grid(std::min<int64_t>((int64_t)n_rows * nch, 2048));
  with_sample_quads(V, nch, [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, none, n_rows, rid, pos, no_rows, logits, V, 0, thr, no_cp, seed,
                       step, temp, nch, b.best, b.bidx);
  });
  hipLaunchKernelGGL(k_sample_rows_final, dim3((n_rows + 3) / 4), dim3(256), 0, st, n_rows, rid, pos, b.best, b.bidx,
                     nch, seed, step, eos, feos, tok);
}

int launch_sample_rows(const float* logits, int n_rows, int V, const int32_t* rid,
                       const int32_t* pos, uint64_t seed, int step, float temp, float top_p, int eos,
                       uint32_t feos, int32_t* tok, hipStream_t st) {
  SampleBufs b{};
  std::vector<void*> owned;
  auto get = [&](void** p, size_t bytes) -> hipError_t {
    hipError_t e = hipMallocAsync(p, bytes, st);
    if (e == hipSuccess) owned.push_back(*p);
    return e;
  };
  auto release = [&]() {
    for (void* q : owned) (void)hipFreeAsync(q, st);
  };
  const bool topp = top_p < 1.0f;
  const size_t winners = (size_t)n_rows * sample_chunks(n_rows, V);
  hipError_t e = get((void**)&b.best, sizeof(float) * winners);
  if (e == hipSuccess) e = get((void**)&b.bidx, sizeof(int32_t) * winners);
  if (e == hipSuccess && topp) e = get((void**)&b.pmax, sizeof(float) * (size_t)n_rows * kTopPChunks);
  if (e == hipSuccess && topp)
    e = get((void**)&b.hist, sizeof(unsigned long long) * (size_t)n_rows * kTopPChunks * kTopPBins);
  if (e == hipSuccess && topp) e = get((void**)&b.state, sizeof(unsigned long long) * 2 * (size_t)n_rows);
  if (e == hipSuccess && topp) e = get((void**)&b.thr, sizeof(uint32_t) * (size_t)n_rows);
  if (e != hipSuccess) {
    release();
    return hip_fail(e, "hipMallocAsync");
  }
  enqueue_sample_rows(b, logits, n_rows, V, rid, pos, seed, step, temp, top_p, eos, feos, tok, st);
  e = hipGetLastError();
  release();
  if (e != hipSuccess) return hip_fail(e, "sample_rows launch");
  e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(e, "sample_rows");
  return SARA_OK;
}

// ---------------------------------------------------------------------------
// The stand-alone sampler without allocation: its buffers live in one static
// device array per GPU (this file's `scratch`, sized for kNoAllocMaxRows rows
// at top_p = 1 and kNoAllocMaxToppRows rows with the top-p passes).  Host code
// never passes the array's name to a kernel: the address each device gives
// for it is looked up once per device and kept.
// ---------------------------------------------------------------------------
namespace {
constexpr size_t kAlign = 256;
constexpr size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
constexpr size_t kOffBest = kAlign;   // the first kAlign bytes are unused
static_assert(kNoAllocMaxRows * kSampleChunks >= 1024, "the winners of sample_chunks fit");
constexpr size_t kOffBidx = kOffBest + align_up(sizeof(float) * (size_t)kNoAllocMaxRows * kSampleChunks);
constexpr size_t kOffPmax = kOffBidx + align_up(sizeof(int32_t) * (size_t)kNoAllocMaxRows * kSampleChunks);
constexpr size_t kOffHist = kOffPmax + align_up(sizeof(float) * (size_t)kNoAllocMaxToppRows * kTopPChunks);
constexpr size_t kOffState =
    kOffHist + align_up(sizeof(unsigned long long) * (size_t)kNoAllocMaxToppRows * kTopPChunks * kTopPBins);
constexpr size_t kOffThr = kOffState + align_up(sizeof(unsigned long long) * 2 * (size_t)kNoAllocMaxToppRows);
constexpr size_t kScratchBytes = kOffThr + align_up(sizeof(uint32_t) * (size_t)kNoAllocMaxToppRows);
static_assert(kScratchBytes == kNoAllocScratchBytes, "scratch layout and its stated size disagree");
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxScratchDevices] = {};
}  // namespace

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// Device address of `scratch` on the current device, looked up on the first
// call on that device.
static int scratch_address(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxScratchDevices) return hip_fail(hipErrorInvalidDevice, "device index");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress");
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return SARA_OK;
}

int launch_sample_rows_noalloc(const float* logits, int n_rows, int V, const int32_t* rid, const int32_t* pos,
                               uint64_t seed, int step, float temp, float top_p, int eos, uint32_t feos,
                               int32_t* tok, hipStream_t st) {
  void* base = nullptr;
  int rc = scratch_address(&base);
  if (rc != SARA_OK) return rc;
  unsigned char* b8 = (unsigned char*)base;
  SampleBufs b{};
  b.best = (float*)(b8 + kOffBest);
  b.bidx = (int32_t*)(b8 + kOffBidx);
  b.pmax = (float*)(b8 + kOffPmax);
  b.hist = (unsigned long long*)(b8 + kOffHist);
  b.state = (unsigned long long*)(b8 + kOffState);
  b.thr = (uint32_t*)(b8 + kOffThr);
  enqueue_sample_rows(b, logits, n_rows, V, rid, pos, seed, step, temp, top_p, eos, feos, tok, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "sample_rows_noalloc launch");
  return SARA_OK;
}

// Largest |gumbel_fast - gumbel_exact| over all 2^24 noise inputs (the
// 24-bit mantissa source of u); non-negative floats order like their bits.
__global__ __launch_bounds__(256) void k_gumbel_check(uint32_t* out) {
  float e = 0.f;
  for (uint32_t m = blockIdx.x * 256 + threadIdx.x; m < (1u << 24); m += gridDim.x * 256) {
    const uint32_t w = m << 8;
    e = fmaxf(e, fabsf(gumbel_fast(w) - gumbel_exact(w)));
  }
  e = wave_max(e);
  if ((threadIdx.x & 63) == 0) atomicMax(out, __float_as_uint(e));
}

int launch_gumbel_check(double* h_out, hipStream_t st) {
  uint32_t* d = nullptr;
  hipError_t e = hipMallocAsync((void**)&d, sizeof(uint32_t), st);
  if (e != hipSuccess) return hip_fail(e, "hipMallocAsync");
  e = hipMemsetAsync(d, 0, sizeof(uint32_t), st);
  if (e != hipSuccess) return hip_fail(e, "hipMemsetAsync");
  hipLaunchKernelGGL(k_gumbel_check, dim3(1024), dim3(256), 0, st, d);
  uint32_t bits = 0;
  e = hipMemcpyAsync(&bits, d, sizeof(uint32_t), hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
  (void)hipFreeAsync(d, st);
  e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(e, "gumbel check");
  float f;
  memcpy(&f, &bits, sizeof(f));
  *h_out = (double)f;
  return SARA_OK;
}

// Copy of a row-major bf16 weight [rows][K] (rows a multiple of 16, K of 64)
// into dst, a matrix of dst_rows rows in the GEMM weight layout, source tile
// j going to destination tile j * tile_mul + tile_add.
int launch_tile_weights(sara_ctx* c, const void* src, void* dst, int rows, int K, int tile_mul, int tile_add,
                        int dst_rows) {
  launch_k(c, c->stream, k_tile_weights, dim3(2048), dim3(256), 0, (const uint16_t*)src, (uint16_t*)dst,
                     rows / 16, K, tile_mul, tile_add, dst_rows / 16);
  return SARA_OK;
}

// Rows of heads head_off.. of a q, k or v weight ([n_rows][K], natural
// order) into the fused q|k|v weight (nqkv rows) in rotation-pair order.
int launch_tile_weights_pairs(sara_ctx* c, const void* src, void* dst, int n_rows, int K, int head_off) {
  launch_k(c, c->stream, k_tile_weights_pairs, dim3(2048), dim3(256), 0, (const uint16_t*)src,
                     (uint16_t*)dst, n_rows, K, head_off, c->hd, c->nqkv / 16);
  return SARA_OK;
}

// norm weights -> fp32 [2L+1][d]
__global__ void k_norm_to_f32_bf16(const uint16_t* __restrict__ src, float* __restrict__ dst, int d) {
  int c = blockIdx.x * 256 + threadIdx.x;
  if (c < d) dst[c] = bf16_to_f32(src[c]);
}

int launch_convert_norms(sara_ctx* c, const void* const* w) {
  const int d = c->d;
  for (int l = 0; l <= 2 * c->L; ++l) {
    const void* src;
    if (l == 2 * c->L) src = w[1 + 9 * c->L];
    else src = w[1 + 9 * (l / 2) + ((l & 1) ? 5 : 0)];
    float* dst = c->norms + (size_t)l * d;
    if (c->md.dtype == SARA_BF16)
      launch_k(c, c->stream, k_norm_to_f32_bf16, dim3((d + 255) / 256), dim3(256), 0,
                         (const uint16_t*)src, dst, d);
    else {
      hipError_t e = hipMemcpyAsync(dst, src, sizeof(float) * d, hipMemcpyDeviceToDevice, c->stream);
      if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync norms");
    }
  }
  return SARA_OK;
}

}  // namespace sara
