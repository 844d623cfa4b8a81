// Prefill of the bf16 models (gfx950): a chunk of prompt tokens through the
// decoder layers.  GEMM inputs are fragment-major (tiled_index), GEMM weights
// k-block-major fragments (wtiled_index), so both operands of a GEMM move to
// LDS as contiguous 1 KiB fragments.
#include <math.h>

#include <algorithm>

#include "gemm_tile.h"
#include "sara_internal.h"

namespace sara {

// ---------------------------------------------------------------------------
// causal prompt attention
// ---------------------------------------------------------------------------
// Block (query tile, KV head g): up to 32 R consecutive tokens of one prompt,
// all G query heads of g.  Wave (head, token subgroup) owns 32 tokens of one
// head as two 16-token MFMA tiles; the NW = G R waves share every 64-key block
// of K and V through LDS.  Keys 0 .. (last token of the tile) are walked from
// 0 in blocks of 64, so a row's result depends on its own context only, not on
// the tile or the chunk it is computed in.
//
// Per 64-key block (two 32-key groups kg) and 16-token tile:
//   S^T = K q^T   (v_mfma_f32_16x16x32_bf16).  The rows of the two K operands
//                 a, b of a group are picked so that lane (token l % 16, grp =
//                 l / 16) receives the scores of keys 32 kg + 8 grp + j, j = 0..3
//                 from a, 4..7 from b: exactly the B operand of the next product
//   online softmax in base 2, one row per lane column (the 4 lanes of a row
//                 exchange maxima; the sums meet at the end); the running maximum
//                 is the base-2 value that was subtracted, so that alpha fits the
//                 weights it rescales; O is rescaled only when some row's moved
//   O^T += V^T P^T  P as a bf16 hi + lo pair (|p - hi - lo| <= 2^-16 p), so PV
//                 has no bf16 rounding point; each lane keeps its own row's O,
//                 so the rescale needs no exchange
// LDS holds the operands in fragment order (64 lanes x 16 bytes), so every
// LDS access is one conflict-free 16 bytes per lane; the next block's fragments
// are loaded into registers while the current one is computed (one barrier a
// block).
//
// Bound by the vector unit and the MFMA about equally (per 16 tokens x 64 keys
// at hd 128: 48 MFMAs = 768 cycles, and 16 exponentials and about 170 other
// vector instructions).  4096 rows of 128-512-token prompts, 12 query heads:
// 36-38 us, where one block per (query row, KV head, 256-token split) and a merge
// pass took 215; three prompts of 1,100-4,590 tokens, 16 heads: 192 us a
// chunk against 873.
template <int HD, int NW>
__global__ __launch_bounds__(NW * 64, 2) void k_attn_prefill(const int4* __restrict__ tiles,
    const uint16_t* __restrict__ qbuf, const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc, int layer,
    int64_t n_blocks, int hq, int hkv, float scale_log2, uint16_t* __restrict__ out) {
  constexpr int NCC = HD / 32, NT = HD / 16;
  constexpr int KF = 4 * NCC, VF = 2 * NT, NF = KF + VF;   // 1 KiB fragments of a key block
  constexpr int FPW = (NF + NW - 1) / NW;                   // fragments a wave stages
  __shared__ u32x4 lds[2][NF][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;
  const int G = hq / hkv;
  const int g = blockIdx.x % hkv;
  const int4 tl = tiles[blockIdx.x / hkv];                  // first row, tokens, first page, first position
  const int row0 = tl.x, cnt = tl.y, t0 = tl.w;
  const int nkeys = t0 + cnt;                               // keys the tile attends (all written)
  const int nkb = (nkeys + 63) >> 6, last_page = (nkeys - 1) >> 4;
  const int head = wave % G;
  const int tb = t0 + 32 * (wave / G);                      // first token of this wave
  const bool live = tb < nkeys;
  const int last_kb = live ? (min(tb + 31, nkeys - 1) >> 6) : -1;
  // staging: fragment f < KF is K (group, operand a/b, dim step), the rest V (group, dim tile)
  const size_t kv_base = (((size_t)layer * n_blocks + tl.z) * hkv + g) * (size_t)(kBlockTok * HD);
  const int pstride = hkv * kBlockTok * HD;
  const uint16_t* src[FPW];
  int pidx[FPW];
#pragma unroll
  for (int j = 0; j < FPW; ++j) {
    const int f = min(wave + NW * j, NF - 1);
    if (f < KF) {
      const int kg = f / (2 * NCC), ab = (f / NCC) & 1, cc = f % NCC;
      const int gg = row >> 2;
      pidx[j] = 2 * kg + (gg >> 1);
      src[j] = kc + kv_base + (8 * (gg & 1) + 4 * ab + (row & 3)) * HD + 32 * cc + 8 * grp;
    } else {
      const int kg = (f - KF) / NT, t = (f - KF) % NT;
      pidx[j] = 2 * kg + (grp >> 1);
      src[j] = vc + kv_base + (16 * t + row) * kBlockTok + 8 * (grp & 1);
    }
  }
  u32x4 stg[FPW];
  auto load_block = [&](int kb) {
#pragma unroll
    for (int j = 0; j < FPW; ++j)   // pages past the last one re-read it (their keys are masked)
      stg[j] = *(const u32x4*)(src[j] + (size_t)min(4 * kb + pidx[j], last_page) * pstride);
  };
  auto store_block = [&](int buf) {
#pragma unroll
    for (int j = 0; j < FPW; ++j)
      if (wave + NW * j < NF) lds[buf][wave + NW * j][lane] = stg[j];
  };
  load_block(0);
  // q operands: token tb + 16 n + row, dims 32 cc + 8 grp
  u32x4 q[2][NCC];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int r = row0 + min(max(tb + 16 * n + row - t0, 0), cnt - 1);
    const u32x4* qp = (const u32x4*)(qbuf + ((size_t)r * hq + g * G + head) * HD + 8 * grp);
#pragma unroll
    for (int cc = 0; cc < NCC; ++cc) q[n][cc] = qp[4 * cc];
  }
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};
  f32x4 o[2][NT];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int t = 0; t < NT; ++t) o[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  store_block(0);
  __syncthreads();
  for (int kb = 0; kb < nkb; ++kb) {
    const int buf = kb & 1;
    if (kb + 1 < nkb) load_block(kb + 1);
    if (kb <= last_kb) {
      f32x4 s[2][4];                                        // [token tile][2 kg + ab]
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[0][e] = s[1][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cc = 0; cc < NCC; ++cc) {
          const bf16x8 kf = __builtin_bit_cast(bf16x8, lds[buf][e * NCC + cc][lane]);
          s[0][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, __builtin_bit_cast(bf16x8, q[0][cc]), s[0][e], 0, 0, 0);
          s[1][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, __builtin_bit_cast(bf16x8, q[1][cc]), s[1][e], 0, 0, 0);
        }
      }
      u32x4 ph[2][2], plo[2][2];                            // [token tile][kg]: 8 probabilities, hi and lo parts
      const bool diag = 64 * kb + 63 > tb;                  // some key may lie past some token
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int tq = tb + 16 * n + row;
        if (diag) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (64 * kb + 32 * (e >> 1) + 8 * grp + 4 * (e & 1) + i > tq) s[n][e][i] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          mx = fmaxf(mx, fmaxf(fmaxf(s[n][e][0], s[n][e][1]), fmaxf(s[n][e][2], s[n][e][3])));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        mx = fmaxf(m[n], mx * scale_log2);
        if (__any(mx > m[n])) {
          const float alpha = __builtin_amdgcn_exp2f(m[n] - mx);
          l[n] *= alpha;
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[n][t][i] *= alpha;
          m[n] = mx;
        }
        float ps = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < 4; i += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s[n][e][i], scale_log2, -mx));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s[n][e][i + 1], scale_log2, -mx));
            ps += p0 + p1;
            const uint32_t hi = pack_bf16(p0, p1);
            const uint32_t lo = pack_bf16(p0 - __uint_as_float(hi << 16), p1 - __uint_as_float(hi & 0xFFFF0000u));
            ph[n][e >> 1][2 * (e & 1) + (i >> 1)] = hi;
            plo[n][e >> 1][2 * (e & 1) + (i >> 1)] = lo;
          }
        l[n] += ps;
      }
      // keys at or past nkeys may hold stale bits in V: their probability is 0, the bits must be too
      const bool tail = 64 * kb + 64 > nkeys;
#pragma unroll
      for (int kg = 0; kg < 2; ++kg) {
        u32x4 vm;
        if (tail) {
          const int left = nkeys - (64 * kb + 32 * kg + 8 * grp);   // valid keys of this lane's eight
#pragma unroll
          for (int w = 0; w < 4; ++w)
            vm[w] = (left > 2 * w ? 0xFFFFu : 0u) | (left > 2 * w + 1 ? 0xFFFF0000u : 0u);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          u32x4 vw = lds[buf][KF + kg * NT + t][lane];
          if (tail) vw &= vm;
          const bf16x8 vf = __builtin_bit_cast(bf16x8, vw);
#pragma unroll
          for (int n = 0; n < 2; ++n) {
            o[n][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, ph[n][kg]), o[n][t], 0, 0, 0);
            o[n][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, plo[n][kg]), o[n][t], 0, 0, 0);
          }
        }
      }
    }
    // the other buffer was last read a block ago, before the previous barrier
    if (kb + 1 < nkb) store_block(buf ^ 1);
    __syncthreads();
  }
  if (!live) return;
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    float ls = l[n];
    ls += __shfl_xor(ls, 16, 64);
    ls += __shfl_xor(ls, 32, 64);
    const float inv = 1.0f / ls;
    // a / ls to fp32 accuracy: one correction of the product (three instructions, a division takes eleven)
    const auto over = [&](float a) { const float q = a * inv; return fmaf(fmaf(-ls, q, a), inv, q); };
    const int tq = tb + 16 * n + row;
    if (tq >= nkeys) continue;
    const int r = row0 + tq - t0, c = (g * G + head) * HD + 4 * grp;
#pragma unroll
    for (int t = 0; t < NT; ++t)
      *(uint2*)(out + tiled_index(r, c + 16 * t, hq * HD)) = make_uint2(pack_bf16(over(o[n][t][0]), over(o[n][t][1])),
                                          pack_bf16(over(o[n][t][2]), over(o[n][t][3])));
  }
}

// ---------------------------------------------------------------------------
// row norms
// ---------------------------------------------------------------------------
// x = RMSNorm(h) * w, fragment-major; EMBED: h is first gathered from the
// embedding of the row's token.  A wave takes 4 rows, 16 lanes each, a lane 8
// consecutive features at a time: 512-byte reads a row, and 64-byte runs of
// the fragment order written (4 rows x 16 bytes).  Memory bound.  KEEP: the row
// stays in registers between its two uses (up to 2048 features).
template <bool EMBED, int VPT, bool KEEP>
__global__ __launch_bounds__(256) void k_rows_norm(int M, const RowDesc* __restrict__ rows,
    const uint16_t* __restrict__ embed, float* __restrict__ h, const float* __restrict__ w, float eps,
    uint16_t* __restrict__ x) {
  constexpr int d = VPT * 128;
  const int lane = threadIdx.x & 63, j = lane & 15;
  const int i = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 4 + (lane >> 4);
  const int ic = min(i, M - 1);                          // lanes past M take part in the row exchanges only
  const uint16_t* er = EMBED ? embed + (size_t)rows[ic].tok * d : nullptr;
  float* hr = h + (size_t)ic * d;
  auto load = [&](int v, f32x4& lo, f32x4& hi) {
    const int c = 8 * (j + 16 * v);
    if constexpr (EMBED) {
      const u32x4 e = *(const u32x4*)(er + c);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        lo[2 * q] = __uint_as_float(e[q] << 16);
        lo[2 * q + 1] = __uint_as_float(e[q] & 0xFFFF0000u);
        hi[2 * q] = __uint_as_float(e[q + 2] << 16);
        hi[2 * q + 1] = __uint_as_float(e[q + 2] & 0xFFFF0000u);
      }
    } else {
      lo = *(const f32x4*)(hr + c);
      hi = *(const f32x4*)(hr + c + 4);
    }
  };
  f32x4 lo[KEEP ? VPT : 1], hi[KEEP ? VPT : 1];
  float ss = 0.f;
  if constexpr (KEEP) {
#pragma unroll
    for (int v = 0; v < VPT; ++v) load(v, lo[v], hi[v]);
#pragma unroll
    for (int v = 0; v < VPT; ++v)
#pragma unroll
      for (int q = 0; q < 4; ++q) ss += lo[v][q] * lo[v][q] + hi[v][q] * hi[v][q];
  } else {
#pragma unroll 8
    for (int v = 0; v < VPT; ++v) {
      load(v, lo[0], hi[0]);
#pragma unroll
      for (int q = 0; q < 4; ++q) ss += lo[0][q] * lo[0][q] + hi[0][q] * hi[0][q];
    }
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  if (i >= M) return;
#pragma unroll KEEP ? VPT : 4
  for (int v = 0; v < VPT; ++v) {
    const int c = 8 * (j + 16 * v);
    const int k = KEEP ? v : 0;
    if constexpr (!KEEP) load(v, lo[0], hi[0]);
    if constexpr (EMBED) {
      *(f32x4*)(hr + c) = lo[k];
      *(f32x4*)(hr + c + 4) = hi[k];
    }
    const f32x4 w0 = *(const f32x4*)(w + c), w1 = *(const f32x4*)(w + c + 4);
    u32x4 p;
    p[0] = pack_bf16(lo[k][0] * inv * w0[0], lo[k][1] * inv * w0[1]);
    p[1] = pack_bf16(lo[k][2] * inv * w0[2], lo[k][3] * inv * w0[3]);
    p[2] = pack_bf16(hi[k][0] * inv * w1[0], hi[k][1] * inv * w1[1]);
    p[3] = pack_bf16(hi[k][2] * inv * w1[2], hi[k][3] * inv * w1[3]);
    *(u32x4*)(x + tiled_index(i, c, d)) = p;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// token subgroups of 32 per tile: 5 to 8 waves whatever the group size
static int attn_subgroups(const sara_ctx* c) { return std::max(1, 8 / c->G); }

// Query tiles of every prefill chunk (consecutive rows of one prompt, tile
// starts at multiples of the tile size within the prompt or at the chunk's
// first row), longest contexts first.
void build_prefill_tiles(sara_ctx* c, const int32_t* pre) {
  const int tq = 32 * attn_subgroups(c);
  c->h_pf_tiles.clear();
  c->h_pf_tile_off.clear();
  int u = 0;
  for (int64_t r0 = 0; r0 < pre[c->U]; r0 += c->prefill_rows) {
    const int64_t r1 = std::min<int64_t>(pre[c->U], r0 + c->prefill_rows);
    c->h_pf_tile_off.push_back((int)c->h_pf_tiles.size());
    while (pre[u + 1] <= r0) ++u;
    for (int v = u; v < c->U && pre[v] < r1; ++v) {
      int64_t r = std::max<int64_t>(r0, pre[v]);
      const int64_t end = std::min<int64_t>(r1, pre[v + 1]);
      while (r < end) {
        const int t = (int)(r - pre[v]);
        const int n = (int)std::min<int64_t>(end - r, tq - t % tq);
        c->h_pf_tiles.push_back(make_int4((int)(r - r0), n, v * c->PB, t));
        r += n;
      }
    }
    std::stable_sort(c->h_pf_tiles.begin() + c->h_pf_tile_off.back(), c->h_pf_tiles.end(),
                     [](const int4& a, const int4& b) { return a.w > b.w; });
  }
  c->h_pf_tile_off.push_back((int)c->h_pf_tiles.size());
}

// upper bound of the tiles of one step
int64_t max_prefill_tiles(const sara_ctx* c) {
  const int tq = 32 * attn_subgroups(c);
  const int64_t rows = (int64_t)c->U * (c->ad.max_prompt - 1);
  return (int64_t)c->U * ((c->ad.max_prompt - 1 + tq - 1) / tq) + rows / c->prefill_rows + 1;
}

void launch_attn_prefill(sara_ctx* c, int chunk, int layer) {
  const int nt = c->h_pf_tile_off[chunk + 1] - c->h_pf_tile_off[chunk];
  const int4* tiles = c->pf_tiles + c->h_pf_tile_off[chunk];
  const float sl2 = (float)(1.4426950408889634 / sqrt((double)c->hd));
  const int nw = c->G * attn_subgroups(c);
#define SARA_AP(HD_, NW_)                                                                                     \
  launch_k(c, c->stream, (k_attn_prefill<HD_, NW_>), dim3(nt * c->hkv), dim3(NW_ * 64), 0, tiles,             \
           (const uint16_t*)c->qbuf, (const uint16_t*)c->kc, (const uint16_t*)c->vc, layer, c->n_blocks, c->hq, \
           c->hkv, sl2, (uint16_t*)c->x)
#define SARA_APH(HD_) \
  switch (nw) { case 5: SARA_AP(HD_, 5); break; case 6: SARA_AP(HD_, 6); break; \
                case 7: SARA_AP(HD_, 7); break; default: SARA_AP(HD_, 8); }
  if (c->hd == 128) { SARA_APH(128) } else { SARA_APH(64) }
#undef SARA_APH
#undef SARA_AP
}

static GemmTileArgs tile_args(const sara_ctx* c, int K) {
  GemmTileArgs a{};
  a.steps = K / 32;
  a.xa = (uint16_t*)c->xa;
  a.rows = c->rows;
  a.rope = c->rope;
  a.qbuf = (uint16_t*)c->qbuf;
  a.kc = (uint16_t*)c->kc;
  a.vc = (uint16_t*)c->vc;
  a.hq = c->hq;
  a.hkv = c->hkv;
  a.n_blocks = c->n_blocks;
  return a;
}

// Whether a GEMM without K splits runs on b 256 x 256 tiles rather than on the
// decode GEMMs' 128 x 128 blocks.  Per 32-wide k step a round of up to 256 tiles takes
// about 0.7 us, the small blocks 0.4 us until the GPU is full and then 0.0054 us a
// tile's worth of them (measured at 1536 -> 17920: 70 tiles 36 us against 25,
// 140 tiles 39 against 42, 280 tiles 76 against 78, 560 tiles 119 against 150).
static bool tiles_pay(int b) { return 0.7 * ((b + 255) / 256) < std::max(0.4, 0.0054 * b); }

// q|k|v of the chunk to qbuf and the KV pages.  kv_only: the last layer's
// queries are not needed (nothing follows its K and V in a prefill).
static void prefill_qkv(sara_ctx* c, const int32_t* M_ptr, int M, int l, bool kv_only) {
  // the small blocks need a pass over fp32 partials for the rotary epilogue:
  // at 64 tiles (2048 rows of 8 column tiles) 57 us with it against 48
  if (tile_blocks(M, c->nqkv) >= 64 || (int64_t)M * c->nqkv > c->ws_floats) {
    GemmTileArgs a = tile_args(c, c->d);
    a.layer = l;
    a.tile0 = kv_only ? c->qdim / 16 : 0;
    if (c->hd == 64) gemm_tile<3>(c, c->x, c->w_qkv[l], M, c->nqkv, c->d, a);
    else gemm_tile<4>(c, c->x, c->w_qkv[l], M, c->nqkv, c->d, a);
    return;
  }
  int sp = 1;
  gemm_bf16(c, c->x, c->w_qkv[l], M_ptr, M, c->nqkv, c->d, sp);
  launch_qkv_epilogue_bf16(c, M_ptr, M, sp, l);
}

// h += X W^T (N = d_model).  Returns the K splits left in ws for the following
// norm to add, 0 when h is complete.
static int prefill_add(sara_ctx* c, const void* X, const void* W, const int32_t* M_ptr, int M, int K) {
  const int b = tile_blocks(M, c->d);
  GemmTileArgs a = tile_args(c, K);
  // Few tiles: the decode GEMMs' blocks with their K splits, below 48 tiles (24
  // for a long K, where each split keeps enough steps to pay for its
  // partials: 24 tiles of 8960 -> 1536 at 1024 rows 45 us against 72).
  if (b < (K >= 4096 ? 24 : 48) && (int64_t)M * c->d <= c->ws_floats) {
    int sp = 1;
    gemm_bf16(c, X, W, M_ptr, M, c->d, K, sp);
    return sp;
  }
  // Otherwise as many splits as keep one round of tiles, at least 16 steps
  // each, while the partials fit.
  int splits = std::min({256 / b, K / 32 / 16, kMaxSplitsDec});
  splits = (int)std::min<int64_t>(splits, c->ws_floats / ((int64_t)M * c->d));
  if (splits <= 1) {
    a.out = c->h;
    gemm_tile<2>(c, X, W, M, c->d, K, a);
    return 0;
  }
  a.out = c->ws;
  a.split_stride = (int64_t)M * c->d;
  const int pairs = K / 64;
  a.steps = 2 * ((pairs + splits - 1) / splits);
  gemm_tile<0>(c, X, W, M, c->d, K, a);
  return (K / 32 + a.steps - 1) / a.steps;
}

template <bool EMBED>
static void rows_norm(sara_ctx* c, int M, const float* w) {
  const dim3 grid((M + 15) / 16);
#define SARA_RN(V_, K_)                                                                                          \
  launch_k(c, c->stream, (k_rows_norm<EMBED, V_, K_>), grid, dim3(256), 0, M, (const RowDesc*)c->rows,           \
           (const uint16_t*)c->embed, c->h, w, c->md.rms_eps, (uint16_t*)c->x)
  switch (c->d / 128) {
    case 4: SARA_RN(4, true); break;
    case 8: SARA_RN(8, true); break;
    case 12: SARA_RN(12, true); break;
    case 16: SARA_RN(16, true); break;
    case 24: SARA_RN(24, false); break;
    default: SARA_RN(32, false); break;
  }
#undef SARA_RN
}

// The M prompt-token rows of a chunk (described in c->rows) through every
// layer, up to the K and V of the last one: its attention and FFN have no
// reader.
void prefill_layers_bf16(sara_ctx* c, const int32_t* M_ptr, int M, int chunk) {
  const size_t d = c->d;
  rows_norm<true>(c, M, c->norms);
  for (int l = 0;; ++l) {
    const bool last = l + 1 == c->L;
    prefill_qkv(c, M_ptr, M, l, last);
    if (last) break;
    launch_attn_prefill(c, chunk, l);
    int sp = prefill_add(c, c->x, c->w_o[l], M_ptr, M, c->qdim);
    const float* nw = c->norms + (2 * l + 1) * d;
    if (sp) residual_norm_bf16(c, M_ptr, M, sp, nw);
    else rows_norm<false>(c, M, nw);
    if (tiles_pay(tile_blocks(M, 2 * c->ffn))) {
      gemm_tile<1>(c, c->x, c->w_gu[l], M, 2 * c->ffn, c->d, tile_args(c, c->d));
    } else {
      gemm_swiglu(c, c->x, c->w_gu[l], M_ptr, M);
    }
    sp = prefill_add(c, c->xa, c->w_d[l], M_ptr, M, c->ffn);
    nw = c->norms + (2 * l + 2) * d;
    if (sp) residual_norm_bf16(c, M_ptr, M, sp, nw);
    else rows_norm<false>(c, M, nw);
  }
}

}  // namespace sara
