// Prefill of the bf16 models (gfx950): a chunk of prompt tokens through the
// decoder layers.  GEMM inputs are fragment-major (tiled_index), GEMM weights
// k-block-major fragments (wtiled_index), so both operands of a GEMM move to
// LDS as contiguous 1 KiB fragments.
#include <math.h>

#include <algorithm>

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
//                 exchange maxima; the sums meet at the end); O is rescaled
//                 only when some row's maximum moved
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
// 36 us, where one block per (query row, KV head, 256-token split) and a merge
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
        float mx = m[n];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          mx = fmaxf(mx, fmaxf(fmaxf(s[n][e][0], s[n][e][1]), fmaxf(s[n][e][2], s[n][e][3])));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if (__any(mx > m[n])) {
          const float alpha = __builtin_amdgcn_exp2f((m[n] - mx) * scale_log2);
          l[n] *= alpha;
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[n][t][i] *= alpha;
          m[n] = mx;
        }
        const float mc = mx * scale_log2;
        float ps = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < 4; i += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s[n][e][i], scale_log2, -mc));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s[n][e][i + 1], scale_log2, -mc));
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
    const int tq = tb + 16 * n + row;
    if (tq >= nkeys) continue;
    const int r = row0 + tq - t0, c = (g * G + head) * HD + 4 * grp;
#pragma unroll
    for (int t = 0; t < NT; ++t)
      *(uint2*)(out + tiled_index(r, c + 16 * t, hq * HD)) = make_uint2(pack_bf16(o[n][t][0] * inv, o[n][t][1] * inv),
                                          pack_bf16(o[n][t][2] * inv, o[n][t][3] * inv));
  }
}

// ---------------------------------------------------------------------------
// GEMM over full tiles
// ---------------------------------------------------------------------------
// out = X W^T on 256 x 256 tiles: 8 waves of 128 rows x 64 weight rows
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation in k order, as the decode
// GEMMs).  Both operands go from memory straight to LDS (global_load_lds, 16
// bytes a lane, fragment order, so the reads are conflict-free) through a ring
// of four 32-wide k stages of 32 KiB.  The waves form two groups, one wave of
// each on every SIMD, that run half a step apart: while one group's MFMAs
// run, the other reads its fragments of the stage and issues loads three
// stages ahead.  Between the phases stands one barrier.
//
// Ring bookkeeping, in phases (group 0 reads stage s in phase 2s, group 1 in
// phase 2s + 1): stage s + 3 is issued in the phase that reads stage s, into
// the slot that stage s - 1 left, last read in phase 2s - 1; every wave waits
// for its own loads of stage s + 1 before the barrier that ends its reading
// phase of stage s, at the latest phase 2s + 1, and stage s + 1 is first read in
// phase 2s + 2.  Past the last stage the loads repeat it into slots that nobody
// reads, so the count of outstanding loads stays exact.
//
// Bound by the matrix cores (and their clock under load): 1.3-1.4 PFLOP/s on
// the prefill shapes (16384^3 library product: 1.6), where 128 x 128 tiles with
// register-staged activations reached 0.57-0.82 and all eight waves in phase on
// the same ring 0.80-0.91.
//
// EPI 0: fp32 partials of K split blockIdx.y to ws[split][M][N].
// EPI 1: SwiGLU over the gate / up tile pairs, fragment-major bf16 [M][N / 2].
// EPI 2: h += out (fp32 residual stream [M][N]).
// EPI 3, 4: q|k|v at head width 64, 128: rotate-half RoPE, q as bf16, k and v to
//           the rows' KV pages (weight rows in rotation-pair order, qkv_pair_col).
struct GemmTileArgs {
  float* out;              // ws or h
  uint16_t* xa;            // EPI 1
  int64_t split_stride;    // EPI 0
  int steps;               // 32-wide k steps per split
  int tile0;               // first 16-row weight tile
  // EPI 3, 4
  const RowDesc* rows;
  const float2* rope;
  uint16_t *qbuf, *kc, *vc;
  int hq, hkv, layer;
  int64_t n_blocks;
};

template <int EPI>
__global__ __launch_bounds__(512, 2) void k_gemm_tile(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
    int M, int N, int K, GemmTileArgs a) {
  constexpr int MT = 8, NT = 4, NW = 8, XF = 2 * MT, NF = XF + 4 * NT, FPW = NF / NW, ST = 4;
  __shared__ u32x4 lds[ST * NF * 64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;
  const int wm = wave >> 2, wn = wave & 3;
  const int ntl = N >> 4, mtl = (M + 15) >> 4;          // 16-row tiles
  // Block -> tile: ids are dealt to the 8 XCDs in turn; each XCD takes a
  // contiguous stretch of an order that walks 4 row tiles by every column
  // tile, so that the 32 blocks running at once on an XCD share few X and W
  // tiles in its L2 (4 x 8: gate|up 1.36 PFLOP/s; 8 x 4 1.34, row tiles alone
  // 1.20).
  int bn, bm;
  {
    const int nb = (ntl - a.tile0 + 15) >> 4, mb = (mtl + 15) >> 4, total = nb * mb;
    const int x = blockIdx.x & 7, per = total >> 3, rem = total & 7;
    const int lin = x * per + min(x, rem) + (blockIdx.x >> 3);
    const int gs = 4 * nb, g = lin / gs, gm = min(4, mb - 4 * g), r = lin - g * gs;
    bm = 4 * g + r % gm;
    bn = r / gm;
  }
  const int tn0 = a.tile0 + 16 * bn, tm0 = 16 * bm;
  const int s0 = blockIdx.y * a.steps;                   // an even step: k blocks are two steps
  const int ns = min(a.steps, (K >> 5) - s0);
  // this wave's FPW fragments of a stage (rows and columns past the end repeat the last tile)
  const uint16_t* base[FPW];
  int blk[FPW];                                          // elements per 64-wide k block
#pragma unroll
  for (int j = 0; j < FPW; ++j) {
    const int f = wave * FPW + j;
    if (f < XF) {
      base[j] = X + ((size_t)min(tm0 + f, mtl - 1) * (K >> 5) + s0) * 512 + lane * 8;
      blk[j] = 1024;
    } else {
      base[j] = W + ((size_t)(s0 >> 1) * ntl + min(tn0 + f - XF, ntl - 1)) * 1024 + lane * 8;
      blk[j] = ntl * 1024;
    }
  }
  auto issue = [&](int s) {
    const int sc = min(s, ns - 1), slot = s % ST;
#pragma unroll
    for (int j = 0; j < FPW; ++j) {
      const uint16_t* p = base[j] + (size_t)(sc >> 1) * blk[j] + (sc & 1) * 512;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                       (__attribute__((address_space(3))) void*)&lds[(slot * NF + wave * FPW + j) * 64],
                                       16, 0, 0);
    }
  };
  // a phase boundary: nothing moves across it
  auto phase = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  f32x4 acc[NT][MT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[n][m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < ST - 1; ++s) issue(s);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ST - 2) * FPW) : "memory");   // stage 0 has landed
  phase();
  if (wave >= 4) phase();                                // the second group runs one phase behind
  for (int s = 0; s < ns; ++s) {
    const u32x4* st = &lds[(s % ST) * NF * 64];
    bf16x8 wf[NT], xf[MT];
#pragma unroll
    for (int n = 0; n < NT; ++n) wf[n] = __builtin_bit_cast(bf16x8, st[(XF + wn * NT + n) * 64 + lane]);
#pragma unroll
    for (int m = 0; m < MT; ++m) xf[m] = __builtin_bit_cast(bf16x8, st[(wm * MT + m) * 64 + lane]);
    issue(s + ST - 1);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((ST - 2) * FPW) : "memory");   // stage s + 1 has landed
    phase();
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[n], xf[m], acc[n][m], 0, 0, 0);
    phase();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the repeated loads, before the block gives its LDS back
  if (wave < 4) phase();
  // lane (row, grp) of acc[n][m]: row 16 m + row of this wave's half, columns 16 n + 4 grp ..+3 of its quarter
  const int tn = tn0 + wn * NT, m0 = (tm0 + wm * MT) * 16 + row;
  if constexpr (EPI == 0 || EPI == 2) {
    float* o = a.out + (EPI == 0 ? (size_t)blockIdx.y * a.split_stride : 0);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      if (m0 + 16 * m >= M) continue;
      float* orow = o + (size_t)(m0 + 16 * m) * N + tn * 16 + 4 * grp;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        if (tn + n >= ntl) continue;
        f32x4 v = acc[n][m];
        if constexpr (EPI == 2) v = *(const f32x4*)(orow + 16 * n) + v;
        *(f32x4*)(orow + 16 * n) = v;
      }
    }
  } else if constexpr (EPI == 1) {
    const int F = N >> 1;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      if (m0 + 16 * m >= M) continue;
#pragma unroll
      for (int n = 0; n < NT; n += 2) {
        if (tn + n >= ntl) continue;
        float r[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float g = acc[n][m][q], u = acc[n + 1][m][q];
          r[q] = g * u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
        }
        *(uint2*)(a.xa + tiled_index(m0 + 16 * m, (tn + n) * 8 + 4 * grp, F)) =
            make_uint2(pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3]));
      }
    }
  } else {
    // the wave's 64 columns lie in one head
    constexpr int HD = EPI == 3 ? 64 : 128, half = HD / 2;
    if (tn >= ntl) return;
    const int h = tn * 16 / HD, j0 = tn % (HD / 16);
    const int lo = grp & 1;
    const bool second = grp >= 2;
    const int nd = (second ? half : 0) + 8 * j0 + 4 * lo;   // natural dim of the lane's first element of n = 0
    if (h < a.hq + a.hkv) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const int mm = min(m0 + 16 * m, M - 1);
        const int pos = a.rows[mm].pos, kv0 = a.rows[mm].kv0;
        const f32x4* cs = (const f32x4*)(a.rope + (size_t)pos * half + 8 * j0 + 4 * lo);
        uint16_t* dst = h < a.hq
            ? a.qbuf + ((size_t)mm * a.hq + h) * HD
            : a.kc + ((((size_t)a.layer * a.n_blocks + kv0 + (pos >> 4)) * a.hkv + (h - a.hq)) * kBlockTok + (pos & 15)) * HD;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const f32x4 c01 = cs[4 * n], c23 = cs[4 * n + 1];   // (cos, sin) of four rotation indices
          const f32x4 v = acc[n][m];
          f32x4 pv;
#pragma unroll
          for (int q = 0; q < 4; ++q) pv[q] = __shfl_xor(v[q], 32, 64);
          if (!second) pv = -pv;
          const uint2 o = make_uint2(pack_bf16(v[0] * c01[0] + pv[0] * c01[1], v[1] * c01[2] + pv[1] * c01[3]),
                                     pack_bf16(v[2] * c23[0] + pv[2] * c23[1], v[3] * c23[2] + pv[3] * c23[3]));
          if (m0 + 16 * m < M) *(uint2*)(dst + nd + 8 * n) = o;
        }
      }
    } else {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const int mm = min(m0 + 16 * m, M - 1);
        const int pos = a.rows[mm].pos, kv0 = a.rows[mm].kv0;
        if (m0 + 16 * m >= M) continue;
        uint16_t* vp = a.vc + (((size_t)a.layer * a.n_blocks + kv0 + (pos >> 4)) * a.hkv + (h - a.hq - a.hkv)) *
                                  (size_t)(HD * kBlockTok) + nd * kBlockTok + (pos & 15);
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const uint32_t p01 = pack_bf16(acc[n][m][0], acc[n][m][1]), p23 = pack_bf16(acc[n][m][2], acc[n][m][3]);
          vp[(8 * n + 0) * kBlockTok] = (uint16_t)(p01 & 0xFFFF);
          vp[(8 * n + 1) * kBlockTok] = (uint16_t)(p01 >> 16);
          vp[(8 * n + 2) * kBlockTok] = (uint16_t)(p23 & 0xFFFF);
          vp[(8 * n + 3) * kBlockTok] = (uint16_t)(p23 >> 16);
        }
      }
    }
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

static int tile_blocks(int M, int N) { return ((M + 255) / 256) * ((N + 255) / 256); }

// Whether a GEMM without K splits runs on b 256 x 256 tiles rather than on the
// decode GEMMs' 128 x 128 blocks.  Per 32-wide k step a round of up to 256 tiles takes
// about 0.7 us, the small blocks 0.4 us until the GPU is full and then 0.0054 us a
// tile's worth of them (measured at 1536 -> 17920: 70 tiles 36 us against 25,
// 140 tiles 39 against 42, 280 tiles 76 against 78, 560 tiles 119 against 150).
static bool tiles_pay(int b) { return 0.7 * ((b + 255) / 256) < std::max(0.4, 0.0054 * b); }

template <int EPI>
static void gemm_tile(sara_ctx* c, const void* X, const void* W, int M, int N, int K, const GemmTileArgs& a) {
  launch_k(c, c->stream, (k_gemm_tile<EPI>), dim3(tile_blocks(M, N - 16 * a.tile0), (K / 32 + a.steps - 1) / a.steps),
           dim3(512), 0, (const uint16_t*)X, (const uint16_t*)W, M, N, K, a);
}

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
