// The 256 x 256 tile GEMM of the bf16 models: every prefill projection of a long
// chunk, and the many-row loop of decode.
#pragma once

#include "sara_internal.h"

namespace sara {

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
// Rows: M of the launch, or (decode, M_ptr set) the live row count read on the
// device; blocks past the live tiles exit at once.  Every output's k order is
// the decode GEMMs' (gemm_mblock), so with the same K splits the results are
// bit-identical to theirs and a row's do not depend on which kernel ran.
//
// Bound by the matrix cores (and their clock under load): 1.2-1.3 PFLOP/s on
// the prefill shapes (16384^3 library product: 1.6; gate|up of 80,000 rows, 1536
// wide: 1.25, a tenth of it the SwiGLU epilogue), where 128 x 128 tiles with
// register-staged activations reached 0.57-0.82 and all eight waves in phase on
// the same ring 0.80-0.91.
//
// EPI 0: fp32 partials of K split blockIdx.y to ws[split][M][N].
// EPI 1: SwiGLU over the gate / up tile pairs, bf16 [M][N / 2], fragment-major like X.
// EPI 2: h += out (fp32 residual stream [M][N]).
// EPI 3, 4: q|k|v at head width 64, 128: rotate-half RoPE, q as bf16, k and v to
//           the rows' KV pages (weight rows in rotation-pair order, qkv_pair_col).
// EPI 5: Gumbel-max over the tile's 256 vocabulary ids (see sample_round).
struct GemmTileArgs {
  const int32_t* M_ptr;    // decode: live rows; null: M of the launch
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
  SampleArgs sample;       // EPI 5
};

template <int NT, int MT, int TC, int T0, bool UNIT>
__device__ __forceinline__ void sample_round(const f32x4 (&acc)[NT][MT], int M, int m_base, int N, int n0,
    const SampleArgs& sa, float temp, uint32_t k0, uint32_t k1, void* xs, int wn, int tid, int chunk);

template <int EPI>
__global__ __launch_bounds__(512, 2) void k_gemm_tile(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
    int M, int N, int K, GemmTileArgs a) {
  constexpr int MT = 8, NT = 4, NW = 8, XF = 2 * MT, NF = XF + 4 * NT, FPW = NF / NW, ST = 4;
  __shared__ u32x4 lds[ST * NF * 64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;
  const int wm = wave >> 2, wn = wave & 3;
  if (a.M_ptr) M = *a.M_ptr;
  const int ntl = N >> 4, mtl = (M + 15) >> 4;          // 16-row tiles
  // Block -> tile: ids are dealt to the 8 XCDs in turn; each XCD takes a
  // contiguous stretch of an order that walks 4 row tiles by every column
  // tile, so that the 32 blocks running at once on an XCD share few X and W
  // tiles in its L2 (gate|up with a shorter SwiGLU: 4 x 8 1.36 PFLOP/s; 8 x 4 1.34,
  // row tiles alone 1.20).
  int bn, bm;
  {
    const int nb = (ntl - a.tile0 + 15) >> 4, mb = (mtl + 15) >> 4, total = nb * mb;
    if ((int)blockIdx.x >= total) return;
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
      const int tile = min(tm0 + f, mtl - 1);
      base[j] = X + ((size_t)tile * (K >> 5) + s0) * 512 + lane * 8;   // rows past M are dropped
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
        const f32x4 r = silu_mul(acc[n][m], acc[n + 1][m]);
        *(uint2*)(a.xa + tiled_index(m0 + 16 * m, (tn + n) * 8 + 4 * grp, F)) =
            make_uint2(pack_bf16(r[0], r[1]), pack_bf16(r[2], r[3]));
      }
    }
  } else if constexpr (EPI == 5) {
    // a row tile a round (more spill); the four waves of a row half meet in LDS
    const CtlParams* cp = a.sample.cp;
    const float temp = cp->temperature;
    uint32_t k0, k1;
    sampler_key(cp->seed, cp->step, k0, k1);
    const int m_base = (tm0 + wm * MT) * 16, tid = threadIdx.x & 255;
    void* red = (char*)lds + wm * 8192;
#define SARA_TS(r, U) sample_round<NT, MT, 1, r, U>(acc, M, m_base, N, tn * 16, a.sample, temp, k0, k1, red, wn, tid, bn);
#define SARA_TS8(U) SARA_TS(0, U) SARA_TS(1, U) SARA_TS(2, U) SARA_TS(3, U) SARA_TS(4, U) SARA_TS(5, U) SARA_TS(6, U) SARA_TS(7, U)
    if (temp == 1.0f) { SARA_TS8(true) } else { SARA_TS8(false) }
#undef SARA_TS8
#undef SARA_TS
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


// tiles of an M x N output, and the launch
inline int tile_blocks(int M, int N) { return ((M + 255) / 256) * ((N + 255) / 256); }

template <int EPI>
static void gemm_tile(sara_ctx* c, const void* X, const void* W, int M, int N, int K, const GemmTileArgs& a) {
  launch_k(c, c->stream, (k_gemm_tile<EPI>),
           dim3(tile_blocks(M, N - 16 * a.tile0), (K / 32 + a.steps - 1) / a.steps), dim3(512), 0, (const uint16_t*)X,
           (const uint16_t*)W, M, N, K, a);
}

}  // namespace sara
