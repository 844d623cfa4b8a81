// Internal declarations of libsara (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/sara.h"

namespace sara {

// ---------------------------------------------------------------------------
// constants
// ---------------------------------------------------------------------------
constexpr int kBlockTok = 16;        // KV page size in tokens
constexpr int kAttnSplit = 256;      // tokens per context split (fp32 VALU attention)
constexpr int kDecPpw = 2;           // KV pages per wave in the decode attention
constexpr int kDecPages = 4 * kDecPpw;  // KV pages per context split in the decode attention
constexpr int kMaxSplitsDec = 12;    // split-K partials of a decode GEMM (summed in one batch; a multiple of 4)
constexpr int kPrefillRows = 4096;   // rows of a prefill chunk
constexpr int kPrefillRowsBf16 = 32768;  // most rows of one of a bf16 model, where memory allows
constexpr int kAttnTile = 64;        // tokens per LDS tile inside a split
constexpr int kSampleChunks = 16;    // vocabulary chunks per sampled row
constexpr int kTopPChunks = 16;      // vocabulary chunks per row in the top-p passes
constexpr int kTopPBins = 2048;      // 11-bit digits of the top-p radix descent
// static scratch of the allocation-free sampler (sara_sample_logits_noalloc)
constexpr int kNoAllocMaxRows = SARA_NOALLOC_MAX_ROWS;
constexpr int kNoAllocMaxToppRows = SARA_NOALLOC_MAX_TOPP_ROWS;
constexpr size_t kNoAllocScratchBytes = SARA_NOALLOC_SCRATCH_BYTES;
constexpr int kCtlThreads = 1024;    // threads of the single-workgroup controller
constexpr int kMaxQueue = 4096;      // pending rollouts held in LDS by the refill
constexpr int kMaxSlots = 4096;
constexpr int kMaxGroup = 8;         // query heads per KV head
constexpr uint64_t kSeedRXor = 0xD1B54A32D192ED03ull;

// ---------------------------------------------------------------------------
// device-side state
// ---------------------------------------------------------------------------
struct Ctl {
  int64_t budget_left, rollouts, tokens;
  int64_t n_dec, n_draw, n_asg, n_fin;
  int32_t next_uid, nA, nC, nAb;
  int32_t qlen, t, done, error;
  int32_t M, dirty, running, pad_;
};

// One query row of a decode or prefill batch.
struct RowDesc {
  int32_t tok;      // input token id
  int32_t pos;      // position of the token (KV append position)
  int32_t plen;     // tokens of the sequence's shared prompt segment (P - 1)
  int32_t slot;     // decode: slot index; prefill: -1
  int32_t rid;      // decode: rollout id uid*k + j
  int32_t gen;      // decode: generated index i
  int32_t uid;
  // KV extents: page ids of a sequence are kv0 + e for its shared prompt
  // segment and kv1 + e for its private segment (decode rows; -1 for prefill
  // rows)
  int32_t kv0;
  int32_t kv1;
};

// An occupied slot, ascending (rebuilt by the refill when slots change): what
// a decode step needs of it besides its generated count and next input token.
struct ActiveRow {
  int32_t slot, uid, j, plen;   // plen: tokens of the shared prompt segment (P - 1)
};

// One work item of the decode attention: context split c of decode row i,
// with the row's page extents and segment lengths, so that an attention
// block needs no further load before its page loads.  n > 1: a split that lies
// wholly in the prompt segment of n rows of one prompt, places i .. i + n - 1 of
// the prompt order.
struct AttnItem {
  int32_t i, c, kv0, kv1;   // row (or place), split, page extents (as in RowDesc)
  int32_t pl, vcnt, n, pad; // prompt positions attended, private positions, rows
};

// One place of the live rows ordered by prompt (rebuilt with the active rows):
// the row, its rank among the rows of its prompt, and how many those are.
struct PromptPlace {
  uint16_t row, rank;
  int32_t n;
};

struct CtlParams;
// Operands of the LM-head GEMM's sampling epilogue.
struct SampleArgs {
  const RowDesc* rows;       // decode rows (rid, gen, slot)
  const CtlParams* cp;       // seed, step index, temperature
  float* logits;             // optional [slots][V] copy of the logits (parity runs), else null
  float* best;               // [vocabulary block][ld] exact best score of the block's ids per row
  int32_t* idx;              // [vocabulary block][ld] its token id
  int ld;                    // row stride of best / idx (>= the live row count)
};

// Parameters every controller kernel reads.
struct CtlParams {
  int32_t B, k, n0, commit_min, U, S, mode, bits, max_new, PB, SB, MAXB, eos, Qcap;
  double tau, a0, b0, prior;
  uint64_t seed;
  int32_t step;
  uint32_t forced_eos;
  float temperature;
  float top_p;                   // < 1: nucleus sampling over fp32 logits
  int32_t has_flen;
  int32_t has_prior;             // per-prompt priors (warm start) in place of (a0, b0, prior)
};

}  // namespace sara

// ---------------------------------------------------------------------------
// host-side context
// ---------------------------------------------------------------------------
struct sara_ctx {
  sara_model_desc md;
  sara_alloc_desc ad;
  hipStream_t stream = nullptr;
  int device = 0;

  // derived sizes
  int L = 0, d = 0, hq = 0, hkv = 0, hd = 0, ffn = 0, V = 0, G = 0, nqkv = 0, qdim = 0;
  int U = 0, k = 0, S = 0, PB = 0, SB = 0, MAXB = 0, max_pos = 0, Qcap = 0;
  int64_t n_blocks = 0;
  int elt = 2;                    // bytes per stored element (2 bf16, 4 fp32)
  int prefill_rows = 0;           // rows per prefill chunk
  int attn_splits_max = 0;
  int dec_splits_max = 0;         // context splits of the decode attention
  int64_t ws_floats = 0;

  // weights (model dtype)
  void* embed = nullptr;
  void* lm_head = nullptr;
  std::vector<void*> w_qkv, w_o, w_gu, w_d;
  float* norms = nullptr;         // [2L+1][d]: attn l, ffn l, final

  // KV cache [L][n_blocks][hkv][16][hd] (V transposed, [hd][16])
  void* kc = nullptr;
  void* vc = nullptr;
  float2* rope = nullptr;         // [max_pos][hd/2] (cos, sin)
  float2* row_rope = nullptr;     // [S][hd/2] (cos, sin) at each decode row's position
  sara::AttnItem* attn_items = nullptr; // [S * dec_splits_max] decode attention work list of the step
  int32_t* attn_nitems = nullptr; // its length
  int attn_dec_grid = 0;          // blocks of the decode attention that are resident at once
  int qkv_spread = 0;             // z blocks sharing a decode batch's tiles in the q|k|v kernel

  // prompt pool (library copies)
  int32_t* tok = nullptr;
  int32_t* off = nullptr;         // [U+1]
  int32_t* pre = nullptr;         // [U+1] prefix sums of (P - 1)
  double* p = nullptr;
  int32_t* flen = nullptr;        // [U*k]
  int has_flen = 0;
  int64_t tok_cap = 0;
  std::vector<int32_t> h_off;
  // query tiles of the prefill attention (bf16 models): (first row in the
  // chunk, tokens, first page, first position); chunk i owns
  // [h_pf_tile_off[i], h_pf_tile_off[i + 1])
  int4* pf_tiles = nullptr;
  std::vector<int4> h_pf_tiles;
  std::vector<int> h_pf_tile_off;

  // controller state
  sara::Ctl* ctl = nullptr;
  int32_t *status = nullptr, *n_iss = nullptr, *n_done = nullptr, *succ = nullptr, *infl = nullptr;
  double* peff = nullptr;
  // history warm start: per-prompt priors of the pool ([U] each) and the
  // caller's prompt-set state (set by sara_set_warm_start)
  double *prior_a = nullptr, *prior_b = nullptr, *prior_p = nullptr;
  const int32_t* warm_ids = nullptr;
  double *warm_a = nullptr, *warm_b = nullptr;
  int32_t warm_n = 0;
  bool warm_step = false;         // the current step began with warm start set
  int32_t *slot_uid = nullptr, *slot_j = nullptr, *slot_gen = nullptr, *fin = nullptr;
  uint64_t* slot_hash = nullptr;
  sara::ActiveRow* active = nullptr;
  sara::PromptPlace* places = nullptr;  // [S] live rows by prompt (bf16 models)
  int32_t *grp_n = nullptr, *grp_at = nullptr;  // [U] live rows of a prompt, its first place
  int32_t* slot_tok = nullptr;    // input token of the slot's next decode step
  uint64_t* queue = nullptr;
  int32_t *out_tok = nullptr, *samp_tok = nullptr, *r_len = nullptr, *r_reward = nullptr;
  int64_t *log_dec = nullptr, *log_draw = nullptr, *log_asg = nullptr, *log_fin = nullptr;
  int64_t cap_dec = 0, cap_draw = 0, cap_asg = 0, cap_fin = 0;

  // activations and workspaces
  sara::RowDesc* rows = nullptr;  // [row_cap]
  int32_t* rows_M = nullptr;      // device row count of the prefill chunk
  int row_cap = 0;
  float* h = nullptr;             // [row_cap][d] residual stream
  void* x = nullptr;              // [row_cap][max(d, qdim)] GEMM input (model dtype)
  void* qbuf = nullptr;           // [row_cap][hq][hd]
  void* xa = nullptr;             // [row_cap][ffn] SwiGLU output (model dtype)
  float* ws = nullptr;            // GEMM partial outputs
  float* attn_part = nullptr;
  float* samp_best = nullptr;
  int32_t* samp_idx = nullptr;
  bool topp = false;              // top_p < 1: nucleus sampler after the LM head
  float* topp_logits = nullptr;   // [S][V] fp32 logits for it (bf16 models)
  float* topp_max = nullptr;      // [S][kTopPChunks] chunk maxima of z
  unsigned long long* topp_hist = nullptr;   // [S][kTopPChunks][kTopPBins] chunk weight histograms
  uint32_t* topp_thr = nullptr;   // [S] key bits of each row's nucleus threshold z* (all of them at the end)
  unsigned long long* topp_above = nullptr;    // [S] weight above the descent's current range
  unsigned long long* topp_target = nullptr;   // [S] target weight t

  // GRPO of committed groups
  int32_t* g_off = nullptr;
  float* g_r = nullptr;
  float* g_adv = nullptr;
  int32_t* g_n = nullptr;         // committed count used for the CSR

  // graph replay: the loop captured with the few-row kernels [0] and, for
  // batches of more than many_rows live rows, the 256 x 256 tile GEMMs [1]
  struct LoopGraph {
    hipGraphExec_t exec = nullptr;
    hipGraph_t graph = nullptr;
    int iters = 0;
  } loop_graph[2];
  int run_M = 0;                  // live rows as last known to the host
  int many_rows = 0;
  bool tile_rows = false;         // launch_decode uses the tile GEMMs (capture of loop_graph[1])
  // forced-token table of the current sara_run, read through memory: the graphs
  // serve every table
  const int32_t** forced_dev = nullptr;
  struct Poll {
    int32_t done[6];              // 2 x (done flag, error word, live rows)
    const int32_t* forced;        // the table of the current sara_run
  };
  Poll* h_poll = nullptr;         // pinned

  std::vector<void*> owned;       // device allocations freed by sara_destroy
  // per-launch profiling of eager decode steps
  struct ProfRec { int cls, N, K, e0, e1; };
  bool prof_enabled = false;
  bool prof_active = false;
  bool capturing = false;
  bool in_prefill = false;
  std::vector<hipEvent_t> prof_events;
  std::vector<ProfRec> prof_recs;
  int prof_next_event = 0;
  int prof_pending = -1;          // event pair reserved for the next launch (-1: none)
  int prof_last = -1;             // event pair of the last profiled launch
  std::vector<sara_kernel_profile> prof_tot;
  sara::CtlParams cp;              // host copy
  sara::CtlParams* cp_dev = nullptr;
  int step_index = 0;
  bool in_step = false;
};

namespace sara {

// one class per kernel (per template instance for the GEMMs, as a kernel
// trace names them), then a breakdown of the GEMMs by weight matrix
enum ProfClass { kPGemmN1, kPGemmGU, kPGemmLM, kPAttn, kPCombine, kPResNorm,
                 kPEmbed, kPSampleP, kPSampleF, kPCopy, kPQkvRope, kPToppMax, kPToppHist, kPToppSel,
                 kPGemmO1, kPGemmQkv, kPGemmO, kPGemmGu, kPGemmD, kPGemmLm, kPNumClasses };
extern const char* const kProfNames[kPNumClasses];
void prof_begin(sara_ctx* c);
void prof_end(sara_ctx* c, int cls, int N = 0, int K = 0);
int prof_collect(sara_ctx* c);

void set_error(const std::string& msg);
int hip_fail(hipError_t e, const char* what);

// Kernel launch on a context's stream.  While a per-kernel profile record is
// open (prof_begin), the launch goes through hipExtLaunchKernelGGL with the
// record's event pair, so the dispatch itself stamps the kernel's start and
// end: the elapsed time is the kernel's own duration, as in a kernel trace.
template <typename F, typename... Args>
static void launch_k(sara_ctx* c, hipStream_t st, F kernel, dim3 grid, dim3 block, uint32_t shm, Args... args) {
  const int p = c->prof_pending;
  if (p >= 0) {
    c->prof_pending = -1;
    c->prof_last = p;
    hipExtLaunchKernelGGL(kernel, grid, block, shm, st, c->prof_events[p], c->prof_events[p + 1], 0u, args...);
  } else {
    hipLaunchKernelGGL(kernel, grid, block, shm, st, args...);
  }
}

// launchers (prefill of bf16 models)
void build_prefill_tiles(sara_ctx* c, const int32_t* pre);
int64_t max_prefill_tiles(const sara_ctx* c);
void prefill_layers_bf16(sara_ctx* c, const int32_t* M_ptr, int M, int chunk);
// model launchers that the prefill shares
int gemm_bf16(sara_ctx* c, const void* X, const void* W, const int32_t* M_ptr, int M, int N, int K, int& splits_out);
void gemm_swiglu(sara_ctx* c, const void* X, const void* W, const int32_t* M_ptr, int M_cap);
void residual_norm_bf16(sara_ctx* c, const int32_t* M_ptr, int M_cap, int sp, const float* w);
void launch_qkv_epilogue_bf16(sara_ctx* c, const int32_t* M_ptr, int M, int sp, int layer);
// launchers (model)
int launch_prefill(sara_ctx* c);
int launch_decode(sara_ctx* c, const int32_t* forced, const int32_t* const* forced_at, float* logits, int model_free);
// launchers (controller)
int launch_reset(sara_ctx* c);
int launch_decide(sara_ctx* c);
int launch_warm_priors(sara_ctx* c);
int launch_warm_update(sara_ctx* c, double lambda);
int launch_refill(sara_ctx* c);
int launch_decide_refill(sara_ctx* c);
int launch_finish(sara_ctx* c, float eps);
int launch_peff(const double* alpha, const double* beta, const int32_t* n, const int32_t* s, int k, int count,
                double* out, hipStream_t st);
int launch_poll(sara_ctx* c, int32_t* d_host);
int launch_grpo(const float* r, const int32_t* off, int n_groups, float eps, float* adv,
                hipStream_t st);
int launch_sample_rows(const float* logits, int n_rows, int V, const int32_t* rid,
                       const int32_t* pos, uint64_t seed, int step, float temp, float top_p, int eos,
                       uint32_t feos, int32_t* tok, hipStream_t st);
int launch_sample_rows_noalloc(const float* logits, int n_rows, int V, const int32_t* rid, const int32_t* pos,
                               uint64_t seed, int step, float temp, float top_p, int eos, uint32_t feos,
                               int32_t* tok, hipStream_t st);
int launch_convert_norms(sara_ctx* c, const void* const* w);
int launch_gumbel_check(double* h_out, hipStream_t st);
int launch_tile_weights(sara_ctx* c, const void* src, void* dst, int rows, int K, int tile_mul, int tile_add,
                        int dst_rows);
int launch_tile_weights_pairs(sara_ctx* c, const void* src, void* dst, int n_rows, int K, int head_off);

// ---------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// Fragment-major ("tiled") layout of a [rows][K] bf16 matrix: for each
// 16-row tile and each 32-wide k step, the 64 lanes' 16-byte MFMA operand
// fragments lie back to back (lane l holds row l % 16, k 8*(l/16)..+8), so
// every fragment load of a wave is one contiguous, fully coalesced 1 KiB read
// and a wave walks its 16 rows as one sequential stream.  The GEMM inputs of
// the bf16 prefill and the decode rows feeding the q|k|v kernel are written
// this way.
__device__ __forceinline__ int64_t tiled_index(int64_t row, int64_t k, int64_t K) {
  const int64_t tile = row >> 4, ks = k >> 5, lane = (row & 15) + 16 * ((k >> 3) & 3);
  return ((tile * (K >> 5) + ks) * 64 + lane) * 8 + (k & 7);
}

// Layout of the bf16 GEMM weights ([rows][K], K a multiple of 64): the same
// 1 KiB fragments, ordered k-block-major.  K is cut into 64-wide blocks; in
// block b the n_tiles 16-row tiles lie back to back, each as its two 32-wide
// k steps.  The waves of a launch walk k at about the same pace, so at any
// moment they read one contiguous stretch of the matrix (spread over every
// HBM channel) instead of n_tiles streams a whole tile row apart, which
// measured 3-18% faster on the decode weight shapes.
__host__ __device__ __forceinline__ int64_t wtiled_index(int64_t row, int64_t k, int64_t n_tiles) {
  const int64_t tile = row >> 4, kb = k >> 6, ks = (k >> 5) & 1, lane = (row & 15) + 16 * ((k >> 3) & 3);
  return (((kb * n_tiles + tile) * 2 + ks) * 64 + lane) * 8 + (k & 7);
}

// two fp32 values rounded (to nearest even) to a bf16 pair, a in the low half
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t b = __float_as_uint(f);
  return (uint16_t)((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
}
template <typename T> __device__ __forceinline__ float ld_f32(const T* p, size_t i);
template <> __device__ __forceinline__ float ld_f32<float>(const float* p, size_t i) { return p[i]; }
template <> __device__ __forceinline__ float ld_f32<uint16_t>(const uint16_t* p, size_t i) {
  return bf16_to_f32(p[i]);
}
template <typename T> __device__ __forceinline__ void st_f32(T* p, size_t i, float v);
template <> __device__ __forceinline__ void st_f32<float>(float* p, size_t i, float v) { p[i] = v; }
template <> __device__ __forceinline__ void st_f32<uint16_t>(uint16_t* p, size_t i, float v) {
  p[i] = f32_to_bf16(v);
}

// Philox4x32-10 (Salmon et al., SC'11): 10 rounds of two 32x32->64 products
// and a Weyl-sequence key schedule.
struct U32x4 { uint32_t x, y, z, w; };
__device__ __forceinline__ U32x4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    // full 64-bit products: one multiply instruction per product on gfx950
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
    const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
    uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  return U32x4{c0, c1, c2, c3};
}
__device__ __forceinline__ void sampler_key(uint64_t seed, int32_t step, uint32_t& k0, uint32_t& k1) {
  k0 = (uint32_t)seed;
  k1 = (uint32_t)(seed >> 32) ^ (uint32_t)step;
}

// silu(g) u = g / (1 + exp(-g)) u.  The exponential e is the hardware's of the
// rounded -g log2(e), and the reciprocal the hardware's; what the argument and
// the sum lost by rounding (l, dl) goes into one correction of the quotient: at
// most 1.4e-7 from silu(g), 3e-8 rms (expf and a division, half as many
// instructions again: 1.8e-7 and 4e-8; without the correction 3.8e-6).  g of
// -88 or less gives 0 (within 2e-36), an infinite one itself (s is then a NaN).
// It costs a pool prefill (256 prompts, width 1536) 22.1 ms against 21.3, and with
// expf and a division 22.6.
__device__ __forceinline__ float silu_mul(float g, float u) {
  constexpr float kL = 1.44269504f, kLlo = 1.92596299e-8f, kLn2 = 0.693147181f;   // log2(e) in two parts
  const float a = __builtin_amdgcn_fmed3f(g, -87.0f, 128.0f);   // no overflow; e < 2^-126 is 0
  const float h = -kL * a, l = fmaf(-kLlo, a, fmaf(-kL, a, -h));
  const float e = __builtin_amdgcn_exp2f(h);
  const float hi = fmaxf(1.0f, e), lo = fminf(1.0f, e), d = hi + lo;
  const float dl = fmaf(e, l * kLn2, lo - (d - hi));
  const float r = __builtin_amdgcn_rcpf(d), t = g * r;
  const float s = fmaf(fmaf(-dl, t, fmaf(-d, t, g)), r, t);
  return fminf(g < -88.0f ? -0.0f : s, fabsf(g)) * u;
}
__device__ __forceinline__ f32x4 silu_mul(f32x4 g, f32x4 u) {
  return f32x4{silu_mul(g[0], u[0]), silu_mul(g[1], u[1]), silu_mul(g[2], u[2]), silu_mul(g[3], u[3])};
}

// SplitMix64 output finalizer (Steele, Lea, Flood, OOPSLA'14).
__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ uint64_t reward_hash_init(uint64_t seed, int32_t step, int32_t uid) {
  return mix64((seed ^ kSeedRXor) ^ mix64(((uint64_t)(uint32_t)step << 32) + (uint64_t)(uint32_t)uid));
}

// Proposition 1 (Eq. peff): posterior predictive probability that the
// completed group of size k is mixed, given n observed rollouts with s
// successes under the prior Beta(a0, b0).  Both saturation terms apply when
// n = 0; a complete unmixed group has probability 0.
__device__ __forceinline__ double peff_dev(int n, int s, int k, double a0, double b0) {
  if (s >= 1 && n - s >= 1) return 1.0;
  int r = k - n;
  if (r <= 0) return 0.0;
  double a = a0 + (double)s, b = b0 + (double)(n - s);
  double lb = lgamma(a) + lgamma(b) - lgamma(a + b);
  double psat = 0.0;
  if (s == 0) psat += exp(lgamma(a) + lgamma(b + r) - lgamma(a + b + r) - lb);
  if (s == n) psat += exp(lgamma(a + r) + lgamma(b) - lgamma(a + b + r) - lb);
  return 1.0 - psat;
}

}  // namespace sara
