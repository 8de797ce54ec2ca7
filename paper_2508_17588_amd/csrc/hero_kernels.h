// Host-callable launchers of the HERO kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

typedef uint16_t bf16_t;

// A kernel that uses more than 64 KB of dynamic LDS must be told so once on every device it runs
// on.  `done` holds one bit per device ordinal (devices past 63 are told on every launch); the
// runtime call is idempotent, so two host threads that meet here at most repeat it.
inline hipError_t allow_dynamic_lds(const void* kern, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? 1ull << dev : 0;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// Every member of the structures below has a value from the start: a launcher that does not know a member yet hands over
// "none", and not what lay on its stack.

// Patch grid of Eq. 4 and the closed-form output offsets of the selection list.
// n_take[class]: tokens taken per patch; class = 2*(clipped bottom row) + (clipped right column).
struct SelectGeom {
  int32_t frames = 0, height = 0, width = 0, n_text = 0;
  int32_t patch_h = 0, patch_w = 0;
  int32_t grid_h = 0, grid_w = 0;  // patches per frame along y / x (ceil)
  int32_t n_patches = 0;           // frames * grid_h * grid_w
  int32_t n_take[4] = {};
  int32_t take_per_full_row = 0;   // picks of one patch-row that is not the last one
  int32_t take_per_frame = 0;
  int32_t n_sel = 0;               // total picks
};

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st);
// clears `seen` (ceil(n_tokens/32) bitmap words and one verdict word) and marks the listed rows;
// verdict bit 0: a row outside [0, n_tokens), bit 1: a row listed twice
hipError_t launch_check_idx(const int32_t* idx, int n_sel, int n_tokens, uint32_t* seen, hipStream_t st);
// mode 0: age priority (largest (age, hash) keys); mode 1: age-weighted sampling without replacement
hipError_t launch_select(const SelectGeom& g, int mode, uint32_t step_salt, int32_t* ages, int32_t* idx,
                         hipStream_t st);
// adaLN modulation of a LayerNorm's output, u * (1 + scale) + shift, with the vectors of the row's
// stream (rows < n_text: text).  scale_v == nullptr: none.
struct LnMod {
  const bf16_t *scale_v = nullptr, *shift_v = nullptr, *scale_t = nullptr, *shift_t = nullptr;
  int32_t n_text = 0;
};
hipError_t launch_gather_ln(const void* x, bool x_fp32, const bf16_t* add, const int32_t* rows, int n_rows,
                            int hidden, const bf16_t* gain, const bf16_t* bias, float eps, bf16_t* out,
                            hipStream_t st, const LnMod& mod = LnMod());

// q / k post-processing (per-head LayerNorm, rotary positions on video rows, softmax scale on q), in place
struct QkPostArgs {
  bf16_t* q = nullptr;           // [n_rows, d]
  bf16_t* k = nullptr;           // [*, d], row rows[i] (or i)
  const int32_t* rows = nullptr;
  int32_t n_rows = 0, d = 0, head_dim = 0, n_text = 0;
  const bf16_t *qn_g = nullptr, *qn_b = nullptr, *kn_g = nullptr, *kn_b = nullptr;  // [head_dim]; qn_g == nullptr: no normalisation
  const float2* rope = nullptr;  // [n_video, head_dim/2] (cos, sin); nullptr: no rotation
  float q_scale = 0.f;
};
hipError_t launch_qk_post(const QkPostArgs& a, hipStream_t st);
hipError_t launch_rope_table(float2* table, int frames, int height, int width, int head_dim, hipStream_t st);
// from_end: the arrays are walked from their last element to their first
hipError_t launch_axpy_features(void* x, bool x_fp32, const bf16_t* s_cur, const bf16_t* s_prev, float alpha,
                                int64_t n_elems, hipStream_t st, bool from_end = false);

// Deep-stack collapse: t = (accumulate ? t : 0) + sum of up to 48 bf16 feature arrays (fp32 result),
// and x += t_cur + (t_cur - t_prev) * alpha (t_prev may be null: x += t_cur).
struct FeatureList {
  const bf16_t* p[48] = {};
  int32_t n = 0;
};
hipError_t launch_sum_features(const FeatureList& fl, float* t, bool accumulate, int64_t n_elems, hipStream_t st);
hipError_t launch_apply_sums(void* x, bool x_fp32, const float* t_cur, const float* t_prev, float alpha,
                             int64_t n_elems, hipStream_t st);
// rows whose age is not 0 (and text rows): x += sum of the listed features; all rows: x += the deep-stack term
// from t_cur / t_prev (both optional; fp32 sums, or the bf16 features of a single layer)
hipError_t launch_end_of_cached_step(void* x, bool x_fp32, const FeatureList& shallow, const int32_t* ages, int n_text,
                                     int hidden, const void* t_cur, const void* t_prev, bool t_fp32, float alpha,
                                     int64_t n_elems, hipStream_t st);

// GEMM epilogues: what happens to act(A W^T + bias)
enum GemmEpilogue {
  EPI_PLAIN = 0,        // C[m, n]                       (ldc = n)
  EPI_GELU = 1,         // C[m, n] = gelu_tanh(.)
  EPI_QKV = 2,          // n < d: Q[m, n];  d <= n < 2d: K[row(m), n-d];  else V^T[n-2d, row(m)]
  EPI_SCATTER = 3,      // S[row(m), n] = .
  EPI_SCATTER_ADD = 4   // S[row(m), n] += .
};

// sums of D and D^2, D = f_next - 2 f_cur + f_prev (fp64), into stats[0..1]; scratch: second_diff_scratch_bytes()
size_t second_diff_scratch_bytes();
hipError_t launch_second_diff_stats(const bf16_t* f_prev, const bf16_t* f_cur, const bf16_t* f_next, int64_t n_elems,
                                    double* scratch, double* stats, bool accumulate, hipStream_t st);

struct GemmArgs {
  const bf16_t* a = nullptr;       // [M, K] row-major
  const bf16_t* w = nullptr;       // [N, K] row-major
  const bf16_t* bias = nullptr;    // [N]
  int32_t m = 0, n = 0, k = 0;
  int32_t epilogue = 0;
  const int32_t* rows = nullptr;   // row(m) = rows ? rows[m] : m   (scatter epilogues)
  bf16_t* c = nullptr;             // PLAIN/GELU: C; QKV: Q [M, d]; SCATTER*: S [*, n]
  bf16_t* k_out = nullptr;         // QKV: K cache [*, d]
  bf16_t* vt_out = nullptr;        // QKV: V^T cache [d, ld_vt]
  int64_t ld_vt = 0;
  int32_t d = 0;                   // QKV: hidden
  float q_scale = 0.f;             // QKV: the Q third is stored multiplied by this (softmax scale folded into Q)
  float* splitk_ws = nullptr;      // optional device scratch for k-split partial sums (nullptr: never split)
  size_t splitk_ws_bytes = 0;
  float* parts = nullptr;          // scratch for the chunks of smaller tiles cut along k, which need arrivals too (nullptr: never cut)
  size_t parts_bytes = 0;
  uint32_t* arrivals = nullptr;    // GEMM_ARRIVALS counters, zero before and after every launch
  void* x = nullptr;               // SCATTER_ADD, optional: x[row(m), :] += the stored (rounded) S[row(m), :]  (Alg. 1 residual add)
  int32_t x_fp32 = 0;              // x holds fp32 (else bf16)
  const bf16_t* gate_v = nullptr;  // SCATTER*, optional: (acc + bias) is multiplied by gate[n] of the row's stream (adaLN gate)
  const bf16_t* gate_t = nullptr;  //   rows (after row(m)) below n_text use gate_t, the others gate_v
  int32_t n_text = 0;
};

constexpr int GEMM_ARRIVALS = 256;
hipError_t launch_gemm(const GemmArgs& g, hipStream_t st);
// the tile launch_gemm takes for this problem, and the chunks along k of the last round's tiles (1: not cut)
void gemm_route(const GemmArgs& g, int* tile_m, int* tile_n, int* k_chunks);

// The rows a GEMM normalises by itself instead of reading them from `a`: LayerNorm of x[row] (+ add[row]) over
// the k channels, as launch_gather_ln computes it.
struct LnInput {
  const void* x = nullptr;
  bool x_fp32 = false;
  const bf16_t* add = nullptr;    // nullptr: none
  const int32_t* rows = nullptr;  // nullptr: row m
  const bf16_t *gain = nullptr, *bias = nullptr;
  float eps = 0.f;
  LnMod mod;
};
// whether one kernel takes LayerNorm and this (QKV or GELU) GEMM faster than two
bool gemm_takes_ln(const GemmArgs& g);
hipError_t launch_gemm_ln(const GemmArgs& g, const LnInput& ln, hipStream_t st);

// Out-projection, LayerNorm, FFN and residual of the listed rows in one kernel (narrow models)
struct TailArgs {
  const bf16_t* o = nullptr;                      // attention output [n_rows, hidden]
  const int32_t* rows = nullptr;                  // nullptr: row m
  int32_t n_rows = 0, hidden = 0, ffn = 0;
  const bf16_t *w_o = nullptr, *b_o = nullptr, *w1 = nullptr, *b1 = nullptr, *w2 = nullptr, *b2 = nullptr;
  const bf16_t *gain = nullptr, *bias = nullptr;  // LayerNorm
  float eps = 0.f;
  LnMod mod;
  const bf16_t *gate1_v = nullptr, *gate1_t = nullptr, *gate2_v = nullptr, *gate2_t = nullptr;  // adaLN gates of the two branches (nullptr: none)
  int32_t n_text = 0;                             // rows below it take the _t vectors
  bf16_t* s = nullptr;                            // stored feature, row rows[m]
  void* x = nullptr;                              // residual stream, read at row rows[m]
  bool x_fp32 = false, add_to_x = false;          // add_to_x: += the stored feature
  float* parts = nullptr;                         // scratch for partial sums (nullptr: the FFN channels are never shared out)
  size_t parts_bytes = 0;
  uint32_t* arrivals = nullptr;                   // NARROW_TAIL_BLOCKS counters, zero before and after every launch
};
constexpr int NARROW_TAIL_ROWS = 16;        // rows of a workgroup
constexpr int NARROW_TAIL_BLOCKS = 256;     // most workgroups that share sums
bool narrow_tail_fits(int n_rows, int hidden, int ffn);
// the workgroups that share the FFN channels of a block of rows, with parts_bytes of `parts` (1: not shared)
int narrow_tail_split(int n_rows, int hidden, size_t parts_bytes);
// bytes of `parts` it can make use of for up to n_rows rows
size_t narrow_tail_parts_bytes(int n_rows, int hidden);
hipError_t launch_narrow_tail(const TailArgs& a, hipStream_t st);

// bytes of `parts` that a layer's GEMM of up to m rows can make use of, however it is cut into smaller tiles
size_t gemm_most_parts_bytes(int m, int n, int k);
// bytes of scratch launch_gemm would use for this problem if it had all it wanted (0: the problem is not cut along k)
size_t gemm_wanted_scratch_bytes(const GemmArgs& g);

struct AttnArgs {
  const bf16_t* q = nullptr;           // [r, n_heads*head_dim]
  const bf16_t* k = nullptr;           // [n_keys, n_heads*head_dim]
  const bf16_t* vt = nullptr;          // [n_heads*head_dim, ld_vt]
  int64_t ld_vt = 0;
  bf16_t* o = nullptr;                 // [r, n_heads*head_dim]
  int32_t r = 0, n_keys = 0, n_heads = 0, head_dim = 0;
  float q_scale = 0.f;                 // scores are exp2(q_scale * q.k): log2(e)/sqrt(head_dim), or 1 if folded into Q
  float* split_ws = nullptr;           // optional device scratch for the partial results of key-split query blocks (nullptr: never split)
  size_t split_ws_bytes = 0;
  uint32_t* fallback_count = nullptr;  // optional device counter (head_dim 64): += 1 per block of 256 queries of one head, however many
                                       // workgroups it has, with row sums beyond the reference-free form's range: recomputed with references
};

hipError_t launch_attention(const AttnArgs& a, hipStream_t st);
// queries per workgroup of the kernel launch_attention takes, and the key ranges of the last round's blocks (1: not cut)
void attention_route(const AttnArgs& a, int* queries, int* key_ranges);
