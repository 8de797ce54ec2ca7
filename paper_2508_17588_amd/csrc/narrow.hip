// What follows attention in a block of a narrow model (at most 256 channels, FFN four times as wide), in one kernel:
// out-projection, residual, LayerNorm, FFN1 with GELU, FFN2 and the residual add (Eq. 2 / Eq. 3 for the listed rows).
// All of it is local to a row, so a workgroup takes 16 rows through the whole chain and only the weights are streamed.
// Where few rows leave the chip idle, 2 or 4 workgroups share a block of rows: each takes a part of the FFN channels
// (and the out-projection and LayerNorm again), and the one that arrives last adds up the parts.
//
// v_mfma_f32_16x16x32_bf16 with the weights as the A operand (lane: weight row lane%16, eight consecutive k starting at
// 8*(lane/16)) and the rows as the B operand (lane: row lane%16, likewise), so that a lane ends up with four consecutive
// channels of one row (accumulator value e: channel 4*(lane/16) + e).  Weights go from global memory to registers in
// batches of 16 weight rows x D of k, NB batches of a wave on their way, and through a place in LDS of the wave's own
// into the operand's order.  The rows' operands lie in LDS, padded by 16 bytes: their reads are free of bank conflicts.
//
// What bounds it: what one CU can stream, about 120 GB/s of weights that lie in the memory-side cache (1.2 MB at 256
// channels), then the latencies of the chain.  It replaces the out-projection, FFN1 and FFN2 kernels (4 + 7 + 8 us on
// 326 rows of 256 channels, each mostly launch and load latency).  A whole layer, before and after: 64 channels, 300
// rows 26.8 -> 18.1 us; 128 channels, 300 rows 29.3 -> 20.8, 2000 rows 38.2 -> 29.4, 16000 rows 174 -> 160; 256 channels,
// 300 rows 33.7 -> 27.6 (32.4 with the FFN channels not shared out), 2000 rows 47.8 -> 40.8, 8000 rows 131 -> 127.
#include <algorithm>
#include <atomic>

#include "hero_device.h"
#include "hero_kernels.h"

namespace {

__device__ __forceinline__ void load4(const float* p, float (&v)[4]) {
  const floatx4_t t = *reinterpret_cast<const floatx4_t*>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = t[e];
}
__device__ __forceinline__ void load4(const bf16_t* p, float (&v)[4]) {
  const u32x2_t t = *reinterpret_cast<const u32x2_t*>(p);
  v[0] = unpack_lo(t[0]); v[1] = unpack_hi(t[0]); v[2] = unpack_lo(t[1]); v[3] = unpack_hi(t[1]);
}
__device__ __forceinline__ void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<floatx4_t*>(p) = floatx4_t{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ void store4(bf16_t* p, const float (&v)[4]) {
  *reinterpret_cast<u32x2_t*>(p) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}

// LDS traffic of this wave is done, then every wave's; loads from global memory stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr int ROWS = NARROW_TAIL_ROWS;
constexpr int NB = 4;         // weight batches of a wave on their way
constexpr int FFN = 4;        // FFN channels for each channel of the stream

// No branch lies between the first load and the last batch, so that every wait is for one batch and leaves the
// others on their way: what is optional (row list, gates, modulation) is loaded from some address in any case.
template <int KD, int WAVES, int SPLIT>
struct NarrowTail {
  static constexpr int D = KD * 64, FS = FFN * D / SPLIT;
  static constexpr int LDS = WAVES * KD * 2048 + ROWS * (D + 8) * 2 + ROWS * (FS + 8) * 2 + FS * 2 + 2 * WAVES * ROWS * 4 + 16;
};

template <int KD, int WAVES, int SPLIT, typename XT>
__global__ __launch_bounds__(WAVES * 64) void narrow_tail_kernel(TailArgs a) {
  constexpr int D = KD * 64, F = FFN * D;
  constexpr int FS = F / SPLIT;                        // FFN channels of this workgroup
  constexpr int TPW = D / 16 / WAVES;                  // output tiles of 16 channels of a wave
  constexpr int NT = FFN * TPW / SPLIT;                // batches of a wave in FFN1 (tiles) and in FFN2 (chunks of D x tiles)
  constexpr int BATCHES = TPW + 2 * NT;                // out-projection, FFN1, FFN2
  constexpr int LD = D + 8, LDH = FS + 8;              // LDS rows, in elements
  constexpr int KF = 2 * KD;                           // fragments (32 of k) in D channels
  static_assert(TPW * WAVES * 16 == D && FS % D == 0 && NT % TPW == 0, "tiles of a wave");
  extern __shared__ u32x4_t smem[];
  struct Lds {
    u32x4_t weights[WAVES][KF * 64];                   // a batch of each wave
    bf16_t rows[ROWS * LD];                            // attention output, then the normalised rows
    bf16_t hid[ROWS * LDH];                            // GELU output
    bf16_t b1[FS];
    float red[2][WAVES][ROWS];
    uint32_t arrived;
  };
  static_assert(sizeof(Lds) == NarrowTail<KD, WAVES, SPLIT>::LDS, "launch");
  Lds& lds = *reinterpret_cast<Lds*>(smem);
  bf16_t *rows_lds = lds.rows, *hid = lds.hid, *b1_lds = lds.b1;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int part = blockIdx.x % SPLIT, row_block = blockIdx.x / SPLIT, r0 = row_block * ROWS;
  const int f0 = part * FS;                            // first FFN channel of this workgroup
  const int mr = min(r0 + m, a.n_rows - 1);            // (rows past the end: computed, not stored)

  // ---- everything that waits for nothing: row number, attention output, FFN1's bias, weights, parameters ----
  const int32_t listed = *(a.rows != nullptr ? a.rows + mr : reinterpret_cast<const int32_t*>(a.b_o));
  constexpr int PIECES = ROWS * D / 8, B1_PIECES = FS / 8;
  const int op = tid % PIECES, bp = tid % B1_PIECES;
  const u32x4_t o_piece = *reinterpret_cast<const u32x4_t*>(a.o + (int64_t)min(r0 + op / (D / 8), a.n_rows - 1) * D + op % (D / 8) * 8);
  const u32x4_t b1_piece = *reinterpret_cast<const u32x4_t*>(a.b1 + f0 + bp * 8);
  static_assert(PIECES <= WAVES * 64 && B1_PIECES <= WAVES * 64, "one piece a thread");

  // a load takes eight rows x 64 of k: neighbouring lanes share a cache line (lanes in the operand's order, 16 rows
  // apart in memory, make 64 requests of it: 38 GB/s a CU instead of 120)
  u32x4_t w[NB][KF];
  const int l8 = lane >> 3, c8 = lane & 7;
  auto fetch = [&](u32x4_t (&dst)[KF], const bf16_t* base, int row0, int ld, int k0) {
    const bf16_t* p = base + (int64_t)(row0 + l8) * ld + k0 + c8 * 8;
#pragma unroll
    for (int f = 0; f < KF; ++f) dst[f] = *reinterpret_cast<const u32x4_t*>(p + (f & 1) * 8 * ld + (f >> 1) * 64);
  };
  // batch b of this wave: out-projection, then FFN1 (both tile by tile), then FFN2 (chunk of D along k, then tile)
  auto fetch_batch = [&](int b) {
    if (b < TPW) fetch(w[b % NB], a.w_o, (wave * TPW + b) * 16, D, 0);
    else if (b < TPW + NT) fetch(w[b % NB], a.w1, f0 + (wave + (b - TPW) * WAVES) * 16, D, 0);
    else if (b < BATCHES) fetch(w[b % NB], a.w2, (wave * TPW + (b - TPW - NT) % TPW) * 16, F, f0 + (b - TPW - NT) / TPW * D);
  };
#pragma unroll
  for (int b = 0; b < TPW; ++b) fetch_batch(b);

  const int64_t src = a.rows != nullptr ? listed : mr;
  const bool text = src < a.n_text;
  const bool gated = a.gate1_v != nullptr, modulated = a.mod.scale_v != nullptr;
  float xv[TPW][4];
  u32x2_t gain[TPW], beta[TPW], b_o[TPW], b_2[TPW], gate1[TPW], gate2[TPW], scale[TPW], shift[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int n = (wave * TPW + t) * 16 + 4 * g;
    auto at = [&](const bf16_t* p) { return *reinterpret_cast<const u32x2_t*>(p + n); };
    b_o[t] = at(a.b_o);
    load4(static_cast<const XT*>(a.x) + src * D + n, xv[t]);
    gain[t] = at(a.gain);
    beta[t] = at(a.bias);
    gate1[t] = at(!gated ? a.b_o : text ? a.gate1_t : a.gate1_v);
    scale[t] = at(!modulated ? a.b_o : text ? a.mod.scale_t : a.mod.scale_v);
    shift[t] = at(!modulated ? a.b_o : text ? a.mod.shift_t : a.mod.shift_v);
    gate2[t] = at(!gated ? a.b_o : text ? a.gate2_t : a.gate2_v);
    b_2[t] = at(a.b2);
  }
#pragma unroll
  for (int b = TPW; b < NB; ++b) fetch_batch(b);
  __builtin_amdgcn_sched_barrier(0);
  *reinterpret_cast<u32x4_t*>(rows_lds + op / (D / 8) * LD + op % (D / 8) * 8) = o_piece;
  *reinterpret_cast<u32x4_t*>(b1_lds + bp * 8) = b1_piece;
  lds_barrier();

  bf16x8_t rf[KF];                                     // the rows as B operand
  auto read_rows = [&](const bf16_t* base, int ld) {
#pragma unroll
    for (int f = 0; f < KF; ++f) rf[f] = *reinterpret_cast<const bf16x8_t*>(base + m * ld + f * 32 + g * 8);
  };
  // the batch goes through LDS into the operand's order; only this wave uses the place, and its LDS operations keep order
  u32x4_t* mine = lds.weights[wave];
  auto mma = [&](const u32x4_t (&wt)[KF], floatx4_t acc) {
#pragma unroll
    for (int f = 0; f < KF; ++f) mine[f * 64 + l8 * 8 + (c8 ^ (((f & 1) * 4 + (l8 >> 1)) & 7))] = wt[f];
    bf16x8_t wf[KF];                                   // 16 rows x 64 of k: row m, chunk 4 (f%2) + g
#pragma unroll
    for (int f = 0; f < KF; ++f)
      wf[f] = *reinterpret_cast<const bf16x8_t*>(&mine[(f >> 1) * 128 + m * 8 + (((f & 1) * 4 + g) ^ ((m >> 1) & 7))]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < KF; ++f) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[f], rf[f], acc, 0, 0, 0);
    return acc;
  };
  auto pair_at = [](const u32x2_t& p, int e) { return e & 1 ? unpack_hi(p[e >> 1]) : unpack_lo(p[e >> 1]); };

  // ---- out-projection ----
  read_rows(rows_lds, LD);
  float feature[TPW][4], y[TPW][4], sum = 0.f;         // (the feature is rounded once, with FFN2's part of it)
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const floatx4_t acc = mma(w[t], floatx4_t{0.f, 0.f, 0.f, 0.f});
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      feature[t][e] = (acc[e] + pair_at(b_o[t], e)) * (gated ? pair_at(gate1[t], e) : 1.0f);
      y[t][e] = xv[t][e] + bf16_to_f32(f32_to_bf16_hw(feature[t][e]));
      sum += y[t][e];
    }
  }
#pragma unroll
  for (int b = 0; b < TPW; ++b) fetch_batch(b + NB);
  __builtin_amdgcn_sched_barrier(0);

  // ---- LayerNorm of the rows: mean, then variance, each over the waves ----
  auto row_total = [&](float v, float (&slot)[WAVES][ROWS]) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (g == 0) slot[wave][m] = v;
    lds_barrier();
    float total = 0.f;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) total += slot[i][m];
    return total;
  };
  const float mean = row_total(sum, lds.red[0]) * (1.0f / D);
  float sq = 0.f;
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) { y[t][e] -= mean; sq += y[t][e] * y[t][e]; }
  const float rstd = rsqrtf(row_total(sq, lds.red[1]) * (1.0f / D) + a.eps);
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int n = (wave * TPW + t) * 16 + 4 * g;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      y[t][e] = y[t][e] * rstd * pair_at(gain[t], e) + pair_at(beta[t], e);
      if (modulated) y[t][e] = y[t][e] * (1.0f + pair_at(scale[t], e)) + pair_at(shift[t], e);
    }
    // (every wave has passed two barriers since it read the attention output from this place)
    *reinterpret_cast<u32x2_t*>(rows_lds + m * LD + n) = u32x2_t{pack_bf16x2_hw(y[t][0], y[t][1]), pack_bf16x2_hw(y[t][2], y[t][3])};
  }
  lds_barrier();

  // ---- FFN1 and GELU ----
  read_rows(rows_lds, LD);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int n = (wave + i * WAVES) * 16 + 4 * g;
    const u32x2_t b = *reinterpret_cast<const u32x2_t*>(b1_lds + n);
    const floatx4_t acc = mma(w[(TPW + i) % NB], floatx4_t{0.f, 0.f, 0.f, 0.f});
    fetch_batch(TPW + i + NB);
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(acc[e] + pair_at(b, e));
    *reinterpret_cast<u32x2_t*>(hid + m * LDH + n) = u32x2_t{pack_bf16x2_hw(v[0], v[1]), pack_bf16x2_hw(v[2], v[3])};
    __builtin_amdgcn_sched_barrier(0);
  }
  lds_barrier();

  // ---- FFN2: chunks of D along k ----
  floatx4_t acc[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) acc[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    if (j % TPW == 0) read_rows(hid + j / TPW * D, LDH);
    acc[j % TPW] = mma(w[(TPW + NT + j) % NB], acc[j % TPW]);
    fetch_batch(TPW + NT + j + NB);
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- the workgroup that arrives last adds up the parts, in their order whichever it is ----
  if constexpr (SPLIT > 1) {
    constexpr int PART = WAVES * 64 * TPW * 16;        // bytes
    const __amdgpu_buffer_rsrc_t rs = parts_rsrc(a.parts + (size_t)row_block * (SPLIT * PART / 4), SPLIT * PART);
#pragma unroll
    for (int t = 0; t < TPW; ++t) store_part(rs, part * PART + (t * WAVES * 64 + tid) * 16, acc[t]);
    if (!last_to_arrive(a.arrivals + row_block, SPLIT, &lds.arrived)) return;
    floatx4_t p[SPLIT][TPW];
#pragma unroll
    for (int c = 0; c < SPLIT; ++c)
#pragma unroll
      for (int t = 0; t < TPW; ++t) p[c][t] = load_part(rs, c * PART + (t * WAVES * 64 + tid) * 16);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
#pragma unroll
      for (int step = 1; step < SPLIT; step *= 2)
#pragma unroll
        for (int c = 0; c < SPLIT; c += 2 * step)
#pragma unroll
          for (int e = 0; e < 4; ++e) p[c][t][e] += p[c + step][t][e];
      acc[t] = p[0][t];
    }
  }

  // ---- the stored feature, and the residual add with it as stored ----
  if (r0 + m >= a.n_rows) return;
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int n = (wave * TPW + t) * 16 + 4 * g;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = (acc[t][e] + pair_at(b_2[t], e)) * (gated ? pair_at(gate2[t], e) : 1.0f) + feature[t][e];
    const u32x2_t out = {pack_bf16x2_hw(v[0], v[1]), pack_bf16x2_hw(v[2], v[3])};
    *reinterpret_cast<u32x2_t*>(a.s + src * D + n) = out;
    if (a.add_to_x) {
      float xo[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) xo[e] = xv[t][e] + pair_at(out, e);
      store4(static_cast<XT*>(a.x) + src * D + n, xo);
    }
  }
}

template <int KD, int WAVES, int SPLIT, typename XT>
hipError_t launch_split(const TailArgs& a, hipStream_t st) {
  static std::atomic<uint64_t> lds_allowed{0};
  auto kern = narrow_tail_kernel<KD, WAVES, SPLIT, XT>;
  constexpr int LDS = NarrowTail<KD, WAVES, SPLIT>::LDS;
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), LDS, lds_allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((a.n_rows + ROWS - 1) / ROWS * SPLIT), dim3(WAVES * 64), LDS, st, a);
  return hipGetLastError();
}

template <int KD, int WAVES, typename XT>
hipError_t launch(const TailArgs& a, hipStream_t st) {
  switch (narrow_tail_split(a.n_rows, a.hidden, a.parts != nullptr ? a.parts_bytes : 0)) {
    case 4: return launch_split<KD, WAVES, 4, XT>(a, st);
    case 2: return launch_split<KD, WAVES, 2, XT>(a, st);
    default: return launch_split<KD, WAVES, 1, XT>(a, st);
  }
}

}  // namespace

// Up to 128 channels a CU holds the weights' way of several workgroups and the kernel is the faster one at every size
// (33000 rows: 64 channels 1287 -> 1195 us for four layers, 128 channels 2396 -> 2300).  Above, it takes the rows in rounds
// of 4096, which pays if the second one is more than half full (256 channels: 8000 rows 522 -> 507, 10000 rows 683 -> 712;
// 192 channels: 5000 rows 269 -> 275, 6500 rows 384 -> 348, 16000 rows the same, 33000 rows 3428 -> 3531).  Wider than
// 256 channels a CU's stream of weights takes longer than the three kernels.
bool narrow_tail_fits(int n_rows, int hidden, int ffn) {
  if (hidden % 64 != 0 || hidden > 256 || ffn != FFN * hidden) return false;
  if (hidden <= 128 || n_rows <= 256 * ROWS) return true;
  return n_rows <= 512 * ROWS && n_rows > 384 * ROWS;
}

// As many parts as keep every workgroup on a CU of its own (at 128 channels and below a CU holds several, but they share
// what it can stream).  256 channels, 300 rows, a layer: 32.4 us in one part, 27.6 in four.
int narrow_tail_split(int n_rows, int hidden, size_t parts_bytes) {
  const int blocks = (n_rows + ROWS - 1) / ROWS;
  for (int split = 4; split > 1; split /= 2)
    if (blocks * split <= NARROW_TAIL_BLOCKS && (size_t)blocks * split * ROWS * hidden * 4 <= parts_bytes) return split;
  return 1;
}

size_t narrow_tail_parts_bytes(int n_rows, int hidden) {
  return (size_t)std::min((n_rows + ROWS - 1) / ROWS * 4, NARROW_TAIL_BLOCKS) * ROWS * hidden * 4;
}

hipError_t launch_narrow_tail(const TailArgs& a, hipStream_t st) {
  if (a.n_rows <= 0) return hipSuccess;
  if (!narrow_tail_fits(a.n_rows, a.hidden, a.ffn)) return hipErrorInvalidValue;
  switch (a.hidden / 64) {
    case 1: return a.x_fp32 ? launch<1, 4, float>(a, st) : launch<1, 4, bf16_t>(a, st);
    case 2: return a.x_fp32 ? launch<2, 8, float>(a, st) : launch<2, 8, bf16_t>(a, st);
    case 3: return a.x_fp32 ? launch<3, 12, float>(a, st) : launch<3, 12, bf16_t>(a, st);
    case 4: return a.x_fp32 ? launch<4, 8, float>(a, st) : launch<4, 8, bf16_t>(a, st);
  }
  return hipErrorInvalidValue;
}
