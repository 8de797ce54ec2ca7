// bf16 MFMA GEMM for the refreshed rows: C = act(A W^T + bias), A [M,K], W [N,K] both
// K-contiguous (QKV projection, out-projection and FFN of Eq. 2 / Eq. 3), fp32 accumulate.
//
// Three kernels, chosen per problem by the expected time of their tiles (choose_tile):
//  * gemm256_kernel, 256 x 256 tiles: large problems; rings of direct global -> LDS loads, k-split of a
//    thin last round;
//  * gemm_halfk_kernel, 128 x 128 to 256 x 128 tiles: problems whose 256 x 256 tiles would leave CUs idle;
//  * gemm_quarterk_kernel, 64 x 64 tiles: problems with few rows or columns, bound by latency along k.
// A fourth, gemm_ln_kernel, normalises the rows itself (narrow models).
// All use v_mfma_f32_32x32x16_bf16 (A fragment: lane holds row lane%32, eight consecutive k starting at
// 8*(lane/32); B fragment likewise for column lane%32; accumulator register i of a lane is row
// 8*(i/4) + 4*(lane/32) + i%4, column lane%32) and walk k in stages of 64: LDS rows of 128 B whose eight
// 16-byte chunks are XOR-swizzled with (row/2)%8, so that fragment reads are free of bank conflicts.
// Loads are bounds-checked by the hardware (rows past M or N read as zero): ragged sizes need no padding.
// Workgroup ids are remapped so that each XCD works on a contiguous range of tiles, walked in groups of
// row tiles, which keeps the panels an XCD streams concurrently small enough for its L2.
// The epilogue adds the bias, applies GELU where asked, and either stores C or scatters rows into the
// feature / K / V^T caches (Eq. 3's merge); the accumulating one (FFN2) also adds the stored feature to x.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "hero_device.h"
#include "hero_kernels.h"

namespace {

// ------------------------------------------------------------------------------------------
// Large problems: 256 x 256 tile, eight waves (two per SIMD) of 128 x 64, K walked in stages of
// 64 through LDS rings (three slots for A, two for W: all 160 KB of a CU) that are filled by
// direct global -> LDS loads (16 bytes per lane).
//
//  * What bounds this kernel is the rate at which a CU's vector cache can keep cache-line
//    requests in flight, so every request must be a whole 128-byte line: a wave-wide load
//    fetches eight rows of 128 bytes (eight consecutive lanes per row).
//  * Two waves per SIMD: a wave whose load waits for the address unit cannot issue MFMAs
//    meanwhile; with a second wave on the SIMD the matrix pipe keeps running.  Each wave issues
//    eight loads in the first quarter of a stage, one per MFMA: its W blocks of the next stage
//    and its A blocks of the stage after that.  The weight panels are shared by every row tile
//    and mostly hit in the caches, so one stage is enough for them; the activation panels
//    stream from HBM (few workgroups read each), and the extra stage of distance takes their
//    misses off the barrier's wait.
//  * LDS layout of a stage: rows of 128 B whose eight 16-byte chunks are XOR-swizzled with
//    (row/2)%8 (conflict-free ds_read_b128 fragment reads).  A direct load writes lane l to
//    byte 16*l of its 1 KB block, i.e. row l/8, chunk slot l%8, so the lane fetches the chunk
//    that belongs in that slot.
//  * One barrier per stage.  Loads complete in issue order, so "all but my four newest" before
//    the barrier of stage t means A and W of stage t are in LDS.  After that barrier every wave
//    holds the fragments of the last k-slice of stage t-1 in registers and has no LDS read
//    outstanding, so the new loads can overwrite the slots of stage t-1 at once (W of t+1 into
//    the other W slot, A of t+2 into the third A slot); they have one and two whole stages
//    (~2000 cycles each) to land.  The fragments of the first slice of stage t are read while the
//    MFMAs of that last slice run, which hides the LDS latency behind the barrier.
//  * The waves accumulate C^T blocks (operands swapped), so a lane owns one row m and four
//    consecutive columns n per accumulator quad.  The epilogue adds the bias, applies the
//    activation, rounds to bf16 and stages the wave's 128 x 64 sub-tile in LDS (8-byte writes,
//    row stride 136 B), then streams it out in 16-byte pieces, one 128-byte line per row.
//    Waves in the V third of the QKV projection keep the operands unswapped and stage the
//    transposed sub-tile, so V^T rows leave the same way.  The accumulating epilogue (FFN2)
//    stages fp32 in two halves and rounds once after adding the cached row.
// ------------------------------------------------------------------------------------------
constexpr int SBK = 64;                       // k elements per stage: one 128-byte line per row
constexpr int RING_B = 2;                     // W slots: its fills run one stage ahead
constexpr int STAGE_BYTES = 256 * SBK * 2;    // one operand, one stage: 32 KB
constexpr int RING_A = 3;                     // A slots: its fills run two stages ahead
constexpr int RING_B_OFF = RING_A * STAGE_BYTES;   // the W ring starts after the A ring
constexpr int CST = 136;                      // bf16 staging: bytes per 64-column row (+8 pad)
constexpr int CSTT = 264;                     // bf16 staging of a transposed sub-tile: 128 columns (+8 pad)
constexpr int CST32 = 264;                    // fp32 staging: bytes per 64-column row (+8 pad)
constexpr int STAGE_REGION = 128 * CST;       // per-wave staging region (17408 B)
constexpr int RING_BYTES = (RING_A + RING_B) * STAGE_BYTES;   // 160 KB
constexpr int GEMM256_LDS = 8 * STAGE_REGION > RING_BYTES ? 8 * STAGE_REGION : RING_BYTES;
static_assert(64 * CST32 <= STAGE_REGION && 64 * CSTT <= STAGE_REGION, "half-tile / transposed tile must fit the staging region");

// Split of the last, partly filled wave of tiles along k.  Tile slots 0 .. full_items-1 are
// whole work items; every later slot is cut into `split` k-chunks whose fp32 partial sums go to a
// workspace (one 256 KB block per chunk, in accumulator order: [i][j][quad][thread] float4) and
// are added up, and sent through the epilogue, by the fix-up kernel.
struct SplitK {
  int32_t full_items;   // tile slots computed whole
  int32_t split;        // k-chunks per remaining tile slot (1: none)
  float* ws;
};

// tile slot -> origin of its bm x bn tile (each XCD owns a contiguous range of tiles, walked in groups of
// group_m row tiles); false for the empty slots that pad the range to a multiple of 8
__device__ __forceinline__ bool tile_origin(int slot, int bm, int bn, int tiles_m, int tiles_n, int per_xcd,
                                            int group_m, int& m0, int& n0) {
  const int p = (slot % 8) * per_xcd + slot / 8;
  if (p >= tiles_m * tiles_n) return false;
  const int group = p / (group_m * tiles_n);
  const int first_m = group * group_m;
  const int gsize = min(tiles_m - first_m, group_m);
  const int in_group = p - group * group_m * tiles_n;
  m0 = (first_m + in_group % gsize) * bm;
  n0 = (in_group / gsize) * bn;
  return true;
}

template <int EPI, int HALVES>
__device__ __forceinline__ void epilogue256(const GemmArgs& g, floatx16_t (&acc)[4][2], int m0, int n0, int wave,
                                            int lane, char* region);

template <int EPI>
__global__ __launch_bounds__(512) void gemm256_kernel(GemmArgs g, int tiles_m, int tiles_n, int per_xcd,
                                                      int group_m, SplitK sk) {
  // ---- workgroup id -> tile slot and k-chunk ----
  int slot = blockIdx.x, chunk = 0, n_chunks = 1;
  if (slot >= sk.full_items) {
    const int r = slot - sk.full_items;
    slot = sk.full_items + r / sk.split;
    chunk = r - (r / sk.split) * sk.split;
    n_chunks = sk.split;
  }
  int m0, n0;
  if (!tile_origin(slot, 256, 256, tiles_m, tiles_n, per_xcd, group_m, m0, n0)) return;

  extern __shared__ u32x4_t smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // waves w and w+4 share a SIMD
  const int wm0 = (wave & 1) * 128, wn0 = (wave >> 1) * 64;
  const int lr = lane & 31, lh = lane >> 5;

  // ---- direct loads: per stage this wave fills A blocks wave+8i and W blocks wave+8i, i = 0..3
  //      (8 rows each); lane l fetches, for row l/8 of the block, the chunk that belongs in
  //      LDS chunk slot l%8 ----
  const uint32_t row_bytes = (uint32_t)g.k * 2u;
  const u32x4_t rsA = rsrc_words(g.a, (uint32_t)g.m * row_bytes);
  const u32x4_t rsB = rsrc_words(g.w, (uint32_t)g.n * row_bytes);
  uint32_t voffA[4], voffB[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = (wave + 8 * i) * 8 + (lane >> 3);
    const int chunk = (lane & 7) ^ ((row >> 1) & 7);
    voffA[i] = (uint32_t)(m0 + row) * row_bytes + chunk * 16;
    voffB[i] = (uint32_t)(n0 + row) * row_bytes + chunk * 16;
  }
  const uint32_t fillA = lds0 + wave * 1024, fillB = lds0 + RING_B_OFF + wave * 1024;
  const int n_stages = g.k / SBK;
  const int stage_begin = chunk * n_stages / n_chunks, stage_end = (chunk + 1) * n_stages / n_chunks;
  auto fill_a = [&](int slot, int stage, int q) {
    lds_fill(rsA, fillA + (uint32_t)slot * STAGE_BYTES + q * 8192, voffA[q], (uint32_t)stage * (SBK * 2));
  };
  auto fill_b = [&](int slot, int stage, int q) {
    lds_fill(rsB, fillB + (uint32_t)slot * STAGE_BYTES + q * 8192, voffB[q], (uint32_t)stage * (SBK * 2));
  };

  // ---- fragment reads: row R, k-chunk c of a stage sits at R*128 + (c ^ ((R/2)%8))*16 ----
  const char* lbase = reinterpret_cast<const char*>(smem);
  const char* fa_ks[4];
  const char* fb_ks[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int off = lr * 128 + (((2 * ks + lh) ^ ((lr >> 1) & 7)) * 16);     // wm0, wn0, 32i are multiples of 16 rows
    fa_ks[ks] = lbase + wm0 * 128 + off;
    fb_ks[ks] = lbase + RING_B_OFF + wn0 * 128 + off;
  }
  auto frag = [&](const char* ks_base, int slot, int i) {
    u32x4_t t = *reinterpret_cast<const u32x4_t*>(ks_base + slot * STAGE_BYTES + i * 4096);
    return *reinterpret_cast<bf16x8_t*>(&t);
  };

  floatx16_t acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // V third of the QKV projection: keep the natural orientation (lanes along n) so that the
  // staged sub-tile is V^T
  const bool natural = (EPI == EPI_QKV) && (n0 + wn0 >= 2 * g.d);

  // Main loop.  Fragment set [1] holds the k-slice consumed first in a stage (the last slice of
  // the previous stage); the four slices of a stage alternate between the sets.
  auto main_loop = [&](auto NAT) {
    constexpr bool NATURAL = decltype(NAT)::value;
    bf16x8_t fa[2][4], fb[2][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      u32x4_t z = {0u, 0u, 0u, 0u};
      fa[1][i] = *reinterpret_cast<bf16x8_t*>(&z);
      if (i < 2) fb[1][i] = *reinterpret_cast<bf16x8_t*>(&z);
    }
    // order in which the 6 fragments of a slice are read (the MFMAs use them in the same order)
    auto read_frag = [&](int set, int slot_a, int slot_b, int ks, int q) {
      switch (q) {
        case 0: fa[set][0] = frag(fa_ks[ks], slot_a, 0); break;
        case 1: fb[set][0] = frag(fb_ks[ks], slot_b, 0); break;
        case 2: fb[set][1] = frag(fb_ks[ks], slot_b, 1); break;
        case 3: fa[set][1] = frag(fa_ks[ks], slot_a, 1); break;
        case 4: fa[set][2] = frag(fa_ks[ks], slot_a, 2); break;
        default: fa[set][3] = frag(fa_ks[ks], slot_a, 3); break;
      }
    };
    auto mma_one = [&](int set, int x) {
      const int i = x >> 1, j = x & 1;
      if (NATURAL) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], fb[set][j], acc[i][j], 0, 0, 0);
      else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
    };
    // one stage: A slot SA and W slot SB hold stage t
    auto stage = [&](auto SLOT_A, auto SLOT_B, int t) {
      constexpr int SA = decltype(SLOT_A)::value, SB = decltype(SLOT_B)::value;
      // All but the four newest fills (A of stage t+1) have landed: A and W of stage t are in LDS.
      // Own fragment reads of stage t-1 are complete; after the barrier the same holds for every
      // wave: stage t is readable, and the slots of stage t-1 are free.
      asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        // MFMAs of slice sl-1 (set (sl+1)&1) while the fragments of slice sl arrive in set sl&1
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          // (after the last stage the same stage is fetched once more into the idle slot: cheaper than
          //  eight branches per stage, and in bounds)
          if (sl == 0) {
            if (x < 4) fill_b(SB ^ 1, min(t + 1, stage_end - 1), x);
            else fill_a((SA + 2) % 3, min(t + 2, stage_end - 1), x - 4);
          }
          if (x < 6) read_frag(sl & 1, SA, SB, sl, x);
          mma_one((sl + 1) & 1, x);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) fill_a(0, stage_begin, q);
#pragma unroll
    for (int q = 0; q < 4; ++q) fill_b(0, stage_begin, q);
#pragma unroll
    for (int q = 0; q < 4; ++q) fill_a(1, min(stage_begin + 1, stage_end - 1), q);
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    for (int t = stage_begin; t < stage_end; t += 6) {
      stage(I0{}, I0{}, t);
      if (t + 1 < stage_end) stage(I1{}, I1{}, t + 1);
      if (t + 2 < stage_end) stage(I2{}, I0{}, t + 2);
      if (t + 3 < stage_end) stage(I0{}, I1{}, t + 3);
      if (t + 4 < stage_end) stage(I1{}, I0{}, t + 4);
      if (t + 5 < stage_end) stage(I2{}, I1{}, t + 5);
    }
    // last slice of the last stage
#pragma unroll
    for (int x = 0; x < 8; ++x) mma_one(1, x);
  };
  if (EPI == EPI_QKV && natural) main_loop(std::true_type{});
  else main_loop(std::false_type{});

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (n_chunks > 1) {
    // partial sums of a k-chunk: 8 KB per store instruction, contiguous over the workgroup
    float* part = sk.ws + ((size_t)(slot - sk.full_items) * sk.split + chunk) * 65536 + tid * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          floatx4_t v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          *reinterpret_cast<floatx4_t*>(part + ((i * 2 + j) * 4 + q) * 2048) = v;
        }
    return;
  }
  __syncthreads();                       // every wave is done with the ring
  epilogue256<EPI, 2>(g, acc, m0, n0, wave, lane, reinterpret_cast<char*>(smem) + wave * STAGE_REGION);
}

// Adds up the k-chunks of the split tiles and sends the sums through the epilogue.  One
// single-wave workgroup per 128 x 64 wave sub-tile (8 per tile), so that even a few dozen split
// tiles spread over the whole chip; the loads of a chunk are independent and in flight together.
// FFN2's epilogue is the longest (S and x are read, added to and written back, row by row) and sets the time: there a wave
// takes half a sub-tile (FFN2 with its fix-up, 17776 rows x 1920 channels 528 -> 518 us, 33976 x 3072 2086 -> 2071).
template <int EPI> constexpr int fixup_waves = EPI == EPI_SCATTER_ADD ? 16 : 8;      // to a tile
template <int EPI>
__global__ __launch_bounds__(64) void gemm256_fixup_kernel(GemmArgs g, int tiles_m, int tiles_n, int per_xcd,
                                                           int group_m, SplitK sk) {
  constexpr int HALVES = fixup_waves<EPI> == 16 ? 1 : 2, LOADS = 16 * HALVES;
  const int tile = blockIdx.x / fixup_waves<EPI>, wave = (blockIdx.x * HALVES / 2) & 7, half = HALVES == 1 ? blockIdx.x & 1 : 0;
  int m0, n0;
  if (!tile_origin(sk.full_items + tile, 256, 256, tiles_m, tiles_n, per_xcd, group_m, m0, n0)) return;
  extern __shared__ u32x4_t smem[];
  const int lane = threadIdx.x;
  floatx16_t acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  const float* part = sk.ws + (size_t)tile * sk.split * 65536 + half * 16 * 2048 + (wave * 64 + lane) * 4;
  for (int c = 0; c < sk.split; ++c, part += 65536) {
    floatx4_t v[LOADS];
#pragma unroll
    for (int x = 0; x < LOADS; ++x) v[x] = __builtin_nontemporal_load(reinterpret_cast<const floatx4_t*>(part + x * 2048));
#pragma unroll
    for (int x = 0; x < LOADS; ++x)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[x >> 3][(x >> 2) & 1][4 * (x & 3) + e] += v[x][e];
  }
  epilogue256<EPI, HALVES>(g, acc, m0 + 64 * half, n0, wave, lane, reinterpret_cast<char*>(smem));
}

template <int EPI, int HALVES>
__device__ __forceinline__ void epilogue256(const GemmArgs& g, floatx16_t (&acc)[4][2], int m0, int n0, int wave,
                                            int lane, char* region) {
  const int wm0 = (wave & 1) * 128, wn0 = (wave >> 1) * 64;
  const int lr = lane & 31, lh = lane >> 5;
  const bool natural = (EPI == EPI_QKV) && (n0 + wn0 >= 2 * g.d);
  const int mw = m0 + wm0, nw = n0 + wn0;            // origin of this wave's sub-tile; region: its LDS staging space

  if (EPI == EPI_QKV && natural) {
    // acc[i][j][4q+e] = C[m = mw + 32i + 8q + 4lh + e][n = nw + 32j + lr]; stage [n][m]
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = nw + 32 * j + lr;
      const float bias = n < g.n ? bf16_to_f32(g.bias[n]) : 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          u32x2_t pk = {pack_bf16x2_hw(acc[i][j][4 * q] + bias, acc[i][j][4 * q + 1] + bias),
                        pack_bf16x2_hw(acc[i][j][4 * q + 2] + bias, acc[i][j][4 * q + 3] + bias)};
          *reinterpret_cast<u32x2_t*>(region + (32 * j + lr) * CSTT + (32 * i + 8 * q + 4 * lh) * 2) = pk;
        }
    }
    if (g.rows != nullptr) {
      // scattered columns (refresh): lanes run along m, so the 64 two-byte stores of one instruction
      // fall into the few cache lines of one V^T row that hold the neighbouring selected tokens
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int m = mw + 64 * half + lane;
        const bool m_ok = m < g.m;
        const int64_t col = m_ok ? (int64_t)g.rows[m] : 0;
#pragma unroll 8
        for (int nl = 0; nl < 64; ++nl) {
          const bf16_t v = *reinterpret_cast<const bf16_t*>(region + nl * CSTT + (64 * half + lane) * 2);
          const int n = nw + nl;
          if (m_ok && n < g.n) g.vt_out[(int64_t)(n - 2 * g.d) * g.ld_vt + col] = v;
        }
      }
      return;
    }
    // contiguous columns (full layer): rows of the region are n (64 of them), 16-byte pieces hold 8 consecutive m
#pragma unroll 4
    for (int it = 0; it < 16; ++it) {
      const int nl = it * 4 + (lane >> 4), piece = lane & 15;
      const u32x2_t lo = *reinterpret_cast<const u32x2_t*>(region + nl * CSTT + piece * 16);
      const u32x2_t hi = *reinterpret_cast<const u32x2_t*>(region + nl * CSTT + piece * 16 + 8);
      const int n = nw + nl, m = mw + piece * 8;
      if (n < g.n && m < g.m) {
        bf16_t* dst = g.vt_out + (int64_t)(n - 2 * g.d) * g.ld_vt;
        if (m + 8 <= g.m) {
          u32x4_t v = {lo[0], lo[1], hi[0], hi[1]};
          *reinterpret_cast<u32x4_t*>(dst + m) = v;
        } else {
          const uint32_t w4[4] = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (m + e < g.m) dst[m + e] = (bf16_t)(w4[e >> 1] >> ((e & 1) * 16));
        }
      }
    }
    return;
  }

  // acc[i][j][4q+e] = C[m = mw + 32i + lr][n = nw + 32j + 8q + 4lh + e]
  const float out_scale = (EPI == EPI_QKV && nw < g.d) ? g.q_scale : 1.0f;
  // destination of element (m, n): base[row(m) * ld + n - n_shift]
  bf16_t* base = g.c;
  int ld = g.n, n_shift = 0;
  bool use_rows = (EPI == EPI_SCATTER || EPI == EPI_SCATTER_ADD) && g.rows != nullptr;
  if (EPI == EPI_QKV) {
    ld = g.d;
    if (nw >= g.d) { base = g.k_out; n_shift = g.d; use_rows = g.rows != nullptr; }
  }
  // bias of the lane's columns: [j][q] holds n = nw + 32j + 8q + 4lh .. +3
  u32x2_t bias4[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = min(nw + 32 * j + 8 * q + 4 * lh, g.n - 4);     // columns past N are never stored
      bias4[j][q] = *reinterpret_cast<const u32x2_t*>(g.bias + n);
    }
  // adaLN gate of the lane's columns, for both streams; the lane's row i picks one.  (Loaded
  // unconditionally, from the bias vector when there is no gate, so that the arrays stay in registers.)
  constexpr bool CAN_GATE = EPI == EPI_SCATTER || EPI == EPI_SCATTER_ADD;
  const bool gated = CAN_GATE && g.gate_v != nullptr;
  u32x2_t gate4_v[2][4], gate4_t[2][4];
  bool text_row[4];
  if (CAN_GATE) {
    const bf16_t* gv = gated ? g.gate_v : g.bias;
    const bf16_t* gt = gated ? g.gate_t : g.bias;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = min(nw + 32 * j + 8 * q + 4 * lh, g.n - 4);
        gate4_v[j][q] = *reinterpret_cast<const u32x2_t*>(gv + n);
        gate4_t[j][q] = *reinterpret_cast<const u32x2_t*>(gt + n);
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = min(mw + 32 * i + lr, g.m - 1);
      text_row[i] = (use_rows ? g.rows[m] : m) < g.n_text;
    }
  }
  auto biased = [&](int i, int j, int q, float* v) {
    v[0] = acc[i][j][4 * q] + unpack_lo(bias4[j][q][0]);
    v[1] = acc[i][j][4 * q + 1] + unpack_hi(bias4[j][q][0]);
    v[2] = acc[i][j][4 * q + 2] + unpack_lo(bias4[j][q][1]);
    v[3] = acc[i][j][4 * q + 3] + unpack_hi(bias4[j][q][1]);
    if (CAN_GATE && gated) {
      const u32x2_t gg = text_row[i] ? gate4_t[j][q] : gate4_v[j][q];
      v[0] *= unpack_lo(gg[0]); v[1] *= unpack_hi(gg[0]);
      v[2] *= unpack_lo(gg[1]); v[3] *= unpack_hi(gg[1]);
    }
  };

  if (EPI == EPI_SCATTER_ADD) {
    // halves of 64 rows staged in fp32; S[row] += . with one rounding
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float v[4];
            biased(2 * h + ii, j, q, v);
            char* dst = region + (32 * ii + lr) * CST32 + (32 * j + 8 * q + 4 * lh) * 4;
            u32x2_t a0 = {__float_as_uint(v[0]), __float_as_uint(v[1])}, a1 = {__float_as_uint(v[2]), __float_as_uint(v[3])};
            *reinterpret_cast<u32x2_t*>(dst) = a0;
            *reinterpret_cast<u32x2_t*>(dst + 8) = a1;
          }
      // 64 rows x 8 pieces of 8 columns
#pragma unroll 4
      for (int it = 0; it < 8; ++it) {
        const int rl = it * 8 + (lane >> 3), piece = lane & 7;
        const char* src = region + rl * CST32 + piece * 32;
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          u32x2_t t = *reinterpret_cast<const u32x2_t*>(src + 8 * e);
          v[2 * e] = __uint_as_float(t[0]); v[2 * e + 1] = __uint_as_float(t[1]);
        }
        const int m = mw + 64 * h + rl, n = nw + piece * 8;
        if (m < g.m && n < g.n) {
          const int64_t row = use_rows ? (int64_t)g.rows[m] : (int64_t)m;
          u32x4_t* d = reinterpret_cast<u32x4_t*>(base + row * ld + n);
          u32x4_t old = *d, out;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            out[e] = pack_bf16x2_hw(v[2 * e] + unpack_lo(old[e]), v[2 * e + 1] + unpack_hi(old[e]));
          *d = out;
          if (g.x != nullptr) {
            // residual add with the feature as stored (rounded), so x matches x += S done afterwards
            if (g.x_fp32) {
              floatx4_t* xp = reinterpret_cast<floatx4_t*>(static_cast<float*>(g.x) + row * ld + n);
              floatx4_t x0 = xp[0], x1 = xp[1];
              x0[0] += unpack_lo(out[0]); x0[1] += unpack_hi(out[0]); x0[2] += unpack_lo(out[1]); x0[3] += unpack_hi(out[1]);
              x1[0] += unpack_lo(out[2]); x1[1] += unpack_hi(out[2]); x1[2] += unpack_lo(out[3]); x1[3] += unpack_hi(out[3]);
              xp[0] = x0; xp[1] = x1;
            } else {
              u32x4_t* xp = reinterpret_cast<u32x4_t*>(static_cast<bf16_t*>(g.x) + row * ld + n);
              u32x4_t xv = *xp, xo;
#pragma unroll
              for (int e = 0; e < 4; ++e)
                xo[e] = pack_bf16x2(unpack_lo(xv[e]) + unpack_lo(out[e]), unpack_hi(xv[e]) + unpack_hi(out[e]));
              *xp = xo;
            }
          }
        }
      }
    }
    return;
  }

#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v[4];
        biased(i, j, q, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (EPI == EPI_QKV) v[e] *= out_scale;
          if (EPI == EPI_GELU) v[e] = gelu_tanh(v[e]);
        }
        u32x2_t pk = {pack_bf16x2_hw(v[0], v[1]), pack_bf16x2_hw(v[2], v[3])};
        *reinterpret_cast<u32x2_t*>(region + (32 * i + lr) * CST + (32 * j + 8 * q + 4 * lh) * 2) = pk;
      }
  // 128 rows x 8 pieces of 8 columns: one 128-byte line per row
#pragma unroll 4
  for (int it = 0; it < 16; ++it) {
    const int rl = it * 8 + (lane >> 3), piece = lane & 7;
    const u32x2_t lo = *reinterpret_cast<const u32x2_t*>(region + rl * CST + piece * 16);
    const u32x2_t hi = *reinterpret_cast<const u32x2_t*>(region + rl * CST + piece * 16 + 8);
    const int m = mw + rl, n = nw + piece * 8;
    if (m < g.m && n < g.n) {
      const int64_t row = use_rows ? (int64_t)g.rows[m] : (int64_t)m;
      u32x4_t v = {lo[0], lo[1], hi[0], hi[1]};
      *reinterpret_cast<u32x4_t*>(base + row * ld + (n - n_shift)) = v;
    }
  }
}

// ------------------------------------------------------------------------------------------
// Smaller problems.  Two kernels whose waves share the k dimension instead of cutting the tile
// further, so that few tiles still keep a CU's matrix pipes and its load path busy; both end in
// stream_tile, which takes the fp32 sums from LDS.
// ------------------------------------------------------------------------------------------

// The tile's fp32 sums lie in LDS as COPIES addends of BM rows of BN + 4 floats (the pad spreads the
// 16-byte accumulator writes of 16 rows over all banks).  All NT threads add the copies in order, apply
// the epilogue and store 16-byte pieces, consecutive lanes along a row; V^T pieces run along m.
// What bounds it is latency: piece after piece, each with its own chain of row number, stored feature and x, took FFN2 of
// 700 rows of 512 channels from 12.4 to 13.3 us, of 1500 x 768 from 26.3 to 28.4, of 8775 x 1920 from 246.7 to 259.0.
template <int EPI, int BM, int BN, int NT, int COPIES>
__device__ __forceinline__ void stream_tile(const GemmArgs& g, const float* tile, int m0, int n0, int tid) {
  constexpr int LDT = BN + 4, PIECES = BN / 8;
  const bool use_rows = EPI != EPI_PLAIN && EPI != EPI_GELU && g.rows != nullptr;
  const int n_rowmajor = EPI == EPI_QKV ? 2 * g.d : g.n;     // columns stored along n
  const bool gated = (EPI == EPI_SCATTER || EPI == EPI_SCATTER_ADD) && g.gate_v != nullptr;
  const bool add_x = EPI == EPI_SCATTER_ADD && g.x != nullptr;
  // BATCH pieces of a thread side by side, everything they need from memory asked for before the first is stored: row
  // numbers, then gates, stored features and x one latency later (addresses past the end are clamped, so that no branch
  // lies between the loads).
  constexpr int PER_THREAD = (BM * PIECES + NT - 1) / NT, BATCH = PER_THREAD < 4 ? PER_THREAD : PER_THREAD % 3 == 0 ? 3 : 4;
  for (int p0 = tid; p0 < BM * PIECES && n0 < n_rowmajor; p0 += BATCH * NT) {
    int ml[BATCH], nl[BATCH], n[BATCH];
    bool ok[BATCH];
    int64_t row[BATCH];
    u32x4_t bias[BATCH], gate[BATCH], old[BATCH];
    u32x4_t xraw[BATCH][2];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int p = p0 + b * NT;
      ml[b] = p / PIECES;
      nl[b] = (p - ml[b] * PIECES) * 8;
      ok[b] = p < BM * PIECES && m0 + ml[b] < g.m && n0 + nl[b] < n_rowmajor;
      ml[b] = min(ml[b], BM - 1);
      n[b] = min(n0 + nl[b], n_rowmajor - 8);
      const int m = min(m0 + ml[b], g.m - 1);
      row[b] = use_rows ? g.rows[m] : m;
    }
    auto at = [](const void* p, int64_t bytes) { return *reinterpret_cast<const u32x4_t*>(static_cast<const char*>(p) + bytes); };
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      bias[b] = at(g.bias, n[b] * 2);
      if (EPI == EPI_SCATTER_ADD) old[b] = at(g.c, (row[b] * g.n + n[b]) * 2);
    }
    if (gated) {
#pragma unroll
      for (int b = 0; b < BATCH; ++b) gate[b] = at(row[b] < g.n_text ? g.gate_t : g.gate_v, n[b] * 2);
    }
    if (add_x && g.x_fp32) {
#pragma unroll
      for (int b = 0; b < BATCH; ++b) {
        xraw[b][0] = at(g.x, (row[b] * g.n + n[b]) * 4);
        xraw[b][1] = at(g.x, (row[b] * g.n + n[b]) * 4 + 16);
      }
    } else if (add_x) {
#pragma unroll
      for (int b = 0; b < BATCH; ++b) xraw[b][0] = at(g.x, (row[b] * g.n + n[b]) * 2);
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      float v[8];
      ResidIO<float>::load8(tile + ml[b] * LDT + nl[b], v);
#pragma unroll
      for (int c = 1; c < COPIES; ++c) {
        float w[8];
        ResidIO<float>::load8(tile + (c * BM + ml[b]) * LDT + nl[b], w);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += w[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) { v[2 * e] += unpack_lo(bias[b][e]); v[2 * e + 1] += unpack_hi(bias[b][e]); }
      if (gated) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[2 * e] *= unpack_lo(gate[b][e]); v[2 * e + 1] *= unpack_hi(gate[b][e]); }
      }
      bf16_t* dst = g.c + row[b] * g.n + n[b];
      if (EPI == EPI_QKV) {
        if (n[b] < g.d) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] *= g.q_scale;
          dst = g.c + (int64_t)(m0 + ml[b]) * g.d + n[b];
        } else {
          dst = g.k_out + row[b] * g.d + (n[b] - g.d);
        }
      }
      if (EPI == EPI_GELU) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = gelu_tanh(v[e]);
      }
      if (EPI == EPI_SCATTER_ADD) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[2 * e] += unpack_lo(old[b][e]); v[2 * e + 1] += unpack_hi(old[b][e]); }
      }
      u32x4_t out;
#pragma unroll
      for (int e = 0; e < 4; ++e) out[e] = pack_bf16x2_hw(v[2 * e], v[2 * e + 1]);
      if (ok[b]) *reinterpret_cast<u32x4_t*>(dst) = out;
      if (add_x) {
        // residual add with the feature as stored (rounded), so x matches x += S done afterwards
        u32x4_t lo, hi;
        if (g.x_fp32) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float f = (e & 1) ? unpack_hi(out[e >> 1]) : unpack_lo(out[e >> 1]), h = (e & 1) ? unpack_hi(out[2 + (e >> 1)]) : unpack_lo(out[2 + (e >> 1)]);
            lo[e] = __float_as_uint(__uint_as_float(xraw[b][0][e]) + f);
            hi[e] = __float_as_uint(__uint_as_float(xraw[b][1][e]) + h);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            lo[e] = pack_bf16x2(unpack_lo(xraw[b][0][e]) + unpack_lo(out[e]), unpack_hi(xraw[b][0][e]) + unpack_hi(out[e]));
        }
        if (ok[b]) {
          char* xp = static_cast<char*>(g.x) + (row[b] * g.n + n[b]) * (g.x_fp32 ? 4 : 2);
          *reinterpret_cast<u32x4_t*>(xp) = lo;
          if (g.x_fp32) *reinterpret_cast<u32x4_t*>(xp + 16) = hi;
        }
      }
    }
  }
  if (EPI == EPI_QKV && n0 + BN > 2 * g.d) {
    auto value = [&](int ml, int nl) {
      float v = tile[ml * LDT + nl];
#pragma unroll
      for (int c = 1; c < COPIES; ++c) v += tile[(c * BM + ml) * LDT + nl];
      return v;
    };
    if (use_rows) {
      // scattered columns: lanes along m, whose tokens are neighbours in a V^T row; a thread's row stays the same from
      // column to column where the threads are a multiple of the rows, and eight columns go side by side
      constexpr int COLS = 8;
      constexpr bool SAME_ROW = NT % BM == 0;
      int64_t token = 0;
      if (SAME_ROW) token = g.rows[min(m0 + tid % BM, g.m - 1)];
      for (int u0 = tid; u0 < BM * BN; u0 += COLS * NT) {
        int nl[COLS], ml[COLS];
        int64_t at[COLS];
        float bias[COLS];
        bool ok[COLS];
#pragma unroll
        for (int i = 0; i < COLS; ++i) {
          const int u = min(u0 + i * NT, BM * BN - 1);
          nl[i] = u / BM;
          ml[i] = u - nl[i] * BM;
          const int n = n0 + nl[i], m = m0 + ml[i];
          ok[i] = u0 + i * NT < BM * BN && m < g.m && n >= 2 * g.d && n < g.n;
          bias[i] = bf16_to_f32(g.bias[min(n, g.n - 1)]);
          at[i] = (int64_t)(n - 2 * g.d) * g.ld_vt + (SAME_ROW ? token : (int64_t)g.rows[min(m, g.m - 1)]);
        }
        bf16_t v[COLS];
#pragma unroll
        for (int i = 0; i < COLS; ++i) v[i] = f32_to_bf16_hw(value(ml[i], nl[i]) + bias[i]);
#pragma unroll
        for (int i = 0; i < COLS; ++i)
          if (ok[i]) g.vt_out[at[i]] = v[i];
      }
    } else {
      // eight columns x BM/8 pieces of eight rows at a time
      for (int u = tid; u < BM / 8 * BN; u += NT) {
        const int nl = u / BM * 8 + u % 8, ml = u / 8 % (BM / 8) * 8, n = n0 + nl, m = m0 + ml;
        if (m >= g.m || n < 2 * g.d || n >= g.n) continue;
        const float b = bf16_to_f32(g.bias[n]);
        bf16_t* dst = g.vt_out + (int64_t)(n - 2 * g.d) * g.ld_vt + m;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = value(ml + e, nl) + b;
        if (m + 8 <= g.m) {
          u32x4_t out;
#pragma unroll
          for (int e = 0; e < 4; ++e) out[e] = pack_bf16x2_hw(v[2 * e], v[2 * e + 1]);
          *reinterpret_cast<u32x4_t*>(dst) = out;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (m + e < g.m) dst[e] = f32_to_bf16_hw(v[e]);
        }
      }
    }
  }
}

// Tiles (of less than 256 x 256) of the last round cut along k: slots 0 .. full_items - 1 are whole work items, the `tiles`
// slots after them are cut in `chunks`, whose sums the workgroup that arrives last adds up (one counter a tile, one block
// of BM x BN floats a chunk).
constexpr int MOST_CHUNKS = 8;
struct Cut {
  int32_t full_items, tiles, chunks;
  float* parts;
  uint32_t* arrivals;
};

// workgroup id -> tile slot and k-chunk: all first chunks of the cut tiles, then all second ones, ..., so that the chunks
// of a tile stay on the XCD that owns its range of tiles (slots are a multiple of 8)
struct CutItem { int slot, chunk, n_chunks; };
__device__ __forceinline__ CutItem cut_item(const Cut& cut) {
  const int r = (int)blockIdx.x - cut.full_items;
  if (r < 0) return {(int)blockIdx.x, 0, 1};
  return {cut.full_items + r % cut.tiles, r / cut.tiles, cut.chunks};
}

// The workgroup's chunk of a tile, PIECES floatx4 of each of NT threads at piece(i) in LDS, becomes part of the tile's
// sum; true for the workgroup that arrives last, which then finds the whole sum there, added in the order of the chunks.
// All chunks' pieces are asked for two at a time: the loads' latency is what this costs.
template <int PIECES, int NT, typename Piece>
__device__ __forceinline__ bool share_sum(const Cut& cut, const CutItem& it, Piece piece, int tid, uint32_t* word) {
  constexpr int PART = PIECES * NT * 16, N = 2;
  const int tile = it.slot - cut.full_items;
  const __amdgpu_buffer_rsrc_t rs = parts_rsrc(cut.parts + (size_t)tile * it.n_chunks * (PART / 4), (uint32_t)it.n_chunks * PART);
#pragma unroll
  for (int i = 0; i < PIECES; ++i) store_part(rs, (uint32_t)it.chunk * PART + (i * NT + tid) * 16, *piece(i));
  if (!last_to_arrive(cut.arrivals + tile, it.n_chunks, word)) return false;
#pragma unroll 2
  for (int h = 0; h < PIECES; h += N) {
    floatx4_t v[MOST_CHUNKS][N];
#pragma unroll
    for (int c = 0; c < MOST_CHUNKS; ++c)
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (c < it.n_chunks) v[c][i] = load_part(rs, (uint32_t)c * PART + ((h + i) * NT + tid) * 16);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      floatx4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < MOST_CHUNKS; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c < it.n_chunks) sum[e] += v[c][i][e];
      *piece(h + i) = sum;
    }
  }
  __syncthreads();
  return true;
}

// BM x BN tile, eight waves: 2 x 2 sub-tiles, each computed by two waves that take one half of every
// 64-wide k stage.  The sub-tile is then large (few LDS reads a flop) with two waves on every SIMD.
// Stages go global -> LDS into a ring of RING slots, filled RING - 1 stages ahead, one barrier a stage;
// a slot holds the BM rows of A, then the BN rows of W, in the layout of the 256 x 256 kernel.
// What bounds it: the fills (48 KB a stage at 192 x 192, two stages on their way; 1.13 PFLOP/s with all
// CUs at work at k = 12288) and, at k = 3072, start-up and epilogue, about 7 of 50 us.  Kernel times of FFN2 after
// the kernel that writes its rows, against 256 x 256 or the earlier 128 x 128 tiles: 4485 rows at hidden 1920
// 174 -> 124 us (192 x 192), 1755 rows at hidden 3072 202 -> 153 (128 x 192), 2925 rows 241, fix-up included, -> 194.
template <int BM, int BN>
struct HalfK {
  static constexpr int STAGE = (BM + BN) * 128;                          // bytes
  static constexpr int RING = 163840 / STAGE < 4 ? 163840 / STAGE : 4;
  static constexpr int TILE_BYTES = BM * (BN + 4) * 4 + 16;               // and a word for last_to_arrive
  static constexpr int LDS = RING * STAGE > TILE_BYTES ? RING * STAGE : TILE_BYTES;
};

template <int BM, int BN, int EPI, bool CUT>
__global__ __launch_bounds__(512) void gemm_halfk_kernel(GemmArgs g, int tiles_m, int tiles_n, int per_xcd, int group_m, Cut cut) {
  using C = HalfK<BM, BN>;
  constexpr int MB = BM / 64, NB = BN / 64;            // 32 x 32 blocks of a wave's BM/2 x BN/2 sub-tile
  constexpr int NF = (BM + BN) / 64;                   // 1 KB fills of a wave per stage
  constexpr int RING = C::RING, STAGE = C::STAGE;
  static_assert(BM % 64 == 0 && BN % 64 == 0 && RING >= 3 && NF <= MB * NB + 2, "tile shape");
  const CutItem it = CUT ? cut_item(cut) : CutItem{(int)blockIdx.x, 0, 1};
  int m0, n0;
  if (!tile_origin(it.slot, BM, BN, tiles_m, tiles_n, per_xcd, group_m, m0, n0)) return;

  extern __shared__ u32x4_t smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);             // waves w and w+4 share a SIMD
  const int wm0 = (wave & 1) * (BM / 2), wn0 = ((wave >> 1) & 1) * (BN / 2), kg = wave >> 2;
  const int lr = lane & 31, lh = lane >> 5;

  // fills: this wave's blocks of eight rows are wave + 8i of the slot's (BM + BN) / 8
  const uint32_t row_bytes = (uint32_t)g.k * 2u;
  const u32x4_t rsA = rsrc_words(g.a, (uint32_t)g.m * row_bytes);
  const u32x4_t rsB = rsrc_words(g.w, (uint32_t)g.n * row_bytes);
  uint32_t voff[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int row = (wave + 8 * i) * 8 + (lane >> 3);
    const int chunk = (lane & 7) ^ ((row >> 1) & 7);
    voff[i] = (uint32_t)(i < BM / 64 ? m0 + row : n0 + row - BM) * row_bytes + chunk * 16;
  }
  const int n_stages = g.k / SBK;
  const int stage_begin = it.chunk * n_stages / it.n_chunks, stage_end = (it.chunk + 1) * n_stages / it.n_chunks;
  auto fill = [&](int slot, int stage, int i) {
    lds_fill(i < BM / 64 ? rsA : rsB, lds0 + wave * 1024 + i * 8192 + (uint32_t)slot * STAGE, voff[i],
             (uint32_t)min(stage, stage_end - 1) * (SBK * 2));           // (past the end: the last stage again, unread)
  };

  const char* lbase = reinterpret_cast<const char*>(smem);
  const char *fa_ks[2], *fb_ks[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int off = lr * 128 + (((4 * kg + 2 * s + lh) ^ ((lr >> 1) & 7)) * 16);
    fa_ks[s] = lbase + wm0 * 128 + off;
    fb_ks[s] = lbase + (BM + wn0) * 128 + off;
  }
  auto frag = [&](const char* base, int slot_off, int i) {
    u32x4_t t = *reinterpret_cast<const u32x4_t*>(base + slot_off + i * 4096);
    return *reinterpret_cast<bf16x8_t*>(&t);
  };

  floatx16_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  bf16x8_t fa[2][MB], fb[2][NB];
  {
    u32x4_t z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < MB; ++i) fa[1][i] = *reinterpret_cast<bf16x8_t*>(&z);
#pragma unroll
    for (int j = 0; j < NB; ++j) fb[1][j] = *reinterpret_cast<bf16x8_t*>(&z);
  }
  auto mma_one = [&](int set, int x) {
    const int i = x / NB, j = x % NB;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int s = 0; s < RING - 1; ++s)
#pragma unroll
    for (int i = 0; i < NF; ++i) fill(s, stage_begin + s, i);
  int slot = 0;
  for (int t = stage_begin; t < stage_end; ++t) {
    // all but the fills of the RING - 2 newest stages have landed: stage t is in LDS; every wave's
    // fragment reads of stage t-1 are complete, so its slot can be filled again
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((RING - 2) * NF) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    const int so = slot * STAGE, refill = slot == 0 ? RING - 1 : slot - 1;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      // MFMAs of the previous slice (set s^1) while the fragments of this one arrive in set s
      constexpr int STEPS = MB * NB > MB + NB ? MB * NB : MB + NB;
#pragma unroll
      for (int x = 0; x < STEPS; ++x) {
        if (s == 0 && x < NF) fill(refill, t + RING - 1, x);
        if (s == 0 && x == STEPS - 1) {
#pragma unroll
          for (int y = STEPS; y < NF; ++y) fill(refill, t + RING - 1, y);
        }
        // A and W fragments alternate: the MFMAs need (0,0), (0,1), ... first
        if (x == 0) fa[s][0] = frag(fa_ks[s], so, 0);
        else if (x <= NB) fb[s][x - 1] = frag(fb_ks[s], so, x - 1);
        else if (x < MB + NB) fa[s][x - NB] = frag(fa_ks[s], so, x - NB);
        if (x < MB * NB) mma_one(s ^ 1, x);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    slot = slot == RING - 1 ? 0 : slot + 1;
  }
#pragma unroll
  for (int x = 0; x < MB * NB; ++x) mma_one(1, x);

  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();                       // every wave is done with the ring, and no fill is in flight
  float* tile = reinterpret_cast<float*>(smem);
  constexpr int LDT = BN + 4;
  float* mine = tile + (wm0 + lr) * LDT + wn0 + 4 * lh;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (kg == half) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            floatx4_t* p = reinterpret_cast<floatx4_t*>(mine + 32 * i * LDT + 32 * j + 8 * q);
            floatx4_t v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            if (half == 1) {
              const floatx4_t o = *p;
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] += o[e];
            }
            *p = v;
          }
    }
    __syncthreads();
  }
  if constexpr (CUT) {
    auto piece = [&](int i) { const int p = i * 512 + tid; return reinterpret_cast<floatx4_t*>(tile + p / (BN / 4) * LDT + p % (BN / 4) * 4); };
    if (it.n_chunks > 1 && !share_sum<BM * BN / 4 / 512, 512>(cut, it, piece, tid, reinterpret_cast<uint32_t*>(tile + BM * LDT))) return;
  }
  stream_tile<EPI, BM, BN, 512, 1>(g, tile, m0, n0, tid);
}

// 64 x 64 tile, four waves, each of which computes the whole tile over its own quarter of k from a
// ring of its own: no barrier until the four partial sums meet in LDS, and at k <= 512 every byte
// a wave needs is requested before it waits for the first.  For problems that leave most CUs without
// a larger tile; what bounds them is the chain of load latencies along k, here a quarter as long.
// Kernel times against 128 x 128 tiles with register staging: FFN2 of 326 rows at hidden 256 30.4 -> 7.4 us, of 691
// rows at hidden 1024 50.3 -> 16.2; QKV of 326 listed rows at hidden 256 14.8 -> 6.9.
constexpr int QK_STAGE = 128 * 128;                      // 64 rows of A, 64 rows of W
constexpr int QK_RING = 2;
constexpr int QK_LDS = 4 * QK_RING * QK_STAGE;
static_assert(4 * 64 * 68 * 4 <= QK_LDS, "the four partial tiles must fit");

template <int EPI, bool CUT>
__global__ __launch_bounds__(256) void gemm_quarterk_kernel(GemmArgs g, int tiles_m, int tiles_n, int per_xcd, int group_m, Cut cut) {
  const CutItem it = CUT ? cut_item(cut) : CutItem{(int)blockIdx.x, 0, 1};
  int m0, n0;
  if (!tile_origin(it.slot, 64, 64, tiles_m, tiles_n, per_xcd, group_m, m0, n0)) return;
  extern __shared__ u32x4_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  char* ring = reinterpret_cast<char*>(smem) + wave * (QK_RING * QK_STAGE);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) void*)ring);

  const uint32_t row_bytes = (uint32_t)g.k * 2u;
  const u32x4_t rsA = rsrc_words(g.a, (uint32_t)g.m * row_bytes);
  const u32x4_t rsB = rsrc_words(g.w, (uint32_t)g.n * row_bytes);
  // rows 8i + lane/8 of either operand; the swizzle term repeats every 16 rows
  uint32_t voffA[2], voffB[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = i * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
    voffA[i] = (uint32_t)(m0 + row) * row_bytes + chunk * 16;
    voffB[i] = (uint32_t)(n0 + row) * row_bytes + chunk * 16;
  }
  const int n_stages = g.k / SBK;
  const int first = it.chunk * n_stages / it.n_chunks, mine = (it.chunk + 1) * n_stages / it.n_chunks - first;
  const int begin = first + wave * mine / 4, end = first + (wave + 1) * mine / 4;
  auto fill = [&](int slot, int stage) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t row16 = (uint32_t)(i >> 1) * 16u * row_bytes;
      lds_fill(rsA, lds0 + slot * QK_STAGE + i * 1024, voffA[i & 1] + row16, (uint32_t)stage * (SBK * 2));
      lds_fill(rsB, lds0 + slot * QK_STAGE + 8192 + i * 1024, voffB[i & 1] + row16, (uint32_t)stage * (SBK * 2));
    }
  };

  floatx16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  if (begin < end) fill(0, begin);
  if (begin + 1 < end) fill(1, begin + 1);
  for (int t = begin; t < end; ++t) {
    const int slot = (t - begin) & 1;
    if (t + 1 < end) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");   // the 16 newest fills are stage t+1
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const char* base = ring + slot * QK_STAGE + lr * 128;
    bf16x8_t fa[4][2], fb[4][2];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int c = ((2 * ks + lh) ^ ((lr >> 1) & 7)) * 16;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        u32x4_t ta = *reinterpret_cast<const u32x4_t*>(base + i * 4096 + c);
        u32x4_t tb = *reinterpret_cast<const u32x4_t*>(base + 8192 + i * 4096 + c);
        fa[ks][i] = *reinterpret_cast<bf16x8_t*>(&ta);
        fb[ks][i] = *reinterpret_cast<bf16x8_t*>(&tb);
      }
    }
    if (t + 2 < end) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                  // the slot has been read
      __builtin_amdgcn_sched_barrier(0);
      fill(slot, t + 2);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
  }
  __syncthreads();                       // every wave has read its last stage: no fill is in flight
  float* tile = reinterpret_cast<float*>(smem);
  float* sums = tile + (wave * 64 + lr) * 68 + 4 * lh;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        floatx4_t v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        *reinterpret_cast<floatx4_t*>(sums + 32 * i * 68 + 32 * j + 8 * q) = v;
      }
  __syncthreads();
  if constexpr (CUT) {
    if (it.n_chunks > 1) {
      // (the waves' quarters are added first, into the first one's place)
      auto piece = [&](int c, int i) { return reinterpret_cast<floatx4_t*>(tile + (c * 64 + i * 16 + tid / 16) * 68 + tid % 16 * 4); };
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        floatx4_t v = *piece(0, i);
#pragma unroll
        for (int c = 1; c < 4; ++c) {
          const floatx4_t w = *piece(c, i);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += w[e];
        }
        *piece(0, i) = v;
      }
      if (!share_sum<4, 256>(cut, it, [&](int i) { return piece(0, i); }, tid, reinterpret_cast<uint32_t*>(tile + 4 * 64 * 68))) return;
      stream_tile<EPI, 64, 64, 256, 1>(g, tile, m0, n0, tid);
      return;
    }
  }
  stream_tile<EPI, 64, 64, 256, 4>(g, tile, m0, n0, tid);
}

// LayerNorm and the 64 x 64 tile in one kernel, for models of at most 256 channels: the whole k extent of both
// operands lies in LDS, W arriving by direct loads while the waves normalise their 64 / WAVES rows each (LPR
// lanes a row, eight elements a lane) and round them to bf16 as the stand-alone LayerNorm does.
// What bounds it: the latency of the row loads and of the two reductions (a wave's rows are reduced side by
// side, step by step), then of the short walk along k.  326 rows, 256 channels: 3.4 (LayerNorm) + 5.8 us (QKV) in two
// launches, 6.9 in one; the interval of the 42-layer model of that size 2430 -> 2215 us, of the 128-channel model 203 -> 171.
template <int EPI, typename XT, int LPR, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void gemm_ln_kernel(GemmArgs g, LnInput ln, int tiles_m, int tiles_n, int per_xcd, int group_m) {
  int m0, n0;
  if (!tile_origin(blockIdx.x, 64, 64, tiles_m, tiles_n, per_xcd, group_m, m0, n0)) return;
  extern __shared__ u32x4_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)smem;
  const int n_stages = g.k / SBK;                      // 64 k elements of 64 rows: 8 KB, swizzled as everywhere here
  char* lds_a = reinterpret_cast<char*>(smem);
  const int w_off = n_stages * 8192;

  // W: blocks of eight rows of one stage, in turn to the waves
  const uint32_t row_bytes = (uint32_t)g.k * 2u;
  const u32x4_t rsB = rsrc_words(g.w, (uint32_t)g.n * row_bytes);
  for (int i = wave; i < n_stages * 8; i += WAVES) {
    const int row = (i & 7) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
    lds_fill(rsB, lds0 + w_off + i * 1024, (uint32_t)(n0 + row) * row_bytes + chunk * 16, (uint32_t)(i >> 3) * (SBK * 2));
  }

  // A: rows of the residual stream (plus the branch feature), normalised
  constexpr int ROWS = 64 / WAVES, PER_PASS = 64 / LPR, BATCH = ROWS / PER_PASS;     // rows of a wave, of a pass; passes
  static_assert(BATCH >= 1 && BATCH * PER_PASS == ROWS, "whole passes");
  const int c = lane % LPR;                            // this lane's 8-element piece of a row
  const bool in_row = c * 8 < g.k;
  float gain[8], bias[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) gain[e] = bias[e] = 0.f;
  if (in_row) {
    ResidIO<bf16_t>::load8(ln.gain + c * 8, gain);
    ResidIO<bf16_t>::load8(ln.bias + c * 8, bias);
  }
  // (bf16 pairs: shift and scale of the video stream, then of the text stream)
  u32x4_t mod[4];
  const bool modulated = ln.mod.scale_v != nullptr;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    mod[i] = u32x4_t{0u, 0u, 0u, 0u};
    const bf16_t* p = i == 0 ? ln.mod.shift_v : i == 1 ? ln.mod.scale_v : i == 2 ? ln.mod.shift_t : ln.mod.scale_t;
    if (modulated && in_row) mod[i] = *reinterpret_cast<const u32x4_t*>(p + c * 8);
  }
  const float inv_k = 1.0f / (float)g.k;
  int src[BATCH];
  float v[BATCH][8], sum[BATCH], sq[BATCH];
#pragma unroll
  for (int p = 0; p < BATCH; ++p) {
    const int m = min(m0 + wave * ROWS + p * PER_PASS + lane / LPR, g.m - 1);   // (rows past m: not stored)
    src[p] = ln.rows ? ln.rows[m] : m;
  }
#pragma unroll
  for (int p = 0; p < BATCH; ++p) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[p][e] = 0.f;
    if (in_row) ResidIO<XT>::load8(static_cast<const XT*>(ln.x) + (int64_t)src[p] * g.k + c * 8, v[p]);
  }
  if (ln.add != nullptr && in_row) {
#pragma unroll
    for (int p = 0; p < BATCH; ++p) {
      float a8[8];
      ResidIO<bf16_t>::load8(ln.add + (int64_t)src[p] * g.k + c * 8, a8);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[p][e] += a8[e];
    }
  }
  // the reductions of the batch go step by step together, so that the latency of one hides the others'
#pragma unroll
  for (int p = 0; p < BATCH; ++p) {
    sum[p] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[p] += v[p][e];
  }
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1)
#pragma unroll
    for (int p = 0; p < BATCH; ++p) sum[p] += __shfl_xor(sum[p], o, 64);
#pragma unroll
  for (int p = 0; p < BATCH; ++p) {
    sq[p] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[p][e] -= sum[p] * inv_k;
      sq[p] += in_row ? v[p][e] * v[p][e] : 0.f;
    }
  }
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1)
#pragma unroll
    for (int p = 0; p < BATCH; ++p) sq[p] += __shfl_xor(sq[p], o, 64);
  if (in_row) {
#pragma unroll
    for (int p = 0; p < BATCH; ++p) {
      const float rstd = rsqrtf(sq[p] * inv_k + ln.eps);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[p][e] = v[p][e] * rstd * gain[e] + bias[e];
      if (modulated) {
        const bool text = src[p] < ln.mod.n_text;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t sh = text ? mod[2][e] : mod[0][e], sc = text ? mod[3][e] : mod[1][e];
          v[p][2 * e] = v[p][2 * e] * (1.0f + unpack_lo(sc)) + unpack_lo(sh);
          v[p][2 * e + 1] = v[p][2 * e + 1] * (1.0f + unpack_hi(sc)) + unpack_hi(sh);
        }
      }
      u32x4_t out;
#pragma unroll
      for (int e = 0; e < 4; ++e) out[e] = pack_bf16x2_hw(v[p][2 * e], v[p][2 * e + 1]);
      const int row = wave * ROWS + p * PER_PASS + lane / LPR;
      *reinterpret_cast<u32x4_t*>(lds_a + (c >> 3) * 8192 + row * 128 + ((c & 7) ^ ((row >> 1) & 7)) * 16) = out;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's part of W is in LDS
  __syncthreads();

  // 2 x 2 sub-tiles, each computed by KG waves that share the slices of 16 along k
  constexpr int KG = WAVES / 4;
  const int wm0 = (wave & 1) * 32, wn0 = ((wave >> 1) & 1) * 32, kg = wave >> 2, n_slices = g.k / 16;
  floatx16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  const char* fa = lds_a + (wm0 + lr) * 128;
  const char* fb = lds_a + w_off + (wn0 + lr) * 128;
  for (int t = kg * n_slices / KG; t < (kg + 1) * n_slices / KG; ++t) {
    const int off = (t >> 2) * 8192 + ((2 * (t & 3) + lh) ^ ((lr >> 1) & 7)) * 16;
    u32x4_t ta = *reinterpret_cast<const u32x4_t*>(fa + off);
    u32x4_t tb = *reinterpret_cast<const u32x4_t*>(fb + off);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8_t*>(&tb), *reinterpret_cast<bf16x8_t*>(&ta), acc, 0, 0, 0);
  }
  __syncthreads();                                     // the sums take the operands' place
  float* tile = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    floatx4_t v = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    *reinterpret_cast<floatx4_t*>(tile + (kg * 64 + wm0 + lr) * 68 + wn0 + 8 * q + 4 * lh) = v;
  }
  __syncthreads();
  stream_tile<EPI, 64, 64, WAVES * 64, KG>(g, tile, m0, n0, tid);
}


// The chip runs 256 workgroups at a time, so the last round of tiles may leave most of it
// idle.  Cutting those n_rem tiles into s k-chunks makes the round take ceil(n_rem*s/256)/s of
// a tile's time, and costs a fix-up pass that moves n_rem*s blocks of 256 KB twice (about
// 0.1*n_rem/stages of a tile's time per chunk, measured).  Take the s that minimises the sum,
// with chunks of at least 16 stages, among those whose partial sums fit ws_bytes.  At the
// 17776-token shapes this cuts FFN2 (k = 12288; 3 rounds + 72 tiles) in 3 and makes it 9 %
// faster; the out-projection (k = 3072, the same tiles) is cut in 2 for 3 %, FFN1 (13 rounds +
// 32 tiles) in 3 for 0.4 %.  Returns the number of k-chunks (1: no cut); *n_rem_out: the tile
// slots of the last round, *share what their round takes in units of a whole one.
int choose_k_split(const GemmArgs& g, size_t ws_bytes, int* n_rem_out, double* share = nullptr) {
  const int tiles_m = (g.m + 255) / 256, tiles_n = (g.n + 255) / 256;
  const int slots = (tiles_m * tiles_n + 7) / 8 * 8;
  const int n_rem = slots - slots / 256 * 256;
  *n_rem_out = n_rem;
  // (the QKV projection is never cut: its k is the hidden size, too short to pay at the supported sizes)
  if (g.epilogue == EPI_QKV || n_rem == 0) return 1;
  const int stages = g.k / SBK;
  const int s_max = (int)std::min<size_t>((size_t)std::min(stages / 16, 8), ws_bytes / ((size_t)n_rem * 262144));
  const double per_chunk = 0.1 * n_rem / stages;
  double best = 1.0;
  int split = 1;
  for (int sp = 2; sp <= s_max; ++sp) {
    const double t = (double)((n_rem * sp + 255) / 256) / sp + per_chunk * sp;
    if (t < best - 0.02) { best = t; split = sp; }
  }
  if (share != nullptr) *share = best;
  return split;
}

hipError_t launch_gemm256(const GemmArgs& g, int split, hipStream_t st) {
  int tiles_m = (g.m + 255) / 256, tiles_n = (g.n + 255) / 256;
  int n_tiles = tiles_m * tiles_n;
  int per_xcd = (n_tiles + 7) / 8;
  const int slots = per_xcd * 8;
  // Row tiles walked together by an XCD.  Operand panels of a long-k problem are several MB each,
  // and a problem with few row tiles gives each XCD only a few groups: both do better with short
  // groups (in-session A/B at the 5B shapes: QKV of 4485 rows 4 % faster with 4, the 17776-row
  // problems with k = 3072 0.5 % faster with 8, 16 is 1-7 % slower everywhere).
  const int group_m = (g.k >= 8192 || tiles_m <= 24) ? 4 : 8;
  const SplitK sk = {split > 1 ? slots / 256 * 256 : slots, split, g.splitk_ws};
  const int n_split_tiles = slots - sk.full_items;
  dim3 grid(sk.full_items + n_split_tiles * sk.split), block(512);
#define HERO_GEMM256_LAUNCH(E)                                                                           \
  do {                                                                                                   \
    auto kern = gemm256_kernel<E>;                                                                       \
    auto fix = gemm256_fixup_kernel<E>;                                                                  \
    static std::atomic<uint64_t> lds_allowed{0};                                                         \
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), GEMM256_LDS, lds_allowed);     \
    if (e != hipSuccess) return e;                                                                       \
    hipLaunchKernelGGL(kern, grid, block, GEMM256_LDS, st, g, tiles_m, tiles_n, per_xcd, group_m, sk);   \
    if (n_split_tiles > 0)                                                                               \
      hipLaunchKernelGGL(fix, dim3(n_split_tiles * fixup_waves<E>), dim3(64), STAGE_REGION, st, g, tiles_m, \
                         tiles_n, per_xcd, group_m, sk);                                                         \
  } while (0)
  switch (g.epilogue) {
    case EPI_PLAIN: HERO_GEMM256_LAUNCH(EPI_PLAIN); break;
    case EPI_GELU: HERO_GEMM256_LAUNCH(EPI_GELU); break;
    case EPI_QKV: HERO_GEMM256_LAUNCH(EPI_QKV); break;
    case EPI_SCATTER: HERO_GEMM256_LAUNCH(EPI_SCATTER); break;
    case EPI_SCATTER_ADD: HERO_GEMM256_LAUNCH(EPI_SCATTER_ADD); break;
    default: return hipErrorInvalidValue;
  }
#undef HERO_GEMM256_LAUNCH
  return hipGetLastError();
}

// A distinct type per kernel, so that each has its own record of the devices it was announced on.
template <typename Kernel, Kernel KERN>
hipError_t launch_tiles(const GemmArgs& g, int bm, int bn, int threads, int lds, int chunks, hipStream_t st) {
  static std::atomic<uint64_t> lds_allowed{0};
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(KERN), lds, lds_allowed);
  if (e != hipSuccess) return e;
  const int tiles_m = (g.m + bm - 1) / bm, tiles_n = (g.n + bn - 1) / bn;
  const int per_xcd = (tiles_m * tiles_n + 7) / 8;
  const int group_m = (g.k >= 8192 || tiles_m <= 24) ? 4 : 8;      // as for the 256 x 256 tiles
  const int slots = per_xcd * 8, full = chunks > 1 ? slots / 256 * 256 : slots;
  const Cut cut = {full, slots - full, chunks, g.parts, g.arrivals};
  hipLaunchKernelGGL(KERN, dim3(full + (slots - full) * chunks), dim3(threads), lds, st, g, tiles_m, tiles_n, per_xcd, group_m, cut);
  return hipGetLastError();
}
using TileKernel = void (*)(GemmArgs, int, int, int, int, Cut);

template <int BM, int BN, bool CUT>
hipError_t launch_halfk(const GemmArgs& g, int split, hipStream_t st) {
  constexpr int LDS = HalfK<BM, BN>::LDS;
  switch (g.epilogue) {
    case EPI_PLAIN: return launch_tiles<TileKernel, gemm_halfk_kernel<BM, BN, EPI_PLAIN, false>>(g, BM, BN, 512, LDS, 1, st);
    case EPI_GELU: return launch_tiles<TileKernel, gemm_halfk_kernel<BM, BN, EPI_GELU, CUT>>(g, BM, BN, 512, LDS, split, st);
    case EPI_QKV: return launch_tiles<TileKernel, gemm_halfk_kernel<BM, BN, EPI_QKV, false>>(g, BM, BN, 512, LDS, 1, st);
    case EPI_SCATTER: return launch_tiles<TileKernel, gemm_halfk_kernel<BM, BN, EPI_SCATTER, CUT>>(g, BM, BN, 512, LDS, split, st);
    case EPI_SCATTER_ADD: return launch_tiles<TileKernel, gemm_halfk_kernel<BM, BN, EPI_SCATTER_ADD, CUT>>(g, BM, BN, 512, LDS, split, st);
    default: return hipErrorInvalidValue;
  }
}
template <int BM, int BN>
hipError_t launch_halfk(const GemmArgs& g, int split, hipStream_t st) {
  return split > 1 ? launch_halfk<BM, BN, true>(g, split, st) : launch_halfk<BM, BN, false>(g, 1, st);
}

template <bool CUT>
hipError_t launch_quarterk(const GemmArgs& g, int split, hipStream_t st) {
  switch (g.epilogue) {
    case EPI_PLAIN: return launch_tiles<TileKernel, gemm_quarterk_kernel<EPI_PLAIN, false>>(g, 64, 64, 256, QK_LDS, 1, st);
    case EPI_GELU: return launch_tiles<TileKernel, gemm_quarterk_kernel<EPI_GELU, CUT>>(g, 64, 64, 256, QK_LDS, split, st);
    case EPI_QKV: return launch_tiles<TileKernel, gemm_quarterk_kernel<EPI_QKV, false>>(g, 64, 64, 256, QK_LDS, 1, st);
    case EPI_SCATTER: return launch_tiles<TileKernel, gemm_quarterk_kernel<EPI_SCATTER, CUT>>(g, 64, 64, 256, QK_LDS, split, st);
    case EPI_SCATTER_ADD: return launch_tiles<TileKernel, gemm_quarterk_kernel<EPI_SCATTER_ADD, CUT>>(g, 64, 64, 256, QK_LDS, split, st);
    default: return hipErrorInvalidValue;
  }
}

template <int EPI, typename XT, int LPR, int WAVES>
hipError_t launch_ln_tiles(const GemmArgs& g, const LnInput& ln, hipStream_t st) {
  static std::atomic<uint64_t> lds_allowed{0};
  auto kern = gemm_ln_kernel<EPI, XT, LPR, WAVES>;
  constexpr int OPERANDS = LPR * 8 * 256, SUMS = WAVES / 4 * 64 * 68 * 4;         // k <= LPR * 8 of both operands
  constexpr int LDS = OPERANDS > SUMS ? OPERANDS : SUMS;
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), LDS, lds_allowed);
  if (e != hipSuccess) return e;
  const int tiles_m = (g.m + 63) / 64, tiles_n = (g.n + 63) / 64;
  const int per_xcd = (tiles_m * tiles_n + 7) / 8;
  hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(WAVES * 64), LDS, st, g, ln, tiles_m, tiles_n, per_xcd, 4);
  return hipGetLastError();
}

template <int EPI, typename XT>
hipError_t launch_ln_epilogue(const GemmArgs& g, const LnInput& ln, hipStream_t st) {
  // up to 128 channels eight waves have little to normalise (16 waves measure the same); of 256 channels 16 waves
  // take a lone workgroup of a CU sooner to its end, and two workgroups of eight a CU that has several:
  // interval of 10 layers, 326 rows 753 against 771 us, 2042 rows 1058 against 1034
  const int64_t tiles = (int64_t)((g.m + 63) / 64) * ((g.n + 63) / 64);
  if (g.k <= 128) return launch_ln_tiles<EPI, XT, 16, 8>(g, ln, st);
  return tiles <= 256 ? launch_ln_tiles<EPI, XT, 32, 16>(g, ln, st) : launch_ln_tiles<EPI, XT, 32, 8>(g, ln, st);
}

enum TileKind { TILE_64, TILE_128, TILE_128x192, TILE_192, TILE_256x128, TILE_256 };

// What a round of at most 256 tiles (one per CU) of a kind takes: fixed + stages * (low .. high) us, the
// rate falling from `low` with a nearly empty chip to `high` with all CUs at work (they share the caches,
// the fabric and the power budget).  Fitted to hero_linear timings on 82 .. 17776 rows, n 256 .. 12288,
// k 256 .. 12288, operands out of the caches; per round at k = 3072, full chip: 64 x 64 11 us, 128 x 128 26,
// 128 x 192 38, 256 x 128 48, 192 x 192 50, 256 x 256 77.
// scatter: what the V^T columns of listed rows (two-byte stores) add to a QKV projection, once, or once for every
// 512 tiles (only a third of the tiles have them, and others run meanwhile); fitted to the kernel times of 118 such
// projections, hidden 256 .. 4096, 82 .. 8775 rows.
// Against the kernel times of every kind on 1325 problems (the block's four GEMMs and hero_linear, hidden 256 .. 4096,
// 50 .. 17776 rows, listed and not, each after the kernel that writes its rows) the kind chosen takes on average
// 0.37 % longer than the best; without `scatter` 0.54 %.
struct TileCost { int bm, bn; float fixed, low, high, scatter; };
constexpr TileCost TILE_COST[] = {{64, 64, 2.2f, 0.17f, 0.18f, 5.f},   {128, 128, 3.5f, 0.31f, 0.48f, 7.5f},
                                  {128, 192, 4.5f, 0.43f, 0.70f, 7.f}, {192, 192, 6.f, 0.65f, 0.91f, 10.5f},
                                  {256, 128, 6.f, 0.55f, 0.87f, 9.5f}, {256, 256, 6.f, 0.72f, 1.48f, 7.5f}};

// What it takes workgroups to share tiles cut along k (us): each stores its part, the last to arrive loads them all past
// the caches, at 35 - 40 GB/s a CU.  fill: work items of the round a CU.  Over 345 problems (out-projection, FFN1 and FFN2
// of 45 .. 8775 rows, hidden 320 .. 3072) and every way to cut them, the kind and cut chosen take 0.7 % longer than the best
// on average, 5.1 % without cuts, and never longer than what is chosen without.  FFN2, kernel times in a layer, uncut and cut
// as it is now: 45 x 1536 19.8 -> 12.7 us (64 x 64 in 4), 84 x 1920 24.4 -> 14.4 (64 x 64 in 4), 700 x 1536 41.0 -> 26.7
// (128 x 128 in 3), 1500 x 3072 148 -> 117 (192 x 192 in 2).
double sharing_cost(const TileCost& c, int split, double fill) {
  const double part = (double)(c.bm * c.bn) / 16384.0;          // in units of 64 KB
  return c.bm == 64 ? 1.0 + 0.8 * split + 1.5 * fill : 2.0 + part * (split + 4.5 * fill);
}

// Stages a chunk of a cut tile has at least: fewer do not cover the start of its pipeline.
constexpr int least_stages(const TileCost& c) { return c.bm == 64 ? 4 : 6; }

struct TileChoice {
  TileKind kind;
  int split;      // chunks along k of the last round's tiles (1: not cut)
};

// The kind with the least expected time.  Small problems take the smallest tiles that still fit one
// round (latency along k bounds them), large ones 256 x 256 (least operand traffic a flop), and in between
// the kind whose tile count fills its last round: e.g. FFN2 of 2925 x 3072 is 144 tiles of 256 x 256 but 256 of
// 192 x 192 (241 us against 194), of 691 x 1024 (k = 4096) 16.2 us on 64 x 64 tiles against 28.3 on 128 x 128.
// A problem that has 128 tiles of 256 x 256 keeps them unless another kind is expected to take 1 % less: less than
// that once took FFN1 of 4485 x 3072 from 296 to 303 us and FFN2 of 17776 x 1920 from 530 to 549, both to 192 x 192.
TileChoice choose_tile(const GemmArgs& g) {
  // (a wave's columns of a 256 x 256 tile must lie inside one of the Q / K / V thirds)
  const bool qkv_split_ok = g.epilogue != EPI_QKV || g.d % 128 == 0;
  const bool scattered = g.epilogue == EPI_QKV && g.rows != nullptr;
  const int stages = g.k / SBK;
  const size_t ws_bytes = g.splitk_ws != nullptr ? g.splitk_ws_bytes : 0;
  TileChoice choice = {TILE_128, 1};
  double best = 1e30;
  for (int kind = TILE_64; kind <= TILE_256; ++kind) {
    if (kind == TILE_256 && !qkv_split_ok) continue;
    const TileCost& c = TILE_COST[kind];
    const int64_t tiles = (int64_t)((g.m + c.bm - 1) / c.bm) * ((g.n + c.bn - 1) / c.bn);
    const double full = c.fixed + stages * c.high;
    // `items` work items of `n` stages, at most one a CU at a time
    auto rounds = [&](int64_t items, double n) {
      const double rem = (double)(items % 256) / 256.0;
      return (double)(items / 256) * (c.fixed + n * c.high) + (rem > 0 ? c.fixed + n * (c.low + rem * (c.high - c.low)) : 0.0);
    };
    double t = rounds(tiles, stages);
    int split = 1;
    if (kind == TILE_256) {
      int n_rem = 0;
      double share = 1.0;
      split = choose_k_split(g, ws_bytes, &n_rem, &share);
      if (split > 1) t = (double)(tiles / 256) * full + share * full;
    } else if (g.parts != nullptr && g.epilogue != EPI_QKV) {
      const int64_t n_rem = (tiles + 7) / 8 * 8 % 256;
      const int least = least_stages(c);
      const double uncut = t;
      for (int s = 2; s <= MOST_CHUNKS && stages / s >= least && n_rem > 0 && n_rem * s * c.bm * c.bn * 4 <= (int64_t)g.parts_bytes; ++s) {
        const double cut = (double)(tiles / 256) * full + rounds(n_rem * s, (double)((stages + s - 1) / s)) +
                           sharing_cost(c, s, (double)(n_rem * s) / 256.0);
        if (cut < t && cut < 0.95 * uncut) { t = cut; split = s; }
      }
    }
    if (scattered) t += c.scatter * std::max(1.0, (double)tiles / 512.0);
    const double margin = kind == TILE_256 && tiles >= 128 ? 1.01 : 1.0;
    if (t <= best * margin) { best = t; choice = {(TileKind)kind, split}; }
  }
  return choice;
}

}  // namespace

size_t gemm_wanted_scratch_bytes(const GemmArgs& g) {
  // stated for 256 x 256 tiles wherever the problem has 128 of them, also where a smaller tile is chosen:
  // what a caller has to provide for a shape does not depend on the timings above
  if (g.m <= 0 || g.n <= 0 || g.k <= 0) return 0;
  if ((int64_t)((g.m + 255) / 256) * ((g.n + 255) / 256) < 128) return 0;
  int n_rem = 0;
  const int split = choose_k_split(g, (size_t)-1, &n_rem);
  return split > 1 ? (size_t)n_rem * split * 262144 : 0;
}

// (the last round has at most 248 tiles: 256 are a whole one)
size_t gemm_most_parts_bytes(int m, int n, int k) {
  size_t most = 0;
  for (int kind = TILE_64; kind < TILE_256; ++kind) {
    const TileCost& c = TILE_COST[kind];
    const int64_t slots = std::min<int64_t>(((int64_t)((m + c.bm - 1) / c.bm) * ((n + c.bn - 1) / c.bn) + 7) / 8 * 8, 248);
    const int chunks = std::min(k / SBK / least_stages(c), MOST_CHUNKS);
    if (chunks > 1) most = std::max(most, (size_t)slots * chunks * c.bm * c.bn * 4);
  }
  return most;
}

hipError_t launch_gemm(const GemmArgs& g, hipStream_t st) {
  if (g.m <= 0 || g.n <= 0) return hipSuccess;
  if (g.k <= 0 || g.k % SBK != 0 || g.n % 64 != 0) return hipErrorInvalidValue;
  if (g.epilogue == EPI_QKV && (g.d % 64 != 0 || g.n != 3 * g.d)) return hipErrorInvalidValue;
  // operands are addressed with 32-bit byte offsets
  if (((int64_t)g.m + 512) * g.k * 2 >= (int64_t)1 << 32 || ((int64_t)g.n + 512) * g.k * 2 >= (int64_t)1 << 32)
    return hipErrorInvalidValue;
  const auto [kind, split] = choose_tile(g);
  switch (kind) {
    case TILE_256: return launch_gemm256(g, split, st);
    case TILE_64: return split > 1 ? launch_quarterk<true>(g, split, st) : launch_quarterk<false>(g, 1, st);
    case TILE_128: return launch_halfk<128, 128>(g, split, st);
    case TILE_128x192: return launch_halfk<128, 192>(g, split, st);
    case TILE_192: return launch_halfk<192, 192>(g, split, st);
    case TILE_256x128: return launch_halfk<256, 128>(g, split, st);
  }
  return hipErrorInvalidValue;
}

void gemm_route(const GemmArgs& g, int* tile_m, int* tile_n, int* k_chunks) {
  const auto [kind, split] = choose_tile(g);
  *tile_m = TILE_COST[kind].bm;
  *tile_n = TILE_COST[kind].bn;
  *k_chunks = split;
}

// Every column tile normalises its rows again, so the line lies where the chip's rounds of tiles cost more in that way
// than a launch and a pass over the rows in between.  Four layers, two kernels against one: 128 channels, FFN 512,
// 17576 rows 807 -> 771 us (2200 tiles), FFN 2048, 2050 rows 216 -> 197 (1056 tiles), but 8126 rows 376 -> 394 (4064)
// and FFN 8192, 17576 rows 1576 -> 1889 (35200); 192 channels, FFN 1536, 1306 rows 186 -> 169 (504), 2050 rows 214 -> 215
// (792); 256 channels, FFN 1024, 1306 rows 182 -> 167 (336), 8126 rows 515 -> 549 (2032); from 320 channels on it loses.
bool gemm_takes_ln(const GemmArgs& g) {
  if (g.epilogue != EPI_QKV && g.epilogue != EPI_GELU) return false;
  const int64_t tiles = (int64_t)((g.m + 63) / 64) * ((g.n + 63) / 64);
  if (g.k <= 128) return tiles <= 1300 + g.m / (g.k <= 64 ? 6 : 4);
  return g.k <= 256 && tiles <= (g.k <= 192 ? 600 : 500) + g.m / 30;
}

hipError_t launch_gemm_ln(const GemmArgs& g, const LnInput& ln, hipStream_t st) {
  if (g.m <= 0 || g.n <= 0) return hipSuccess;
  if (!gemm_takes_ln(g) || g.k <= 0 || g.k % SBK != 0 || g.n % 64 != 0) return hipErrorInvalidValue;
  if (g.epilogue == EPI_QKV && (g.d % 64 != 0 || g.n != 3 * g.d)) return hipErrorInvalidValue;
  if (g.epilogue == EPI_QKV) return ln.x_fp32 ? launch_ln_epilogue<EPI_QKV, float>(g, ln, st) : launch_ln_epilogue<EPI_QKV, bf16_t>(g, ln, st);
  return ln.x_fp32 ? launch_ln_epilogue<EPI_GELU, float>(g, ln, st) : launch_ln_epilogue<EPI_GELU, bf16_t>(g, ln, st);
}
