// Block-scaled NVFP4 GEMM with BF16 output for gfx950.
//
//   out[m][n] = bf16( fp32( aA * aB * sum_k (sA qA)[m][k] (sB qB)[n][k] + bias[n] ) )
//
// How the E4M3-per-16 scales are applied.  CDNA4's scaled matrix
// instructions take one power-of-two (E8M0) scale per 32 K-elements, while an
// NVFP4 element decodes to q * s with an E4M3 s: up to 2 + 4 = 6 significant
// bits per operand, more than any FP4/FP6/FP8 matrix input carries.  So the
// operands stay packed (0.5 B/element codes + 1/16 B/element scales) in HBM
// and L2, and each element is dequantized exactly to FP16 (q * s has at most
// 6 significant bits and lies in [2^-10, 2688]) before the FP16 matrix cores
// (v_mfma_f32_32x32x16_f16, FP32 accumulation) consume it.  Every product
// (sA qA)(sB qB) is exact; only the FP32 sums, the epilogue FMA and the BF16
// rounding round.  The per-tensor scales and the bias are applied once, in
// the epilogue.
//
// The dequantization is two instructions per pair of elements: the hardware
// FP4 converter (which applies only the exponent of its scale operand) with
// scale 2^8 gives 256 q exactly in FP16, and one packed FP16 multiply by the
// E4M3 byte shifted into an FP16 bit pattern (which reads as s * 2^-8, the
// two formats' mantissa fields being aligned and E4M3 subnormals landing on
// FP16 subnormals) gives q * s exactly.
//
// Two kernels:
//   nvfp4_gemm_lane_kernel (nearly every K; lane_takes): codes travel
//     from HBM into LDS by DMA and each wave dequantizes its own MFMA operands
//     in registers, so LDS carries 0.5 B/element of codes instead of 2 B of
//     FP16 per operand read; with too few tiles for one 256 x 256 tile per
//     CU it runs on 128 x 128 tiles; a last round of at most a quarter of
//     the CUs' worth of 256 x 256 tiles runs in a second launch as their
//     128 x 128 quadrants (launch_gemm_quad), and otherwise a last round of
//     at most half the CUs' worth as two K halves per tile (SplitK);
//   nvfp4_gemm_kernel (the rest): the workgroup converts each stage once
//     into FP16 tiles in LDS, which all waves read.
// Few tokens take one of two kernels of their own, chosen here by estimated
// time: 64 x 64 tiles (gemm_small.hip; K % 128 == 0, at most one tile per
// CU) or 32 x 32 tiles with the K stages dealt to the four waves of a
// workgroup (gemm_wavek.hip).
#include <type_traits>

#include "device_common.h"
#include "nvfp4_gemm_common.h"
#include "solfp4.h"
#include "kernels.h"

namespace solfp4 {

// ---------------------------------------------------------------------------
// nvfp4_gemm_kernel: workgroup-shared dequantization, any K % 16 == 0.
//
// Per K stage each pair of threads owns one row of the A tile and one row of
// the B tile, each thread converting 32 codes of each to FP16 and storing
// them to LDS, where all eight waves read their MFMA operands: each element
// is converted once per 256 x 256 output tile.  Tiling: 8 waves (2 x 4, two
// per SIMD so one wave's waits are covered by the other's MFMAs), each wave
// owning 128 x 64 (4 x 2 MFMA tiles of 32 x 32); K advances 64 elements
// (4 NVFP4 blocks) per stage.  LDS holds two stages of FP16 A and B tiles
// (rows padded to 144 bytes: conflict-free 16-byte row accesses).  Packed
// codes for stage s+2 are fetched into registers while stage s runs its
// MFMAs and stage s+1 is converted into the other LDS buffer, so each stage
// ends with a single barrier.  The two threads of a row load its 32 code
// bytes (and 4 scale bytes) with one coalesced request.  The MFMA's first
// operand is the weight tile, so each lane's accumulators hold runs of 4
// consecutive output columns of one row; one lane swap with the partner 32
// lanes away turns them into 16-byte runs for the stores.

constexpr int kBM = 256;
constexpr int kBN = 256;
constexpr int kBK = 64;                       // K elements per stage
constexpr int kBlocksPerStage = kBK / 16;     // NVFP4 blocks per row per stage
constexpr int kRowHalves = kBK + 8;           // padded LDS row (144 bytes)
constexpr int kGemmThreads = 512;
constexpr int kWaveTileM = 128;
constexpr int kWaveTileN = 64;
constexpr int kFragsM = kWaveTileM / 32;      // 32x32 MFMA tiles per wave, along M
constexpr int kFragsN = kWaveTileN / 32;      // and along N
constexpr int kSteps = kBK / 16;              // MFMA K-steps per stage

struct Smem {
  _Float16 a[2][kBM * kRowHalves];
  _Float16 b[2][kBN * kRowHalves];
  uint16_t bias[kBN];
};

// 8 E2M1 codes (element 2j in the low nibble of byte j) times the block
// scale, as 4 words of FP16 pairs (elements 2j, 2j+1); s2 holds s * 2^-8 in
// both halves.
__device__ __forceinline__ void dequant8(uint32_t w, uint32_t s2, uint32_t (&d)[4]) {
  const half2_t s = as_h2(s2);
  d[0] = h2_as_u32(__builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 0) * s);
  d[1] = h2_as_u32(__builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 1) * s);
  d[2] = h2_as_u32(__builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 2) * s);
  d[3] = h2_as_u32(__builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 3) * s);
}

// One thread's share of a stage: half a row of one operand, 32 codes (16
// bytes, two NVFP4 blocks).  Scales arrive separately, four stages at a time.
struct HalfRow {
  uint4 c;
};

// Buffer resources for one operand's 256-row tile: rows past the end of the
// matrix fall outside num_records and read as zeros (code 0 with scale 0:
// the value 0), so no load needs a branch.
struct TileSrc {
  __amdgpu_buffer_rsrc_t codes, scales;
  uint32_t code_off, scale_off;   // this thread's half row / row, in bytes
};

__device__ __forceinline__ TileSrc make_tile_src(const uint8_t* codes, const uint8_t* scales,
                                                 int64_t row0, int64_t rows, int64_t K, int t) {
  const int64_t valid = min<int64_t>(rows - row0, 256);
  const int r = t >> 1, h = t & 1;
  TileSrc s;
  s.codes = uniform_rsrc(codes + row0 * (K / 2), valid * (K / 2));
  s.scales = uniform_rsrc(scales + row0 * (K / 16), valid * (K / 16));
  s.code_off = (uint32_t)(r * (K / 2) + 16 * h);
  s.scale_off = (uint32_t)(r * (K / 16));
  return s;
}

// Load this thread's 16 code bytes of `stage`.  kFast: K % 64 == 0 (every
// stage full, 16-byte offsets aligned).  Otherwise two 8-byte loads, and
// blocks past K are zeroed.
template <bool kFast>
__device__ __forceinline__ void load_codes(HalfRow& r, const TileSrc& src, int64_t K, int stage,
                                           int h) {
  const uint32_t co = src.code_off + (uint32_t)stage * (kBK / 2);
  if (kFast) {
    const u32x4_t a = __builtin_amdgcn_raw_buffer_load_b128(src.codes, co, 0, 0);
    r.c = make_uint4(a.x, a.y, a.z, a.w);
  } else {
    const int64_t kb_left = K / 16 - (int64_t)stage * kBlocksPerStage - 2 * h;
    u32x2_t blk[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      blk[j] = __builtin_amdgcn_raw_buffer_load_b64(src.codes, co + 8 * j, 0, 0);
      blk[j] = j < kb_left ? blk[j] : u32x2_t{0, 0};
    }
    r.c = make_uint4(blk[0].x, blk[0].y, blk[1].x, blk[1].y);
  }
}

// The row's 16 scale bytes for stages 4g .. 4g+3 (both threads of a row load
// the same bytes: one coalesced request).  Byte 4j + b is block b of stage
// 4g + j.  Blocks past K are zeroed.
template <bool kFast>
__device__ __forceinline__ u32x4_t load_scales(const TileSrc& src, int64_t K, int g) {
  const uint32_t so = src.scale_off + (uint32_t)g * 16;
  if (kFast && (K / 16) % 16 == 0) {
    return __builtin_amdgcn_raw_buffer_load_b128(src.scales, so, 0, 0);
  } else if (kFast) {
    // 4-byte aligned (K % 64 == 0); stages past K read other rows or zeros
    // and are never converted into a used buffer
    u32x4_t v;
    v.x = __builtin_amdgcn_raw_buffer_load_b32(src.scales, so, 0, 0);
    v.y = __builtin_amdgcn_raw_buffer_load_b32(src.scales, so + 4, 0, 0);
    v.z = __builtin_amdgcn_raw_buffer_load_b32(src.scales, so + 8, 0, 0);
    v.w = __builtin_amdgcn_raw_buffer_load_b32(src.scales, so + 12, 0, 0);
    return v;
  } else {
    const int64_t kb_left = K / 16 - (int64_t)g * 16;
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t b = __builtin_amdgcn_raw_buffer_load_b8(src.scales, so + i, 0, 0);
      w[i / 4] |= (i < kb_left ? b : 0u) << (8 * (i % 4));
    }
    return u32x4_t{w[0], w[1], w[2], w[3]};
  }
}

// Convert block j (0 or 1) of a half row (scale bytes of its two blocks in
// sc2) and store its 16 FP16 values.  The
// E4M3 scale byte shifted into an FP16 bit pattern reads as s * 2^-8 (the
// two formats align their mantissa fields, and E4M3 subnormals become FP16
// subnormals); one exact multiply by 2^8 restores s.
__device__ __forceinline__ void convert_block(const HalfRow& r, uint32_t sc2, int j,
                                              _Float16* dst) {
  const uint32_t c = (sc2 >> (8 * j)) & 0xFFu;
  const uint32_t s2 = (c << 7) | (c << 23);   // s * 2^-8 in both FP16 halves
  const uint32_t w0 = j == 0 ? r.c.x : r.c.z;
  const uint32_t w1 = j == 0 ? r.c.y : r.c.w;
  uint32_t d[4], e[4];
  dequant8(w0, s2, d);
  dequant8(w1, s2, e);
  *reinterpret_cast<uint4*>(dst + 16 * j) = make_uint4(d[0], d[1], d[2], d[3]);
  *reinterpret_cast<uint4*>(dst + 16 * j + 8) = make_uint4(e[0], e[1], e[2], e[3]);
}

// Scheduling of one K-step segment (after its operand reads are fenced
// off): each of the 8 MFMAs is followed by up to 5 VALU instructions of the
// next stage's conversion, and the conversion's 2 LDS stores go last, so the
// conversion runs in the shadow of the matrix pipeline.
__device__ __forceinline__ void interleave_step() {
#pragma unroll
  for (int i = 0; i < kFragsM * kFragsN; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
    __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);   // VALU
    if (i >= 6) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);    // DS write
  }
}

template <bool kFast, bool kVecOut>
__global__ __launch_bounds__(kGemmThreads, 1) void nvfp4_gemm_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const float* __restrict__ a_gs, const uint8_t* __restrict__ b_codes,
    const uint8_t* __restrict__ b_scales, const float* __restrict__ b_gs,
    const uint16_t* __restrict__ bias, uint16_t* __restrict__ out, int64_t M, int64_t N,
    int64_t K) {
  __shared__ Smem smem;

  const int tiles_m = (int)((M + kBM - 1) / kBM);
  const int tiles_n = (int)((N + kBN - 1) / kBN);
  int tm, tn;
  tile_coords(tiles_m, tiles_n, tm, tn);
  const int64_t m0 = (int64_t)tm * kBM;
  const int64_t n0 = (int64_t)tn * kBN;

  const int t = threadIdx.x;
  const int lane = t & (kWave - 1);
  const int wave = t / kWave;
  const int wm = wave >> 2;
  const int wn = wave & 3;
  const int li = lane & 31;
  const int lg = lane >> 5;
  const int h = t & 1;

  floatx16_t acc[kFragsN][kFragsM];
#pragma unroll
  for (int i = 0; i < kFragsN; ++i)
#pragma unroll
    for (int j = 0; j < kFragsM; ++j) acc[i][j] = floatx16_t{};

  const int nstages = (int)((K + kBK - 1) / kBK);
  const TileSrc src_a = make_tile_src(a_codes, a_scales, m0, M, K, t);
  const TileSrc src_b = make_tile_src(b_codes, b_scales, n0, N, K, t);
  // this thread's half row in an LDS stage buffer
  const int my = (t >> 1) * kRowHalves + 32 * h;
  // this thread's two scale bytes of stage s sit in word s%4 of its group's
  // scale registers, at byte offset 2h
  const int sshift = 16 * h;
  HalfRow ca[2], cb[2];
  u32x4_t sa4[2], sb4[2];
  // prologue: scales of stages 0-7, codes of stages 0-1; stage 0 converted
  // into buffer 0
  sa4[0] = load_scales<kFast>(src_a, K, 0);
  sb4[0] = load_scales<kFast>(src_b, K, 0);
  sa4[1] = load_scales<kFast>(src_a, K, 1);
  sb4[1] = load_scales<kFast>(src_b, K, 1);
  load_codes<kFast>(ca[0], src_a, K, 0, h);
  load_codes<kFast>(cb[0], src_b, K, 0, h);
  load_codes<kFast>(ca[1], src_a, K, 1, h);
  load_codes<kFast>(cb[1], src_b, K, 1, h);
  convert_block(ca[0], sa4[0].x >> sshift, 0, &smem.a[0][my]);
  convert_block(ca[0], sa4[0].x >> sshift, 1, &smem.a[0][my]);
  convert_block(cb[0], sb4[0].x >> sshift, 0, &smem.b[0][my]);
  convert_block(cb[0], sb4[0].x >> sshift, 1, &smem.b[0][my]);
  // the tile's bias (+0 without one: fma(alpha, acc, +0) == alpha * acc for
  // every accumulator, which never holds -0)
  if (t < kBN) smem.bias[t] = bias && n0 + t < N ? bias[n0 + t] : (uint16_t)0;
  __syncthreads();

  // One stage, branch free.  P = s % 8 selects the register sets: codes of
  // stage s+1 (converted now into buffer cur^1) are in set (P+1)%2 and the
  // loads of stage s+2 go to set P%2; scales of stage s+1 are in group set
  // ((P+1)/4)%2, and at P == 0 / P == 4 the scales of the group after next
  // are fetched into the set the previous group used.  Past the last stage
  // the loads read zeros or unused data and the conversion fills the buffer
  // nobody reads again.
  auto run_stage = [&](auto phase, int s) {
    constexpr int P = decltype(phase)::value;
    constexpr int kc = P & 1;              // code set loaded now (stage s+2)
    constexpr int kn = (P + 1) & 1;        // code set converted now (stage s+1)
    constexpr int gn = ((P + 1) >> 2) & 1; // scale set of stage s+1
    constexpr int wn_ = (P + 1) & 3;       // word of stage s+1 in its group
    const int cur = s & 1;
    if (P == 0 || P == 4) {
      constexpr int gl = P == 0 ? 1 : 0;   // set receiving group s/4 + 1
      sa4[gl] = load_scales<kFast>(src_a, K, s / 4 + 1);
      sb4[gl] = load_scales<kFast>(src_b, K, s / 4 + 1);
    }
    load_codes<kFast>(ca[kc], src_a, K, s + 2, h);
    load_codes<kFast>(cb[kc], src_b, K, s + 2, h);
    const uint32_t sca = sa4[gn][wn_] >> sshift;
    const uint32_t scb = sb4[gn][wn_] >> sshift;
    const _Float16* sa = smem.a[cur] + (wm * kWaveTileM + li) * kRowHalves + 8 * lg;
    const _Float16* sb = smem.b[cur] + (wn * kWaveTileN + li) * kRowHalves + 8 * lg;
    _Float16* na = &smem.a[cur ^ 1][my];
    _Float16* nb = &smem.b[cur ^ 1][my];
    half8_t af[2][kFragsM], bf[2][kFragsN];
#pragma unroll
    for (int f = 0; f < kFragsM; ++f) af[0][f] = *reinterpret_cast<const half8_t*>(sa + f * 32 * kRowHalves);
#pragma unroll
    for (int f = 0; f < kFragsN; ++f) bf[0][f] = *reinterpret_cast<const half8_t*>(sb + f * 32 * kRowHalves);
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
      const int c = st & 1;
      // operand reads for the next K-step go out first: they have this
      // step's MFMAs to complete
      if (st + 1 < kSteps) {
#pragma unroll
        for (int f = 0; f < kFragsM; ++f)
          af[c ^ 1][f] = *reinterpret_cast<const half8_t*>(sa + f * 32 * kRowHalves + 16 * (st + 1));
#pragma unroll
        for (int f = 0; f < kFragsN; ++f)
          bf[c ^ 1][f] = *reinterpret_cast<const half8_t*>(sb + f * 32 * kRowHalves + 16 * (st + 1));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int fn = 0; fn < kFragsN; ++fn)
#pragma unroll
        for (int fm = 0; fm < kFragsM; ++fm)
          acc[fn][fm] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf[c][fn], af[c][fm], acc[fn][fm], 0, 0, 0);
      // a quarter of the next stage's conversion per K-step
      if (st == 0) convert_block(ca[kn], sca, 0, na);
      if (st == 1) convert_block(ca[kn], sca, 1, na);
      if (st == 2) convert_block(cb[kn], scb, 0, nb);
      if (st == 3) convert_block(cb[kn], scb, 1, nb);
      interleave_step();
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  };

  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  using P2 = std::integral_constant<int, 2>;
  using P3 = std::integral_constant<int, 3>;
  using P4 = std::integral_constant<int, 4>;
  using P5 = std::integral_constant<int, 5>;
  using P6 = std::integral_constant<int, 6>;
  using P7 = std::integral_constant<int, 7>;
  int s = 0;
  for (; s + 8 <= nstages; s += 8) {
    run_stage(P0{}, s);
    run_stage(P1{}, s + 1);
    run_stage(P2{}, s + 2);
    run_stage(P3{}, s + 3);
    run_stage(P4{}, s + 4);
    run_stage(P5{}, s + 5);
    run_stage(P6{}, s + 6);
    run_stage(P7{}, s + 7);
  }
  const int rest = nstages - s;
  if (rest > 0) run_stage(P0{}, s);
  if (rest > 1) run_stage(P1{}, s + 1);
  if (rest > 2) run_stage(P2{}, s + 2);
  if (rest > 3) run_stage(P3{}, s + 3);
  if (rest > 4) run_stage(P4{}, s + 4);
  if (rest > 5) run_stage(P5{}, s + 5);
  if (rest > 6) run_stage(P6{}, s + 6);

  // epilogue: out = bf16(fp32(fma(alpha, acc, bias))), alpha = aA * aB in
  // FP32.  Lane (li, lg) holds, per MFMA tile, row m = li and the column runs
  // 8k + 4lg .. 8k + 4lg + 3 (k = 0..3); swapping halves with the lane 32
  // apart gives each lane two runs of 8 consecutive columns (16-byte
  // stores).  Stores go through a buffer resource covering the tile's valid
  // rows, so rows past M are dropped by the hardware range check; columns
  // past N get an offset beyond the range.
  const float alpha = a_gs[0] * b_gs[0];
  const __amdgpu_buffer_rsrc_t ro = uniform_rsrc(out + m0 * N, min<int64_t>(M - m0, kBM) * N * 2);
#pragma unroll
  for (int fm = 0; fm < kFragsM; ++fm) {
    const uint32_t mrow = (uint32_t)((wm * kWaveTileM + fm * 32 + li) * N);
#pragma unroll
    for (int fn = 0; fn < kFragsN; ++fn) {
      const int nb = wn * kWaveTileN + fn * 32;
      float v[16];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint2 b2 = *reinterpret_cast<const uint2*>(&smem.bias[nb + 8 * k + 4 * lg]);
        const float bv[4] = {__uint_as_float(b2.x << 16), __uint_as_float(b2.x & 0xFFFF0000u),
                             __uint_as_float(b2.y << 16), __uint_as_float(b2.y & 0xFFFF0000u)};
#pragma unroll
        for (int q = 0; q < 4; ++q) v[4 * k + q] = __builtin_fmaf(alpha, acc[fn][fm][4 * k + q], bv[q]);
      }
      uint32_t p[4][2];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        p[k][0] = pack_bf16(v[4 * k], v[4 * k + 1]);
        p[k][1] = pack_bf16(v[4 * k + 2], v[4 * k + 3]);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t r[4];   // 8 columns starting at nb + 16 h + 8 lg
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const auto x = __builtin_amdgcn_permlane32_swap(p[2 * h][d], p[2 * h + 1][d], false, false);
          r[d] = x[0];
          r[2 + d] = x[1];
        }
        const int64_t n = n0 + nb + 16 * h + 8 * lg;
        store_run8<kVecOut>(ro, mrow, n, N, r);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// nvfp4_gemm_lane_kernel: lane-side dequantization, any K % 16 == 0.
//
// Tiling and data movement follow the MXFP4 GEMM: a 2 kWN x 2 kWN output
// tile per workgroup of 4 waves (one per SIMD), each wave owning kWM x kWN:
// 128 x 128 (4 x 4 MFMA tiles of 32 x 32, 256 FP32 accumulators per lane), or,
// for GEMMs with too few 256 x 256 tiles to fill the chip, 64 x 64 (a quarter
// of the work per workgroup) or 128 x 64.  In the last form (kGroups == 2) the
// four waves are two groups that each hold sums of the whole 128 x 128 tile:
// group kg takes stages kg, kg + 2, ..., both groups' codes of a row arrive as
// one 128-byte line, and the groups add their sums through LDS at the end.
// K advances 128
// elements (64 code bytes per row) per stage; codes go from global memory
// straight into four LDS stage buffers by DMA, three stages ahead, each lane
// quad reading the 64 contiguous bytes of one row, stored as [row][piece] x
// 16 bytes with the piece order of row r swizzled by (r >> 2) & 3 (no bank
// conflicts on the operand reads).
//
// Each wave turns its own operands into FP16 in registers.  The order of K
// inside a stage is free as long as both operands use the same one, so lane
// group g (lanes 32g .. 32g+31) of K-step j supplies the 8 elements
// 32 p + 8 (j % 4) .. +7 with p = g for j < 4 and p = 2 + g after: one
// 16-byte LDS read of a row's piece p feeds four K-steps, and the 8 elements
// of a K-step always sit in one NVFP4 block.  Scales are staged through LDS
// already as FP16 patterns (s * 2^-8, two blocks per word), so a lane reads
// the word of its row and piece and a packed multiply with the half selected
// by op_sel applies the block scale.  Per K-step a 128 x 128 wave tile converts 8
// fragments (64 VALU instructions) under 16 MFMAs.

// kFull: K % 128 == 0, every stage lies inside the rows and a stage's 8
// scale bytes per row are one aligned 8-byte load.  Otherwise (any other
// K % 16 == 0) the last stage is partial: its code pieces past K read bytes
// of the next row (or zeros past the tile), which stay harmless because the
// scales of those blocks are set to zero (E2M1 codes are all finite, and
// q * 0 = 0).  A row's scales then start at any byte offset; the 8-byte load
// works at any alignment, but the buffer range check drops a whole 4-byte
// word that straddles the end of the range, so a load never starts closer
// than 8 bytes to the end: the one lane whose stage reaches past the
// operand's last scale byte (the last row, last stage) starts early and
// shifts its bytes down when it parks them.
template <bool kVecOut, bool kFull, int kWM, int kWN, int kGroups>
__global__ __launch_bounds__(kLThreads, 1) void nvfp4_gemm_lane_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const float* __restrict__ a_gs, const uint8_t* __restrict__ b_codes,
    const uint8_t* __restrict__ b_scales, const float* __restrict__ b_gs,
    const uint16_t* __restrict__ bias, uint16_t* __restrict__ out, int64_t M, int64_t N,
    int64_t K, SplitK split) {
  constexpr int kT = 2 * kWN;                // output tile edge (M and N)
  constexpr int kFrA = kWM / 32;             // 32 x 32 MFMA tiles per wave tile, along M
  constexpr int kFrB = kWN / 32;             // and along N
  constexpr int kWaves = 2 * (kT / kWM);     // waves of a group
  constexpr int kTh = kWaves * kWave;        // threads of a group
  static_assert(kWN == 128 || kWN == 64, "tile edge 256 or 128");
  static_assert(kTh * kGroups == kLThreads, "one wave per SIMD");
  static_assert(kGroups == 1 || (kGroups == 2 && kFrB == 2), "a column fragment per group");
  constexpr int kStage = kT * kLRowBytes;    // one operand, one stage
  constexpr int kArr = kGroups * kStage;     // one stage buffer: a stage of every group
  constexpr int kGw = kT / 16 / kWaves;      // 16-row DMA groups per wave and operand
  constexpr int kDma = 2 * kGw;              // DMA instructions per wave and stage
  // one array per stage buffer and operand, so the compiler can tell the
  // buffer being filled by DMA from the one being read
  __shared__ __attribute__((aligned(1024))) uint8_t la0[kArr], la1[kArr],
      la2[kArr], la3[kArr];
  __shared__ __attribute__((aligned(1024))) uint8_t lb0[kArr], lb1[kArr],
      lb2[kArr], lb3[kArr];
  __shared__ uint32_t lsc_all[kGroups][2][2][kT * kLScaleStride];   // [group][stage parity][operand][row, word]
  __shared__ uint16_t lbias[kT];
  // this wave's group (kGroups == 2: group kg takes stages kg, kg + 2, ...)
  const int kg = kGroups == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kTh);
  uint32_t (&lsc)[2][2][kT * kLScaleStride] = lsc_all[kg];
  uint8_t* const abuf[kLBufs] = {la0, la1, la2, la3};
  uint8_t* const bbuf[kLBufs] = {lb0, lb1, lb2, lb3};

  const int tiles_m = (int)((M + kT - 1) / kT);
  const int tiles_n = (int)((N + kT - 1) / kT);
  // workgroups past split.dp_tiles each take one K range of a remainder tile
  const int sub = (int)blockIdx.x - split.dp_tiles;
  const int rem = sub < 0 ? -1 : sub / split.splits;
  const int part_idx = sub < 0 ? 0 : sub - rem * split.splits;
  int tm, tn;
  const int tile_id = sub < 0 ? (int)blockIdx.x : split.dp_tiles + rem;
  if constexpr (kT == 128) {
    if (split.quad_base >= 0) {
      // quadrant tile_id % 4 of 256 x 256 tile quad_base + tile_id / 4
      tile_coords_at(split.quad_base + tile_id / 4, (int)((M + 255) / 256), (int)((N + 255) / 256),
                     tm, tn);
      tm = 2 * tm + ((tile_id >> 1) & 1);
      tn = 2 * tn + (tile_id & 1);
      if ((int64_t)tm * kT >= M || (int64_t)tn * kT >= N) return;   // quadrant outside the output
    } else {
      tile_coords_at(tile_id, tiles_m, tiles_n, tm, tn);
    }
  } else {
    tile_coords_at(tile_id, tiles_m, tiles_n, tm, tn);
  }
  const int64_t m0 = (int64_t)tm * kT;
  const int64_t n0 = (int64_t)tn * kT;
  const int all_stages = (int)((K + kLBK - 1) / kLBK);
  const int s_first = sub < 0 ? 0 : part_idx * split.stages;
  const int nstages = sub < 0 ? all_stages : min(all_stages - s_first, split.stages);
  // stages each group runs (the second one's last may lie past the range: its
  // scales are zeroed)
  const int my_stages = (nstages + kGroups - 1) / kGroups;

  const int t = kGroups == 1 ? (int)threadIdx.x : (int)threadIdx.x & (kTh - 1);   // thread of the group
  const int lane = t & (kWave - 1);
  const int wave = t / kWave;
  const int wm = wave >> 1;   // 0 where a wave tile spans the tile's rows
  const int wn = wave & 1;
  const int li = lane & 31;
  const int g = lane >> 5;

  const int64_t row_bytes = K / 2;
  const int64_t scale_row = K / 16;
  const int64_t valid_a = min<int64_t>(M - m0, kT);
  const int64_t valid_b = min<int64_t>(N - n0, kT);
  const __amdgpu_buffer_rsrc_t rca = uniform_rsrc(a_codes + m0 * row_bytes, valid_a * row_bytes);
  const __amdgpu_buffer_rsrc_t rcb = uniform_rsrc(b_codes + n0 * row_bytes, valid_b * row_bytes);
  // !kFull: the scale ranges hold at least 8 bytes (a last tile of one to
  // three rows of a short K starts 8 bytes early; the host sends operands
  // with fewer than 8 scale bytes in all elsewhere); two groups only run K
  // ranges of 16 stages and more, whose rows hold more than the 16 bytes of
  // their loads
  const uint32_t back_a = !kFull && kGroups == 1 && valid_a * scale_row < 8 ? 8 : 0;
  const uint32_t back_b = !kFull && kGroups == 1 && valid_b * scale_row < 8 ? 8 : 0;
  const __amdgpu_buffer_rsrc_t rsa =
      uniform_rsrc(a_scales + m0 * scale_row - back_a, valid_a * scale_row + back_a);
  const __amdgpu_buffer_rsrc_t rsb =
      uniform_rsrc(b_scales + n0 * scale_row - back_b, valid_b * scale_row + back_b);

  // code DMA, one group: wave w fills 16-row groups kGw w .. kGw w + kGw - 1
  // of each operand; lane quad l/4 reads the 64 bytes of row l/4 of the group,
  // lane l's 16 bytes land in slot l of the group's 1 KB.  Two groups: an
  // instruction covers 8 rows of both groups' stages, 128 contiguous bytes
  // each (slot c of row r holds piece c ^ ((r >> 1) & 7): no bank conflicts)
  const int any_wave = kWaves * kg + wave;   // of the workgroup's four
  const int dma_r = kGroups == 1 ? lane >> 2 : lane >> 3;
  const int piece = kGroups == 1 ? (lane & 3) ^ ((dma_r >> 2) & 3) : (lane & 7) ^ (dma_r >> 1);
  constexpr int kDmaRows = 16 / kGroups;     // rows an instruction covers
  const uint32_t dma_row = (uint32_t)((kDmaRows * kGw * any_wave + dma_r) * row_bytes);
  const uint32_t dma_k = (uint32_t)(s_first * kLRowBytes);
  // byte offset of instruction j's first stage (odd ones of two groups: the
  // row's bit 3 moves the pieces by four)
  const uint32_t dma_off[2] = {dma_row + dma_k + 16 * piece,
                               dma_row + dma_k + 16 * (kGroups == 1 ? piece : piece ^ 4)};
  const uint32_t group_stride = (uint32_t)(kDmaRows * row_bytes);
  // scale staging, one group: thread t moves the 8 scale bytes of tile row t
  // of A and B (threads past the tile's rows load zeros out of range and
  // store nothing).  Two groups: a thread of group 0 moves the 16 bytes of a
  // row of A that cover both groups' stages, one of group 1 a row of B
  const uint32_t sg_off = (uint32_t)(t * scale_row + 8 * s_first);
  const uint32_t sg_a = sg_off + back_a, sg_b = sg_off + back_b;
  const uint32_t sg_u = kg == 0 ? sg_a : sg_b;
  const __amdgpu_buffer_rsrc_t rsu =
      uniform_rsrc(kg == 0 ? a_scales + m0 * scale_row - back_a : b_scales + n0 * scale_row - back_b,
                   kg == 0 ? valid_a * scale_row + back_a : valid_b * scale_row + back_b);
  // operand slots of this lane: row r of the tile lives in group r / 16 at
  // byte (r % 16) * 64 + 16 * (piece ^ ((r % 16) >> 2)); lane group g reads
  // piece g in K-steps 0-3 and piece 2 + g in K-steps 4-7 (two groups: row r
  // at byte 128 r, pieces 4 kg .. 4 kg + 3)
  const int swz = kGroups == 1 ? ((li & 15) >> 2) & 3 : (li >> 1) & 7;
  constexpr int kFragBytes = 2048 * kGroups;   // 32 rows
  const int rd_a = (wm * kWM >> 4) * (kFragBytes / 2) +
                   (kGroups == 1 ? (li >> 4) * 1024 + (li & 15) * 64 : li * 128);
  const int rd_b = (wn * kWN >> 4) * (kFragBytes / 2) +
                   (kGroups == 1 ? (li >> 4) * 1024 + (li & 15) * 64 : li * 128);
  const int q_off[2] = {16 * ((4 * kg + g) ^ swz), 16 * ((4 * kg + 2 + g) ^ swz)};
  // and its scale words: word p of a row holds the patterns of blocks 2p, 2p+1
  const int rs_a = (wm * kWM + li) * kLScaleStride + g;
  const int rs_b = (wn * kWN + li) * kLScaleStride + g;

  // the tile's bias (+0 without one: fma(alpha, acc, +0) == alpha * acc for
  // every accumulator, which never holds -0); parked in LDS once the
  // prologue's loads are out, so its latency overlaps theirs
  constexpr bool kAllRows = kT == kTh;   // every thread stages one tile row
  const bool row_thread = kAllRows || t < kT;
  const uint16_t bias_v = bias && row_thread && n0 + t < N ? bias[n0 + t] : (uint16_t)0;

  floatx16_t acc[kFrB][kFrA];
#pragma unroll
  for (int i = 0; i < kFrB; ++i)
#pragma unroll
    for (int j = 0; j < kFrA; ++j) acc[i][j] = floatx16_t{};

  uint32_t sca[2][kFrA][2], scb[2][kFrB][2];   // [stage parity][frag][half stage]
  u32x4_t ca[2][kFrA], cb[2][kFrB];            // code pieces, [half stage][frag]
  half8_t oa[2][kFrA], ob[2][kFrB];            // FP16 operands, [K-step parity][frag]

  // group j of the DMA of `stage` (2 of its kDma instructions) into buffer
  // `buf`.  A stage's bytes past K are those of later rows or zeros, computed
  // under zero scales.
  auto dma_part = [&](int buf, int stage, int j) {
    // (stages that will not be computed get offsets out of range, which
    // fetch nothing: three stages a tile, about 1% of 18432 x 9216 x 3072)
    const uint32_t adv = stage < my_stages ? (uint32_t)stage * (kGroups * kLRowBytes) : 0x80000000u;
    const uint32_t off = dma_off[j & 1] + adv + j * group_stride;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rca, (lds_ptr_t)(abuf[buf] + (kGw * any_wave + j) * 1024), 16, off, 0, 0, 1);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rcb, (lds_ptr_t)(bbuf[buf] + (kGw * any_wave + j) * 1024), 16, off, 0, 0, 1);
  };
  auto dma_stage = [&](int buf, int stage) {
#pragma unroll
    for (int j = 0; j < kGw; ++j) dma_part(buf, stage, j);
  };
  // one stage's scale bytes of this thread's A and B rows, in flight (two
  // groups: both groups' stages of one row)
  constexpr uint32_t kSBytes = 8 * kGroups;      // bytes a load takes
  const uint32_t lim_a = (uint32_t)(valid_a * scale_row) + back_a - kSBytes;
  const uint32_t lim_b = (uint32_t)(valid_b * scale_row) + back_b - kSBytes;
  const uint32_t lim_u = kg == 0 ? lim_a : lim_b;
  struct ScaleFetch {
    u32x2_t a, b;
  };
  auto fetch_scales = [&](ScaleFetch& f, int stage) {
    if constexpr (kGroups == 1) {
      const uint32_t oa = sg_a + 8 * stage, ob = sg_b + 8 * stage;
      f.a = __builtin_amdgcn_raw_buffer_load_b64(rsa, kFull ? oa : min(oa, lim_a), 0, 0);
      f.b = __builtin_amdgcn_raw_buffer_load_b64(rsb, kFull ? ob : min(ob, lim_b), 0, 0);
    } else {
      const uint32_t ou = sg_u + 16 * stage;
      const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rsu, kFull ? ou : min(ou, lim_u), 0, 0);
      f.a = u32x2_t{v.x, v.y};
      f.b = u32x2_t{v.z, v.w};
    }
  };
  // scale bytes of `stage` (fetched earlier into f) into set `set`, as FP16
  // patterns; blocks at or past K/16 get scale 0
  auto store_scales = [&](ScaleFetch& f, int set, int stage) {
    u32x2_t ga = f.a, gb = f.b;
    if (!kFull && kGroups == 1) {
      const int valid = (int)scale_row - 8 * (s_first + stage);   // blocks inside K
      if (valid < 8) {
        const uint32_t oa = sg_a + 8 * stage, ob = sg_b + 8 * stage;
        const uint64_t keep = valid <= 0 ? 0ull : (~0ull >> (64 - 8 * valid));
        ga = __builtin_bit_cast(u32x2_t, (__builtin_bit_cast(uint64_t, ga) >> (8 * (oa - min(oa, lim_a)) & 63)) & keep);
        gb = __builtin_bit_cast(u32x2_t, (__builtin_bit_cast(uint64_t, gb) >> (8 * (ob - min(ob, lim_b)) & 63)) & keep);
      }
    }
    if (!kFull && kGroups == 2) {
      // blocks inside K and inside this workgroup's K range
      const int valid = min((int)scale_row - 8 * s_first, 8 * nstages) - 16 * stage;
      if (valid < 16) {
        const uint32_t ou = sg_u + 16 * stage;
        const uint32_t early = 8 * (ou - min(ou, lim_u));   // bits; below 128 where valid > 0
        uint64_t lo = __builtin_bit_cast(uint64_t, ga), hi = __builtin_bit_cast(uint64_t, gb);
        if (early & 64) { lo = hi; hi = 0; }
        if (early & 63) {
          lo = (lo >> (early & 63)) | (hi << (64 - (early & 63)));
          hi >>= early & 63;
        }
        lo &= valid >= 8 ? ~0ull : valid <= 0 ? 0ull : ~0ull >> (64 - 8 * valid);
        hi &= valid <= 8 ? 0ull : ~0ull >> (128 - 8 * valid);
        ga = __builtin_bit_cast(u32x2_t, lo);
        gb = __builtin_bit_cast(u32x2_t, hi);
      }
    }
    if (row_thread) {
      uint32_t* da = &lsc_all[0][set][kGroups == 1 ? 0 : kg][t * kLScaleStride];
      uint32_t* db = &lsc_all[kGroups - 1][set][kGroups == 1 ? 1 : kg][t * kLScaleStride];
      da[0] = scale_patterns(ga.x, false);
      da[1] = scale_patterns(ga.x, true);
      da[2] = scale_patterns(ga.y, false);
      da[3] = scale_patterns(ga.y, true);
      db[0] = scale_patterns(gb.x, false);
      db[1] = scale_patterns(gb.x, true);
      db[2] = scale_patterns(gb.y, false);
      db[3] = scale_patterns(gb.y, true);
    }
  };
  // this lane's scale words of `stage` (its 4 A rows and 4 B rows, both pieces)
  auto read_scales = [&](uint32_t (&da)[kFrA][2], uint32_t (&db)[kFrB][2], int stage) {
    const int set = stage & 1;
#pragma unroll
    for (int f = 0; f < kFrA; ++f) {
      da[f][0] = lsc[set][0][rs_a + f * 32 * kLScaleStride];
      da[f][1] = lsc[set][0][rs_a + f * 32 * kLScaleStride + 2];
      if (f >= kFrB) continue;
      db[f][0] = lsc[set][1][rs_b + f * 32 * kLScaleStride];
      db[f][1] = lsc[set][1][rs_b + f * 32 * kLScaleStride + 2];
    }
  };
  auto read_codes = [&](int half, int buf) {
#pragma unroll
    for (int f = 0; f < kFrA; ++f) {
      ca[half][f] = *reinterpret_cast<const u32x4_t*>(abuf[buf] + rd_a + f * kFragBytes + q_off[half]);
      if (f < kFrB) cb[half][f] = *reinterpret_cast<const u32x4_t*>(bbuf[buf] + rd_b + f * kFragBytes + q_off[half]);
    }
  };
  // K-step j of a stage (scale words ss) into operand set d
  auto convert = [&](auto step, const uint32_t (&ssa)[kFrA][2],
                     const uint32_t (&ssb)[kFrB][2], int d) {
    constexpr int j = decltype(step)::value;
    constexpr int h = j >> 2, w = j & 3;
#pragma unroll
    for (int f = 0; f < kFrA; ++f) {
      const half2_t xa = as_h2(ssa[f][h]);
      const half2_t sa = (w & 2) ? __builtin_shufflevector(xa, xa, 1, 1) : __builtin_shufflevector(xa, xa, 0, 0);
      oa[d][f] = dequant_step(ca[h][f][w], sa);
      if (f >= kFrB) continue;
      const half2_t xb = as_h2(ssb[f][h]);
      const half2_t sb = (w & 2) ? __builtin_shufflevector(xb, xb, 1, 1) : __builtin_shufflevector(xb, xb, 0, 0);
      ob[d][f] = dequant_step(cb[h][f][w], sb);
    }
  };
  // (boustrophedon: consecutive MFMAs share an operand also where fn moves
  // on, so fewer operand bits are read and toggle: 256 x 256 tiles 0.4-0.7%,
  // 18432 x 9216 x 3072 829.1 -> 823.5 us; 128 x 128 tiles 2-3%, 1024 x 3072 x
  // 3072 26.3 -> 25.6; the MXFP4 kernel gains nothing by it)
  auto mfma_step = [&](int d) {
#pragma unroll
    for (int fn = 0; fn < kFrB; ++fn)
#pragma unroll
      for (int i = 0; i < kFrA; ++i) {
        const int fm = (fn & 1) ? kFrA - 1 - i : i;
        acc[fn][fm] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ob[d][fn], oa[d][fm], acc[fn][fm], 0, 0, 0);
      }
  };
  // a K-step's MFMAs, each followed by its share of the VALU instructions of
  // the next K-step's conversion (8 a fragment) and of the step's kR pairs of
  // LDS reads, kV memory loads and kW LDS writes (one of each per MFMA for the
  // 128 x 128 wave tile, two for 128 x 64, four for 64 x 64)
  auto interleave = [&](auto reads, auto vmem, auto writes) {
    constexpr int kR = decltype(reads)::value, kV = decltype(vmem)::value,
                  kW = decltype(writes)::value;
    constexpr int kMfma = kFrA * kFrB;
    constexpr int kPer = 16 / kMfma;
#pragma unroll
    for (int i = 0; i < kMfma; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                          // MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 8 * (kFrA + kFrB) / kMfma, 0);                   // VALU
      if (i * kPer < kR) __builtin_amdgcn_sched_group_barrier(0x100, 2 * kPer, 0);   // DS read
      if (i * kPer < kV) __builtin_amdgcn_sched_group_barrier(0x020, kPer, 0);       // VMEM read
      if (i * kPer < kW) __builtin_amdgcn_sched_group_barrier(0x200, kPer, 0);       // DS write
    }
  };

  using I0 = std::integral_constant<int, 0>;
  using I4 = std::integral_constant<int, 4>;
  using I8 = std::integral_constant<int, 8>;
  using I12 = std::integral_constant<int, 12>;
  using J0 = std::integral_constant<int, 0>;
  using J1 = std::integral_constant<int, 1>;
  using J2 = std::integral_constant<int, 2>;
  using J3 = std::integral_constant<int, 3>;
  using J4 = std::integral_constant<int, 4>;
  using J5 = std::integral_constant<int, 5>;
  using J6 = std::integral_constant<int, 6>;
  using J7 = std::integral_constant<int, 7>;

  constexpr int kSL = 3 - kGroups;   // vector-memory instructions of one scale fetch (but for one stage of one lane)
  // prologue: the scales of stages 0-2, then the codes of stages 0-2, all go
  // out first; the scales of stages 0 and 1 are parked in LDS as they land
  // (each store waits only for its own, older loads), stage 2's stay in
  // registers; once stages 0 and 1 have landed (only stage 2's DMA, the
  // youngest loads, may still be in flight), the first half stage's codes
  // and the scales of stage 0 are read and K-step 0 converted.  The second
  // barrier keeps stage 0 from parking stage 2's scales over set 0 before
  // every wave has read it.
  ScaleFetch sf, sf0, sf1;   // sf: the stage in flight during the main loop
  fetch_scales(sf0, 0);
  fetch_scales(sf1, 1);
  fetch_scales(sf, 2);
  dma_stage(0, 0);
  dma_stage(1, 1);
  dma_stage(2, 2);
  if (row_thread) lbias[t] = bias_v;
  store_scales(sf0, 0, 0);
  store_scales(sf1, 1, 1);
  wait_counts<kDma, 0>();
  __builtin_amdgcn_s_barrier();
  read_scales(sca[0], scb[0], 0);
  read_codes(0, 0);
  wait_counts<63, 0>();
  __builtin_amdgcn_s_barrier();
  convert(J0{}, sca[0], scb[0], 0);

  // Stage s with P = s % 4 (buffer P, scale parity C = P % 2).  K-steps 0
  // .. kGw-1 issue the DMA of stage s+3 into buffer (P + 3) % 4 (last read in
  // stage s-1); K-step 0 parks the scales of stage s+2 in set C (last read in stage s-1,
  // next read in stage s+1) and fetches those of stage s+3, and reads this
  // stage's second code half; K-step 4 reads the next stage's first code
  // half and scales; K-step 7 converts the next stage's K-step 0.  The
  // barrier that ends stage s waits for this wave's DMA of stage s+2, so in
  // stage s+1 both its own buffer and the next one are complete.
  auto run_stage = [&](auto phase, int s) {
    constexpr int P = decltype(phase)::value;
    constexpr int C = P & 1;
    __builtin_amdgcn_sched_barrier(0);
    // the scale loads go out before the DMA, so the wait that ends the stage
    // can count the DMA alone (the compiler may merge the scale loads into
    // fewer instructions than written)
    store_scales(sf, C, s + 2);
    fetch_scales(sf, s + 3);
    // the DMA of stage s+3 goes out a group (2 instructions) per K-step over
    // K-steps 0 .. kGw-1: issued at once, the 8 instructions of a 128 x 128
    // wave tile filled the texture addresser's queues and held up the MFMA
    // issue behind them (3% slower)
    using I2 = std::integral_constant<int, 2>;
    dma_part((P + 3) % kLBufs, s + 3, 0);
    read_codes(1, P);
    mfma_step(0);
    convert(J1{}, sca[C], scb[C], 1);
    interleave(I4{}, std::integral_constant<int, 2 + kSL>{}, I8{});
    __builtin_amdgcn_sched_barrier(0);
    dma_part((P + 3) % kLBufs, s + 3, 1);
    mfma_step(1);
    convert(J2{}, sca[C], scb[C], 0);
    interleave(I0{}, I2{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    if (kGw > 2) dma_part((P + 3) % kLBufs, s + 3, 2);
    mfma_step(0);
    convert(J3{}, sca[C], scb[C], 1);
    interleave(I0{}, std::integral_constant<int, (kGw > 2 ? 2 : 0)>{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    if (kGw > 3) dma_part((P + 3) % kLBufs, s + 3, 3);
    mfma_step(1);
    convert(J4{}, sca[C], scb[C], 0);
    interleave(I0{}, std::integral_constant<int, (kGw > 3 ? 2 : 0)>{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    read_codes(0, (P + 1) % kLBufs);
    read_scales(sca[C ^ 1], scb[C ^ 1], s + 1);
    mfma_step(0);
    convert(J5{}, sca[C], scb[C], 1);
    interleave(I12{}, I0{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(1);
    convert(J6{}, sca[C], scb[C], 0);
    interleave(I0{}, I0{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(0);
    convert(J7{}, sca[C], scb[C], 1);
    interleave(I0{}, I0{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(1);
    convert(J0{}, sca[C ^ 1], scb[C ^ 1], 0);
    interleave(I0{}, I0{}, I0{});
    __builtin_amdgcn_sched_barrier(0);
    // this stage's kDma DMA instructions, the last vector-memory operations
    // it issued, may stay in flight; everything older (the DMA of stage s+2
    // and this stage's scale loads) is complete
    wait_counts<kDma, 0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  using P2 = std::integral_constant<int, 2>;
  using P3 = std::integral_constant<int, 3>;
  // !kFull: a last stage of at most 64 elements runs its first four K-steps
  // only (both lane groups' pieces 0 and 1); its scales, first code half and
  // K-step 0 operands are in registers already.  One instance with the scale
  // set selected (two, by parity, doubled the accumulators and spilled 1 KB
  // a lane).  8192 x 6720 x 2240, half a stage of 17.5: 249 -> 238 us.
  auto run_half = [&](bool odd) {
    uint32_t ha[kFrA][2], hb[kFrB][2];
#pragma unroll
    for (int f = 0; f < kFrA; ++f) {
      ha[f][0] = odd ? sca[1][f][0] : sca[0][f][0];
      ha[f][1] = 0;
      if (f >= kFrB) continue;
      hb[f][0] = odd ? scb[1][f][0] : scb[0][f][0];
      hb[f][1] = 0;
    }
    mfma_step(0);
    convert(J1{}, ha, hb, 1);
    mfma_step(1);
    convert(J2{}, ha, hb, 0);
    mfma_step(0);
    convert(J3{}, ha, hb, 1);
    mfma_step(1);
  };
  const bool half_tail = !kFull && kGroups == 1 && s_first + nstages == all_stages && scale_row - 8 * (int64_t)(all_stages - 1) <= 4;
  const int whole_stages = my_stages - (half_tail ? 1 : 0);
  int s = 0;
  for (; s + 4 <= whole_stages; s += 4) {
    run_stage(P0{}, s);
    run_stage(P1{}, s + 1);
    run_stage(P2{}, s + 2);
    run_stage(P3{}, s + 3);
  }
  {
    const int rest = whole_stages - s;
    if (rest > 0) run_stage(P0{}, s);
    if (rest > 1) run_stage(P1{}, s + 1);
    if (rest > 2) run_stage(P2{}, s + 2);
    if (!kFull && half_tail) run_half((rest & 1) != 0);
  }
  // no DMA may still be writing LDS when the workgroup ends
  wait_counts<0, 0>();

  // kGroups == 2: both groups hold sums of the whole tile.  Group kg keeps
  // column fragment kg of each wave tile, hands the other one over through
  // the stage buffers (16 KB a wave, free now) and adds what it gets, so the
  // epilogue is shared too.
  constexpr int kFnOwn = kGroups == 1 ? kFrB : 1;
  if constexpr (kGroups == 2) {
    static_assert(kFrA * 4 * 1024 <= kArr, "a wave's fragments fit one stage buffer");
    __syncthreads();   // no other wave's DMA may still be writing LDS
    uint8_t* const slab0 = (wave == 0 ? la0 : la1) + 16 * lane;
    uint8_t* const slab1 = (wave == 0 ? lb0 : lb1) + 16 * lane;
    uint8_t* const mine = kg == 0 ? slab0 : slab1;
    const uint8_t* const theirs = kg == 0 ? slab1 : slab0;
#pragma unroll
    for (int fm = 0; fm < kFrA; ++fm)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        u32x4_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a0 = acc[0][fm][4 * q + e], a1 = acc[1][fm][4 * q + e];
          v[e] = __float_as_uint(kg == 0 ? a1 : a0);
          acc[0][fm][4 * q + e] = kg == 0 ? a0 : a1;
        }
        *reinterpret_cast<u32x4_t*>(mine + (4 * fm + q) * 1024) = v;
      }
    __syncthreads();
#pragma unroll
    for (int fm = 0; fm < kFrA; ++fm)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(theirs + (4 * fm + q) * 1024);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][fm][4 * q + e] += __uint_as_float(v[e]);
      }
  }

  if (sub >= 0) {
    // One of the two K halves of a remainder tile: park the FP32
    // accumulators in the workspace; the second of the tile's two
    // workgroups to finish adds the other half's sums to its own (FP32
    // addition is commutative, so the result does not depend on which one
    // that is) and runs the epilogue.  The partial sums are written and read
    // with the sc1 cache policy (written through to memory, read past this
    // XCD's L2), so they are coherent across XCDs without writing back or
    // invalidating whole L2 caches; a half's stores are complete before its
    // workgroup counts itself in.  Lane-major 16-byte slots: each store or
    // load instruction covers 1 KB.
    constexpr int kSlots = kFnOwn * kFrA * 4;       // 16-byte slots per lane
    constexpr uint32_t kSlotBytes = 16 * kWave;     // one slot of a wave
    constexpr uint32_t kHalfBytes = 4 * kSlots * kSlotBytes;   // one half's partial tile
    constexpr int kSc1 = 16;                        // cache policy bits: sc1
    const __amdgpu_buffer_rsrc_t rp = uniform_rsrc(
        reinterpret_cast<const uint8_t*>(split.part) + (size_t)rem * 2 * kHalfBytes,
        (int64_t)2 * kHalfBytes);
    const uint32_t lane_off = (uint32_t)any_wave * kSlots * kSlotBytes + 16u * lane;
#pragma unroll
    for (int fn = 0; fn < kFnOwn; ++fn)
#pragma unroll
      for (int fm = 0; fm < kFrA; ++fm)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const floatx16_t& a = acc[fn][fm];
          const u32x4_t v = {__float_as_uint(a[4 * q]), __float_as_uint(a[4 * q + 1]),
                             __float_as_uint(a[4 * q + 2]), __float_as_uint(a[4 * q + 3])};
          __builtin_amdgcn_raw_buffer_store_b128(
              v, rp, lane_off + part_idx * kHalfBytes + ((fn * kFrA + fm) * 4 + q) * kSlotBytes, 0, kSc1);
        }
    __shared__ int last_flag;
    wait_counts<0, 0>();   // this thread's partial sums have reached memory
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint64_t mine = kSplitToken ^ (uint64_t)(2 * rem + part_idx);
      const uint64_t before = __hip_atomic_exchange(&split.slots[rem], mine, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
      last_flag = before == (mine ^ 1u);   // the other half's token: it finished first
      if (last_flag)
        __hip_atomic_store(&split.slots[rem], (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last_flag) return;
    // The other half's sums come in through LDS, whose stage buffers are
    // free now: each wave moves its own slots by DMA (no registers held
    // while the loads are in flight), half of them at a time into two of
    // the stage buffers, then reads each slot back and adds it.
    constexpr int kPerBuf = kArr / 1024;   // 1 KB slots per stage buffer
    constexpr int kPass = kSlots / 2;
    static_assert(kSlots % 2 == 0 && kPass <= 2 * kPerBuf, "slots per pass");
    uint8_t* const lds_lo = any_wave == 0 ? la0 : any_wave == 1 ? la2 : any_wave == 2 ? lb0 : lb2;
    uint8_t* const lds_hi = any_wave == 0 ? la1 : any_wave == 1 ? la3 : any_wave == 2 ? lb1 : lb3;
    const uint32_t other = lane_off + (1 - part_idx) * kHalfBytes;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
      for (int i = 0; i < kPass; ++i) {
        uint8_t* const dst = (i < kPerBuf ? lds_lo : lds_hi) + (i % kPerBuf) * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rp, (lds_ptr_t)dst, 16,
                                                 other + (pass * kPass + i) * kSlotBytes, 0, 0, kSc1);
      }
      wait_counts<0, 0>();
#pragma unroll
      for (int i = 0; i < kPass; ++i) {
        const int slot = pass * kPass + i;
        const int fn = slot / (4 * kFrA), fm = (slot / 4) % kFrA, q = slot % 4;
        const uint8_t* const src = (i < kPerBuf ? lds_lo : lds_hi) + (i % kPerBuf) * 1024 + 16 * lane;
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(src);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[fn][fm][4 * q + e] += __uint_as_float(v[e]);
      }
    }
  }

  // epilogue: out = bf16(fp32(fma(alpha, acc, bias))), alpha = aA * aB in
  // FP32.  Lane (li, g) holds, per MFMA tile, row m = li and the column runs
  // 8k + 4g .. 8k + 4g + 3 (k = 0..3); swapping halves with the lane 32 apart
  // gives each lane two runs of 8 consecutive columns (16-byte stores).
  // Stores go through a buffer resource covering the tile's valid rows, so
  // rows past M are dropped by the hardware range check; columns past N get
  // an offset beyond the range.
  const float alpha = a_gs[0] * b_gs[0];
  const __amdgpu_buffer_rsrc_t ro = uniform_rsrc(out + m0 * N, valid_a * N * 2);
#pragma unroll
  for (int fm = 0; fm < kFrA; ++fm) {
    const uint32_t mrow = (uint32_t)((wm * kWM + fm * 32 + li) * N);
#pragma unroll
    for (int fn = 0; fn < kFnOwn; ++fn) {
      const int nb = wn * kWN + (kGroups == 1 ? fn : kg) * 32;
      float v[16];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint2 b2 = *reinterpret_cast<const uint2*>(&lbias[nb + 8 * k + 4 * g]);
        const float bv[4] = {__uint_as_float(b2.x << 16), __uint_as_float(b2.x & 0xFFFF0000u),
                             __uint_as_float(b2.y << 16), __uint_as_float(b2.y & 0xFFFF0000u)};
#pragma unroll
        for (int q = 0; q < 4; ++q) v[4 * k + q] = __builtin_fmaf(alpha, acc[fn][fm][4 * k + q], bv[q]);
      }
      uint32_t p[4][2];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        p[k][0] = pack_bf16(v[4 * k], v[4 * k + 1]);
        p[k][1] = pack_bf16(v[4 * k + 2], v[4 * k + 3]);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t r[4];   // 8 columns starting at nb + 16 h + 8 g
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const auto x = __builtin_amdgcn_permlane32_swap(p[2 * h][d], p[2 * h + 1][d], false, false);
          r[d] = x[0];
          r[2 + d] = x[1];
        }
        const int64_t n = n0 + nb + 16 * h + 8 * g;
        store_run8<kVecOut>(ro, mrow, n, N, r);
      }
    }
  }
}

// Compute units of the current device (256 on MI355X), queried once per
// device.
int device_cu_count() {
  constexpr int kMaxDevices = 64;
  static int cached[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  int v = __atomic_load_n(&cached[dev], __ATOMIC_RELAXED);
  if (v <= 0) {
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
      v = 256;
    __atomic_store_n(&cached[dev], v, __ATOMIC_RELAXED);
  }
  return v;
}

// Whether 128 x 128 tiles finish sooner than 256 x 256 ones: one workgroup
// per CU at a time, so a launch takes about ceil(tiles / CUs) rounds of one
// tile's time, and a small tile takes kSmallTileCost of a large one's
// (measured; ideal would be 1/4).
bool small_tiles_pay(int64_t tiles256, int64_t tiles128) {
#ifndef SOLFP4_SMALL_TILE_COST
#define SOLFP4_SMALL_TILE_COST 0.46
#endif
  const int64_t cus = device_cu_count();
  const double big = (double)((tiles256 + cus - 1) / cus);
  const double small = (double)((tiles128 + cus - 1) / cus) * SOLFP4_SMALL_TILE_COST;
  return small < big;
}

// Quadrants of the last round split in K halves from this many stages on
// (measured: 8 stages 0.92x of whole quadrants, 18 stages 1.01x, 24-96
// stages 1.05-1.10x).
constexpr int64_t kQuadHalvesMinStages = 16;

SplitPlan plan_split(int64_t tiles, int64_t nstages, double fixed_cost, double part_cost,
                     size_t part_tile_bytes, bool quad_ok) {
  SplitPlan plan;
  plan.dp_tiles = tiles;
  plan.stages = nstages;
  const int64_t cus = device_cu_count();
  const int64_t rem = tiles % cus;
  if (rem == 0) return plan;
  if (quad_ok && tiles > cus && 4 * rem <= cus) {
    plan.quad = true;
    plan.rem_tiles = rem;
    plan.dp_tiles = tiles - rem;
    if (8 * rem <= cus && nstages >= kQuadHalvesMinStages) {
      const int64_t quads = 4 * rem;
      plan.splits = 2;
      plan.stages = (nstages + 1) / 2;
      plan.bytes = ((size_t)quads * 8 + 255) / 256 * 256 + (size_t)quads * 2 * (part_tile_bytes / 4);
    }
    return plan;
  }
  if (nstages < 2) return plan;
  // two K halves per remainder tile (the kernels add exactly two), when
  // both halves of every remainder tile fit in one round
  if (2 * rem > cus) return plan;
  const double whole = (double)nstages + fixed_cost;
  const double halves = (double)((nstages + 1) / 2) + fixed_cost + 2.0 * part_cost;
  if (!(halves < whole)) return plan;
  plan.stages = (nstages + 1) / 2;
  plan.splits = 2;
  plan.rem_tiles = rem;
  plan.dp_tiles = tiles - rem;
  plan.bytes = ((size_t)rem * 8 + 255) / 256 * 256 + (size_t)(rem * plan.splits) * part_tile_bytes;
  return plan;
}

SplitK split_args(const SplitPlan& plan, void* workspace) {
  SplitK a{};
  a.dp_tiles = (int)plan.dp_tiles;
  a.splits = (int)plan.splits;
  a.stages = (int)plan.stages;
  if (plan.active()) {
    a.slots = static_cast<uint64_t*>(workspace);
    a.part = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) +
                                      ((size_t)plan.rem_tiles * 8 + 255) / 256 * 256);
  }
  return a;
}

// Timing estimates in units of one K stage of the NVFP4 lane kernel
// (measured about 5.1k cycles on a busy chip): prologue plus epilogue of a
// tile about 3.3 stages; writing one 256 KB partial tile, or reading one
// back, with every remainder workgroup doing so at once, 2-3.5 stages.
#ifndef SOLFP4_SPLIT_FIXED
#define SOLFP4_SPLIT_FIXED 3.3
#endif
#ifndef SOLFP4_SPLIT_PART
#define SOLFP4_SPLIT_PART 2.5
#endif
// The same for 128 x 128 tiles, in units of their own (latency-bound) stage:
// fitted to the measured gain of the split on the 128-token 3072 -> 3072
// (1.32x), 128-token 1152 -> 1152 at K = 4608 (1.49x), 512-token 2240 ->
// 2240 (1.16x) and 128-token 1152 -> 1152 (none) layers.
#ifndef SOLFP4_SPLIT_FIXED_SMALL
#define SOLFP4_SPLIT_FIXED_SMALL 9.0
#endif
#ifndef SOLFP4_SPLIT_PART_SMALL
#define SOLFP4_SPLIT_PART_SMALL 2.0
#endif

// What the lane kernel can take: all but operands with fewer than 8 scale
// bytes, the size of its scale loads.
static bool lane_can_take(int64_t M, int64_t N, int64_t K) { return M * K >= 128 && N * K >= 128; }

// What it takes: nearly all of that (K % 32 == 16: the shared kernel reads
// such rows a byte of scales at a time and has no smaller tile; 934 x 1789 x
// 1680 84.5 -> 20 us, 4000 x 4000 x 2064 112 -> 74, 400 x 1000 x 9744 329 ->
// 42, 8192 x 6720 x 208 70 -> 55, x 144 64.8 -> 51, x 80 58.6 -> 44, 2930 x
// 2235 x 144 23.2 -> 13.1, 300 x 300 x 48 8.4 -> 6.4).  The shared kernel
// keeps, on unsplit 256 x 256 tiles, K = 16 and 48 in one round (4096 x 4096
// x 48 15.5 us against 16.3; 704 tiles 31.3 against 30.2) and K % 128 == 64
// below 1024, where the half last stage weighs most (shared against lane: 4096
// x 4096 x 64 14.0 and 15.9, x 320 20.4 and 21.7, x 832 33.7 and 34.5, x 1088
// 40.1 and 39.3; 8192 x 4096 x 832 63.4 and 66.1, x 1088 77.2 and 75.7; 8192 x
// 5600 x 320 46.6 and 47.3, x 576 67.1 and 66.4, x 1088 107 and 101, x 2240
// 192 and 177; outputs 8192 wide are faster on the lane kernel at any K, 8192 x
// 8192 x 320 72.6 and 64.3, which this line leaves).
static bool lane_takes(int64_t M, int64_t N, int64_t K, bool small, bool split_or_quad) {
  if (!lane_can_take(M, N, K)) return false;
  if (small || split_or_quad) return true;
  if (K == 16 || K == 48) return ((M + 255) / 256) * ((N + 255) / 256) > device_cu_count();
  return K % kLBK != 64 || K > 1024;
}

// The tiles, and how the lane kernel splits the last round of them (it is
// the one that splits, on either tile size).
static SplitPlan gemm_plan(int64_t M, int64_t N, int64_t K, bool* small_out) {
  SplitPlan plan;
  const bool lane_ok = lane_can_take(M, N, K);
  const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256);
  const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128);
  const bool small = lane_ok && small_tiles_pay(t256, t128);
  if (small_out) *small_out = small;
  plan.dp_tiles = small ? t128 : t256;
  if (!lane_ok) return plan;
  const int64_t nstages = (K + kLBK - 1) / kLBK;
  if (small)
    return plan_split(t128, nstages, SOLFP4_SPLIT_FIXED_SMALL, SOLFP4_SPLIT_PART_SMALL, 128 * 128 * 4,
                      false);
  return plan_split(t256, nstages, SOLFP4_SPLIT_FIXED, SOLFP4_SPLIT_PART, 256 * 256 * 4, true);
}

size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) {
  if (M <= 0 || N <= 0 || K <= 0 || use_small_gemm(M, N, K) || use_wavek_gemm(M, N, K)) return 0;
  return gemm_plan(M, N, K, nullptr).bytes;
}

void describe_gemm(int64_t M, int64_t N, int64_t K, bool with_workspace, int* kernel, int* tile,
                   int64_t* workgroups, int* splits) {
  if (use_wavek_gemm(M, N, K)) {
    *kernel = SOLFP4_KERNEL_NVFP4_WAVEK;
    *tile = 32;
    *splits = 1;
    *workgroups = ((M + 31) / 32) * ((N + 31) / 32);
    return;
  }
  if (use_small_gemm(M, N, K)) {
    *kernel = SOLFP4_KERNEL_NVFP4_SMALL;
    *tile = 64;
    *splits = 1;
    *workgroups = ((M + 63) / 64) * ((N + 63) / 64);
    return;
  }
  bool small = false;
  SplitPlan plan = gemm_plan(M, N, K, &small);
  const bool split = plan.active() && with_workspace;
  const bool lane = lane_takes(M, N, K, small, split || plan.quad);
  *kernel = lane ? SOLFP4_KERNEL_NVFP4_LANE : SOLFP4_KERNEL_NVFP4_SHARED;
  *tile = small ? 128 : 256;
  *splits = split ? (int)plan.splits : 1;
  const int64_t tiles = small ? ((M + 127) / 128) * ((N + 127) / 128)
                              : ((M + 255) / 256) * ((N + 255) / 256);
  if (plan.quad)
    *workgroups = plan.dp_tiles + 4 * plan.rem_tiles * (split ? plan.splits : 1);
  else
    *workgroups = split ? plan.dp_tiles + plan.rem_tiles * plan.splits : tiles;
}

// The small-tile kernel takes the shapes whose 64 x 64 tiles fit in one
// round (one workgroup per CU).  Measured against the 128 x 128 / 256 x 256
// kernels, graph-replayed: 128 x 1152 x 1152 6.96 vs 11.46 us, 128 x 3072 x
// 3072 13.3 vs 17.8, 768 x 1152 x 1152 7.4 vs 11.6; past one round it loses
// (384 x 3072 x 3072 0.96x, 1024 x 3072 x 3072 0.85x, 128 x 9216 x 3072
// 0.95x) or gains little (1024 x 1152 x 1152 1.16x at 288 tiles).
bool use_small_gemm(int64_t M, int64_t N, int64_t K) {
  if (K % kLBK != 0 || M <= 0 || N <= 0 || K <= 0) return false;
  const int64_t t64 = ((M + 63) / 64) * ((N + 63) / 64);
  return t64 <= device_cu_count();
}

// Few tokens with K % 128 != 0, which the small-tile kernel does not take:
// whether the wave-K kernel is estimated faster than the 128 x 128 lane
// kernel.  Microseconds, fitted on one box to 30 shapes of 1 to 5000 tokens
// and K = 176 to 12272.  Wave-K: a lone workgroup as below, each further one
// on a CU adding 0.45 + 0.025 per stage of a wave of a lone one's time (long
// K is held by operand traffic).  Lane: 2.5 + 1.1 per stage, or with its
// tiles in two K halves 6.5 + 1 per stage of a half + 0.03 per tile.
// Measured, lane -> wave-K: 16 x 5600 x 2240 15.8 -> 5.5 us, 122 x 326 x
// 5600 30.3 -> 9.1, 777 x 1235 x 1040 13.9 -> 9.5, 700 x 700 x 5600 27.5 ->
// 16.0, 2000 x 100 x 11600 47.2 -> 16.0; kept on the lane kernel: 256 x 6720
// x 2240 (18.6 against 19.9), 200 x 9728 x 2416 (23.8 against 29.0), 1500 x
// 1500 x 1648 (18.4 against 23.6), 1024 x 2240 x 5600 (44 against 57).
static bool ragged_wavek_pays(int64_t M, int64_t N, int64_t K) {
  const int64_t cus = device_cu_count();
  const int64_t stages = (K + kLBK - 1) / kLBK;
  const double mine = (double)((stages + 3) / 4);
  const int64_t t32 = ((M + 31) / 32) * ((N + 31) / 32);
  const double per_cu = (double)((t32 + cus - 1) / cus);
  const double wavek = (1.0 + (0.45 + 0.025 * mine) * (per_cu - 1.0)) * (2.83 + 0.52 * mine);
  const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128);
  if (!lane_can_take(M, N, K) || t128 > cus) return false;
  bool small = false;
  const SplitPlan plan = gemm_plan(M, N, K, &small);
  const double lane = plan.active() ? 6.5 + (double)plan.stages + 0.03 * (double)t128
                                    : 2.5 + 1.1 * (double)stages;
  return wavek < lane;
}

// Among the shapes the small-tile kernel takes, the wave-K kernel (32 x 32
// tiles, each workgroup's K stages dealt to its four waves) where its
// estimated time is lower.  Its LDS lets two workgroups share a CU, so a
// launch of t tiles puts ceil(t / CUs) of them on the busiest CU, and each
// one past the first adds 0.52 of a lone workgroup's time (two at once run
// 1.28-1.6x as long as one alone, longer K towards the top).  A lone
// workgroup costs a fixed part plus one per stage of its longest wave; the
// 64 x 64 kernel never takes more than one round here.  The costs, in
// microseconds, are fitted to measurements on one box (50 launches per
// timing): the 64 x 64 kernel 3.35 + 0.40 per stage, the wave-K kernel
// 2.83 + 0.52 per stage (128 x 1152 x 1152 6.9 -> 4.4 us, 128 x 3072 x 12288
// 42.4 -> 23.6 at 384 tiles, 256 x 3072 x 3072 13.7 -> 12.4 at 768; kept on
// 64 x 64 tiles: 512 x 2048 x 2048, 10.6 against 11.9 at 1024 tiles).  On
// 15 shapes of 7 to 512 tokens the estimate picks the faster kernel on all
// but one, 128 x 6144 x 1536, where wave-K would be 3% faster.
// Past one round of 64 x 64 tiles it still takes outputs at most 32 wide (or
// tall), of which a 128 x 128 tile would be three quarters padding: 20000 x 32
// x 3072 23.9 -> 13.5 us, 17000 x 16 x 9728 63.5 -> 30.8; at K = 256 the two
// are alike, and at 33 to 64 wide it loses (26574 x 48 x 2432 0.95x).
// K % 128 != 0: ragged_wavek_pays (128 x 1152 x 1120, lane -> wave-K: 12.4 ->
// 6.1 us; 256 x 1152 x 1120 12.4 -> 5.7, 384 x 2432 x 1120 12.8 -> 9.3).
bool use_wavek_gemm(int64_t M, int64_t N, int64_t K) {
  if (M <= 0 || N <= 0 || K <= 0) return false;
  if (K % kLBK != 0) return K > kLBK && ragged_wavek_pays(M, N, K);
  if (!use_small_gemm(M, N, K)) return (M <= 32 || N <= 32) && K >= 4 * kLBK;
  const int64_t cus = device_cu_count();
  const int64_t t32 = ((M + 31) / 32) * ((N + 31) / 32);
  const int64_t stages = K / kLBK;
  const double small = 3.35 + 0.40 * (double)stages;
  const double per_cu = (double)((t32 + cus - 1) / cus);
  const double wavek = (1.0 + 0.52 * (per_cu - 1.0)) * (2.83 + 0.52 * (double)((stages + 3) / 4));
  return wavek < small;
}

hipError_t launch_gemm(const uint8_t* a_codes, const uint8_t* a_scales, const float* a_gs,
                       const uint8_t* b_codes, const uint8_t* b_scales, const float* b_gs,
                       const uint16_t* bias, uint16_t* out, int64_t M, int64_t N, int64_t K,
                       void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (M == 0 || N == 0) return hipSuccess;
  if (use_wavek_gemm(M, N, K))
    return launch_gemm_wavek(a_codes, a_scales, a_gs, b_codes, b_scales, b_gs, bias, out, M, N, K,
                             stream);
  if (use_small_gemm(M, N, K))
    return launch_gemm_small(a_codes, a_scales, a_gs, b_codes, b_scales, b_gs, bias, out, M, N, K,
                             nullptr, stream);
  return launch_gemm_regular(a_codes, a_scales, a_gs, b_codes, b_scales, b_gs, bias, out, M, N, K,
                             workspace, workspace_bytes, stream);
}

// Whether K ranges of `range` stages are whole in pairs (the two wave groups
// of a 128 x 128 tile then need no masking).
static bool whole_pairs(int64_t K, int64_t range) { return K % (2 * kLBK) == 0 && range % 2 == 0; }

// Wave groups of a 128 x 128 tile.  Two of them run a stage in 0.62 us
// against 0.82 (6 operand fragments converted per 8 MFMAs and not 4 per 4,
// half the cache lines touched), but start up 0.3 us later, add their sums
// (1-1.3 us) and leave room for one workgroup per CU.  So: from 16 stages
// per K range in whole pairs or 26 of any kind where every workgroup has a
// CU to itself, from 48 otherwise.  Measured, one group -> two: 1024 x 3072 x
// 2048 20.1 -> 19.2 us, x 3072 25.1 -> 23.3, 1000 x 2432 x 3712 28.3 -> 27.5, x
// 9728 67.4 -> 55.9, 2048 x 3072 x 12288 145.7 -> 135.9; in K halves 512 x 3072
// x 9728 40.4 -> 36.0; quadrants of 4608 x 4096 x 12288 346.6 -> 340.6.  Kept
// on one: 333 x 7296 x 2432 (22.4 against 22.7), 1024 x 3072 x 1024, 1024 x
// 5600 x 2240 (34.9 against 39.6), 2000 x 2240 x 5600 (66.8 against 67.5).
static int lane_groups(int64_t workgroups, int64_t K, int64_t range) {
  if (workgroups > device_cu_count()) return range >= 48 ? 2 : 1;
  return range >= (whole_pairs(K, range) ? 16 : 26) ? 2 : 1;
}

// One launch of the lane kernel: `wt` the wave tile's edge, `groups` of four
// waves each.
static hipError_t launch_lane(int wt, int groups, dim3 grid, const uint8_t* a_codes,
                              const uint8_t* a_scales, const float* a_gs, const uint8_t* b_codes,
                              const uint8_t* b_scales, const float* b_gs, const uint16_t* bias,
                              uint16_t* out, int64_t M, int64_t N, int64_t K, const SplitK& split,
                              hipStream_t stream) {
  const bool vec = N % 8 == 0;
  const bool full = groups == 1 ? K % kLBK == 0 : whole_pairs(K, split.stages);
#define SOLFP4_LANE_LAUNCH(V, F, WM, WN, G)                                                   \
  launch_kernel(nvfp4_gemm_lane_kernel<V, F, WM, WN, G>, grid, dim3(kLThreads), stream, a_codes, \
                a_scales, a_gs, b_codes, b_scales, b_gs, bias, out, M, N, K, split)
#define SOLFP4_LANE_PICK(WM, WN, G)                              \
  (vec && full ? SOLFP4_LANE_LAUNCH(true, true, WM, WN, G)      \
   : full      ? SOLFP4_LANE_LAUNCH(false, true, WM, WN, G)     \
   : vec       ? SOLFP4_LANE_LAUNCH(true, false, WM, WN, G)     \
               : SOLFP4_LANE_LAUNCH(false, false, WM, WN, G))
  if (wt == 128) return SOLFP4_LANE_PICK(128, 128, 1);
  if (groups == 2) return SOLFP4_LANE_PICK(128, 64, 2);
  return SOLFP4_LANE_PICK(64, 64, 1);
#undef SOLFP4_LANE_PICK
#undef SOLFP4_LANE_LAUNCH
}

// The whole tiles in one launch of 256 x 256 tiles, then the last round's
// tiles as four 128 x 128 quadrants each (their K halves added through the
// workspace when the plan splits them).  The quadrants run the same MFMAs
// per output element in the same order as whole tiles (or, split, as two K
// halves of a whole tile) while one wave group runs them; from lane_groups'
// thresholds on, even and odd stages are summed apart, and results agree with
// whole tiles to FP32 summation error.  Measured on one box against the
// one-launch plans: shapes with one round plus 8 to 64 tiles 1.04-1.20x (K =
// 256 to 12288), 18432 x 9216 x 3072 1.017x.
static hipError_t launch_gemm_quad(const uint8_t* a_codes, const uint8_t* a_scales,
                                   const float* a_gs, const uint8_t* b_codes,
                                   const uint8_t* b_scales, const float* b_gs,
                                   const uint16_t* bias, uint16_t* out, int64_t M, int64_t N,
                                   int64_t K, const SplitPlan& plan, void* workspace,
                                   hipStream_t stream) {
  const int all_stages = (int)((K + kLBK - 1) / kLBK);
  SplitK whole{};
  whole.dp_tiles = (int)plan.dp_tiles;
  whole.splits = 1;
  whole.stages = all_stages;
  const int64_t quads = 4 * plan.rem_tiles;
  SplitK tail{};
  tail.quad_base = (int)plan.dp_tiles;
  if (plan.active()) {
    tail.dp_tiles = 0;
    tail.splits = (int)plan.splits;
    tail.stages = (int)plan.stages;
    tail.slots = static_cast<uint64_t*>(workspace);
    tail.part = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) +
                                         ((size_t)quads * 8 + 255) / 256 * 256);
  } else {
    tail.dp_tiles = (int)quads;
    tail.splits = 1;
    tail.stages = all_stages;
  }
  if (plan.dp_tiles > 0) {
    const hipError_t e = launch_lane(128, 1, dim3((unsigned)plan.dp_tiles), a_codes, a_scales, a_gs,
                                     b_codes, b_scales, b_gs, bias, out, M, N, K, whole, stream);
    if (e != hipSuccess) return e;
  }
  const int groups = lane_groups(quads * tail.splits, K, tail.stages);
  return launch_lane(64, groups, dim3((unsigned)(quads * tail.splits)), a_codes, a_scales, a_gs,
                     b_codes, b_scales, b_gs, bias, out, M, N, K, tail, stream);
}

hipError_t launch_gemm_regular(const uint8_t* a_codes, const uint8_t* a_scales, const float* a_gs,
                               const uint8_t* b_codes, const uint8_t* b_scales, const float* b_gs,
                               const uint16_t* bias, uint16_t* out, int64_t M, int64_t N, int64_t K,
                               void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (M == 0 || N == 0) return hipSuccess;
  const int64_t tiles = ((M + kBM - 1) / kBM) * ((N + kBN - 1) / kBN);
  const dim3 grid((unsigned)tiles);
  const bool vec = N % 8 == 0;
  // Kernel choice as in gemm_plan (at K = 5600, where the shared kernel
  // must take its unaligned path, the lane kernel is 1.46x faster).
  bool small = false;
  SplitPlan plan = gemm_plan(M, N, K, &small);
  if (plan.active() && (workspace == nullptr || workspace_bytes < plan.bytes)) {
    // no room: every tile (or quadrant) whole
    const bool quad = plan.quad;
    const int64_t rem = plan.rem_tiles;
    plan = SplitPlan{};
    plan.dp_tiles = small ? ((M + 127) / 128) * ((N + 127) / 128) : ((M + 255) / 256) * ((N + 255) / 256);
    plan.stages = (K + kLBK - 1) / kLBK;
    if (quad) {
      plan.quad = true;
      plan.rem_tiles = rem;
      plan.dp_tiles -= rem;
    }
  }
  if (plan.quad)
    return launch_gemm_quad(a_codes, a_scales, a_gs, b_codes, b_scales, b_gs, bias, out, M, N, K,
                            plan, workspace, stream);
  if (lane_takes(M, N, K, small, plan.active())) {
    const SplitK split = split_args(plan, workspace);
    const dim3 lgrid((unsigned)(plan.dp_tiles + plan.rem_tiles * plan.splits));
    const int groups = small ? lane_groups(lgrid.x, K, split.stages) : 1;
    return launch_lane(small ? 64 : 128, groups, lgrid, a_codes, a_scales, a_gs, b_codes, b_scales, b_gs, bias, out, M, N, K, split, stream);
  }
  const dim3 block(kGemmThreads);
  const bool fast = K % kBK == 0;
#define SOLFP4_SHARED_LAUNCH(F, V)                                                             \
  launch_kernel(nvfp4_gemm_kernel<F, V>, grid, block, stream, a_codes, a_scales, a_gs, b_codes, \
                b_scales, b_gs, bias, out, M, N, K)
  if (fast && vec) return SOLFP4_SHARED_LAUNCH(true, true);
  if (fast) return SOLFP4_SHARED_LAUNCH(true, false);
  if (vec) return SOLFP4_SHARED_LAUNCH(false, true);
  return SOLFP4_SHARED_LAUNCH(false, false);
#undef SOLFP4_SHARED_LAUNCH
}

}  // namespace solfp4
