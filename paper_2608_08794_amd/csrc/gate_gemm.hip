// Gate GEMM of the direct audio-visual distance (Section 3.1, "Gated fine
// pass"; the fine-pass term of Eq. 2): for every visual token i of a clip
// whose gate fired, max_j x_A[j] . x_V[i] / |x_A[j]|, from C = X_A X_V^T on
// bf16 MFMA with fp32 accumulation.  This is the kernel for bf16 inputs
// whose dim is a multiple of 64; k_gate_gemm_any below covers the rest.
//
// Each workgroup owns a tile of 32 BI x 256 (audio rows x visual columns; BI
// is 8 unless fewer rows fill the chip better, see gate_gemm256_tiles); its
// eight waves (two per SIMD) own 16 BI x 64 blocks as BI x 4 blocks of
// v_mfma_f32_16x16x32_bf16, so with BI = 8 a wave reads 12 fragments from
// LDS per 32 MFMAs.  K streams through two 64-element LDS stages (2 x 64 KiB
// with BI = 8), filled by 16-byte direct-to-LDS loads; the 128-byte rows are stored with their
// 16-byte chunks XOR-swizzled by the row index, so the fragment reads of
// consecutive rows hit distinct banks without padding.  Every output
// element sums K in order, 32 elements per MFMA, whatever its tile.  The
// epilogue scales by the inverse audio norms and folds the column maxima
// into order-preserving keys with atomicMax.
//
// What bounds it is power: at the long clips' sizes the clock falls to
// 1.5-1.7 GHz, and the rate follows the energy of a product rather than its
// schedule.  In registers alone the 16x16x32 form sustains 2.07 PFLOP/s and
// the 32x32x16 form 1.82 (with every fragment read from LDS 1.86 and 1.68),
// because it moves half as many accumulator bytes per product.  A 290 s clip
// (7250 x 83520 x 3584) takes 3.33 ms (1.30 PFLOP/s) against 3.62 with
// 32x32x16, a 60 s clip 158 us against 176.  Four waves of 128 x 128 (a third
// fewer LDS reads) took 4.06 ms: one wave per SIMD leaves its waits bare.
//
// Workgroups are dealt to the eight XCDs round-robin by index, so the host
// lists the tiles so that each XCD gets a run of column blocks of one band
// of at most eight row tiles, and the workgroups resident on one XCD share
// both operands in that XCD's L2: a band's audio rows and a few column
// blocks of visual rows.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "dynamics_plan.hpp"

namespace apack {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(1))) void* glb_ptr_t;

constexpr int kTileN = 256;                    // columns per workgroup
constexpr int kK = kGemm256K;                  // K elements per LDS stage
constexpr int kRowB = kK * 2;                  // bytes of one row per stage
constexpr int kChunks = kRowB / 16;            // 16-byte chunks per row
constexpr int kWaves = 8;
constexpr int kWN = 4;                         // waves along the visual columns
constexpr int kBJ = kTileN / kWN / 16;         // 16-column blocks per wave
static_assert(kK == 64, "two 32-element slices per stage");

// Shape of a tile of 32 BI rows.
template <int BI>
struct TileGeom {
  static constexpr int kTileM = kWaves / kWN * BI * 16;
  static constexpr int kOpA = kTileM * kRowB, kOpB = kTileN * kRowB;   // operands' bytes per stage
  static constexpr int kStageB = kOpA + kOpB;
  // LDS stages: a stage of few rows carries too little arithmetic to cover
  // the latency of its loads, so they run further ahead (bi = 2: 49 us with
  // two stages, 35 with four).
  static constexpr int kStages = 160 * 1024 / kStageB < 4 ? 160 * 1024 / kStageB : 4;
  static constexpr int kReads = BI + kBJ;      // fragments of one 32-element K slice
  static constexpr int kMfmas = BI * kBJ;      // MFMAs of one slice
  // 1 KiB loads per wave and stage.  Where the waves do not share the audio
  // rows evenly, the last load is issued by more than one wave (the same
  // bytes to the same place).
  static constexpr int kLoadsA = (kOpA / 1024 + kWaves - 1) / kWaves, kLoadsB = kOpB / 1024 / kWaves;
  static constexpr int kLoads = kLoadsA + kLoadsB;
  // MFMAs from one fragment read, and from one load, to the next.
  static constexpr int kReadStep = kMfmas >= 2 * kReads ? 2 : 1;
  static constexpr int kLoadStep = kMfmas >= 3 * kLoads ? 3 : kMfmas >= 2 * kLoads ? 2 : 1;
  static_assert(kMfmas >= kReads && kMfmas >= kLoads && kStages >= 2, "slots of the K-slice schedule");
};
constexpr int kXcds = 8;

// Chunk c of row r sits at chunk c ^ swz(r).  A 16-byte LDS read is served
// sixteen lanes at a time across 64 four-byte banks (256 bytes); the
// sixteen consecutive rows those lanes read must then fill the 256 bytes
// once.  Rows share a 256-byte window kRowsPer256 at a time, so the XOR key
// is the row's index among the rows that fall on the same banks.
constexpr int kRowsPer256 = 256 / kRowB;
__device__ __forceinline__ int swz(int r) { return (r / kRowsPer256) & (kChunks - 1); }

// One operand's stage: rows r0, r0 + 1, ... (clamped to the last valid row),
// elements [k0, k0 + kK).  Load j fills LDS bytes [1024 j, 1024 j + 1024);
// lane l's 16 bytes land at row r = (1024 j + 16 l) / kRowB, chunk c, and
// come from global chunk c ^ swz(r).  The result is lane l's byte offset of
// load j from the stage's first byte (row r0, element k0), the same for
// every stage, so a stage only moves the scalar base.
__device__ __forceinline__ uint32_t load_offset(int64_t r0, int64_t n_rows, int dim, int j, int lane) {
  const int byte = j * 1024 + lane * 16;
  const int r = byte / kRowB;
  const int c = ((byte % kRowB) >> 4) ^ swz(r);
  const int64_t left = n_rows - 1 - r0;
  const int rr = left < r ? (int)left : r;
  return (uint32_t)rr * (uint32_t)dim * 2u + (uint32_t)c * 16u;
}

// p as a scalar (it is the same in every lane), so that the loads that add a
// per-lane offset to it take the scalar-base form.
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}

// MFMA operand of rows row .. row+15 (row a multiple of 16 plus lane % 16)
// and K elements [32 ks, 32 ks + 32): lane l holds 8 elements at
// 32 ks + 8 (l / 16).
__device__ __forceinline__ bf16x8 lds_frag(const char* lds, int row, int ks, int lane) {
  const int c = (ks * 4 + (lane >> 4)) ^ swz(row);
  return *reinterpret_cast<const bf16x8*>(lds + row * kRowB + c * 16);
}

// e such that 2^-e takes a row of squared norm nn to a norm in [1, 2), kept
// where 2^e and 2^-e are normal floats (a row of smaller or larger norm comes
// within 2^-23 and 2^8 of that); an all-zero row stays all zero.
__device__ __forceinline__ int row_exponent(double nn) {
  const int e = ((int)((uint64_t)__double_as_longlong(nn) >> 52 & 0x7FF) - 1023) >> 1;
  return min(max(e, -126), 126);
}
__device__ __forceinline__ float exp2_int(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }

// Inverse norms of audio rows m0 .. m0 + M - 1 (0 for a zero row, -inf past
// the clip's audio, so those rows never win), of the scaled rows if SCALED.
template <int M, bool SCALED>
__device__ __forceinline__ void inverse_norms(float* inv, const double* na, int64_t m0, int64_t n_a, int tid) {
  for (int r = tid; r < M; r += kWaves * 64) {
    float s = -INFINITY;
    if (m0 + r < n_a) {
      const double nn = na[m0 + r];
      const double up = SCALED ? (double)exp2_int(row_exponent(nn)) : 1.0;
      s = nn > 0.0 ? (float)(1.0 / sqrt(nn) * up) : 0.0f;
    }
    inv[r] = s;
  }
}

// Largest scaled product of each of a wave's columns, merged into the keys:
// acc[i][j][e] of lane l is row 16 i + 4(l/16) + e of inv and column
// n0 + 16 j + l%16.  SCALED: the products are of scaled rows, and nv holds the
// columns' squared norms; a column of infinite norm (whose parts are NaN) gets
// +inf, as its products with the unsplit values would have.
template <bool SCALED, int BI, int BJ>
__device__ __forceinline__ void column_maxima(const f32x4 (&acc)[BI][BJ], const float* inv, int lane, int64_t n0,
                                              int64_t n_v, const double* nv, uint32_t* maxkey) {
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float s = inv[i * 16 + 4 * (lane >> 4) + e];
        m = fmaxf(m, s == -INFINITY ? -INFINITY : acc[i][j][e] * s);
      }
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    const int64_t col = n0 + j * 16 + (lane & 15);
    if constexpr (SCALED) {
      const double nn = nv[min(col, n_v - 1)];
      m = nn == (double)INFINITY ? INFINITY : m * exp2_int(row_exponent(nn));
    }
    if (lane < 16 && col < n_v && m > -INFINITY) atomicMax(&maxkey[col], order_key(m));
  }
}

template <int BI>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gate_gemm256(
    const ClipDev* __restrict__ clips, const GemmTileDev* __restrict__ tiles, int dim, const uint16_t* __restrict__ xv,
    const uint16_t* __restrict__ xa, const double* __restrict__ na, uint32_t* __restrict__ maxkey) {
  using G = TileGeom<BI>;
  constexpr int kBI = BI, kStageB = G::kStageB, kOpA = G::kOpA, kReads = G::kReads, kMfmas = G::kMfmas,
                kLoads = G::kLoads;
  constexpr int S = G::kStages;
  __shared__ __attribute__((aligned(16))) char lds[S * kStageB];
  const GemmTileDev tl = tiles[blockIdx.x];
  if (tl.clip < 0) return;  // padding of an XCD's share
  const ClipDev c = clips[tl.clip];
  if (!c.gate) return;
  const int64_t n_a = c.n_audio, n_v = (int64_t)c.n_frames * c.per_frame;
  const uint16_t* A = xa + c.aud_off * dim;
  const uint16_t* B = xv + c.vis_off * dim;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / kWN, wn = wave % kWN;

  f32x4 acc[kBI][kBJ];
#pragma unroll
  for (int i = 0; i < kBI; ++i)
#pragma unroll
    for (int j = 0; j < kBJ; ++j) acc[i][j] = f32x4{};

  const int n_k = dim / kK;
  const char* base_a = reinterpret_cast<const char*>(A + row_start(tl.m0, dim));
  const char* base_b = reinterpret_cast<const char*>(B + row_start(tl.n0, dim));
  // Load l of this wave's share of a stage: audio rows first.
  int at[kLoads];         // LDS byte of the load within the stage
  uint32_t off[kLoads];   // this lane's offset from its base
#pragma unroll
  for (int l = 0; l < kLoads; ++l) {
    const bool audio = l < G::kLoadsA;
    const int j = audio ? min(wave + kWaves * l, kOpA / 1024 - 1) : wave + kWaves * (l - G::kLoadsA);
    at[l] = (audio ? 0 : kOpA) + j * 1024;
    off[l] = audio ? load_offset(tl.m0, n_a, dim, j, lane) : load_offset(tl.n0, n_v, dim, j, lane);
  }
  auto issue_load = [&](char* stage, const char* ga, const char* gb, int l) {
    __builtin_amdgcn_global_load_lds((glb_ptr_t)((l < G::kLoadsA ? ga : gb) + off[l]), (lds_ptr_t)(stage + at[l]), 16, 0,
                                     0);
  };
  auto issue = [&](int k_stage) {
#pragma unroll
    for (int l = 0; l < kLoads; ++l)
      issue_load(lds + k_stage * kStageB, base_a + (size_t)k_stage * kRowB, base_b + (size_t)k_stage * kRowB, l);
  };
  // Fragments of the slice in hand and of the next one; read r of a slice in
  // the order its MFMAs first need them: fa[0], fb[0 ..], fa[1 ..].
  bf16x8 fa[2][kBI], fb[2][kBJ];
  const int row_a = wm * kBI * 16 + (lane & 15), row_b = wn * kBJ * 16 + (lane & 15);
  auto read = [&](const char* stage, int ks, int r) {
    if (r >= 1 && r <= kBJ)
      fb[ks][r - 1] = lds_frag(stage + kOpA, row_b + 16 * (r - 1), ks, lane);
    else
      fa[ks][r == 0 ? 0 : r - kBJ] = lds_frag(stage, row_a + 16 * (r == 0 ? 0 : r - kBJ), ks, lane);
  };
  // The first S stages (issue takes a stage below S); stage 0 is awaited.
#pragma unroll
  for (int p = 0; p < S; ++p)
    if (p < n_k) issue(p);
  if (n_k >= S)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * kLoads) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int r = 0; r < kReads; ++r) read(lds, 0, r);
  __builtin_amdgcn_sched_barrier(0);
  // One stage, its two slices' MFMAs back to back.  Slice 0's run over the
  // reads of slice 1; then every wave waits for its loads of stage it + 1
  // (issued S - 1 stages ago) and its last reads of stage it, so that past
  // the barrier stage it + 1 is whole and this stage's buffer is free; slice
  // 1's MFMAs run over the first reads of stage it + 1 and the loads of stage
  // it + S.  The scheduling barriers hold one fragment read behind every
  // second MFMA and one load behind every third (with BI = 8): loads issued in a burst
  // stop the MFMAs behind them (spaced every MFMA 169 us on the 60 s clip,
  // second 162, third 158, fourth 158; every second one is 1% faster on the
  // 290 s clip, every fourth 4% slower).
  int buf = 0;   // it % S
  auto stage = [&](int it, auto load_tag, auto next_tag) {
    constexpr bool kLoad = decltype(load_tag)::value, kNext = decltype(next_tag)::value;
    char* cur = lds + buf * kStageB;
    buf = buf + 1 == S ? 0 : buf + 1;
    const char* next = lds + buf * kStageB;
    const char* next_a = uniform_ptr(base_a + (size_t)(it + S) * kRowB);
    const char* next_b = uniform_ptr(base_b + (size_t)(it + S) * kRowB);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if (ks == 1 && kNext) {
        if constexpr (kLoad)   // the loads of the S - 2 stages after it + 1 stay in flight
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * kLoads) : "memory");
        else
          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int g = 0; g < kMfmas; ++g) {
        const int i = g / kBJ, j = g % kBJ;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
        if (g % G::kReadStep == 0 && g / G::kReadStep < kReads && (ks == 0 || kNext)) {
          read(ks == 0 ? cur : next, ks ^ 1, g / G::kReadStep);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (ks == 1 && kLoad && (g + 1) % G::kLoadStep == 0 && g / G::kLoadStep < kLoads) {
          issue_load(cur, next_a, next_b, g / G::kLoadStep);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int it = 0;
  for (; it + S < n_k; ++it) stage(it, std::true_type{}, std::true_type{});
  for (; it + 1 < n_k; ++it) stage(it, std::false_type{}, std::true_type{});
  stage(it, std::false_type{}, std::false_type{});

  // Epilogue.  Inverse audio norms of the tile's rows in LDS (-inf past the
  // clip's audio, so those rows never win); acc[i][j][e] of lane l is audio
  // row 16 (kBI wm + i) + 4(l/16) + e, visual column 16 (kBJ wn + j) + l%16.
  __syncthreads();
  float* inv = reinterpret_cast<float*>(lds);
  inverse_norms<G::kTileM, false>(inv, na + c.aud_off, tl.m0, n_a, tid);
  __syncthreads();
  column_maxima<false>(acc, inv + wm * kBI * 16, lane, tl.n0 + wn * kBJ * 16, n_v, nullptr, maxkey + c.vis_off);
}

// ---------------------------------------------------------------------------
// The same product for fp32 inputs, and for bf16 inputs of any dim (a
// multiple of 8): tiles of 256 x 128, eight waves of 64 x 64, the operands
// staged through registers into two LDS buffers.
//
// fp32: each row is scaled by the power of two that takes its norm to [1, 2)
// (row_exponent; undone in the epilogue), then each value is split into three
// bf16 parts, x = h + m + l (each part the rounded remainder of the last:
// 8 + 8 + 8 significand bits).  The split is exact for values of at least
// 2^-102 of the row's norm, whose last parts are normal bf16; smaller ones
// lose less than 2^-125 of the norm.  The distance is a cosine, so rows of any
// magnitude keep the same bits (unscaled, rows near 2^-118 had lost up to 6e-3
// of a value).  The scaling is one product per value in place of a clamp that
// unscaled first parts need.  x y is summed as
// h h, and l h + h l + m h + m m + h m in accumulators of their own, on the
// bf16 matrix cores: six MFMAs of 32 elements in fp32.  What is left out (m l,
// l m, l l) is below 2^-25 of the product.  The large sum is rounded K / 32
// times where v_mfma_f32_32x32x2_f32 rounds it K / 2 times, the small one at
// 2^-8 of its size.  (With all six in one accumulator every product of every
// step was rounded to the large sum: on one-signed rows up to twice the error
// of the fp32 unit.)  Error of 1 - distance against 64 bits, rms over four
// sets of random / one-signed / wide-ranging rows, here and on
// v_mfma_f32_32x32x2_f32, in 1e-8: dim 264 1.8 / 12 / 3.9 and 5.2 / 25 / 8.5,
// 2048 1.4 / 21 / 2.8 and 4.6 / 89 / 25, 3584 1.5 / 35 / 3.2 and 4.5 / 80 / 26,
// 16384 1.5 / 55 / 3.3 and 4.6 / 183 / 58.  The fp32 MFMA peaks at 157 TFLOP/s;
// six bf16 ones leave room for twice that: 1500 x 17280 x 2048 takes 638 us
// against 1148 (644 with one accumulator), and 1500 x 17280 x 1288 in bf16 129
// against 141 (128 x 128 tiles on 32x32x16 MFMAs).  The second accumulators
// fit because the second parts are read into the third ones' registers; sums
// of a step added to one set of accumulators by the vector ALU were as exact
// and 5-8% slower.
// Parts are kept as planes of 64-byte LDS rows (32 elements), so a fragment
// read once serves two or three products.
// ---------------------------------------------------------------------------
constexpr int kAnyM = 256, kAnyN = 128;        // tile rows (audio) and columns (visual)
constexpr int kAnyRows = kAnyM + kAnyN;
constexpr int kAnyB = 4;                       // 16-row (and 16-column) blocks per wave
constexpr int kAnyWN = kAnyN / (kAnyB * 16);   // waves along the columns
constexpr int kSubB = kAnyRows * 64;           // one plane of one 32-element slice

template <class T> struct AnyGeom;
template <> struct AnyGeom<uint16_t> {
  static constexpr int planes = 1, slices = 2;
};
template <> struct AnyGeom<float> {
  static constexpr int planes = 3, slices = 1;
};

// Eight consecutive elements in flight, and their parts as eight bf16 each.
template <class T> struct Unit;
template <> struct Unit<uint16_t> {
  uint4 u;
  __device__ __forceinline__ void load(const uint16_t* p) { u = *reinterpret_cast<const uint4*>(p); }
  __device__ __forceinline__ void parts(bool valid, float, uint4 (&out)[1]) const {
    out[0] = valid ? u : make_uint4(0, 0, 0, 0);
  }
};
template <> struct Unit<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = reinterpret_cast<const float4*>(p)[0];
    b = reinterpret_cast<const float4*>(p)[1];
  }
  // Two bf16 (round to nearest even) packed, and what they leave of the pair.
  static __device__ __forceinline__ uint32_t split(const float x, const float y, float& rx, float& ry) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const bf16x2 h = __builtin_convertvector(f32x2{x, y}, bf16x2);
    uint32_t w;
    __builtin_memcpy(&w, &h, 4);
    rx = x - __uint_as_float(w << 16);
    ry = y - __uint_as_float(w & 0xFFFF0000u);
    return w;
  }
  __device__ __forceinline__ void parts(bool valid, float scale, uint4 (&out)[3]) const {
    const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float x = valid ? v[2 * i] * scale : 0.0f, y = valid ? v[2 * i + 1] * scale : 0.0f;
#pragma unroll
      for (int p = 0; p < 3; ++p) w[p][i] = split(x, y, x, y);
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) out[p] = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
  }
};

template <class T>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gate_gemm_any(
    const ClipDev* __restrict__ clips, const GemmTileDev* __restrict__ tiles, int dim, const T* __restrict__ xv,
    const T* __restrict__ xa, const double* __restrict__ nv, const double* __restrict__ na,
    uint32_t* __restrict__ maxkey) {
  constexpr bool kScaled = sizeof(T) == 4;   // rows scaled before they are split
  constexpr int NP = AnyGeom<T>::planes, KS = AnyGeom<T>::slices;
  constexpr int kStep = 32 * KS, kBufB = KS * NP * kSubB;
  constexpr int kUnits = kAnyRows * 4 * KS / (kWaves * 64);   // 8-element units per thread per step
  static_assert(kAnyRows * 4 * KS % (kWaves * 64) == 0 && kAnyM * 4 % (kWaves * 64) == 0, "whole units per thread");
  __shared__ __attribute__((aligned(16))) char lds[2 * kBufB];
  const GemmTileDev tl = tiles[blockIdx.x];
  if (tl.clip < 0) return;  // padding of an XCD's share
  const ClipDev c = clips[tl.clip];
  if (!c.gate) return;
  const int64_t n_a = c.n_audio, n_v = (int64_t)c.n_frames * c.per_frame;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / kAnyWN, wn = wave % kAnyWN;

  // Unit i of this thread: row (tid + 512 i) / 4 of slice i / (kUnits / KS),
  // chunk tid % 4; audio rows first (clamped to the clip's last rows).
  const int chunk = tid & 3;
  const T* row[kUnits / KS];
  float scale[kUnits / KS];
#pragma unroll
  for (int i = 0; i < kUnits / KS; ++i) {
    const int r = (tid >> 2) + i * (kWaves * 16);
    const int64_t at = r < kAnyM ? c.aud_off + min(tl.m0 + (int64_t)r, n_a - 1)
                                 : c.vis_off + min(tl.n0 + (int64_t)(r - kAnyM), n_v - 1);
    row[i] = (r < kAnyM ? xa : xv) + row_start(at, dim);
    scale[i] = kScaled ? exp2_int(-row_exponent((r < kAnyM ? na : nv)[at])) : 1.0f;
  }
  Unit<T> raw[kUnits];
  auto gload = [&](int k0) {
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
      raw[u].load(row[u % (kUnits / KS)] + min(k0 + 32 * (u / (kUnits / KS)) + chunk * 8, dim - 8));
  };
  auto lstore = [&](int k0, char* buf) {
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
      const int ks = u / (kUnits / KS), r = (tid >> 2) + (u % (kUnits / KS)) * (kWaves * 16);
      uint4 part[NP];
      raw[u].parts(k0 + 32 * ks + chunk * 8 < dim, scale[u % (kUnits / KS)], part);
#pragma unroll
      for (int p = 0; p < NP; ++p)
        *reinterpret_cast<uint4*>(buf + (ks * NP + p) * kSubB + r * 64 + ((chunk ^ (r >> 2)) & 3) * 16) = part[p];
    }
  };
  // Fragment of rows row .. row + 15: chunk c of row r sits at c ^ (r / 4),
  // so sixteen consecutive rows fill 256 bytes once.
  auto frag = [&](const char* sub, int r) {
    return *reinterpret_cast<const bf16x8*>(sub + r * 64 + (((lane >> 4) ^ (r >> 2)) & 3) * 16);
  };

  f32x4 acc[kAnyB][kAnyB], low[kAnyB][kAnyB];   // low: the sum of the small products (fp32 inputs)
#pragma unroll
  for (int i = 0; i < kAnyB; ++i)
#pragma unroll
    for (int j = 0; j < kAnyB; ++j) acc[i][j] = low[i][j] = f32x4{};
  const int n_k = (dim + kStep - 1) / kStep;
  const int row_a = wm * kAnyB * 16 + (lane & 15), row_b = kAnyM + wn * kAnyB * 16 + (lane & 15);
  gload(0);
  lstore(0, lds);
  gload(kStep);
  for (int it = 0; it < n_k; ++it) {
    // Every wave's share of step it is in LDS, and the other buffer is no
    // longer read; the loads of step it + 1 stay in flight.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const char* buf = lds + (it & 1) * kBufB;
    bf16x8 fa[KS * NP][kAnyB], fb[KS * NP][kAnyB];
    auto read_a = [&](int p) {
#pragma unroll
      for (int i = 0; i < kAnyB; ++i) fa[p][i] = frag(buf + p * kSubB, row_a + 16 * i);
    };
    auto read_b = [&](int p) {
#pragma unroll
      for (int i = 0; i < kAnyB; ++i) fb[p][i] = frag(buf + p * kSubB, row_b + 16 * i);
    };
    auto product = [&](int pa, int pb, f32x4 (&sum)[kAnyB][kAnyB]) {
#pragma unroll
      for (int i = 0; i < kAnyB; ++i)
#pragma unroll
        for (int j = 0; j < kAnyB; ++j)
          sum[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[pa][i], fb[pb][j], sum[i][j], 0, 0, 0);
    };
    if constexpr (NP == 3) {
      read_a(2);
      read_b(0);
      read_a(0);
      read_b(2);
    } else {
#pragma unroll
      for (int p = KS - 1; p >= 0; --p) {
        read_a(p);
        read_b(p);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // The next step is split and stored under this step's products.
    lstore((it + 1) * kStep, lds + ((it + 1) & 1) * kBufB);
    gload((it + 2) * kStep);
    if constexpr (NP == 3) {
      // The second parts are read as the third ones' registers come free.
      product(2, 0, low);
      read_a(1);
      product(0, 2, low);
      read_b(1);
      product(1, 0, low);
      product(1, 1, low);
      product(0, 1, low);
      product(0, 0, acc);
#pragma unroll
      for (int g = 0; g < 6 * kAnyB * kAnyB; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);   // two VALU instructions
        if (g >= 15 && g < 15 + kAnyB) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
        if (g >= 31 && g < 31 + kAnyB) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    } else {
#pragma unroll
      for (int p = 0; p < KS; ++p) product(p, p, acc);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // Epilogue, as above: acc[i][j][e] of lane l is audio row
  // 16 (kAnyB wm + i) + 4(l/16) + e, visual column 16 (kAnyB wn + j) + l%16.
  __syncthreads();
  float* inv = reinterpret_cast<float*>(lds);
  if constexpr (NP == 3) {
#pragma unroll
    for (int i = 0; i < kAnyB; ++i)
#pragma unroll
      for (int j = 0; j < kAnyB; ++j) acc[i][j] += low[i][j];
  }
  inverse_norms<kAnyM, kScaled>(inv, na + c.aud_off, tl.m0, n_a, tid);
  __syncthreads();
  column_maxima<kScaled>(acc, inv + wm * kAnyB * 16, lane, tl.n0 + wn * kAnyB * 16, n_v, nv + c.vis_off,
                         maxkey + c.vis_off);
}

}  // namespace

constexpr int kCUs = 256;
constexpr double kRoundCost = 5.0;

// One tile per workgroup, of tile_m audio rows by tile_n visual columns; a
// list that its padding takes past `most` goes without.
static std::vector<GemmTileDev> gate_gemm_tiles(const std::vector<ClipDev>& clips, int tile_m, int tile_n,
                                                int64_t most) {
  // A clip's row tiles are cut into bands of at most kBandRows (as even as
  // possible); a band's tiles, column block after column block, are cut into
  // eight runs of equal length, one per XCD.  A tall clip's audio then passes
  // through each XCD's L2 once per band and column block rather than once per
  // column block, and no XCD gets more tiles than its share: whole column
  // blocks to each had given some 35 of a 45 s clip's 255 tiles to an XCD's
  // 32 compute units, a second round (144 us; 87 now).
  constexpr int kBandRows = 8;
  std::vector<std::vector<GemmTileDev>> share(kXcds);
  int first = 0;   // XCD of the band's first run
  for (size_t s = 0; s < clips.size(); ++s) {
    const ClipDev& c = clips[s];
    const int64_t nv = (int64_t)c.n_frames * c.per_frame;
    if (nv == 0 || c.n_audio == 0) continue;
    const int mb = (int)((c.n_audio + tile_m - 1) / tile_m), nb = (int)((nv + tile_n - 1) / tile_n);
    const int n_band = (mb + kBandRows - 1) / kBandRows;
    for (int b = 0; b < n_band; ++b, first = (first + 1) % kXcds) {
      const int m0 = (int)((int64_t)b * mb / n_band), rows = (int)((int64_t)(b + 1) * mb / n_band) - m0;
      const int64_t n_tiles = (int64_t)rows * nb;
      for (int64_t t = 0; t < n_tiles; ++t)
        share[(first + t * kXcds / n_tiles) % kXcds].push_back(
            {(int32_t)s, (m0 + (int)(t % rows)) * tile_m, (int)(t / rows) * tile_n, 0});
    }
  }
  size_t rounds = 0;
  for (auto& q : share) rounds = std::max(rounds, q.size());
  std::vector<GemmTileDev> out;
  out.reserve(rounds * kXcds);
  for (size_t r = 0; r < rounds; ++r)
    for (int x = 0; x < kXcds; ++x) out.push_back(r < share[x].size() ? share[x][r] : GemmTileDev{-1, 0, 0, 0});
  // Trailing padding only costs empty workgroups; drop it.
  while (!out.empty() && out.back().clip < 0) out.pop_back();
  if ((int64_t)out.size() > most)
    out.erase(std::remove_if(out.begin(), out.end(), [](const GemmTileDev& t) { return t.clip < 0; }), out.end());
  return out;
}

// Rows per tile (32 bi) of a call: the tiles run in rounds of one per compute
// unit, and a round of tiles of bi blocks costs about bi + kRoundCost (a part
// is paid whatever the rows: the visual operand's loads and reads, filling
// the pipeline, the epilogue), so a part-empty round is weighed against
// smaller tiles.  Measured on 3584-d clips, us with bi = 8 and as chosen:
// 4 s 68 and 36 (bi 2), 20 s 70 and 35 (2), 30 s 72 and 49 (4), 45 s 87 and 87
// (8), 60 s 158 and 149 (7), 100 s 412 and 409 (8); a round takes 77 us with
// bi 8, 73 with 7, 60 with 6, 55 with 5, 48 with 4, 40 with 3 and 33 with 2.
std::vector<GemmTileDev> gate_gemm256_tiles(const std::vector<ClipDev>& clips, int64_t most, int* bi_out) {
  int best = 8;
  double best_cost = 0.0;
  for (int bi = 8; bi >= 2; --bi) {
    int64_t n = 0;
    for (const ClipDev& c : clips)
      n += ((c.n_audio + 32 * bi - 1) / (32 * bi)) * (((int64_t)c.n_frames * c.per_frame + kTileN - 1) / kTileN);
    const double cost = (double)((n + kCUs - 1) / kCUs) * (bi + kRoundCost);
    if (bi == 8 || (n <= most && cost < best_cost)) {   // tiles of 256 x 256 are never more than `most`
      best = bi;
      best_cost = cost;
    }
  }
  *bi_out = best;
  return gate_gemm_tiles(clips, 32 * best, kTileN, most);
}
std::vector<GemmTileDev> gate_gemm_any_tiles(const std::vector<ClipDev>& clips, int64_t most) {
  return gate_gemm_tiles(clips, kAnyM, kAnyN, most);
}

apack_status launch_gate_gemm256(const ClipDev* clips, const GemmTileDev* tiles, int64_t n_tiles, int bi, int dim,
                                 const uint16_t* xv, const uint16_t* xa, const double* na, uint32_t* maxkey,
                                 hipStream_t stream) {
  if (n_tiles == 0) return APACK_OK;
  auto kernel = bi == 8   ? k_gate_gemm256<8>
                : bi == 7 ? k_gate_gemm256<7>
                : bi == 6 ? k_gate_gemm256<6>
                : bi == 5 ? k_gate_gemm256<5>
                : bi == 4 ? k_gate_gemm256<4>
                : bi == 3 ? k_gate_gemm256<3>
                          : k_gate_gemm256<2>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)n_tiles), dim3(kWaves * 64), 0, stream, clips, tiles, dim, xv, xa, na,
                     maxkey);
  return launch_status("k_gate_gemm256");
}

apack_status launch_gate_gemm_any(const ClipDev* clips, const GemmTileDev* tiles, int64_t n_tiles, int dim, bool bf16,
                                  const void* xv, const void* xa, const double* nv, const double* na, uint32_t* maxkey,
                                  hipStream_t stream) {
  if (n_tiles == 0) return APACK_OK;
  const dim3 grid((unsigned)n_tiles), block(kWaves * 64);
  if (bf16)
    hipLaunchKernelGGL(k_gate_gemm_any<uint16_t>, grid, block, 0, stream, clips, tiles, dim,
                       static_cast<const uint16_t*>(xv), static_cast<const uint16_t*>(xa), nv, na, maxkey);
  else
    hipLaunchKernelGGL(k_gate_gemm_any<float>, grid, block, 0, stream, clips, tiles, dim, static_cast<const float*>(xv),
                       static_cast<const float*>(xa), nv, na, maxkey);
  return launch_status("k_gate_gemm_any");
}

}  // namespace apack
