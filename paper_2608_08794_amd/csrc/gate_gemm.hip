// Gate GEMM of the direct audio-visual distance (Section 3.1, "Gated fine
// pass"; the fine-pass term of Eq. 2): for every visual token i of a clip
// whose gate fired, max_j x_A[j] . x_V[i] / |x_A[j]|, from C = X_A X_V^T on
// bf16 MFMA with fp32 accumulation.  This is the kernel for bf16 inputs
// whose dim is a multiple of 64; k_gate_gemm in dynamics.hip covers the rest.
//
// Each workgroup owns a 256 x 256 tile (audio rows x visual columns); its
// eight waves (two per SIMD) own 128 x 64 blocks as 8 x 4 blocks of
// v_mfma_f32_16x16x32_bf16, so a wave reads 12 fragments from LDS per 32
// MFMAs.  K streams through two 64-element LDS stages (2 x 64 KiB), filled
// by 16-byte direct-to-LDS loads; the 128-byte rows are stored with their
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
// lists the tiles so that each XCD gets whole column blocks of one band of
// at most eight row tiles, and the workgroups resident on one XCD share
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

constexpr int kTile = 256;                     // rows and columns per workgroup
constexpr int kK = kGemm256K;                  // K elements per LDS stage
constexpr int kRowB = kK * 2;                  // bytes of one row per stage
constexpr int kChunks = kRowB / 16;            // 16-byte chunks per row
constexpr int kOpB = kTile * kRowB;            // one operand's stage
constexpr int kStageB = 2 * kOpB;
constexpr int kWaves = 8;
constexpr int kWN = 4;                         // waves along the visual columns
constexpr int kBI = kTile / (kWaves / kWN) / 16;  // 16-row blocks per wave
constexpr int kBJ = kTile / kWN / 16;             // 16-column blocks per wave
constexpr int kReads = kBI + kBJ;                 // fragments of one 32-element K slice
constexpr int kMfmas = kBI * kBJ;                 // MFMAs of one slice
constexpr int kLoadsPerWave = kOpB / 1024 / kWaves;  // 1 KiB loads per wave per operand
static_assert(kK == 64 && kMfmas >= 2 * kReads && kMfmas >= 3 * 2 * kLoadsPerWave, "slots of the K-slice schedule");
constexpr int kXcds = 8;

// Chunk c of row r sits at chunk c ^ swz(r).  A 16-byte LDS read is served
// sixteen lanes at a time across 64 four-byte banks (256 bytes); the
// sixteen consecutive rows those lanes read must then fill the 256 bytes
// once.  Rows share a 256-byte window kRowsPer256 at a time, so the XOR key
// is the row's index among the rows that fall on the same banks.
constexpr int kRowsPer256 = 256 / kRowB;
__device__ __forceinline__ int swz(int r) { return (r / kRowsPer256) & (kChunks - 1); }

// One operand's stage: rows r0 .. r0+255 (clamped to the last valid row),
// elements [k0, k0 + kK).  Load j fills LDS bytes [1024 j, 1024 j + 1024);
// lane l's 16 bytes land at row r = (1024 j + 16 l) / kRowB, chunk c, and
// come from global chunk c ^ swz(r).  off[i] is lane l's byte offset of load
// i from the stage's first byte (row r0, element k0), the same for every
// stage, so a stage only moves the scalar base.
__device__ __forceinline__ void operand_offsets(int64_t r0, int64_t n_rows, int dim, int wave, int lane,
                                                uint32_t (&off)[kLoadsPerWave]) {
#pragma unroll
  for (int i = 0; i < kLoadsPerWave; ++i) {
    const int j = wave * kLoadsPerWave + i;
    const int byte = j * 1024 + lane * 16;
    const int r = byte / kRowB;
    const int c = ((byte % kRowB) >> 4) ^ swz(r);
    const int64_t left = n_rows - 1 - r0;
    const int rr = left < r ? (int)left : r;
    off[i] = (uint32_t)rr * (uint32_t)dim * 2u + (uint32_t)c * 16u;
  }
}

// Load l of a wave's share of a stage (l < kLoadsPerWave: audio, else visual).
__device__ __forceinline__ void issue_load(char* stage, const char* base_a, const char* base_b,
                                           const uint32_t (&off_a)[kLoadsPerWave],
                                           const uint32_t (&off_b)[kLoadsPerWave], int wave, int l) {
  const int i = l % kLoadsPerWave, j = wave * kLoadsPerWave + i;
  if (l < kLoadsPerWave)
    __builtin_amdgcn_global_load_lds((glb_ptr_t)(base_a + off_a[i]), (lds_ptr_t)(stage + j * 1024), 16, 0, 0);
  else
    __builtin_amdgcn_global_load_lds((glb_ptr_t)(base_b + off_b[i]), (lds_ptr_t)(stage + kOpB + j * 1024), 16, 0, 0);
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

// Inverse norms of audio rows m0 .. m0 + M - 1 (0 for a zero row, -inf past
// the clip's audio, so those rows never win).
template <int M>
__device__ __forceinline__ void inverse_norms(float* inv, const double* na, int64_t m0, int64_t n_a, int tid) {
  for (int r = tid; r < M; r += kWaves * 64) {
    float s = -INFINITY;
    if (m0 + r < n_a) {
      const double nn = na[m0 + r];
      s = nn > 0.0 ? (float)(1.0 / sqrt(nn)) : 0.0f;
    }
    inv[r] = s;
  }
}

// Largest scaled product of each of a wave's columns, merged into the keys:
// acc[i][j][e] of lane l is row 16 i + 4(l/16) + e of inv and column
// n0 + 16 j + l%16.
template <int BI, int BJ>
__device__ __forceinline__ void column_maxima(const f32x4 (&acc)[BI][BJ], const float* inv, int lane, int64_t n0,
                                              int64_t n_v, uint32_t* maxkey) {
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
    if (lane < 16 && col < n_v && m > -INFINITY) atomicMax(&maxkey[col], order_key(m));
  }
}

__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gate_gemm256(
    const ClipDev* __restrict__ clips, const GemmTileDev* __restrict__ tiles, int dim, const uint16_t* __restrict__ xv,
    const uint16_t* __restrict__ xa, const double* __restrict__ na, uint32_t* __restrict__ maxkey) {
  __shared__ __attribute__((aligned(16))) char lds[2 * kStageB];
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
  uint32_t off_a[kLoadsPerWave], off_b[kLoadsPerWave];
  operand_offsets(tl.m0, n_a, dim, wave, lane, off_a);
  operand_offsets(tl.n0, n_v, dim, wave, lane, off_b);
  const char* base_a = reinterpret_cast<const char*>(A + tl.m0 * dim);
  const char* base_b = reinterpret_cast<const char*>(B + tl.n0 * dim);
  auto issue = [&](int k_stage) {
#pragma unroll
    for (int l = 0; l < 2 * kLoadsPerWave; ++l)
      issue_load(lds + (k_stage & 1) * kStageB, base_a + (size_t)k_stage * kRowB, base_b + (size_t)k_stage * kRowB, off_a,
                 off_b, wave, l);
  };
  // Fragments of the slice in hand and of the next one; read r of a slice in
  // the order its MFMAs first need them: fa[0], fb[0 ..], fa[1 ..].
  bf16x8 fa[2][kBI], fb[2][kBJ];
  const int row_a = wm * kBI * 16 + (lane & 15), row_b = wn * kBJ * 16 + (lane & 15);
  auto read = [&](const char* stage, int ks, int r) {
    if (r >= 1 && r <= kBJ)
      fb[ks][r - 1] = lds_frag(stage + kOpB, row_b + 16 * (r - 1), ks, lane);
    else
      fa[ks][r == 0 ? 0 : r - kBJ] = lds_frag(stage, row_a + 16 * (r == 0 ? 0 : r - kBJ), ks, lane);
  };
  issue(0);
  if (n_k > 1) {
    issue(1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kLoadsPerWave) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int r = 0; r < kReads; ++r) read(lds, 0, r);
  __builtin_amdgcn_sched_barrier(0);
  // One stage, its two slices' MFMAs back to back.  Slice 0's run over the
  // reads of slice 1; then every wave waits for its loads of stage it + 1
  // (issued one stage ago) and its last reads of stage it, so that past the
  // barrier stage it + 1 is whole and this stage's buffer is free; slice 1's
  // MFMAs run over the first reads of stage it + 1 and the loads of stage
  // it + 2.  The scheduling barriers hold one fragment read behind every
  // second MFMA and one load behind every third: loads issued in a burst
  // stop the MFMAs behind them (spaced every MFMA 169 us on the 60 s clip,
  // second 162, third 158, fourth 158; every second one is 1% faster on the
  // 290 s clip, every fourth 4% slower).
  auto stage = [&](int it, auto load_tag, auto next_tag) {
    constexpr bool kLoad = decltype(load_tag)::value, kNext = decltype(next_tag)::value;
    char* cur = lds + (it & 1) * kStageB;
    const char* next = lds + ((it + 1) & 1) * kStageB;
    const char* next_a = uniform_ptr(base_a + (size_t)(it + 2) * kRowB);
    const char* next_b = uniform_ptr(base_b + (size_t)(it + 2) * kRowB);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if (ks == 1 && kNext) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int g = 0; g < kMfmas; ++g) {
        const int i = g / kBJ, j = g % kBJ;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
        if (g % 2 == 0 && g / 2 < kReads && (ks == 0 || kNext)) {
          read(ks == 0 ? cur : next, ks ^ 1, g / 2);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (ks == 1 && kLoad && g % 3 == 2 && g / 3 < 2 * kLoadsPerWave) {
          issue_load(cur, next_a, next_b, off_a, off_b, wave, g / 3);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int it = 0;
  for (; it + 2 < n_k; ++it) stage(it, std::true_type{}, std::true_type{});
  if (it + 1 < n_k) stage(it++, std::false_type{}, std::true_type{});
  stage(it, std::false_type{}, std::false_type{});

  // Epilogue.  Inverse audio norms of the tile's rows in LDS (-inf past the
  // clip's audio, so those rows never win); acc[i][j][e] of lane l is audio
  // row 16 (kBI wm + i) + 4(l/16) + e, visual column 16 (kBJ wn + j) + l%16.
  __syncthreads();
  float* inv = reinterpret_cast<float*>(lds);
  inverse_norms<kTile>(inv, na + c.aud_off, tl.m0, n_a, tid);
  __syncthreads();
  column_maxima(acc, inv + wm * kBI * 16, lane, tl.n0 + wn * kBJ * 16, n_v, maxkey + c.vis_off);
}

// ---------------------------------------------------------------------------
// The same product for fp32 inputs, and for bf16 inputs of any dim (a
// multiple of 8): tiles of 256 x 128, eight waves of 64 x 64, the operands
// staged through registers into two LDS buffers.
//
// fp32: each value is split into three bf16 parts, x = h + m + l exactly
// (each part the rounded remainder of the last: 8 + 8 + 8 significand bits),
// and x y is summed as l h + h l + m m + m h + h m + h h on the bf16 matrix
// cores, six MFMAs of 32 elements in fp32.  What is left out (m l, l m, l l)
// is below 2^-25 of the product, and a sum of K products is rounded 6 K / 32
// times where v_mfma_f32_32x32x2_f32 rounds it K / 2 times.  Error of the
// largest cosine against 64 bits, rms over random, one-signed and
// wide-ranging rows, this and that: dim 264 1.8-2.0e-7 and 2.4-2.9e-7, 2048
// 4.3-5.7e-7 and 6.5-7.5e-7, 3584 5.2-7.5e-7 and 8.1-9.6e-7, 16384 1.1-1.5e-6
// and 1.8-2.0e-6.  The fp32 MFMA peaks at 157 TFLOP/s; six bf16 ones leave
// room for twice that: 1500 x 17280 x 2048 takes 654 us against 1148, and
// 1500 x 17280 x 1288 in bf16 129 against 141 (128 x 128 tiles on 32x32x16
// MFMAs).
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
  __device__ __forceinline__ void parts(bool valid, uint4 (&out)[1]) const {
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
  static __device__ __forceinline__ uint32_t split(float x, float y, float& rx, float& ry) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const bf16x2 h = __builtin_convertvector(f32x2{x, y}, bf16x2);
    uint32_t w;
    __builtin_memcpy(&w, &h, 4);
    rx = x - __uint_as_float(w << 16);
    ry = y - __uint_as_float(w & 0xFFFF0000u);
    return w;
  }
  __device__ __forceinline__ void parts(bool valid, uint4 (&out)[3]) const {
    const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // The largest finite bf16 bounds the first part, so it never rounds to
      // infinity.
      constexpr float kTop = 3.3895313892515355e38f;
      float x = valid ? v[2 * i] : 0.0f, y = valid ? v[2 * i + 1] : 0.0f, rx, ry, t0, t1;
      w[0][i] = split(__builtin_amdgcn_fmed3f(x, -kTop, kTop), __builtin_amdgcn_fmed3f(y, -kTop, kTop), t0, t1);
      rx = x - __uint_as_float(w[0][i] << 16);
      ry = y - __uint_as_float(w[0][i] & 0xFFFF0000u);
      w[1][i] = split(rx, ry, t0, t1);
      w[2][i] = split(t0, t1, rx, ry);
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) out[p] = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
  }
};

template <class T>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gate_gemm_any(
    const ClipDev* __restrict__ clips, const GemmTileDev* __restrict__ tiles, int dim, const T* __restrict__ xv,
    const T* __restrict__ xa, const double* __restrict__ na, uint32_t* __restrict__ maxkey) {
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
#pragma unroll
  for (int i = 0; i < kUnits / KS; ++i) {
    const int r = (tid >> 2) + i * (kWaves * 16);
    row[i] = r < kAnyM ? xa + (c.aud_off + min(tl.m0 + (int64_t)r, n_a - 1)) * dim
                       : xv + (c.vis_off + min(tl.n0 + (int64_t)(r - kAnyM), n_v - 1)) * dim;
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
      raw[u].parts(k0 + 32 * ks + chunk * 8 < dim, part);
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

  f32x4 acc[kAnyB][kAnyB];
#pragma unroll
  for (int i = 0; i < kAnyB; ++i)
#pragma unroll
    for (int j = 0; j < kAnyB; ++j) acc[i][j] = f32x4{};
  const int n_k = (dim + kStep - 1) / kStep;
  const int row_a = wm * kAnyB * 16 + (lane & 15), row_b = kAnyM + wn * kAnyB * 16 + (lane & 15);
  auto products = [&](const bf16x8 (&fa)[kAnyB], const bf16x8 (&fb)[kAnyB]) {
#pragma unroll
    for (int i = 0; i < kAnyB; ++i)
#pragma unroll
      for (int j = 0; j < kAnyB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
  };
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
#pragma unroll
    for (int p = KS * NP - 1; p >= 0; --p)
#pragma unroll
      for (int i = 0; i < kAnyB; ++i) {
        fa[p][i] = frag(buf + p * kSubB, row_a + 16 * i);
        fb[p][i] = frag(buf + p * kSubB, row_b + 16 * i);
      }
    __builtin_amdgcn_sched_barrier(0);
    // The next step is split and stored under this step's products.
    lstore((it + 1) * kStep, lds + ((it + 1) & 1) * kBufB);
    gload((it + 2) * kStep);
    if constexpr (NP == 3) {
      products(fa[2], fb[0]);
      products(fa[0], fb[2]);
      products(fa[1], fb[1]);
      products(fa[1], fb[0]);
      products(fa[0], fb[1]);
      products(fa[0], fb[0]);
    } else {
#pragma unroll
      for (int p = 0; p < KS; ++p) products(fa[p], fb[p]);
    }
    if constexpr (NP == 3) {
#pragma unroll
      for (int g = 0; g < 6 * kAnyB * kAnyB; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);   // two VALU instructions
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // Epilogue, as above: acc[i][j][e] of lane l is audio row
  // 16 (kAnyB wm + i) + 4(l/16) + e, visual column 16 (kAnyB wn + j) + l%16.
  __syncthreads();
  float* inv = reinterpret_cast<float*>(lds);
  inverse_norms<kAnyM>(inv, na + c.aud_off, tl.m0, n_a, tid);
  __syncthreads();
  column_maxima(acc, inv + wm * kAnyB * 16, lane, tl.n0 + wn * kAnyB * 16, n_v, maxkey + c.vis_off);
}

}  // namespace

// One tile per workgroup, of tile_m audio rows by tile_n visual columns.
static std::vector<GemmTileDev> gate_gemm_tiles(const std::vector<ClipDev>& clips, int tile_m, int tile_n) {
  // A clip's row tiles are cut into bands of at most kBandRows (as even as
  // possible); per band, column blocks (clip, n0) are dealt to the XCDs in
  // turn, and an XCD's share lists the band's row tiles of its blocks, block
  // after block.  A tall clip's audio then passes through each XCD's L2 once
  // per band and column block rather than once per column block.
  constexpr int kBandRows = 8;
  std::vector<std::vector<GemmTileDev>> share(kXcds);
  int next = 0;
  for (size_t s = 0; s < clips.size(); ++s) {
    const ClipDev& c = clips[s];
    const int64_t nv = (int64_t)c.n_frames * c.per_frame;
    if (nv == 0 || c.n_audio == 0) continue;
    const int mb = (int)((c.n_audio + tile_m - 1) / tile_m), nb = (int)((nv + tile_n - 1) / tile_n);
    const int n_band = (mb + kBandRows - 1) / kBandRows;
    for (int b = 0; b < n_band; ++b) {
      const int m0 = b * mb / n_band, m1 = (b + 1) * mb / n_band;
      for (int n = 0; n < nb; ++n, next = (next + 1) % kXcds)
        for (int m = m0; m < m1; ++m) share[next].push_back({(int32_t)s, m * tile_m, n * tile_n, 0});
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
  return out;
}

std::vector<GemmTileDev> gate_gemm256_tiles(const std::vector<ClipDev>& clips) {
  return gate_gemm_tiles(clips, kTile, kTile);
}
std::vector<GemmTileDev> gate_gemm_any_tiles(const std::vector<ClipDev>& clips) {
  return gate_gemm_tiles(clips, kAnyM, kAnyN);
}

apack_status launch_gate_gemm256(const ClipDev* clips, const GemmTileDev* tiles, int64_t n_tiles, int dim,
                                 const uint16_t* xv, const uint16_t* xa, const double* na, uint32_t* maxkey,
                                 hipStream_t stream) {
  if (n_tiles == 0) return APACK_OK;
  hipLaunchKernelGGL(k_gate_gemm256, dim3((unsigned)n_tiles), dim3(kWaves * 64), 0, stream, clips, tiles, dim, xv, xa,
                     na, maxkey);
  return launch_status("k_gate_gemm256");
}

apack_status launch_gate_gemm_any(const ClipDev* clips, const GemmTileDev* tiles, int64_t n_tiles, int dim, bool bf16,
                                  const void* xv, const void* xa, const double* na, uint32_t* maxkey,
                                  hipStream_t stream) {
  if (n_tiles == 0) return APACK_OK;
  const dim3 grid((unsigned)n_tiles), block(kWaves * 64);
  if (bf16)
    hipLaunchKernelGGL(k_gate_gemm_any<uint16_t>, grid, block, 0, stream, clips, tiles, dim,
                       static_cast<const uint16_t*>(xv), static_cast<const uint16_t*>(xa), na, maxkey);
  else
    hipLaunchKernelGGL(k_gate_gemm_any<float>, grid, block, 0, stream, clips, tiles, dim, static_cast<const float*>(xv),
                       static_cast<const float*>(xa), na, maxkey);
  return launch_status("k_gate_gemm_any");
}

}  // namespace apack
