// The projection after attention, y = x W^T + b (paper Section 3.5 and Appendix A.4: the
// truncated V/O weights stay dense, so this is a plain bf16 GEMM of the attention output with
// the output weight), as hand-written MFMA kernels for gfx950.
//
// x bf16 [M, K], W bf16 [N, K] (the nn.Linear layout), bias bf16 [N] or none, y bf16 [M, N];
// float32 accumulation, the bias added in float32, one rounding to bf16 (nearest even).  Both
// kernels use v_mfma_f32_32x32x16_bf16 with W rows on the MFMA's M side and x rows on its N
// side, so each lane finishes with one row of y and runs of 4 consecutive columns (8-byte
// stores).  Both operands are k-contiguous in memory and in LDS: a 64-wide k step of a tile is
// rows of 128 bytes whose eight 16-byte chunks are XOR-swizzled by (row >> 1) & 7, so that the
// fragment reads (32 rows at one chunk) hit distinct banks.  Rows past M or N read the last row
// and are not stored.
//
// linear_kernel_pc (every K below 2^22): four waves multiply, four load straight into an LDS ring; four
// tile sizes, chosen by the cost rule of linear_plan.hpp.
//
// linear_kernel (longer rows, whose tiles 32-bit offsets cannot address, or outputs of which no other
// tile fits one launch): 4 waves, a 128 x 128 tile of y^T, two work-groups per compute unit, wave w
// owning a 64 x 64 quarter as 2 x 2 blocks.  The k steps are double buffered: the global loads of step s + 1 are in flight in registers while step
// s is multiplied, then written to the other LDS buffer before the step's one barrier.  Chunks
// past K read as zeros.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "linear_plan.hpp"

namespace unstep {
namespace {

constexpr int kThreads = 256;
constexpr int kBM = 128;                 // x rows (columns of y^T) per work-group
constexpr int kBN = 128;                 // W rows (columns of y) per work-group
constexpr int kBK = kLinearBK;           // k per step
constexpr int kRowBytes = kBK * 2;       // one tile row in LDS
constexpr int kTileBytes = kBN * kRowBytes;
constexpr int kChunks = kRowBytes / 16;  // 16-byte chunks per tile row
constexpr int kLoads = kTileBytes / 16 / kThreads;   // chunks per thread per operand per step
constexpr int kXcds = 8;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;

__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

struct LinearArgs {
  const uint16_t* x;
  const uint16_t* w;
  const uint16_t* bias;
  uint16_t* y;
  int32_t M, N, K;
  int32_t tiles_m, tiles_n;
};

// Global loads of one k step: thread t fetches chunks t + 256 j (j < kLoads) of the W tile and
// of the x tile (chunk c = row c / 8, 16-byte piece c % 8).  Returns zeros past K.
__device__ __forceinline__ void load_step(const LinearArgs& a, int32_t n0, int32_t m0, int32_t k0, int tid,
                                          u32x4_t (&wr)[kLoads], u32x4_t (&xr)[kLoads]) {
#pragma unroll
  for (int j = 0; j < kLoads; ++j) {
    const int c = tid + kThreads * j;
    const int row = c / kChunks, piece = c % kChunks;
    const int32_t k = k0 + piece * 8;
    const bool in_k = k < a.K;
    const int32_t nr = min(n0 + row, a.N - 1), mr = min(m0 + row, a.M - 1);
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    wr[j] = in_k ? *reinterpret_cast<const u32x4_t*>(a.w + int64_t(nr) * a.K + k) : zero;
    xr[j] = in_k ? *reinterpret_cast<const u32x4_t*>(a.x + int64_t(mr) * a.K + k) : zero;
  }
}

__device__ __forceinline__ void store_step(uint8_t* lw, uint8_t* lx, int tid, const u32x4_t (&wr)[kLoads],
                                           const u32x4_t (&xr)[kLoads]) {
#pragma unroll
  for (int j = 0; j < kLoads; ++j) {
    const int c = tid + kThreads * j;
    const int row = c / kChunks, piece = c % kChunks;
    const int off = row * kRowBytes + ((piece ^ swz(row)) * 16);
    *reinterpret_cast<lds_u32x4_t*>(reinterpret_cast<uintptr_t>(lw + off)) = wr[j];
    *reinterpret_cast<lds_u32x4_t*>(reinterpret_cast<uintptr_t>(lx + off)) = xr[j];
  }
}

__global__ __launch_bounds__(kThreads, 2) void linear_kernel(LinearArgs a) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[2][2][kTileBytes];   // [buffer][W, x]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave >> 1, wm = wave & 1;
  const int col = lane & 31, half = lane >> 5;

  // XCD-aware numbering: hardware work-group i runs on XCD i % 8; each XCD gets a contiguous
  // range of tiles, n fastest, so the work-groups of an XCD share x row blocks in its L2
  const int32_t G = gridDim.x;
  const int32_t xcd = blockIdx.x % kXcds;
  const int32_t g = xcd * (G / kXcds) + min(xcd, G % kXcds) + blockIdx.x / kXcds;
  const int32_t tn = g % a.tiles_n, tm = g / a.tiles_n;
  const int32_t n0 = tn * kBN, m0 = tm * kBM;

  // fragment read offsets within a tile: row wn*64 + nb*32 + col (W) or wm*64 + mb*32 + col (x),
  // chunk 2 kk + half; rows 32 apart share the swizzle, so nb / mb is an immediate offset
  int w_off[4], x_off[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int rw = wn * 64 + col, rx = wm * 64 + col;
    w_off[kk] = rw * kRowBytes + (((2 * kk + half) ^ swz(rw)) * 16);
    x_off[kk] = rx * kRowBytes + (((2 * kk + half) ^ swz(rx)) * 16);
  }

  f32x16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16_t{};

  const int32_t steps = (a.K + kBK - 1) / kBK;
  u32x4_t wr[kLoads], xr[kLoads];
  load_step(a, n0, m0, 0, tid, wr, xr);
  store_step(lds[0][0], lds[0][1], tid, wr, xr);
  __syncthreads();
  for (int32_t s = 0; s < steps; ++s) {
    const int buf = s & 1;
    if (s + 1 < steps) load_step(a, n0, m0, (s + 1) * kBK, tid, wr, xr);
    const uint8_t* lw = lds[buf][0];
    const uint8_t* lx = lds[buf][1];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8_t fw[2], fx[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        fw[b] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const lds_u32x4_t*>(
                                                 reinterpret_cast<uintptr_t>(lw + w_off[kk] + b * 32 * kRowBytes)));
        fx[b] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const lds_u32x4_t*>(
                                                 reinterpret_cast<uintptr_t>(lx + x_off[kk] + b * 32 * kRowBytes)));
      }
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
          acc[nb][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[nb], fx[mb], acc[nb][mb], 0, 0, 0);
    }
    // the other buffer was last read in step s - 1, which every wave finished before the
    // barrier that ended it; the barrier below publishes the new contents for step s + 1
    if (s + 1 < steps) store_step(lds[buf ^ 1][0], lds[buf ^ 1][1], tid, wr, xr);
    __syncthreads();
  }

  // epilogue: lane holds y[m][n .. n + 3] for m = m0 + wm*64 + mb*32 + col and the four runs
  // n = n0 + wn*64 + nb*32 + 8 g + 4 half, g = 0..3
  typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int mb = 0; mb < 2; ++mb) {
    const int32_t m = m0 + wm * 64 + mb * 32 + col;
    if (m >= a.M) continue;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int32_t n = n0 + wn * 64 + nb * 32 + 8 * gq + 4 * half;
        if (n >= a.N) continue;      // N is a multiple of 8: a run of 4 is all in or all out
        bf16x4_t r;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float v = acc[nb][mb][4 * gq + e];
          if (a.bias) v += __uint_as_float(uint32_t(a.bias[n + e]) << 16);
          r[e] = (__bf16)v;
        }
        *reinterpret_cast<bf16x4_t*>(a.y + int64_t(m) * a.N + n) = r;
      }
  }
}

// ---- direct-to-LDS staging: waves 0-3 multiply, waves 4-7 load ------------------------------------
//
// Multiplying wave w (one per SIMD) owns a quarter of the tile (n half w / 2, m half w % 2) as
// NB x MB blocks of 32 x 32.  The loading waves bring a stage, the 64-wide k step of both operands
// (W rows, then x rows, 128 bytes each), from global memory into the ring with
// global_load_lds_dwordx4: a load is 1 KB = 8 rows, lane l lands in row l / 8, physical chunk l % 8,
// so it fetches logical chunk (l % 8) ^ swz(row).  Issuing such a load stalls the issuing wave, so
// keeping the loads off the multiplying waves keeps their MFMA stream going.  When K is no multiple
// of 64 the last stage is read through a buffer descriptor and the chunks past K take an offset
// outside it, which reads as zero.
//
// What bounds it: the stream of operands into LDS.  One compute unit draws at most ~105 GB/s (about
// 46 bytes per clock) however few of them run, and all together ~12 TB/s with the two larger tiles,
// 15 with 64 x 128 and 19 with 64 x 64 (two work-groups per unit).  So a launch wants the largest
// tile that still gives every compute unit one, and a small launch wants small tiles: many units
// drawing at once, each with a deep ring (several stages in flight hide the ~1 us that a first
// touch takes).  Measured (us, against a 128 x 256 tile for K a multiple of 64 and linear_kernel
// otherwise): [1560, 1536] x [1536, 1536]^T 18.1 -> 13.3 (156 tiles of 128 x 128); [72, 1536] x
// [1536, 1536]^T 16.0 -> 6.7; [1365, 1032] x [1000, 1032]^T 26.7 -> 10.4; [64, 12288] x
// [1536, 12288]^T 102 -> 36.
//
// Two barrier placements.  Mid: the work-group's barrier of stage s comes before its last 16-wide k
// step; past it stage s + 1 has landed, so its first fragments are read during that k step and the
// MFMA stream does not wait for LDS at the stage's edge, but a slot is refilled one barrier later
// and the ring holds one stage less in flight.  Otherwise: the barrier follows the stage's last
// MFMAs.  With three 48 KB stages the deeper prefetch is worth more ([4680, 1536] x [1536, 1536]^T:
// 24.4 us against 26.4 with Mid); the smaller tiles have five or more stages and take Mid.
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) bf16x4_t lds_bf16x4_t;

constexpr int kPCThreads = 512;

// A kBN (W rows) x kBM (x rows) tile, a ring of kSt stages.
template <int kBN_, int kBM_, int kSt_, bool kMid_>
struct Tile {
  static constexpr int BN = kBN_, BM = kBM_, BK = kBK, St = kSt_;
  static constexpr bool Mid = kMid_;                       // barrier before a stage's last k step (else after it)
  static constexpr int Row = BK * 2;                       // bytes of a tile row
  static constexpr int Chunks = Row / 16;
  static constexpr int Stage = (BN + BM) * Row;            // W rows, then x rows
  static constexpr int RowsPerLoad = 1024 / Row;           // rows of one load instruction of a wave
  static constexpr int WLoads = BN / RowsPerLoad / 4;      // per loader wave and stage
  static constexpr int XLoads = BM / RowsPerLoad / 4;
  static constexpr int Loads = WLoads + XLoads;
  static constexpr int NB = BN / 64, MB = BM / 64;         // 32 x 32 blocks per multiplying wave
  static constexpr int KK = BK / 16;                       // MFMA k steps per stage
  static constexpr int YPitch = BN * 2 + 16;               // y staging rows
  static constexpr int Lds = St * Stage;
  static_assert(BM * YPitch <= Lds && Lds <= 160 * 1024, "LDS");
  static_assert((St - 2) * Loads <= 63, "vmcnt range: a prologue waits with St - 2 stages in flight");
};

// Workgroup barrier; at most kLeft of this wave's LDS reads are still in flight.
template <int kLeft>
__device__ __forceinline__ void big_barrier() {
  asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" ::"n"(kLeft) : "memory");
}

// Wait until at most n (0 .. kMax) stages of kL loads are in flight.
template <int kL, int kMax>
__device__ __forceinline__ void wait_stages(int n) {
  if constexpr (kMax > 0) {
    if (n < kMax) {
      wait_stages<kL, kMax - 1>(n);
      return;
    }
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kL * kMax) : "memory");
}

// A loader wave's view of its share of a stage.
template <class T>
struct Loader {
  const uint16_t* w;           // first tile row of W and of x, at k of the next stage
  const uint16_t* x;
  uint32_t wbytes, xbytes;     // from there to the end of the tile's last row
  uint32_t off[T::Loads];      // the lane's byte offset, per load; rows past the matrix read its last row
  int32_t kc[T::Loads];        // k of the lane's chunk within the stage
  uint32_t ldsw, ldsx;         // LDS address of this wave's first W and x row in stage 0
};

// The next stage into ring slot `slot`.  The loads' scalar bases must come from the scalar unit: an
// SGPR written by a VALU instruction would need 5 wait states before a vector-memory read of it,
// which the compiler does not insert ahead of inline assembly.  (An M0 write needs one.)
template <class T>
__device__ __forceinline__ void load_stage(Loader<T>& l, int slot, int32_t k0, int32_t K) {
  const uint32_t dw = l.ldsw + slot * T::Stage, dx = l.ldsx + slot * T::Stage;
  if (k0 + T::BK <= K) {
#pragma unroll
    for (int j = 0; j < T::Loads; ++j) {
      const uint32_t m0 = j < T::WLoads ? dw + j * 1024 : dx + (j - T::WLoads) * 1024;
      asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(l.off[j]), "s"(j < T::WLoads ? l.w : l.x), "{m0}"(m0) : "memory");
    }
  } else {
    // the last stage when K is no multiple of BK: chunks past K take an offset outside the buffer,
    // which reads as zero
#pragma unroll
    for (int j = 0; j < T::Loads; ++j) {
      const bool is_w = j < T::WLoads;
      const uint64_t base = uint64_t(uintptr_t(is_w ? l.w : l.x));
      const u32x4_t rsrc = {uint32_t(base), uint32_t(base >> 32), is_w ? l.wbytes : l.xbytes, 0x00020000u};
      const uint32_t m0 = is_w ? dw + j * 1024 : dx + (j - T::WLoads) * 1024;
      const uint32_t off = k0 + l.kc[j] < K ? l.off[j] : 0x80000000u;
      asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(off), "s"(rsrc), "{m0}"(m0) : "memory");
    }
  }
  l.w += T::BK;
  l.x += T::BK;
  l.wbytes -= T::Row;
  l.xbytes -= T::Row;
}

template <class T>
__device__ __forceinline__ void load_loop(const LinearArgs& a, uint32_t lds0, int lw, int lane, int32_t n0, int32_t m0, int32_t steps) {
  const int32_t wrows = min(a.N - n0, T::BN), xrows = min(a.M - m0, T::BM);
  Loader<T> l;
  l.w = a.w + int64_t(n0) * a.K;
  l.x = a.x + int64_t(m0) * a.K;
  l.wbytes = uint32_t(wrows) * uint32_t(a.K) * 2u;
  l.xbytes = uint32_t(xrows) * uint32_t(a.K) * 2u;
#pragma unroll
  for (int j = 0; j < T::Loads; ++j) {
    const bool is_w = j < T::WLoads;
    const int row = (is_w ? lw * T::WLoads + j : lw * T::XLoads + j - T::WLoads) * T::RowsPerLoad + lane / T::Chunks;
    const int chunk = (lane % T::Chunks) ^ swz(row);
    l.off[j] = uint32_t(min(row, (is_w ? wrows : xrows) - 1)) * uint32_t(a.K) * 2u + uint32_t(chunk) * 16u;
    l.kc[j] = chunk * 8;
  }
  l.ldsw = lds0 + lw * T::WLoads * 1024;
  l.ldsx = lds0 + T::BN * T::Row + lw * T::XLoads * 1024;
#pragma unroll
  for (int t = 0; t < T::St - 1; ++t)
    if (t < steps) load_stage<T>(l, t, t * T::BK, a.K);
  wait_stages<T::Loads, T::St - 2>(min(T::St - 1, steps) - 1);
  big_barrier<0>();                            // stage 0 has landed
  int slot = T::St - 1;
  for (int32_t s = 0; s < steps; ++s) {
    if (T::Mid) {
      if (s + 1 < steps) wait_stages<T::Loads, T::St - 3>(min(s + T::St - 2, steps - 1) - (s + 1));
      big_barrier<0>();                        // stage s + 1 has landed, stage s - 1 has been read
    }
    if (s + T::St - 1 < steps) load_stage<T>(l, slot, (s + T::St - 1) * T::BK, a.K);
    if (!T::Mid) {
      if (s + 1 < steps) wait_stages<T::Loads, T::St - 2>(min(s + T::St - 1, steps - 1) - (s + 1));
      big_barrier<0>();                        // stage s + 1 has landed, stage s has been read
    }
    slot = slot + 1 == T::St ? 0 : slot + 1;
  }
}

template <class T>
__device__ __forceinline__ void multiply(const LinearArgs& a, uint32_t lds0, int lw, int lane, int32_t n0, int32_t m0, int32_t steps) {
  constexpr int NB = T::NB, MB = T::MB, KK = T::KK, F = NB + MB;
  const int wn = lw >> 1, wm = lw & 1;
  const int col = lane & 31, half = lane >> 5;

  // this lane's bias values, loaded before the loop so that their latency is hidden (N is a
  // multiple of 8: a run of 4 is all in or all out)
  u32x2_t bq[NB][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const int32_t n = n0 + wn * 32 * NB + nb * 32 + 8 * gq + 4 * half;
      bq[nb][gq] = (a.bias && n < a.N) ? *reinterpret_cast<const u32x2_t*>(a.bias + n) : u32x2_t{0u, 0u};
    }

  uint32_t w_off[KK], x_off[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int rw = wn * 32 * NB + col, rx = wm * 32 * MB + col;
    w_off[kk] = lds0 + rw * T::Row + (((2 * kk + half) ^ swz(rw)) * 16);
    x_off[kk] = lds0 + T::BN * T::Row + rx * T::Row + (((2 * kk + half) ^ swz(rx)) * 16);
  }
  auto frag = [&](uint32_t cur, int kk, int i) {
    const uint32_t addr = i < NB ? w_off[kk] + cur + i * 32 * T::Row : x_off[kk] + cur + (i - NB) * 32 * T::Row;
    return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const lds_u32x4_t*>(uintptr_t(addr)));
  };

  f32x16_t acc[NB][MB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[i][j] = f32x16_t{};

  bf16x8_t fr[2][F];
  big_barrier<0>();                            // stage 0 has landed
  if (T::Mid)
#pragma unroll
    for (int i = 0; i < F; ++i) fr[0][i] = frag(0, 0, i);
  uint32_t cur = 0;
  for (int32_t s = 0; s < steps; ++s) {
    const uint32_t nxt = cur + T::Stage == uint32_t(T::Lds) ? 0u : cur + T::Stage;
    if (!T::Mid) {
#pragma unroll
      for (int i = 0; i < F; ++i) fr[0][i] = frag(cur, 0, i);
      __builtin_amdgcn_sched_group_barrier(0x100, F, 0);
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      // before the last k step: stage s + 1 has landed (its first fragments are read below), and
      // every fragment of stage s - 1 has been read
      if (T::Mid && kk == KK - 1) {
        __builtin_amdgcn_sched_barrier(0);
        big_barrier<F>();
      }
#pragma unroll
      for (int i = 0; i < NB * MB; ++i) {
        const int nb = i / MB, mb = i % MB;
        acc[nb][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[kk & 1][nb], fr[kk & 1][NB + mb], acc[nb][mb], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        constexpr int per = (F + NB * MB - 1) / (NB * MB);
#pragma unroll
        for (int r = 0; r < per; ++r)
          if (i * per + r < F && (T::Mid || kk + 1 < KK)) {
            fr[(kk + 1) & 1][i * per + r] = kk + 1 < KK ? frag(cur, kk + 1, i * per + r) : frag(nxt, 0, i * per + r);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
      }
    }
    cur = nxt;
    if (!T::Mid) big_barrier<0>();
  }
  if (T::Mid) big_barrier<0>();                // every wave has read the ring

  // lane holds y[m][n .. n + 3] for tile row wm*32*MB + mb*32 + col and tile columns
  // wn*32*NB + nb*32 + 8 gq + 4 half; rows past M or N are not stored
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int r = wm * 32 * MB + mb * 32 + col;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int cn = wn * 32 * NB + nb * 32 + 8 * gq + 4 * half;
        bf16x4_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t b2 = bq[nb][gq][e >> 1];
          const float bias = __uint_as_float((e & 1) ? (b2 & 0xffff0000u) : (b2 << 16));
          v[e] = (__bf16)(acc[nb][mb][4 * gq + e] + bias);
        }
        *reinterpret_cast<lds_bf16x4_t*>(uintptr_t(lds0 + uint32_t(r * T::YPitch + cn * 2))) = v;
      }
  }
}

template <class T>
__global__ __launch_bounds__(kPCThreads, 1) void linear_kernel_pc(LinearArgs a) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[T::Lds];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // XCD-aware numbering: as in linear_kernel
  const int32_t G = gridDim.x;
  const int32_t xcd = blockIdx.x % kXcds;
  const int32_t g = xcd * (G / kXcds) + min(xcd, G % kXcds) + blockIdx.x / kXcds;
  const int32_t tn = g % a.tiles_n, tm = g / a.tiles_n;
  const int32_t n0 = tn * T::BN, m0 = tm * T::BM;
  const uint32_t lds0 = uint32_t(uintptr_t((__attribute__((address_space(3))) void*)lds));
  const int32_t steps = (a.K + T::BK - 1) / T::BK;
  if (wave >= 4) {
    load_loop<T>(a, lds0, wave - 4, lane, n0, m0, steps);
    if (T::Mid) big_barrier<0>();
  } else {
    multiply<T>(a, lds0, wave, lane, n0, m0, steps);
  }
  big_barrier<0>();                            // the y tile is in LDS (the ring is free)

  // all 8 waves store the tile in 16-byte pieces that cover whole row runs
  constexpr int kPieces = T::BN / 8, kRows = kPCThreads / kPieces;
  const int c = tid % kPieces;
  const int32_t n = n0 + 8 * c;
#pragma unroll
  for (int i = 0; i < T::BM / kRows; ++i) {
    const int r = tid / kPieces + kRows * i;
    const int32_t m = m0 + r;
    const u32x4_t v = *reinterpret_cast<const lds_u32x4_t*>(uintptr_t(lds0 + uint32_t(r * T::YPitch + c * 16)));
    if (m < a.M && n < a.N) *reinterpret_cast<u32x4_t*>(a.y + int64_t(m) * a.N + n) = v;
  }
}

template <class T>
hipError_t launch_pc(const LinearArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(linear_kernel_pc<T>, dim3(unsigned(int64_t(a.tiles_m) * a.tiles_n)), dim3(kPCThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_linear(const uint16_t* x, const uint16_t* w, const uint16_t* bias, uint16_t* y, int32_t M,
                         int32_t N, int32_t K, hipStream_t stream) {
  const LinearTile t = linear_plan(M, N, K);
  const LinearArgs a{x, w, bias, y, M, N, K, t.tiles_m, t.tiles_n};
  if (!t.fits) return hipErrorInvalidConfiguration;
  if (!t.staged) {
    if (t.bm == 256) return launch_pc<Tile<128, 256, 3, false>>(a, stream);
    if (t.bn == 128) return launch_pc<Tile<128, 128, 5, true>>(a, stream);
    if (t.bm == 128) return launch_pc<Tile<64, 128, 6, true>>(a, stream);
    return launch_pc<Tile<64, 64, 5, true>>(a, stream);
  }
  const int64_t tiles = int64_t(t.tiles_m) * t.tiles_n;
  hipLaunchKernelGGL(linear_kernel, dim3(unsigned(tiles)), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace unstep
