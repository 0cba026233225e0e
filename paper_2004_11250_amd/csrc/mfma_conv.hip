// mfma_conv.hip -- a pruned 3x3 layer in bf16 on the bf16 matrix cores.
//
// Regrouping filters by pattern to feed the matrix cores (one dense
// contraction per (filter group, pattern) over the channels where some filter
// of the group uses the pattern) does not shrink the work when patterns are
// assigned independently per kernel: a channel lands in most groups' sets, so
// the contraction over all (tap, channel) pairs -- the layer's masked dense
// conv, A[o][(t, c)] = w[o][c][t] where tap t is in kernel (o, c)'s pattern
// and the kernel is kept, else 0 -- is the tightest matrix-core form.  It does
// 9 c_in c_out MACs per pixel instead of the surviving ones (about 4.5x more
// at half the kernels kept), on units with 16x the vector rate in bf16
// (2.5 PFLOP/s dense against 157 TFLOP/s), so it wins for most bf16 layers of
// 32 channels and more (512 -> 512 at 28 x 28 26 us against 30 on the lean
// kernel, at 14 x 14 21 against 17) and loses on the smallest maps, where its
// long reduction over a few tiles leaves the chip idle; the planner picks per
// layer.
//
// Each call expands the blob into A in the caller's scratch
// (pp_mfma_expand_kernel: original filter order, in the matrix cores' operand
// order, and the bias in original order) and runs an implicit GEMM
// C[o][pixel] = sum_k A[o][k] B[k][pixel], with B read from the staged input
// (never stored).  Products of bf16 values are exact in fp32; sums are fp32;
// the epilogue (bias, ReLU, accumulate, PixelShuffle(2), 2 x 2 max pool)
// rounds once to bf16, as the vector kernels do.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "conv_pp_kernel.hpp"

namespace pp {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct MTiles {
  uint32_t m_tiles, tiles_x, tiles_y;
};

constexpr uint32_t kOut = 0x80000000u;   // byte offset of an element outside a tensor (reads zero)

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// lo and hi in bf16, rounded to nearest even
__device__ __forceinline__ uint32_t cvt_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}
__device__ __forceinline__ float bf16_val(uint32_t u) { return __uint_as_float(u << 16); }   // of the low half
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

// One thread per (slot group g, slot s, input channel c), channel fastest:
// the 9 taps of kernel (perm[8 g + s], c) into A (zeros for taps off
// the pattern and for pruned kernels), and the slot's bias into bo[o].  Every
// (filter, channel) pair is written exactly once.  Offsets read from the
// device blob are clamped (a pattern id past the library reads as pruned, a
// weight index past n_wt as zero).
__global__ __launch_bounds__(256) void pp_mfma_expand_kernel(ConvParams a, uint16_t* __restrict__ am,
                                                             float* __restrict__ bo) {
  const long gid = static_cast<long>(blockIdx.x) * 256 + threadIdx.x;
  if (gid >= static_cast<long>(a.n_groups) * 8 * a.c_in) return;
  const int c = static_cast<int>(gid % a.c_in);
  const long gs = gid / a.c_in;   // 8 g + s
  const int s = static_cast<int>(gs & 7);
  const uint32_t o = reinterpret_cast<const uint32_t*>(a.blob + a.off_perm)[gs];
  if (o >= static_cast<uint32_t>(a.c_out)) return;   // padding slot
  const size_t gc = static_cast<size_t>(gs >> 3) * a.c_in + c;
  const uint8_t* code = a.blob + a.off_codes + gc * 8;
  const uint16_t* masks = reinterpret_cast<const uint16_t*>(a.blob + a.off_masks);
  const uint32_t wo = reinterpret_cast<const uint32_t*>(a.blob + a.off_woff)[gc];
  const uint32_t kept = wo >> 24;
  auto mask_of = [&](int q) -> uint32_t {
    const uint32_t id = code[q];
    return ((kept >> q) & 1u) && id < static_cast<uint32_t>(a.n_patterns) ? masks[id] & 0x1FFu : 0u;
  };
  // the slot's first weight: after the kept slots before it (bf16 kernels
  // are padded to an even element count)
  uint32_t idx = wo & 0xFFFFFFu;
  for (int q = 0; q < s; ++q) idx += (static_cast<uint32_t>(__builtin_popcount(mask_of(q))) + 1u) & ~1u;
  const uint32_t m = mask_of(s);
  const uint16_t* w = reinterpret_cast<const uint16_t*>(a.blob + a.off_w);
  // operand order (see pp_mfma_conv_kernel): blocks of 32 filters, each [16 channels][tap][half][row][8 channels]
  const uint32_t mb = o >> 5, rows = min(32u, static_cast<uint32_t>(a.c_out) - 32u * mb);
  uint16_t* dst = am + static_cast<size_t>(mb) * 32 * 9 * a.c_in +
                  ((static_cast<size_t>(c >> 4) * 18 + ((c >> 3) & 1)) * rows + (o & 31)) * 8 + (c & 7);
  for (int t = 0; t < 9; ++t) {
    uint16_t v = 0;
    if ((m >> t) & 1u) {
      v = idx < a.n_wt ? w[idx] : static_cast<uint16_t>(0);
      if (v == 0) v = 0x8000u;   // a stored zero: +0 is left for taps that are not there
      ++idx;
    }
    dst[static_cast<size_t>(t) * 16 * rows] = v;
  }
  if (c == 0) bo[o] = reinterpret_cast<const float*>(a.blob + a.off_bias)[gs];
}

// Pairs of bf16 for the NaN repair (see pp_mfma_conv_kernel): per half, 1 for
// a non-finite value (huge) or for a weight that is there (bits other than
// +0), the sign of an infinity (of any weight but zero and NaN), and the
// value with 1 of its sign in the place of an infinity or NaN.
template <class F>
__device__ __forceinline__ uint32_t halves(uint32_t u, F f) {
  return f(u & 0xFFFFu) | f(u >> 16) << 16;
}
__device__ __forceinline__ uint32_t one_of_sign(uint32_t h) { return (h & 0x8000u) | 0x3F80u; }
__device__ __forceinline__ bool is_huge(uint32_t h) { return (h & 0x7F80u) == 0x7F80u; }
__device__ __forceinline__ uint32_t count_huge(uint32_t u) {
  return halves(u, [](uint32_t h) { return is_huge(h) ? 0x3F80u : 0u; });
}
__device__ __forceinline__ uint32_t sign_inf(uint32_t u) {
  return halves(u, [](uint32_t h) { return (h & 0x7FFFu) == 0x7F80u ? one_of_sign(h) : 0u; });
}
__device__ __forceinline__ uint32_t without_huge(uint32_t u) {
  return halves(u, [](uint32_t h) { return is_huge(h) ? one_of_sign(h) : h; });
}
__device__ __forceinline__ uint32_t count_kept(uint32_t u) {
  return halves(u, [](uint32_t h) { return h ? 0x3F80u : 0u; });
}
__device__ __forceinline__ uint32_t sign_weight(uint32_t u) {
  return halves(u, [](uint32_t h) { return (h & 0x7FFFu) - 1u < 0x7F80u ? one_of_sign(h) : 0u; });
}

// lgkmcnt(0), then the workgroup barrier: LDS traffic is complete, global
// loads stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Tile geometry.  A workgroup is 4 waves, WM along the filters and 4 / WM
// along the pixels; a wave owns MB blocks of 32 filters by TN blocks of 32
// pixels.  The pixel tile is TH x TW outputs of one image; its input halo
// (HR x HC) is staged CB channels at a time as [pixel][channel], PITCH bytes
// a pixel (16 more than the channels need: neighbouring pixels' 16-byte
// pieces then fall on different banks).
template <int WM, int MB, int TN, int CB, int TW_, int S, int D>
struct MGeo {
  static constexpr int WN = 4 / WM, BM = 32 * MB * WM, NBLK = WN * TN, BN = 32 * NBLK;
  static constexpr int TW = TW_, TH = BN / TW, RPB = 32 / TW;   // rows of a 32-pixel block
  static constexpr int HR = (TH - 1) * S + 2 * D + 1;
  static constexpr int HC = ((TW - 1) * S + 2 * D + 1 + 1 + 1) / 2 * 2;   // from an even column: one more, even
  static constexpr int PITCH = 2 * CB + 16;
  static constexpr int BUF = HR * HC * PITCH;                  // bytes of one staged block
  static constexpr int LDS = 2 * BUF;
};

// What bounds it and why this form: the contraction needs 9 c_in k per
// output, and gathering B per tap from NCHW (2-byte loads, one per element
// and tap) was bound by the load instructions.  Here a channel block's halo
// is read from memory once, transposed in registers (8 channels of a pixel
// pair: eight 4-byte loads, eight byte permutes, two 16-byte LDS writes) and
// read by all nine taps as shifted 16-byte LDS reads.  The weights never
// touch LDS: every wave reads its own filters', so a k-step costs a unit's
// cache 4 MB KB.  The 64 x 128 tile therefore takes one block of filters by
// two of pixels per wave (with two by one, all four waves read the same
// filters: bound by that cache, also with four
// times the waves; 512 -> 512 at 14 x 14 28.7 -> 22.3, 256 -> 256 at 56 x 56
// 17.4 -> 14.0, 64 -> 64 at 224 x 224 12.6 -> 9.9, 512 -> 512 stride 2 at 32 x
// 32 41.8 -> 36.4), its pixel operands read two k-steps ahead (3 % of those).
// They lie in memory in operand order (one contiguous KB per 32
// filters x 16 k), so each operand is one coalesced 16-byte load per lane,
// issued PF k-steps ahead; k runs channel block by channel block of 16, tap
// by tap inside.  Measured (bf16, us, per-tap gather -> this): 64 -> 64 at
// 270 x 480 37 -> 19, 64 -> 256 at 540 x 960 with the shuffle 317 -> 170,
// 512 -> 512 on 8 x 32 x 32 62 -> 39 (dilation 2 83 -> 37): 35-40 % of the
// 2.5 PFLOP/s peak on the large ones, 0.8-1.0 of what a large library
// matrix product reaches on the card (1.15).  What is left is the weights'
// way through each unit's cache (a tile half as large takes 1.4x), and on
// small grids the wait for each channel block's input.
// PX2: the halo is staged by pixel pairs (even image width, no upsample),
// else pixel by pixel; with PP_UPSAMPLE2 the conv's input is the nearest x2
// upsampling of x.
template <int WM, int MB, int TN, int CB, int TW_, int S, int D, bool PX2>
__global__ __launch_bounds__(256, 2) void pp_mfma_conv_kernel(ConvParams a, const uint16_t* __restrict__ am,
                                                               const float* __restrict__ bias, MTiles mt) {
  using M = MGeo<WM, MB, TN, CB, TW_, S, D>;
  constexpr int KS = CB / 16 * 9;        // k-steps (16 deep) of a channel block
  constexpr int PF = TN < 4 && KS % 6 == 0 ? 6 : 3;   // weights in flight ahead, in k-steps (divides KS)
  constexpr int BD = MB == 1 ? 2 : 1;    // pixel operands read ahead, in k-steps
  constexpr int PW = PX2 ? 2 : 1;        // pixels per staged item
  constexpr int NPC = M::HC / PW;        // items across
  constexpr int ITEMS = NPC * M::HR * (CB / 8);
  constexpr int NIT = (ITEMS + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint8_t smem[M::LDS];
  __shared__ float bias_s[M::BM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wv % WM, wn = wv / WM;

  // block -> (image, tile, filter tile): filter tiles of one pixel tile are neighbours on one XCD
  uint32_t blk = kern::xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t mtile = blk % mt.m_tiles;
  blk /= mt.m_tiles;
  const uint32_t txi = blk % mt.tiles_x;
  blk /= mt.tiles_x;
  const uint32_t tyi = blk % mt.tiles_y;
  const uint32_t img = blk / mt.tiles_y;
  const int oy0 = tyi * M::TH, ox0 = txi * M::TW;
  const int iy0 = oy0 * S - a.pad, ixw = ox0 * S - a.pad;
  const int ix0 = ixw & ~1, sh = ixw & 1;   // the staged columns start at an even one

  for (int i = tid; i < M::BM; i += 256) {
    const int o = mtile * M::BM + i;
    bias_s[i] = o < a.c_out ? bias[o] : 0.0f;
  }

  // input: per-item byte offsets within a channel block (kOut: outside the image)
  const bool up = !PX2 && (a.flags & PP_UPSAMPLE2) != 0;
  const int hs = up ? a.h / 2 : a.h, wsd = up ? a.w / 2 : a.w;   // stored input size
  const uint32_t hw = static_cast<uint32_t>(hs) * wsd;
  const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.x), static_cast<short>(0), static_cast<int>(static_cast<uint32_t>(a.n) * a.c_in * hw * 2),
      0x00020000);
  uint32_t xoff[NIT], loff[NIT];
#pragma unroll
  for (int t = 0; t < NIT; ++t) {
    const int e = tid + 256 * t;
    const int pc = e % NPC, q = e / NPC, hr = q % M::HR, oct = q / M::HR;
    const int gy = iy0 + hr, gx = ix0 + PW * pc;
    const bool ok = e < ITEMS && gy >= 0 && gy < a.h && gx >= 0 && gx < a.w;
    const uint32_t el = up ? static_cast<uint32_t>(gy >> 1) * wsd + (gx >> 1) : static_cast<uint32_t>(gy) * wsd + gx;
    xoff[t] = ok ? (static_cast<uint32_t>(img) * a.c_in * hw + 8u * oct * hw + el) * 2u : kOut;
    // items past the tile's last write over its first pixels' padding bytes (nobody reads those)
    loff[t] = e < ITEMS ? (hr * M::HC + PW * pc) * M::PITCH + 16 * oct : 2 * CB;
  }
  uint32_t rb[NIT][8];
  auto fetch = [&](int cb) __attribute__((always_inline)) {
    const uint32_t c2 = static_cast<uint32_t>(cb) * CB * hw * 2u;
#pragma unroll
    for (int t = 0; t < NIT; ++t)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if constexpr (PX2)
          rb[t][j] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, xoff[t], static_cast<int>(c2 + j * hw * 2u), 0);
        else
          rb[t][j] = __builtin_amdgcn_raw_buffer_load_b16(xrsrc, xoff[t], static_cast<int>(c2 + j * hw * 2u), 0);
      }
  };
  auto put = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NIT; ++t) {
      uint8_t* d = smem + buf * M::BUF + loff[t];
      uint32_t lo[4], hi[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        lo[k] = __builtin_amdgcn_perm(rb[t][2 * k + 1], rb[t][2 * k], 0x05040100u);
        hi[k] = __builtin_amdgcn_perm(rb[t][2 * k + 1], rb[t][2 * k], 0x07060302u);
      }
      *reinterpret_cast<uint4*>(d) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
      if constexpr (PX2) {
        if ((t + 1) * 256 <= ITEMS || tid + 256 * t < ITEMS)
          *reinterpret_cast<uint4*>(d + M::PITCH) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
      }
    }
  };

  // weights: block of 32 filters mb holds, per k-step, [half][row][8 k] of its
  // R = min(32, c_out - 32 mb) rows; a row past them reads zero
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(am), static_cast<short>(0), a.c_out * 9 * a.c_in * 2, 0x00020000);
  uint32_t aoff[MB], astep[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int mb = mtile * (M::BM / 32) + wm * MB + i;
    const int rows = min(32, a.c_out - 32 * mb);
    const int row = lane & 31;
    aoff[i] = row < rows ? static_cast<uint32_t>(mb) * 32u * 18u * a.c_in + ((lane >> 5) * rows + row) * 16u : kOut;
    astep[i] = rows > 0 ? 32u * rows : 0u;
  }
  const int nblk = a.c_in / CB;
  const uint32_t last_step = static_cast<uint32_t>(nblk) * KS - 1;
  typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
  u32x4v ar[PF][MB];
  auto load_a = [&](int slot, uint32_t step) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
      ar[slot][i] = __builtin_bit_cast(
          u32x4v, __builtin_amdgcn_raw_buffer_load_b128(arsrc, aoff[i], static_cast<int>(step * astep[i]), 0));
  };

  // pixel operands: this lane's pixel of the wave's first block, tap (0, 0)
  const int lp = lane & 31;
  const int prow = wn * TN * M::RPB + lp / M::TW, pcol = lp % M::TW;
  const uint32_t lbase = (prow * S * M::HC + pcol * S + sh) * M::PITCH + (lane >> 5) * 16;

  f32x16 acc[MB][TN];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x16{};

  fetch(0);
#pragma unroll
  for (int s = 0; s < PF; ++s) load_a(s, s);
  put(0);
  lds_barrier();
#pragma unroll 1
  for (int cb = 0; cb < nblk; ++cb) {
    const bool more = cb + 1 < nblk;
    {
      const uint8_t* bsrc = smem + (cb & 1) * M::BUF + lbase;
      auto read_b = [&](int s, bf16x8 (&bv)[TN]) __attribute__((always_inline)) {
        const int h = s / 9, t = s % 9, ky = t / 3, kx = t % 3;
#pragma unroll
        for (int j = 0; j < TN; ++j)
          bv[j] = *reinterpret_cast<const bf16x8*>(bsrc + ((ky * D + j * M::RPB * S) * M::HC + kx * D) * M::PITCH + h * 32);
      };
      bf16x8 bv[BD + 1][TN];
#pragma unroll
      for (int s = 0; s < BD; ++s) read_b(s, bv[s]);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        // (loads return in order: issued any earlier, the next block's input would hold up the weights behind it)
        if (s == KS - PF && more) fetch(cb + 1);
        if (s + BD < KS) read_b(s + BD, bv[(s + BD) % (BD + 1)]);
        bf16x8 av[MB];
#pragma unroll
        for (int i = 0; i < MB; ++i) av[i] = __builtin_bit_cast(bf16x8, ar[s % PF][i]);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[s % (BD + 1)][j], acc[i][j], 0, 0, 0);
        // the ring's next k-step (past the last one that one again: nothing outside the weights is read)
        const int ns = s + PF;
        load_a(s % PF, min(static_cast<uint32_t>(cb * KS + ns), last_step));
        // (left to itself the scheduler sinks the weight loads to their use, a step's wait each)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (more) put((cb & 1) ^ 1);   // that buffer's last readers passed the previous barrier
    lds_barrier();
  }

  // where the lane's accumulators lie, worked out anew (held over the loop they would cost it registers)
  const int ln = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int brow = wn * TN * M::RPB + (ln & 31) / M::TW, bcol = (ln & 31) % M::TW;

  // A pruned tap's zero weight times an infinity of the input is NaN, where the
  // vector kernels never read that tap.  Outputs that came out NaN (found by one
  // FMA per accumulator pair: NaN stays, a false alarm only costs the look; 0.5 %
  // of a 128 x 256 tile) are contracted again, a wave's 32 x 32 block at a time
  // with its operands straight from memory: first how many products of taps that
  // are there are infinite or NaN, and the signs of the infinite ones; then, where
  // that leaves it open, the sum with those inputs out of it.  A last channel of
  // NaN, us against the call without it: 512 -> 512 at 28 x 28 259 (27), 64 -> 256
  // at 540 x 960 1984 (198), 64 -> 64 at 270 x 480 143 (17): about ten times,
  // whatever the input (the loads' latency), and nothing held over the loop above.
  float probe = 0.0f;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; r += 2) probe = __builtin_fmaf(acc[i][j][r], acc[i][j][r + 1], probe);
  if (__builtin_expect(__any(probe != probe), 0)) {
#pragma unroll 1
    for (int b = 0; b < MB * TN; ++b) {
      uint32_t bad = 0;   // bit r: accumulator r of block b is NaN
#pragma unroll
      for (int k = 0; k < MB * TN; ++k)
        if (b == k) {
#pragma unroll
          for (int r = 0; r < 16; ++r) bad |= acc[k / TN][k % TN][r] != acc[k / TN][k % TN][r] ? 1u << r : 0u;
        }
      const int oy = oy0 + brow + b % TN * M::RPB, ox = ox0 + bcol;
      if (!__any(bad)) continue;
      const int mb = mtile * (M::BM / 32) + wm * MB + b / TN;
      const int rows = min(32, a.c_out - 32 * mb);
      const uint32_t ao = (ln & 31) < rows
                              ? static_cast<uint32_t>(mb) * 32u * 18u * a.c_in + ((ln >> 5) * rows + (ln & 31)) * 16u
                              : kOut;
      const uint32_t as = rows > 0 ? 32u * rows : 0u;
      // op(weights, inputs) for every 16-deep k-step of the block, the loads of as
      // many channel blocks at a time as the registers hold beside acc, and where
      // they hold all three sums in one walk
      constexpr int RU = CB == 64 ? 4 : 2;
      constexpr bool kOnce = CB == 64;
      auto steps = [&](auto op) __attribute__((always_inline)) {
#pragma unroll 1
        for (int t = 0; t < 9; ++t) {
          const int gy = oy * S - a.pad + t / 3 * D, gx = ox * S - a.pad + t % 3 * D;
          const bool ok = gy >= 0 && gy < a.h && gx >= 0 && gx < a.w;
          const uint32_t el = up ? static_cast<uint32_t>(gy >> 1) * wsd + (gx >> 1) : static_cast<uint32_t>(gy) * wsd + gx;
          const uint32_t xo = ok ? (static_cast<uint32_t>(img) * a.c_in * hw + 8u * (ln >> 5) * hw + el) * 2u : kOut;
#pragma unroll 1
          for (uint32_t c = 0; c < static_cast<uint32_t>(a.c_in); c += 16 * RU) {
            u32x4v wt[RU], xv[RU];
#pragma unroll
            for (int q = 0; q < RU; ++q) {
              wt[q] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(
                                                     arsrc, ao, static_cast<int>(((c >> 4) + q) * 9u * as + t * as), 0));
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                const uint32_t at = (c + 16 * q + 2 * k) * hw * 2u;
                const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(xrsrc, xo, static_cast<int>(at), 0);
                const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(xrsrc, xo, static_cast<int>(at + hw * 2u), 0);
                xv[q][k] = (lo & 0xFFFFu) | hi << 16;
              }
            }
#pragma unroll
            for (int q = 0; q < RU; ++q) op(wt[q], xv[q]);
          }
        }
      };
      auto each = [](u32x4v v, auto f) { return __builtin_bit_cast(bf16x8, (u32x4v{f(v[0]), f(v[1]), f(v[2]), f(v[3])})); };
      // n products, d of them +inf less those -inf (all of one sign only if n = |d|); sum: without those inputs
      f32x16 n = f32x16{}, d = f32x16{}, sum = f32x16{};
      auto count = [&](u32x4v w, u32x4v x) __attribute__((always_inline)) {
        n = __builtin_amdgcn_mfma_f32_32x32x16_bf16(each(w, count_kept), each(x, count_huge), n, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(each(w, sign_weight), each(x, sign_inf), d, 0, 0, 0);
      };
      auto add = [&](u32x4v w, u32x4v x) __attribute__((always_inline)) {
        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), each(x, without_huge), sum, 0, 0, 0);
      };
      if constexpr (kOnce) {
        steps([&](u32x4v w, u32x4v x) __attribute__((always_inline)) {
          count(w, x);
          add(w, x);
        });
      } else {
        steps(count);
      }
      uint32_t plus = 0, minus = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        plus |= n[r] + d[r] != 0.0f ? 1u << r : 0u;
        minus |= n[r] - d[r] != 0.0f ? 1u << r : 0u;
      }
      if (!kOnce && __any(bad & ~(plus & minus))) steps(add);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if ((plus >> r) & 1u) sum[r] += __builtin_inff();
        if ((minus >> r) & 1u) sum[r] -= __builtin_inff();
      }
#pragma unroll
      for (int k = 0; k < MB * TN; ++k)
        if (b == k) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            acc[k / TN][k % TN][r] = (bad >> r) & 1u ? sum[r] : acc[k / TN][k % TN][r];
        }
    }
  }

  // accumulator r of block (i, j), lane l, is C[8 (r / 4) + 4 (l / 32) + r % 4][l % 32] of the block.
  // A row's address is a wave-uniform base (filter 8 (r / 4) + r % 4) plus a
  // 32-bit lane offset (4 filters for the upper half of the wave, and the pixel).
  const bool relu = (a.flags & PP_RELU) != 0;
  const int ex = ox0 + bcol;
  const size_t plane = static_cast<size_t>(a.ho) * a.wo;
  uint16_t* __restrict__ y = static_cast<uint16_t*>(a.y) + static_cast<size_t>(img) * a.c_out * plane;
  const uint32_t half4 = (ln >> 5) * 4, odd = ln & 1;
  const int ob = mtile * M::BM + wm * MB * 32;   // the wave's first filter
  auto act2 = [&](int i, int j, int r) __attribute__((always_inline)) -> uint32_t {   // rows r, r + 1, in bf16
    const int ol = (wm * MB + i) * 32 + 8 * (r >> 2) + half4 + (r & 3);
    float v0 = acc[i][j][r] + bias_s[ol], v1 = acc[i][j][r + 1] + bias_s[ol + 1];
    if (relu) {
      v0 = fmaxf(v0, 0.0f);
      v1 = fmaxf(v1, 0.0f);
    }
    return cvt_bf16x2(v0, v1);
  };
  const bool shuf = (a.flags & PP_PIXSHUF2) != 0, y4 = reinterpret_cast<uintptr_t>(a.y) % 4 == 0;
  const bool pool = (a.flags & PP_MAXPOOL2) != 0;
  const bool accum = (a.flags & PP_ACCUMULATE) != 0;
  // (the plain stores first: on the smallest grids a jump over the others costs 1 to 5 %)
  if (__builtin_expect(!pool && !shuf && a.wo % 2 == 0 && y4, 1)) {
    // columns in pairs: an even lane stores filter o of its and its
    // neighbour's pixel, the neighbour filter o + 1 of both (4-byte stores)
    const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int ey = oy0 + brow + j * M::RPB;
      const bool valid = ey < a.ho && ex < a.wo;
      const uint32_t voff = ((half4 + odd) * static_cast<uint32_t>(plane) + static_cast<uint32_t>(ey) * a.wo + ex - odd) * 2u;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        auto at = [&](int r) __attribute__((always_inline)) {
          return reinterpret_cast<uint32_t*>(
              reinterpret_cast<uint8_t*>(y + static_cast<size_t>(ob + 32 * i + 8 * (r >> 2) + (r & 3)) * plane) + voff);
        };
        auto in = [&](int r) __attribute__((always_inline)) {
          return valid && ob + 32 * i + 8 * (r >> 2) + (r & 3) + static_cast<int>(half4 + odd) < a.c_out;
        };
        uint32_t old[8];
        if (accum) {
#pragma unroll
          for (int r = 0; r < 16; r += 2) old[r / 2] = in(r) ? *at(r) : 0u;
        }
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const uint32_t u = act2(i, j, r);
          const uint32_t nb = __builtin_amdgcn_mov_dpp(u, 0xB1, 0xF, 0xF, true);   // lanes 1, 0, 3, 2 of each four
          uint32_t t = __builtin_amdgcn_perm(nb, u, sel);
          // PP_ACCUMULATE: y = y + act(...), the activated value rounded to bf16 first
          if (accum)
            t = cvt_bf16x2(bf16_val(old[r / 2]) + bf16_val(t), bf16_hi(old[r / 2]) + bf16_hi(t));
          if (in(r)) *at(r) = t;
        }
      }
    }
    return;
  }
  if (__builtin_expect(!shuf && !pool, 1)) {
    // odd widths and a y that starts between dwords: 2-byte stores
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int ey = oy0 + brow + j * M::RPB;
      if (ey >= a.ho || ex >= a.wo) continue;
      const uint32_t voff = (half4 * static_cast<uint32_t>(plane) + static_cast<uint32_t>(ey) * a.wo + ex) * 2u;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const uint32_t u = act2(i, j, r);
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const int os = ob + 32 * i + 8 * (r >> 2) + (r & 3) + k;
            if (os + static_cast<int>(half4) >= a.c_out) break;
            uint16_t* d = reinterpret_cast<uint16_t*>(reinterpret_cast<uint8_t*>(y + static_cast<size_t>(os) * plane) + voff);
            const uint32_t b = k ? u >> 16 : u & 0xFFFFu;
            *d = static_cast<uint16_t>(accum ? cvt_bf16x2(bf16_val(*d) + bf16_val(b), 0.0f) : b);
          }
        }
    }
    return;
  }
  if (shuf && y4) {
    // PixelShuffle(2): filters o, o + 1 (o even; accumulators r, r + 1)
    // land in adjacent columns 2 ex, 2 ex + 1 of one output row: one
    // 4-byte store per pair (c_out is a multiple of 4)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int ey = oy0 + brow + j * M::RPB;
      if (ey >= a.ho || ex >= a.wo) continue;
      const uint32_t voff = (half4 * static_cast<uint32_t>(plane) + (2u * ey) * 2u * a.wo + 2u * ex) * 2u;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const int os = ob + 32 * i + 8 * (r >> 2);   // multiple of 8
          uint8_t* row = reinterpret_cast<uint8_t*>(y + static_cast<size_t>(os) * plane + (r & 2) * a.wo);
          if (os + static_cast<int>(half4) < a.c_out) *reinterpret_cast<uint32_t*>(row + voff) = act2(i, j, r);
        }
    }
    return;
  }
  if (pool) {
    // the 2 x 2 max of the values the plain store would write: columns of a
    // window are neighbouring lanes, its rows two of the wave's pixel blocks
    // (32 columns across) or lanes 16 apart (16 across).  The even lane of a
    // window stores filter o, the odd one filter o + 1.
    static_assert(M::TW == 32 ? TN % 2 == 0 : M::RPB == 2, "a wave holds whole windows");
    const uint32_t pw = a.wo / 2, pplane = pw * (a.ho / 2u);
    uint16_t* __restrict__ yp = static_cast<uint16_t*>(a.y) + static_cast<size_t>(img) * a.c_out * pplane;
    auto max2 = [](uint32_t u, uint32_t v) __attribute__((always_inline)) -> uint32_t {
      return __float_as_uint(fmaxf(bf16_val(u), bf16_val(v))) >> 16 | __float_as_uint(fmaxf(bf16_hi(u), bf16_hi(v)));
    };
    auto across = [&](uint32_t u) __attribute__((always_inline)) -> uint32_t {
      return max2(u, __builtin_amdgcn_mov_dpp(u, 0xB1, 0xF, 0xF, true));   // lanes 1, 0, 3, 2 of each four
    };
#pragma unroll
    for (int j = 0; j < TN; j += M::TW == 32 ? 2 : 1) {
      const int ey = oy0 + brow + j * M::RPB;   // the window's first row, in the lanes that store
      const bool valid = (M::TW == 32 || (ln & 16) == 0) && ey + 1 < a.ho && (ex | 1) < a.wo;
      // (one lane pointer walking the filters: an address per row would take the scalar registers)
      int o = ob + half4 + odd;
      uint16_t* d = yp + static_cast<size_t>(o) * pplane + (static_cast<uint32_t>(ey) >> 1) * pw + (static_cast<uint32_t>(ex) >> 1);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          uint32_t v = across(act2(i, j, r));
          if constexpr (M::TW == 32)
            v = max2(v, across(act2(i, j + 1, r)));
          else
            v = max2(v, __shfl_xor(v, 16));
          if (valid && o < a.c_out) *d = static_cast<uint16_t>(odd ? v >> 16 : v);
          const int next = r & 2 ? 6 : 2;   // filters 0, 2, 8, 10, 16, ... of the block
          o += next;
          d += static_cast<size_t>(next) * pplane;
        }
    }
    return;
  }
  {
    // the shuffle into a y that starts between dwords: two 2-byte stores
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int ey = oy0 + brow + j * M::RPB;
      if (ey >= a.ho || ex >= a.wo) continue;
      const uint32_t voff = (half4 * static_cast<uint32_t>(plane) + (2u * ey) * 2u * a.wo + 2u * ex) * 2u;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const int os = ob + 32 * i + 8 * (r >> 2);
          uint16_t* d = reinterpret_cast<uint16_t*>(
              reinterpret_cast<uint8_t*>(y + static_cast<size_t>(os) * plane + (r & 2) * a.wo) + voff);
          if (os + static_cast<int>(half4) >= a.c_out) continue;
          const uint32_t u = act2(i, j, r);
          d[0] = static_cast<uint16_t>(u);
          d[1] = static_cast<uint16_t>(u >> 16);
        }
    }
  }
}

size_t a_bytes(const ConvParams& p) {
  return (static_cast<size_t>(p.c_out) * 9 * p.c_in * 2 + 255) / 256 * 256;
}

// workgroups of a layer in tiles of bm filters x (th x tw) outputs
long tiles(const ConvParams& p, int bm, int th, int tw) {
  return static_cast<long>((p.c_out + bm - 1) / bm) * ((p.ho + th - 1) / th) * ((p.wo + tw - 1) / tw) * p.n;
}

// Tiles (filters x pixels; timed on MI355X, bf16, us): the weights cross
// each compute unit's caches once per wave, so larger tiles are better as
// long as every unit still gets one or two workgroups.
//   128 x 256 from 512 such tiles (64 -> 256 at 270 x 480: 44, 128 x 128 47;
//     512 -> 512 on 8 x 32 x 32, 128 tiles: 60 against 37)
//   128 x 128 from 192 (that layer; 128 -> 256 on 8 x 64 x 64: 23, 64 x 128 33)
//   64 x 256 for at most 64 filters from 400 (64 -> 64 at 270 x 480: 18, 64 x 128 21)
//   64 x 128 below (128 -> 128 at 128 x 128: 12.3, 128 x 128 14)
// 128 x 128 stages 64 channels at a time when c_in is a multiple of 64 (one workgroup per
// unit: half the waits for a block's input; 512 -> 512: 37 against 39), and
// 64 x 128 does from 128 channels on grids of at most one workgroup per unit
// (512 -> 512 at 28 x 28 26.2 against 27.9; 64 -> 64 with dilation 2 at 256 x 256 14.7
// against 11.8: not below, where two workgroups per unit come first).  The
// 128-pixel tiles are 4 x 32 or 8 x 16 outputs, whichever covers the map with fewer tiles.
// Every tile sums in the same order: the choice never changes a result's bits.
enum Form { kS2, kS2Wide, k128x256, k64x256, k128x128, k64x128 };

bool is_tall(const ConvParams& p) { return tiles(p, 128, 8, 16) < tiles(p, 128, 4, 32); }   // 8 x 16 covers the map with fewer

Form choose_form(const ConvParams& p) {
  const bool wide = p.c_out > 64, d1 = p.dil == 1;
  if (p.stride == 2) return d1 && wide && tiles(p, 128, 4, 32) >= 192 ? kS2Wide : kS2;
  if (d1 && wide && tiles(p, 128, 8, 32) >= 512) return k128x256;
  if (d1 && !wide && tiles(p, 64, 8, 32) >= 400) return k64x256;
  return wide && std::min(tiles(p, 128, 8, 16), tiles(p, 128, 4, 32)) >= 192 ? k128x128 : k64x128;
}

template <int WM, int MB, int TN, int CB, int TW, int S, int D>
hipError_t launch_tiles(const ConvParams& p, const uint16_t* am, const float* bo, hipStream_t st) {
  using M = MGeo<WM, MB, TN, CB, TW, S, D>;
  static_assert(M::LDS + M::BM * 4 <= 160 * 1024, "staging buffers fit the LDS");
  MTiles t;
  t.m_tiles = (p.c_out + M::BM - 1) / M::BM;
  t.tiles_x = (p.wo + M::TW - 1) / M::TW;
  t.tiles_y = (p.ho + M::TH - 1) / M::TH;
  const size_t blocks = static_cast<size_t>(t.m_tiles) * t.tiles_x * t.tiles_y * p.n;
  if (blocks < 1 || blocks > 0x7FFFFFFFu) return hipErrorInvalidConfiguration;
  const dim3 grid(static_cast<uint32_t>(blocks));
  // pixel pairs: rows of whole 4-byte words (an upsampled input reads each stored pixel twice)
  const bool px2 = p.w % 2 == 0 && !(p.flags & PP_UPSAMPLE2) && reinterpret_cast<uintptr_t>(p.x) % 4 == 0;
  if (px2)
    hipLaunchKernelGGL((pp_mfma_conv_kernel<WM, MB, TN, CB, TW, S, D, true>), grid, dim3(256), 0, st, p, am, bo, t);
  else
    hipLaunchKernelGGL((pp_mfma_conv_kernel<WM, MB, TN, CB, TW, S, D, false>), grid, dim3(256), 0, st, p, am, bo, t);
  return hipGetLastError();
}

}  // namespace

bool mfma_eligible(const ConvParams& p) {
  if (p.c_in < 32 || p.c_in % 32 != 0 || p.c_out < 1) return false;   // (staged 32 channels at a time)
  if (p.stride < 1 || p.stride > 2 || p.dil < 1 || p.dil > 2 || p.pad < 0) return false;
  const bool up = (p.flags & PP_UPSAMPLE2) != 0;
  if (up && (p.h % 2 || p.w % 2)) return false;
  // 32-bit byte offsets below 2^30 (2^31 marks an element outside a tensor
  // and the loads add the channel offset to it)
  const size_t hw = static_cast<size_t>(up ? p.h / 2 : p.h) * (up ? p.w / 2 : p.w);
  return static_cast<size_t>(p.n) * p.c_in * hw * 2 < (size_t{1} << 30) &&
         static_cast<size_t>(p.c_out) * 9 * p.c_in * 2 < (size_t{1} << 30);
}

// A workgroup's time is linear in c_in (what bounds it is the weights' way
// through its unit's cache, the same for every channel), and workgroups past
// one per unit queue.  us per input channel, measured on MI355X: 64 x 128
// 0.036 (512 -> 512 at 14 x 14 21.2, 256 -> 256 at 56 x 56 13.4, 64 -> 64 at
// 224 x 224, 392 tiles, 9.9), 128 x 128 0.0625 (512 -> 512 on 8 x 32 x 32
// 37), 64 x 256 0.105, 128 x 256 0.16 (64 -> 256 at 540 x 960 170), stride 2
// 0.062 (512 -> 512 at 32 x 32 36.4), its 128 x 128 0.1; 5 us to launch, fill
// and drain.
double mfma_time(const ConvParams& p) {
  double us = 0.036;
  long t = std::min(tiles(p, 64, 8, 16), tiles(p, 64, 4, 32));
  switch (choose_form(p)) {
    case kS2: us = 0.062, t = tiles(p, 64, 4, 32); break;
    case kS2Wide: us = 0.1, t = tiles(p, 128, 4, 32); break;
    case k128x256: us = 0.16, t = tiles(p, 128, 8, 32); break;
    case k64x256: us = 0.105, t = tiles(p, 64, 8, 32); break;
    case k128x128: us = 0.0625, t = std::min(tiles(p, 128, 8, 16), tiles(p, 128, 4, 32)); break;
    case k64x128: break;
  }
  return (5.0 + us * p.c_in * std::max(1.0, t / 256.0)) * 1e-6;
}

size_t mfma_bytes(const ConvParams& p) { return a_bytes(p) + static_cast<size_t>(p.c_out) * sizeof(float); }

hipError_t launch_mfma_expand(const ConvParams& p, void* out, hipStream_t st) {
  if (!out || reinterpret_cast<uintptr_t>(out) % 256) return hipErrorInvalidValue;
  uint16_t* am = static_cast<uint16_t*>(out);
  float* bo = reinterpret_cast<float*>(static_cast<uint8_t*>(out) + a_bytes(p));
  const long ex = static_cast<long>(p.n_groups) * 8 * p.c_in;
  hipLaunchKernelGGL(pp_mfma_expand_kernel, dim3(static_cast<uint32_t>((ex + 255) / 256)), dim3(256), 0, st, p, am, bo);
  return hipGetLastError();
}

hipError_t launch_mfma_conv(const ConvParams& p, hipStream_t st) {
  if (!mfma_eligible(p) || !p.part || reinterpret_cast<uintptr_t>(p.part) % 256) return hipErrorInvalidValue;
  const uint16_t* am = reinterpret_cast<const uint16_t*>(p.part);
  const float* bo = reinterpret_cast<const float*>(reinterpret_cast<const uint8_t*>(p.part) + a_bytes(p));
  // PP_PREPARED: the workspace already holds the expansion (pp_conv2d_prepare)
  if (!(p.flags & PP_PREPARED)) {
    const hipError_t e = launch_mfma_expand(p, p.part, st);
    if (e != hipSuccess) return e;
  }
  const bool d1 = p.dil == 1;
  switch (choose_form(p)) {
    case kS2: return d1 ? launch_tiles<2, 1, 2, 16, 32, 2, 1>(p, am, bo, st) : launch_tiles<2, 1, 2, 16, 32, 2, 2>(p, am, bo, st);
    case kS2Wide: return launch_tiles<2, 2, 2, 32, 32, 2, 1>(p, am, bo, st);
    case k128x256: return launch_tiles<2, 2, 4, 32, 32, 1, 1>(p, am, bo, st);
    case k64x256: return launch_tiles<1, 2, 2, 32, 32, 1, 1>(p, am, bo, st);
    case k128x128:
      if (p.c_in % 64 == 0) {
        if (is_tall(p)) return d1 ? launch_tiles<2, 2, 2, 64, 16, 1, 1>(p, am, bo, st) : launch_tiles<2, 2, 2, 64, 16, 1, 2>(p, am, bo, st);
        return d1 ? launch_tiles<2, 2, 2, 64, 32, 1, 1>(p, am, bo, st) : launch_tiles<2, 2, 2, 64, 32, 1, 2>(p, am, bo, st);
      }
      if (is_tall(p)) return d1 ? launch_tiles<2, 2, 2, 32, 16, 1, 1>(p, am, bo, st) : launch_tiles<2, 2, 2, 32, 16, 1, 2>(p, am, bo, st);
      return d1 ? launch_tiles<2, 2, 2, 32, 32, 1, 1>(p, am, bo, st) : launch_tiles<2, 2, 2, 32, 32, 1, 2>(p, am, bo, st);
    case k64x128: break;
  }
  if (p.c_in % 64 == 0 && p.c_in >= 128 && tiles(p, 64, is_tall(p) ? 8 : 4, is_tall(p) ? 16 : 32) <= 256) {
    if (is_tall(p)) return d1 ? launch_tiles<2, 1, 2, 64, 16, 1, 1>(p, am, bo, st) : launch_tiles<2, 1, 2, 64, 16, 1, 2>(p, am, bo, st);
    return d1 ? launch_tiles<2, 1, 2, 64, 32, 1, 1>(p, am, bo, st) : launch_tiles<2, 1, 2, 64, 32, 1, 2>(p, am, bo, st);
  }
  if (is_tall(p)) return d1 ? launch_tiles<2, 1, 2, 32, 16, 1, 1>(p, am, bo, st) : launch_tiles<2, 1, 2, 32, 16, 1, 2>(p, am, bo, st);
  return d1 ? launch_tiles<2, 1, 2, 32, 32, 1, 1>(p, am, bo, st) : launch_tiles<2, 1, 2, 32, 32, 1, 2>(p, am, bo, st);
}

}  // namespace pp
