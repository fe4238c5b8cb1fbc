// x2 super-sampling network (Sec. 3.4, end; Sec. 4.1: GlassNet renders at the
// training resolution and a small CNN, fed by full-resolution G-buffers from
// the rasterizer, doubles it).  Layers: bilinear x2 of the render (half-pixel
// centres, clamped sources) joined with the 14 G-buffer planes, conv 3x3
// 17 -> 32 + ReLU, conv 3x3 32 -> 32 + ReLU, conv 1x1 32 -> 3, plus the
// upsampled render; 3x3 convs zero-padded to keep the size.
//
// One fused kernel per call (sr_forward_kernel), both 3x3 convs as implicit
// GEMMs with the weights as the 16-row operand (two tiles of 16 output
// channels) and 16 pixels as the columns, fp32 operands split in three on the
// bf16 matrix cores (fp32_core.h), fp32 sums.  A 256-thread block owns a 16 x
// 16 output tile:
//   stage 0  the 17-channel input over the tile plus a two-pixel halo, split,
//            into LDS (upsampling on the fly);
//   stage 1  conv1 + ReLU over the tile plus a one-pixel halo (324 positions,
//            21 column tiles of 16), split, into the same LDS, zero outside
//            the image as conv2's padding requires;
//   stage 2  conv2 + ReLU, one output row of 16 pixels per column tile, then
//            the 1x1 head: each lane holds 8 of the 32 channels of its pixel,
//            and two cross-lane sums complete the 3 outputs; plus the
//            upsampled render.
// The backward recomputes the hidden layers with the fp32 instruction
// (sr_recompute_kernel): its ReLU masks must not move by a rounding.
#include <algorithm>

#include "fp32_core.h"

namespace gn {
namespace {

using f32::f32x4;
using f32::u32x4;
using f32::Split;

constexpr int kC = kSrWidth;          // hidden channels
constexpr int kIn = kSrIn;            // 3 upsampled + 14 G-buffer channels
constexpr int kInP = 20;              // input channels padded to a multiple of 4
constexpr int kT = 16;                // output tile edge
constexpr int kE0 = kT + 4;           // staged input edge (two-pixel halo)
constexpr int kE1 = kT + 2;           // conv1 output edge (one-pixel halo)
constexpr int kP1 = kE1 * kE1;        // conv1 positions per tile (324)
constexpr int kA1Stride = 336;        // LDS floats per conv1 output channel
constexpr int kThreads = 256;
constexpr int kS1 = 9 * kInP / 4;     // conv1 K steps (45)
constexpr int kS2 = 9 * kC / 4;       // conv2 K steps (72)
constexpr int kN1 = (kP1 + 15) / 16;  // conv1 column tiles (21)
// Re-laid weights.  Floats, for the recompute and the head: A1 [kS1][2][64],
// b1 [32], A2 [kS2][2][64], b2 [32], w3 [3][32], b3 [3].  Then (16-byte
// aligned) split fragments [step][channel tile][part][lane][16 bytes]: conv1,
// conv2, and conv2's transpose (input and output channels swapped, taps
// mirrored) for the backward.
constexpr int kOffB1 = kS1 * 2 * 64;
constexpr int kOffA2 = kOffB1 + kC;
constexpr int kOffB2 = kOffA2 + kS2 * 2 * 64;
constexpr int kOffW3 = kOffB2 + kC;
constexpr int kOffB3 = kOffW3 + kSrOut * kC;
constexpr int kWtFp32 = kOffB3 + kSrOut;
constexpr int kOffSplit = (kWtFp32 + 3) / 4 * 4;
// K-steps of 32 of the split convs.  conv2: one tap, 32 channels.  conv1: steps
// 0-3 two taps of channels 0-15, step 4 tap 8 of those and the nine taps of
// channel 16.
constexpr int kQ1 = 5, kQ2 = 9, kQFloats = 2 * 3 * 64 * 4;
constexpr int kOffF1 = kOffSplit, kOffF2 = kOffF1 + kQ1 * kQFloats, kOffF2T = kOffF2 + kQ2 * kQFloats;
static_assert(kOffF2T + kQ2 * kQFloats == kSrWtFloats, "re-laid weight size");
static_assert(kA1Stride >= kP1 && kA1Stride % 64 == 16, "conv1 output channel stride");

// packed weights -> MFMA operand order.  fp32 fragment (s, mt, lane): output
// channel 16 mt + lane % 16, K index 4 s + lane / 16 = tap * C + channel.
__global__ __launch_bounds__(kThreads) void sr_relayout_kernel(const float *__restrict__ w,
                                                               float *__restrict__ wt) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  const float *w1 = w, *b1 = w1 + kC * kIn * 9, *w2 = b1 + kC, *b2 = w2 + kC * kC * 9;
  const float *w3 = b2 + kC, *b3 = w3 + kSrOut * kC;
  if (i >= kWtFp32) {
    // split fragments, a thread per lane: row 16 mt + lane % 16, K index
    // 8 (lane / 16) + e
    const int j = i - kWtFp32, l = j % 64, mt = (j / 64) % 2, g = l / 16;
    const int o = 16 * mt + l % 16;
    int q = j / 128;
    if (q >= kQ1 + 2 * kQ2) return;
    u32x4 *dst = (u32x4 *)(wt + kOffSplit + q * kQFloats) + mt * 3 * 64 + l;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (q < kQ1) {
        const int c = 8 * (g & 1) + e, tap = 2 * q + (g >> 1);
        const int t16 = 8 * (g - 2) + e;       // step 4's upper half: channel 16, tap t16
        if (q < 4 || g < 2) x[e] = w1[(o * kIn + c) * 9 + tap];
        else x[e] = t16 < 9 ? w1[(o * kIn + 16) * 9 + t16] : 0.0f;
      } else if (q < kQ1 + kQ2) {
        x[e] = w2[(o * kC + 8 * g + e) * 9 + q - kQ1];
      } else {
        x[e] = w2[((8 * g + e) * kC + o) * 9 + 8 - (q - kQ1 - kQ2)];
      }
    }
    const Split sp = f32::split8(x);
    dst[0] = sp.hi;
    dst[64] = sp.mid;
    dst[128] = sp.lo;
    return;
  }
  float v;
  if (i < kOffB1) {
    const int s = i / 128, mt = (i / 64) % 2, l = i % 64;
    const int k = 4 * s + l / 16, tap = k / kInP, c = k % kInP, o = 16 * mt + l % 16;
    v = c < kIn ? w1[(o * kIn + c) * 9 + tap] : 0.0f;
  } else if (i < kOffA2) {
    v = b1[i - kOffB1];
  } else if (i < kOffB2) {
    const int j = i - kOffA2;
    const int s = j / 128, mt = (j / 64) % 2, l = j % 64;
    const int k = 4 * s + l / 16, tap = k / kC, c = k % kC, o = 16 * mt + l % 16;
    v = w2[(o * kC + c) * 9 + tap];
  } else if (i < kOffW3) {
    v = b2[i - kOffB2];
  } else if (i < kOffB3) {
    v = w3[i - kOffW3];
  } else {
    v = b3[i - kOffB3];
  }
  wt[i] = v;
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// LDS staging with many loads in flight: element e < N of a block goes to
// dst(e) from byte offset off(e) of the buffer behind r (kOutside, past the
// buffer's bound, reads zero: the callers' zero padding).  Loads guarded by a
// branch or followed by a select on their value are each waited for before
// the next one issues; these are neither, so the compiler issues a group of
// them before the first store.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr uint32_t kOutside = 0x80000000u;   // past every bound (resources stay under 2 GiB)
__device__ __forceinline__ rsrc_t make_rsrc(const void *base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0,
                                           (int)std::min<int64_t>(bytes, kOutside), 0x00020000);
}

// One float at byte `off` (kOutside: zero) of a plane at the uniform byte
// offset `plane`: the planes cost no vector arithmetic.
__device__ __forceinline__ float load1(rsrc_t r, uint32_t off, uint32_t plane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, plane, 0));
}

template <int N, class Off, class Dst>
__device__ __forceinline__ void stage(int tid, rsrc_t r, Off off, Dst dst) {
  constexpr int kIt = (N + kThreads - 1) / kThreads, kG = 8;
  // groups of kG loads, then their kG stores (in program order: the
  // compiler does not move a buffer load above an LDS store)
  for (int i0 = 0; i0 < kIt; i0 += kG) {
    float v[kG];
#pragma unroll
    for (int j = 0; j < kG; ++j) {
      const int e = min(tid + (i0 + j) * kThreads, N - 1);
      v[j] = i0 + j < kIt
                 ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off(e), 0, 0))
                 : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < kG; ++j) {
      const int e = tid + (i0 + j) * kThreads;
      if (i0 + j < kIt && (N % kThreads == 0 || e < N)) *dst(e) = v[j];
    }
  }
}

// The render's 3 channels upsampled x2 into LDS over a square window of edge
// E at (y0, x0) of the output image: element e < 3 E^2 is channel e / E^2,
// row (e / E) % E, column e % E.  Output pixel (Y, X) samples source
// position (Y + 0.5) / 2 - 0.5: rows Y/2 - 1 and Y/2 at weights 1/4 and 3/4
// for even Y, rows (Y-1)/2 and (Y+1)/2 at 3/4 and 1/4 for odd Y (clamped
// into the image); likewise for columns.  Outside the image
// the four source offsets are past the buffer's bound, so the loads read
// zeros and the blend is zero; groups of 4 elements issue their 16 loads
// before any store.
struct UpTap {
  uint32_t o[4];   // source elements within a plane, from its row y0 on
  float fx, fy;
};
__device__ __forceinline__ UpTap up_tap(int Y, int X, int y0, int h, int w) {
  const int sy = (Y >> 1) - ((Y & 1) ? 0 : 1), sx = (X >> 1) - ((X & 1) ? 0 : 1);
  const int ya = max(sy, 0) - y0, yb = min(sy + 1, h - 1) - y0;
  const int xa = max(sx, 0), xb = min(sx + 1, w - 1);
  return {{(uint32_t)(ya * w + xa), (uint32_t)(ya * w + xb), (uint32_t)(yb * w + xa),
           (uint32_t)(yb * w + xb)},
          (X & 1) ? 0.25f : 0.75f,
          (Y & 1) ? 0.25f : 0.75f};
}
__device__ __forceinline__ float up_blend(const float (&v)[4], float fx, float fy) {
  const float top = (1.0f - fx) * v[0] + fx * v[1];
  const float bot = (1.0f - fx) * v[2] + fx * v[3];
  return (1.0f - fy) * top + fy * bot;
}

template <int E>
__device__ __forceinline__ void stage_up(int tid, rsrc_t rlo, int h, int w, int y0, int x0,
                                         float *dst) {
  constexpr int N = 3 * E * E, kIt = (N + kThreads - 1) / kThreads, kG = 4;
  const int H = 2 * h, W = 2 * w;
  for (int i0 = 0; i0 < kIt; i0 += kG) {
    float v[kG][4], fx[kG], fy[kG];
#pragma unroll
    for (int j = 0; j < kG; ++j) {
      const int e = min(tid + (i0 + j) * kThreads, N - 1);
      const int c = e / (E * E), Y = y0 + (e / E) % E, X = x0 + e % E;
      const bool ok = i0 + j < kIt && Y >= 0 && Y < H && X >= 0 && X < W;
      const int sy = (Y >> 1) - ((Y & 1) ? 0 : 1), sx = (X >> 1) - ((X & 1) ? 0 : 1);
      fy[j] = (Y & 1) ? 0.25f : 0.75f;
      fx[j] = (X & 1) ? 0.25f : 0.75f;
      const int ya = max(sy, 0), yb = min(sy + 1, h - 1), xa = max(sx, 0), xb = min(sx + 1, w - 1);
      const uint32_t base = (uint32_t)(c * h * w);
      const uint32_t o[4] = {base + ya * w + xa, base + ya * w + xb, base + yb * w + xa,
                             base + yb * w + xb};
#pragma unroll
      for (int k = 0; k < 4; ++k)
        v[j][k] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rlo, ok ? 4 * o[k] : kOutside, 0, 0));
    }
#pragma unroll
    for (int j = 0; j < kG; ++j) {
      const int e = tid + (i0 + j) * kThreads;
      if (i0 + j < kIt && (N % kThreads == 0 || e < N)) {
        const float top = (1.0f - fx[j]) * v[j][0] + fx[j] * v[j][1];
        const float bot = (1.0f - fx[j]) * v[j][2] + fx[j] * v[j][3];
        dst[e] = (1.0f - fy[j]) * top + fy[j] * bot;
      }
    }
  }
}

// ---- convolutions with split operands ----------------------------------
// Activations in LDS: planes of 16-byte records, one per position, each 8
// channels of one of the three parts, so 16 neighbouring columns read
// consecutive records.
constexpr int kRec = 16;

__device__ __forceinline__ Split lds_split(const uint8_t *p, int part) {
  return Split{*(const u32x4 *)p, *(const u32x4 *)(p + part), *(const u32x4 *)(p + 2 * part)};
}
__device__ __forceinline__ void store_split(uint8_t *p, int part, const Split &s) {
  *(u32x4 *)p = s.hi;
  *(u32x4 *)(p + part) = s.mid;
  *(u32x4 *)(p + 2 * part) = s.lo;
}

// Four channels: half of a record.
__device__ __forceinline__ void store_split4(uint8_t *p, int part, const float (&v)[4]) {
  const float x[8] = {v[0], v[1], v[2], v[3], 0.f, 0.f, 0.f, 0.f};
  const Split s = f32::split8(x);
  *(uint2 *)p = uint2{s.hi[0], s.hi[1]};
  *(uint2 *)(p + part) = uint2{s.mid[0], s.mid[1]};
  *(uint2 *)(p + 2 * part) = uint2{s.lo[0], s.lo[1]};
}

// acc[jj] += conv over STEPS K-steps for this wave's column tiles wave + 4 jj
// below ntiles; src(jj, s) is the LDS record of part 0.  A step's weights, 6
// KiB, come from L2 a step ahead (the first step's in a[0], by conv_first) and
// serve all of the wave's tiles.  FRESH: as SplitPipe's.
typedef u32x4 ConvWeights[2][6];
__device__ __forceinline__ void conv_first(ConvWeights &a, const float *frags, int lane) {
#pragma unroll
  for (int e = 0; e < 6; ++e) a[0][e] = ((const u32x4 *)frags)[lane + e * 64];
}

template <int NJ, int STEPS, bool FRESH, class Src>
__device__ __forceinline__ void conv_split(f32x4 (&acc)[NJ][2], ConvWeights &a, const float *frags,
                                           int part, int ntiles, int lane, int wave, Src src) {
  const u32x4 *f = (const u32x4 *)frags + lane;
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    if (s + 1 < STEPS) {
#pragma unroll
      for (int e = 0; e < 6; ++e) a[(s + 1) & 1][e] = f[((s + 1) * 6 + e) * 64];
    }
    const u32x4(&w)[6] = a[s & 1];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      if (wave + 4 * jj >= ntiles) continue;
      const Split b = lds_split(src(jj, s), part);
      f32x4 c0 = FRESH ? f32::zero4() : acc[jj][0], c1 = FRESH ? f32::zero4() : acc[jj][1];
      // the two channel tiles in turn: each product waits for the sum before it
      c0 = f32::mma_bf16(w[2], b.hi, c0);
      c1 = f32::mma_bf16(w[5], b.hi, c1);
      c0 = f32::mma_bf16(w[0], b.lo, c0);
      c1 = f32::mma_bf16(w[3], b.lo, c1);
      c0 = f32::mma_bf16(w[1], b.mid, c0);
      c1 = f32::mma_bf16(w[4], b.mid, c1);
      c0 = f32::mma_bf16(w[1], b.hi, c0);
      c1 = f32::mma_bf16(w[4], b.hi, c1);
      c0 = f32::mma_bf16(w[0], b.mid, c0);
      c1 = f32::mma_bf16(w[3], b.mid, c1);
      c0 = f32::mma_bf16(w[0], b.hi, c0);
      c1 = f32::mma_bf16(w[3], b.hi, c1);
      acc[jj][0] = FRESH ? acc[jj][0] + c0 : c0;
      acc[jj][1] = FRESH ? acc[jj][1] + c1 : c1;
    }
  }
}

// conv2's operand (the forward's a1, the backward's dz2): [part][channel / 8]
// [position], over the tile and a one-pixel halo.
constexpr int kPartH = 4 * kP1 * kRec;
constexpr int kNJ1f = (kN1 + 3) / 4;   // conv1 column tiles per wave (6)

// The split forward's LDS: conv1's operand, per part channels 0-15 [half]
// [position], then channel 16's nine taps at every conv1 position: taps 0-7,
// and tap 8 with seven zeros.  a1 takes its place.
constexpr int kE2 = kE0 * kE0, kTapRec = 2 * kE2, kTap8Rec = kTapRec + kP1;
constexpr int kPartX = (kTap8Rec + kP1) * kRec;
static_assert(kPartH <= kPartX, "a1 fits the input's place");

// What bounds it: per tile and CU 12k cycles of matrix-core work (21 x 5 + 16 x
// 9 steps of 12 products) and as many of vector work (splitting the input and
// a1 in three, the upsampling), which two workgroups per CU overlap in part.
// One 256^2 -> 512^2 call: 49 us, 90 on the fp32 instruction (33k cycles of
// matrix-core work per tile).
__global__ __launch_bounds__(kThreads, 2) void sr_forward_kernel(
    const float *__restrict__ wt, const float *__restrict__ lowres,
    const float *__restrict__ gbuf, float *__restrict__ out, int h, int w) {
  __shared__ __attribute__((aligned(16))) uint8_t x_s[3 * kPartX];   // 69.5 KB
  __shared__ float up_s[kSrOut * kE2], c16_s[kE2];           // 6.3 KB
  const int H = 2 * h, W = 2 * w;
  const int f = blockIdx.z;
  const int oy0 = blockIdx.y * kT, ox0 = blockIdx.x * kT;
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int col = lane % 16, grp = lane / 16;
  const int64_t plane_lo = (int64_t)h * w, plane_hi = (int64_t)H * W;

  ConvWeights a;
  // stage 0: a thread per input position (400: two rounds), all of its loads
  // before the first use
  {
    constexpr int kG = kIn - 3;
    // a resource per plane, over the rows the tile reads: offsets stay small
    // whatever the frame's size
    const int y0 = max(oy0 - 2, 0), y1 = min(oy0 + kT + 2, H);
    const int s0 = max(y0 / 2 - 1, 0), s1 = min((y1 - 1) / 2 + 1, h - 1) + 1;
    const float *g0 = gbuf + (int64_t)f * kG * plane_hi + (int64_t)y0 * W;
    const float *lo0 = lowres + (int64_t)f * 3 * plane_lo + (int64_t)s0 * w;
    const int64_t g_bytes = 4 * (int64_t)(y1 - y0) * W, lo_bytes = 4 * (int64_t)(s1 - s0) * w;
    float gv[2][kG], uv[2][3][4], fx[2], fy[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int P = tid + r * kThreads, Y = oy0 - 2 + P / kE0, X = ox0 - 2 + P % kE0;
      const bool ok = P < kE2 && Y >= 0 && Y < H && X >= 0 && X < W;
      const uint32_t px = ok ? 4 * ((uint32_t)(Y - y0) * W + X) : kOutside;
#pragma unroll
      for (int c = 0; c < kG; ++c) gv[r][c] = load1(make_rsrc(g0 + c * plane_hi, g_bytes), px, 0);
      const UpTap u = up_tap(Y, X, s0, h, w);
      fx[r] = u.fx;
      fy[r] = u.fy;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t o = ok ? 4 * u.o[k] : kOutside;
#pragma unroll
        for (int c = 0; c < 3; ++c) uv[r][c][k] = load1(make_rsrc(lo0 + c * plane_lo, lo_bytes), o, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int P = tid + r * kThreads;
      if (P >= kE2) continue;
      float x[17];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        x[c] = up_blend(uv[r][c], fx[r], fy[r]);
        up_s[c * kE2 + P] = x[c];
      }
#pragma unroll
      for (int c = 0; c < kG; ++c) x[3 + c] = gv[r][c];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = x[8 * hf + e];
        store_split(x_s + (hf * kE2 + P) * kRec, kPartX, f32::split8(v));
      }
      c16_s[P] = x[16];
    }
    __syncthreads();
    conv_first(a, wt + kOffF1, lane);
    // channel 16's taps at every conv1 position
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int q = tid + r * kThreads;
      if (q >= kP1) continue;
      const float *src = c16_s + (q / kE1) * kE0 + q % kE1;
      float v[8], v8[8] = {};
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = src[(e / 3) * kE0 + e % 3];
      v8[0] = src[2 * kE0 + 2];
      store_split(x_s + (kTapRec + q) * kRec, kPartX, f32::split8(v));
      store_split(x_s + (kTap8Rec + q) * kRec, kPartX, f32::split8(v8));
    }
  }
  __syncthreads();

  // stage 1: conv1 + ReLU over the tile and a one-pixel halo
  {
    f32x4 acc[kNJ1f][2];
    int pos[kNJ1f], q[kNJ1f];
#pragma unroll
    for (int jj = 0; jj < kNJ1f; ++jj) {
      q[jj] = 16 * (wave + 4 * jj) + col;
      const int qq = min(q[jj], kP1 - 1);   // columns past the last position are discarded
      pos[jj] = (qq / kE1) * kE0 + qq % kE1;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) acc[jj][mt] = *(const f32x4 *)(wt + kOffB1 + 16 * mt + 4 * grp);
    }
    conv_split<kNJ1f, kQ1, false>(acc, a, wt + kOffF1, kPartX, kN1, lane, wave, [&](int jj, int s) {
      // lane groups 0, 1: channels 0-7, 8-15 of tap 2 s; 2, 3: of tap 2 s + 1,
      // in the last step channel 16's taps
      const int t0 = 2 * s, t1 = 2 * s + 1;
      const int o0 = (t0 / 3) * kE0 + t0 % 3, o1 = (t1 / 3) * kE0 + t1 % 3;
      const int base = (grp & 1) * kE2 + pos[jj];
      if (s < kQ1 - 1) return x_s + (base + (grp < 2 ? o0 : o1)) * kRec;
      const int tap = kTapRec + (grp & 1) * kP1 + min(q[jj], kP1 - 1);
      return x_s + (grp < 2 ? base + o0 : tap) * kRec;
    });
    __syncthreads();   // every wave has read the input: a1 takes its place
    conv_first(a, wt + kOffF2, lane);
#pragma unroll
    for (int jj = 0; jj < kNJ1f; ++jj) {
      if (q[jj] >= kP1) continue;
      const int Y = oy0 - 1 + q[jj] / kE1, X = ox0 - 1 + q[jj] % kE1;
      const bool inside = Y >= 0 && Y < H && X >= 0 && X < W;
      const float most = inside ? __builtin_inff() : 0.0f;   // ReLU, and zero outside
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_fmed3f(acc[jj][mt][i], 0.0f, most);
        store_split4(x_s + ((2 * mt + (grp >> 1)) * kP1 + q[jj]) * kRec + (grp & 1) * 8, kPartH, v);
      }
    }
  }
  __syncthreads();

  // stage 2: conv2 + ReLU, the 1x1 head and the residual; one row per tile
  f32x4 acc[4][2];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj)
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) acc[jj][mt] = *(const f32x4 *)(wt + kOffB2 + 16 * mt + 4 * grp);
  conv_split<4, kQ2, false>(acc, a, wt + kOffF2, kPartH, kT, lane, wave, [&](int jj, int s) {
    return x_s + (grp * kP1 + (wave + 4 * jj + s / 3) * kE1 + col + s % 3) * kRec;
  });
  f32x4 w3[kSrOut][2];
#pragma unroll
  for (int k = 0; k < kSrOut; ++k)
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) w3[k][mt] = *(const f32x4 *)(wt + kOffW3 + k * kC + 16 * mt + 4 * grp);
  const int kout = min(grp, kSrOut - 1);
  const float b3 = wt[kOffB3 + kout];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    float y[kSrOut];
#pragma unroll
    for (int k = 0; k < kSrOut; ++k) {
      float p = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p = fmaf(w3[k][0][i], fmaxf(acc[jj][0][i], 0.0f), p);
        p = fmaf(w3[k][1][i], fmaxf(acc[jj][1][i], 0.0f), p);
      }
      p += __shfl_xor(p, 16);
      p += __shfl_xor(p, 32);
      y[k] = p;
    }
    // lanes of group k < 3 write output channel k of pixel col
    const int ty = wave + 4 * jj, Y = oy0 + ty, X = ox0 + col;
    if (grp < kSrOut && Y < H && X < W) {
      const float yk = grp == 0 ? y[0] : (grp == 1 ? y[1] : y[2]);
      out[(int64_t)f * kSrOut * plane_hi + kout * plane_hi + (int64_t)Y * W + X] =
          up_s[kout * kE2 + (ty + 2) * kE0 + col + 2] + b3 + yk;
    }
  }
}

// The backward's recompute: relu(z1) and relu(z2) of the tile's own pixels to
// a1_out, a2_out [n][32][2h][2w], on the fp32 matrix cores (16x16x4), K
// tap-major (k = tap * C + channel): each 4-wide K step reads four channels of
// one tap, an LDS address per lane that is a constant offset from a per-tile
// base, and each wave's weights stay in registers.
__global__ __launch_bounds__(kThreads, 2) void sr_recompute_kernel(
    const float *__restrict__ wt, const float *__restrict__ lowres,
    const float *__restrict__ gbuf, int h, int w, float *__restrict__ a1_out,
    float *__restrict__ a2_out) {
  __shared__ float in_s[kInP * kE0 * kE0];   // 32.0 KB
  __shared__ float a1_s[kC * kA1Stride];     // 43.0 KB

  const int H = 2 * h, W = 2 * w;
  const int f = blockIdx.z;
  const int oy0 = blockIdx.y * kT, ox0 = blockIdx.x * kT;
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const int col = lane % 16, grp = lane / 16;
  const int64_t plane_lo = (int64_t)h * w, plane_hi = (int64_t)H * W;
  const float *lo_f = lowres + (int64_t)f * 3 * plane_lo;
  const float *g_f = gbuf + (int64_t)f * (kIn - 3) * plane_hi;

  // stage 0: the input over the tile and a two-pixel halo (zero outside the
  // image and in the three padding channels)
  {
    constexpr int E2 = kE2;
    auto inside = [&](int e) {
      const int Y = oy0 - 2 + (e / kE0) % kE0, X = ox0 - 2 + e % kE0;
      return Y >= 0 && Y < H && X >= 0 && X < W;
    };
    auto pix = [&](int e) {
      return (int64_t)(oy0 - 2 + (e / kE0) % kE0) * W + ox0 - 2 + e % kE0;
    };
    // the 14 G-buffer channels, the upsampled render, the padding channels
    const rsrc_t rg = make_rsrc(g_f, 4 * (kIn - 3) * plane_hi);
    stage<(kIn - 3) * E2>(
        tid, rg,
        [&](int e) {
          return inside(e) ? (uint32_t)(4 * ((e / E2) * plane_hi + pix(e))) : kOutside;
        },
        [&](int e) { return in_s + 3 * E2 + e; });
    stage_up<kE0>(tid, make_rsrc(lo_f, 4 * 3 * plane_lo), h, w, oy0 - 2, ox0 - 2, in_s);
    for (int e = tid; e < (kInP - kIn) * E2; e += kThreads) in_s[kIn * E2 + e] = 0.0f;
  }

  // stage 1: conv1 + ReLU over the tile and a one-pixel halo
  {
    float a[kS1][2];
#pragma unroll
    for (int s = 0; s < kS1; ++s) {
      a[s][0] = wt[(2 * s) * 64 + lane];
      a[s][1] = wt[(2 * s + 1) * 64 + lane];
    }
    float bias[2][4];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) bias[mt][i] = wt[kOffB1 + 16 * mt + 4 * grp + i];
    __syncthreads();
    for (int j = wave; j < kN1; j += kThreads / 64) {
      const int q = 16 * j + col;
      const int qq = min(q, kP1 - 1);  // the 12 columns past the last position are discarded
      const float *src = in_s + grp * kE0 * kE0 + (qq / kE1) * kE0 + qq % kE1;
      f32x4 acc0 = {0.0f, 0.0f, 0.0f, 0.0f}, acc1 = acc0;
#pragma unroll
      for (int s = 0; s < kS1; ++s) {
        const int tap = s / (kInP / 4), c4 = 4 * (s % (kInP / 4));
        const float b = src[c4 * kE0 * kE0 + (tap / 3) * kE0 + tap % 3];
        acc0 = mfma4(a[s][0], b, acc0);
        acc1 = mfma4(a[s][1], b, acc1);
      }
      if (q < kP1) {
        const int Y = oy0 - 1 + q / kE1, X = ox0 - 1 + q % kE1;
        const bool inside = Y >= 0 && Y < H && X >= 0 && X < W;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a1_s[(4 * grp + i) * kA1Stride + q] = inside ? fmaxf(acc0[i] + bias[0][i], 0.0f) : 0.0f;
          a1_s[(16 + 4 * grp + i) * kA1Stride + q] =
              inside ? fmaxf(acc1[i] + bias[1][i], 0.0f) : 0.0f;
        }
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < kC * kT * kT; e += kThreads) {
    const int o = e / (kT * kT), p = e % (kT * kT);
    const int Y = oy0 + p / kT, X = ox0 + p % kT;
    if (Y < H && X < W)
      a1_out[((int64_t)f * kC + o) * plane_hi + (int64_t)Y * W + X] =
          a1_s[o * kA1Stride + (p / kT + 1) * kE1 + p % kT + 1];
  }

  // stage 2: conv2 + ReLU, one row per column tile
  float a[kS2][2];
#pragma unroll
  for (int s = 0; s < kS2; ++s) {
    a[s][0] = wt[kOffA2 + (2 * s) * 64 + lane];
    a[s][1] = wt[kOffA2 + (2 * s + 1) * 64 + lane];
  }
  float bias[2][4];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) bias[mt][i] = wt[kOffB2 + 16 * mt + 4 * grp + i];
  for (int ty = wave; ty < kT; ty += kThreads / 64) {
    const float *src = a1_s + grp * kA1Stride + ty * kE1 + col;
    f32x4 acc0 = {0.0f, 0.0f, 0.0f, 0.0f}, acc1 = acc0;
#pragma unroll
    for (int s = 0; s < kS2; ++s) {
      const int tap = s / (kC / 4), c4 = 4 * (s % (kC / 4));
      const float b = src[c4 * kA1Stride + (tap / 3) * kE1 + tap % 3];
      acc0 = mfma4(a[s][0], b, acc0);
      acc1 = mfma4(a[s][1], b, acc1);
    }
    const int Y = oy0 + ty, X = ox0 + col;
    if (Y < H && X < W) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float *dst = a2_out + ((int64_t)f * kC + 4 * grp + i) * plane_hi + (int64_t)Y * W + X;
        dst[0] = fmaxf(acc0[i] + bias[0][i], 0.0f);
        dst[16 * plane_hi] = fmaxf(acc1[i] + bias[1][i], 0.0f);
      }
    }
  }
}

// ---------------------------------------------------------------- backward
// The weight gradient of sum(dy * out), after a recompute of the forward that
// saves a1 = relu(z1) and a2 = relu(z2) (the masks z > 0 are a > 0):
//   dz2 = [a2 > 0] W3^T dy                       per pixel
//   dz1 = [a1 > 0] (conv2's transpose of dz2)    per pixel, 3x3 neighbourhood
//   dW3 = sum dy a2^T, dW2 = sum dz2 (a1 window)^T, dW1 = sum dz1 (x window)^T
// per persistent workgroup into one row of fp32 partials, then fp32 sums of
// those rows, in groups and then over the groups, each in a fixed order
// (deterministic).  dz2 is made where it is used, from a2 and dy (its own
// kernel took 44 us of a 16 x 128^2 call and 134 MB).  The transposed conv runs
// with split operands on the bf16 matrix cores, the conv weight gradients on
// the fp32 ones: their operands are shifted windows of pixels, which bf16
// fragments of eight neighbours cannot start at any pixel.

// dz2 of one pixel and channel o: [a2 > 0] (W3^T dy)[o].
__device__ __forceinline__ float dz2_of(const float *w3, int o, float a2, float d0, float d1,
                                        float d2) {
  const float g = fmaf(w3[o], d0, fmaf(w3[kC + o], d1, w3[2 * kC + o] * d2));
  return a2 > 0.0f ? g : 0.0f;
}

// dz1[c][Y][X] = [a1 > 0] sum_o sum_tap W2[o][c][tap] dz2[o][Y + 1 - ty][X + 1 - tx]:
// a zero-padded 3x3 correlation of dz2 with conv2's transpose (taps mirrored),
// on the matrix cores exactly as the forward's conv2: dz2 over the tile and a
// one-pixel halo, made from a2 and dy while it is staged, split, in LDS.
// What bounds it: 440 MB of a2, a1 and dz1 for 16 x 128^2, read and written in
// step with the matrix-core work (27% of its 182 us; 260 us on the fp32
// instruction, plus dz2's kernel).
__global__ __launch_bounds__(kThreads, 2) void sr_bwd_dz1_kernel(
    const float *__restrict__ wt, const float *__restrict__ dy, const float *__restrict__ a2,
    const float *__restrict__ a1, float *__restrict__ dz1, int H, int W) {
  __shared__ __attribute__((aligned(16))) uint8_t d_s[3 * kPartH];   // 60.8 KB
  const int f = blockIdx.z, oy0 = blockIdx.y * kT, ox0 = blockIdx.x * kT;
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int col = lane % 16, grp = lane / 16;
  const int64_t plane = (int64_t)H * W;
  const uint32_t pl = 4 * (uint32_t)plane;
  // a tile's dz1 is computed with the sign of its place, and each K-step of the
  // conv is summed by itself (FRESH): the bf16 instruction rounds its sums
  // towards minus infinity, by a fraction of an ulp that a gradient's sum over the
  // pixels would collect (3e-6 over 2^16 of them; 3e-7 as it is)
  const float sign =
      f32::sign_of(blockIdx.x) * f32::sign_of(blockIdx.y) * f32::sign_of(blockIdx.z);
  ConvWeights a;
  conv_first(a, wt + kOffF2T, lane);
  // a1 at the lane's outputs, requested ahead of the rest
  float m[4][2][4];
  const rsrc_t r1 = make_rsrc(a1 + (int64_t)f * kC * plane, 4 * kC * plane);
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const int Y = oy0 + wave + 4 * jj, X = ox0 + col;
    const uint32_t px = Y < H && X < W ? 4 * (4 * grp * (uint32_t)plane + (uint32_t)Y * W + X) : kOutside;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) m[jj][mt][i] = load1(r1, px, (16 * mt + i) * pl);
  }
  {
    // a wave takes 8 channels of all positions, its w3 in scalar registers
    constexpr int kIt = (kP1 + 63) / 64, kG = 3;   // 6 rounds, 3 in flight
    const rsrc_t ra = make_rsrc(a2 + ((int64_t)f * kC + 8 * wave) * plane, 4 * 8 * plane);
    const rsrc_t rd = make_rsrc(dy + (int64_t)f * kSrOut * plane, 4 * kSrOut * plane);
    const float *w3 = wt + kOffW3 + 8 * wave;
    static_assert(kIt % kG == 0, "whole groups");
    for (int i0 = 0; i0 < kIt; i0 += kG) {
      float v[kG][8], d[kG][3];
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        const int q = lane + 64 * (i0 + j), Y = oy0 - 1 + q / kE1, X = ox0 - 1 + q % kE1;
        const bool ok = q < kP1 && Y >= 0 && Y < H && X >= 0 && X < W;
        const uint32_t px = ok ? 4 * ((uint32_t)Y * W + X) : kOutside;
#pragma unroll
        for (int c = 0; c < 8; ++c) v[j][c] = load1(ra, px, c * pl);
#pragma unroll
        for (int c = 0; c < kSrOut; ++c) d[j][c] = load1(rd, px, c * pl);
      }
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        const int q = lane + 64 * (i0 + j);
#pragma unroll
        for (int c = 0; c < 8; ++c)
          v[j][c] = sign * dz2_of(w3, c, v[j][c], d[j][0], d[j][1], d[j][2]);
        if (q < kP1) store_split(d_s + (wave * kP1 + q) * kRec, kPartH, f32::split8(v[j]));
      }
    }
  }
  __syncthreads();
  f32x4 acc[4][2];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) acc[jj][0] = acc[jj][1] = f32::zero4();
  conv_split<4, kQ2, true>(acc, a, wt + kOffF2T, kPartH, kT, lane, wave, [&](int jj, int s) {
    return d_s + (grp * kP1 + (wave + 4 * jj + s / 3) * kE1 + col + s % 3) * kRec;
  });
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const int Y = oy0 + wave + 4 * jj, X = ox0 + col;
    if (Y >= H || X >= W) continue;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dz1[((int64_t)f * kC + 16 * mt + 4 * grp + i) * plane + (int64_t)Y * W + X] =
            m[jj][mt][i] > 0.0f ? sign * acc[jj][mt][i] : 0.0f;
  }
}

// Per-tile partial sums of every weight's gradient, in the packed order.
// The two conv gradients are GEMMs over the tile's 256 pixels on the matrix
// cores: dW[o][(c, tap)] = sum_p dz[o][p] act[c][p + tap], with dz (32 x 256)
// as the 16-row operand, held in registers, and the activation windows
// (columns (c, tap) in packed order, c * 9 + tap) gathered from LDS.  One
// more column reads a plane of ones: its sums are the bias gradients
// sum_p dz[o][p].
constexpr int kDzStride = kT * kT + 4;   // LDS row of dz: rows land in distinct banks
// floats: dz rows, the activation windows, the plane of ones (two workgroups per CU)
constexpr int kWgLds = kC * kDzStride + kC * kP1 + kP1;

// dz_s rows (32 x 256, stride kDzStride) against the windows of act_s
// (channels of kP1 floats, the tile plus a one-pixel halo) and, as column
// ncol, against ones_s, added to acc: column tile j = wave + 4 jj of 16.
template <int NJ>
__device__ __forceinline__ void wgrad_gemm(const float *dz_s, const float *act_s,
                                           const float *ones_s, int ncol, f32x4 (&acc)[NJ][2],
                                           int lane, int wave) {
  const int col = lane % 16, grp = lane / 16;
  // the wave's column tiles; a tile past the last column repeats the ones
  // column (its sums are never stored)
  const float *src[NJ];
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) {
    const int n = min(16 * (wave + (kThreads / 64) * jj) + col, ncol);
    const int c = n / 9, tap = n % 9;
    src[jj] = n == ncol ? ones_s + grp : act_s + c * kP1 + (tap / 3) * kE1 + tap % 3 + grp;
  }
#pragma unroll 4
  for (int s = 0; s < kT * kT / 4; ++s) {
    // pixel p = 4 s + grp: row s / 4, column 4 (s % 4) + grp
    const float a0 = dz_s[col * kDzStride + 4 * s + grp];
    const float a1 = dz_s[(16 + col) * kDzStride + 4 * s + grp];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      const float b = src[jj][(s / 4) * kE1 + 4 * (s % 4)];
      acc[jj][0] = mfma4(a0, b, acc[jj][0]);
      acc[jj][1] = mfma4(a1, b, acc[jj][1]);
    }
  }
}

// Column n < ncol to out[row * ncol + n], the ones column to bias[row].
template <int NJ>
__device__ __forceinline__ void wgrad_store(const f32x4 (&acc)[NJ][2], int ncol,
                                            float *__restrict__ out, float *__restrict__ bias,
                                            int lane, int wave) {
  const int col = lane % 16, grp = lane / 16;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) {
    const int n = 16 * (wave + (kThreads / 64) * jj) + col;
    if (n > ncol) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float *d0 = n < ncol ? out + (4 * grp + i) * ncol + n : bias + 4 * grp + i;
      float *d1 = n < ncol ? out + (16 + 4 * grp + i) * ncol + n : bias + 16 + 4 * grp + i;
      *d0 = acc[jj][0][i];
      *d1 = acc[jj][1][i];
    }
  }
}

constexpr int kNJ2 = (kC * 9 / 16 + 1 + 3) / 4;    // conv2 column tiles (19) per wave (5)
constexpr int kNJ1 = (kIn * 9 + 1 + 15) / 16;      // conv1 column tiles (10)
constexpr int kNJ1w = (kNJ1 + 3) / 4;              // per wave (3)
static_assert((kC * 9 + 1 + 15) / 16 <= 4 * kNJ2, "conv2 columns and the ones column");

// A tile's planes by way of registers: C channels at the thread's own pixel, or
// over the tile and a one-pixel halo, position tid and then the 68 positions
// past kThreads, channel by channel.  tile: first row and column.
constexpr int kPast = kP1 - kThreads;
constexpr int halo_loads(int C) { return C + (C * kPast + kThreads - 1) / kThreads; }

struct TilePos {
  int f, y0, x0;
};

__device__ __forceinline__ uint32_t image_offset(int Y, int X, int H, int W) {
  return Y >= 0 && Y < H && X >= 0 && X < W ? 4 * ((uint32_t)Y * W + X) : kOutside;
}

template <int C>
__device__ __forceinline__ void fetch_own(float (&v)[C], rsrc_t r, TilePos t, int tid, int H, int W) {
  const uint32_t px = image_offset(t.y0 + tid / kT, t.x0 + tid % kT, H, W), pl = 4 * (uint32_t)(H * W);
#pragma unroll
  for (int c = 0; c < C; ++c) v[c] = load1(r, px, c * pl);
}

template <int C>
__device__ __forceinline__ void fetch_halo(float (&v)[halo_loads(C)], rsrc_t r, TilePos t, int tid,
                                           int H, int W) {
  auto at = [&](int q) { return image_offset(t.y0 - 1 + q / kE1, t.x0 - 1 + q % kE1, H, W); };
  const uint32_t px = at(tid), pl = 4 * (uint32_t)(H * W);
#pragma unroll
  for (int c = 0; c < C; ++c) v[c] = load1(r, px, c * pl);
#pragma unroll
  for (int i = C; i < halo_loads(C); ++i) {
    const int e = tid + (i - C) * kThreads;
    const uint32_t o = at(kThreads + e % kPast);
    v[i] = load1(r, e < C * kPast && o != kOutside ? o + e / kPast * pl : kOutside, 0);
  }
}

template <int C>
__device__ __forceinline__ void put_halo(float *dst, const float (&v)[halo_loads(C)], int tid) {
#pragma unroll
  for (int c = 0; c < C; ++c) dst[c * kP1 + tid] = v[c];
#pragma unroll
  for (int i = C; i < halo_loads(C); ++i) {
    const int e = tid + (i - C) * kThreads;
    if (e < C * kPast) dst[e / kPast * kP1 + kThreads + e % kPast] = v[i];
  }
}

// Persistent: workgroup b takes tiles b, b + gridDim.x, ... (in that order)
// and keeps its running sums of every weight gradient in registers, written
// once to partial[b].  Each phase's planes are requested a phase ahead.
//
// What bounds it: the fp32 matrix instruction (549k of 970k cycles at 16 x
// 128^2), in phases that the two workgroups of a CU overlap in part.  404 us; 441
// with each phase's planes staged between barriers, element by element.
__global__ __launch_bounds__(kThreads, 2) void sr_bwd_wgrad_kernel(
    const float *__restrict__ lowres, const float *__restrict__ gbuf, const float *__restrict__ dy,
    const float *__restrict__ a1, const float *__restrict__ a2, const float *__restrict__ dz1,
    const float *__restrict__ w3, float *__restrict__ partial, int n, int h, int w) {
  __shared__ float buf[kWgLds];   // 76.1 KB
  const int H = 2 * h, W = 2 * w;
  const int tx_n = (W + kT - 1) / kT, ty_n = (H + kT - 1) / kT;
  const int ntiles = n * tx_n * ty_n;
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int col = lane % 16, grp = lane / 16;
  const int64_t plane = (int64_t)H * W, plane_lo = (int64_t)h * w;
  const int64_t fb = 4 * kC * plane;   // bytes of one frame's 32 planes
  constexpr int kOffW2 = kC * kIn * 9 + kC, kOffB2p = kOffW2 + kC * kC * 9;
  constexpr int kOffW3p = kOffB2p + kC, kOffB3p = kOffW3p + kSrOut * kC;
  constexpr int P = kT * kT, kG = kIn - 3;
  static_assert(P == kThreads, "a thread per pixel");
  f32x4 acc2[kNJ2][2] = {}, acc1[kNJ1w][2] = {};
  // the head on waves 0..2: column tile `wave` of [a2^T | 1] against dy
  f32x4 acc_h = {0.f, 0.f, 0.f, 0.f};
  float *dz_s = buf, *act_s = buf + kC * kDzStride, *ones_s = buf + kC * kDzStride + kC * kP1;
  for (int e = tid; e < kP1; e += kThreads) ones_s[e] = 1.0f;
  auto tile_pos = [&](int t) {
    return TilePos{t / (tx_n * ty_n), ((t / tx_n) % ty_n) * kT, (t % tx_n) * kT};
  };
  float v2[kC], vy[kSrOut];            // a2 and dy at the thread's pixel
  auto fetch_head = [&](TilePos tp, int tid) {
    fetch_own<kC>(v2, make_rsrc(a2 + (int64_t)tp.f * kC * plane, fb), tp, tid, H, W);
    fetch_own<kSrOut>(vy, make_rsrc(dy + (int64_t)tp.f * kSrOut * plane, 4 * kSrOut * plane), tp,
                      tid, H, W);
  };
  fetch_head(tile_pos(blockIdx.x), tid);
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const TilePos tp = tile_pos(t);
    // opaque per tile: what derives from the thread's index would otherwise be
    // hoisted and take the registers
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid % 64, col = lane % 16, grp = lane / 16;
    // phase 0: the head, dW3[k][o] = sum_p dy[k][p] a2[o][p] and b3[k] =
    // sum_p dy[k][p] on the matrix cores: dy (3 rows of 16) the row operand,
    // [a2^T | 1] (33 of 48 columns) the column operand, over the tile's own
    // pixels (zero outside the image).  a2 [32][256] in dz_s, which becomes dz2
    // there, dy_s [3][256] in the activations' place.
    float *dy_s = act_s;
    float va[halo_loads(kC)];
    fetch_halo<kC>(va, make_rsrc(a1 + (int64_t)tp.f * kC * plane, fb), tp, tid, H, W);
#pragma unroll
    for (int o = 0; o < kC; ++o) dz_s[o * kDzStride + tid] = v2[o];
#pragma unroll
    for (int k = 0; k < kSrOut; ++k) dy_s[k * P + tid] = vy[k];
    __syncthreads();
    if (wave < 3) {
      const int nc = 16 * wave + col;            // column: a2 channel, 32 = ones
#pragma unroll 8
      for (int s = 0; s < P / 4; ++s) {
        const int p = 4 * s + grp;
        const float av = col < kSrOut ? dy_s[col * P + p] : 0.0f;
        const float bv = nc < kC ? dz_s[nc * kDzStride + p] : (nc == kC ? 1.0f : 0.0f);
        acc_h = mfma4(av, bv, acc_h);
      }
    }
    __syncthreads();
    // phase A: conv2.  dz_s [32][256] = dz2 over the tile's own pixels and
    // act_s [32][18][18] = a1 over the tile and a one-pixel halo; zero
    // outside the image.
#pragma unroll
    for (int o = 0; o < kC; ++o) dz_s[o * kDzStride + tid] = dz2_of(w3, o, v2[o], vy[0], vy[1], vy[2]);
    put_halo<kC>(act_s, va, tid);
    __syncthreads();
    float vd[kC], vx[halo_loads(kG)];
    fetch_own<kC>(vd, make_rsrc(dz1 + (int64_t)tp.f * kC * plane, fb), tp, tid, H, W);
    fetch_halo<kG>(vx, make_rsrc(gbuf + (int64_t)tp.f * kG * plane, 4 * kG * plane), tp, tid, H, W);
    __builtin_amdgcn_sched_barrier(0);
    wgrad_gemm<kNJ2>(dz_s, act_s, ones_s, kC * 9, acc2, lane, wave);
    __syncthreads();
    // phase B: conv1.  dz_s = dz1 over the tile's own pixels, x_s
    // [17][18][18] = the input over the tile and a one-pixel halo.
    float *x_s = act_s;
#pragma unroll
    for (int o = 0; o < kC; ++o) dz_s[o * kDzStride + tid] = vd[o];
    put_halo<kG>(x_s + 3 * kP1, vx, tid);
    stage_up<kE1>(tid, make_rsrc(lowres + (int64_t)tp.f * 3 * plane_lo, 4 * 3 * plane_lo), h, w,
                  tp.y0 - 1, tp.x0 - 1, x_s);
    __syncthreads();
    if (t + (int)gridDim.x < ntiles) fetch_head(tile_pos(t + gridDim.x), tid);
    __builtin_amdgcn_sched_barrier(0);
    wgrad_gemm<kNJ1w>(dz_s, x_s, ones_s, kIn * 9, acc1, lane, wave);
    __syncthreads();
  }
  float *out = partial + (int64_t)blockIdx.x * kSrParams;
  wgrad_store<kNJ2>(acc2, kC * 9, out + kOffW2, out + kOffB2p, lane, wave);
  wgrad_store<kNJ1w>(acc1, kIn * 9, out, out + kC * kIn * 9, lane, wave);
  // head: lane (col, grp) holds rows 4 grp + i (outputs k) of column 16 wave + col
  if (wave < 3 && grp == 0) {
    const int nc = 16 * wave + col;
#pragma unroll
    for (int i = 0; i < kSrOut; ++i) {
      if (nc < kC) out[kOffW3p + i * kC + nc] = acc_h[i];
      else if (nc == kC) out[kOffB3p + i] = acc_h[i];
    }
  }
}

// grad_w[i] = sum over rows of partial[row][i] in fp32, in two fixed-order
// stages (deterministic): groups of kRedGroup consecutive rows, then the
// groups in order.
constexpr int kRedGroup = 64;

__global__ __launch_bounds__(kThreads) void sr_bwd_group_sum_kernel(
    const float *__restrict__ partial, int tiles, float *__restrict__ groups) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= kSrParams) return;
  const int t0 = blockIdx.y * kRedGroup, t1 = min(t0 + kRedGroup, tiles);
  float s = 0.0f;
  for (int t = t0; t < t1; ++t) s += partial[(int64_t)t * kSrParams + i];
  groups[(int64_t)blockIdx.y * kSrParams + i] = s;
}

__global__ __launch_bounds__(kThreads) void sr_bwd_reduce_kernel(const float *__restrict__ groups,
                                                                 int ngroups, float *__restrict__ gw) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= kSrParams) return;
  float s = 0.0f;
  for (int g = 0; g < ngroups; ++g) s += groups[(int64_t)g * kSrParams + i];
  gw[i] = s;
}

}  // namespace

static void launch_relayout(const float *w, float *wt, hipStream_t stream) {
  constexpr int items = kWtFp32 + (kQ1 + 2 * kQ2) * 2 * 64;
  hipLaunchKernelGGL(sr_relayout_kernel, dim3((items + kThreads - 1) / kThreads), dim3(kThreads), 0,
                     stream, w, wt);
}

hipError_t launch_sr_forward(const float *w, float *wt, const float *lowres, const float *gbuf,
                             float *out, int n, int h, int w_lo, hipStream_t stream) {
  launch_relayout(w, wt, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((2 * w_lo + kT - 1) / kT), (unsigned)((2 * h + kT - 1) / kT),
                  (unsigned)n);
  hipLaunchKernelGGL(sr_forward_kernel, grid, dim3(kThreads), 0, stream, wt, lowres, gbuf, out, h,
                     w_lo);
  return hipGetLastError();
}

// Persistent workgroups of the weight-gradient kernel (two per CU).
constexpr int kWgBlocks = 512;

static int64_t wgrad_blocks(int n, int h, int w) {
  const int64_t tiles = (int64_t)n * ((2 * h + kT - 1) / kT) * ((2 * w + kT - 1) / kT);
  return std::min<int64_t>(tiles, kWgBlocks);
}

size_t sr_backward_workspace_bytes(int n, int h, int w) {
  const int64_t px = (int64_t)n * 4 * h * w;
  const int64_t rows = wgrad_blocks(n, h, w);
  const int64_t groups = (rows + kRedGroup - 1) / kRedGroup;
  return sizeof(float) * (size_t)(3 * kC * px + (rows + groups) * kSrParams);
}

hipError_t launch_sr_backward(const float *w, float *wt, const float *lowres, const float *gbuf,
                              const float *dy, float *gw, int n, int h, int w_lo, float *ws,
                              hipStream_t stream) {
  const int H = 2 * h, W = 2 * w_lo;
  const int64_t plane = (int64_t)H * W, px = (int64_t)n * plane;
  float *a1 = ws, *a2 = a1 + kC * px, *dz1 = a2 + kC * px;
  float *partial = dz1 + kC * px;
  launch_relayout(w, wt, stream);
  const dim3 tiles((unsigned)((W + kT - 1) / kT), (unsigned)((H + kT - 1) / kT), (unsigned)n);
  hipLaunchKernelGGL(sr_recompute_kernel, tiles, dim3(kThreads), 0, stream, wt, lowres, gbuf, h,
                     w_lo, a1, a2);
  hipLaunchKernelGGL(sr_bwd_dz1_kernel, tiles, dim3(kThreads), 0, stream, wt, dy, a2, a1, dz1, H, W);
  // persistent workgroups; each writes one row of partial sums
  const int nblocks = (int)wgrad_blocks(n, h, w_lo);
  hipLaunchKernelGGL(sr_bwd_wgrad_kernel, dim3((unsigned)nblocks), dim3(kThreads), 0, stream,
                     lowres, gbuf, dy, a1, a2, dz1, wt + kOffW3, partial, n, h, w_lo);
  const int ngroups = (nblocks + kRedGroup - 1) / kRedGroup;
  // the group sums follow the partials
  float *groups = partial + (int64_t)nblocks * kSrParams;
  const unsigned pblocks = (kSrParams + kThreads - 1) / kThreads;
  hipLaunchKernelGGL(sr_bwd_group_sum_kernel, dim3(pblocks, (unsigned)ngroups), dim3(kThreads), 0,
                     stream, partial, nblocks, groups);
  hipLaunchKernelGGL(sr_bwd_reduce_kernel, dim3(pblocks), dim3(kThreads), 0, stream, groups,
                     ngroups, gw);
  return hipGetLastError();
}

}  // namespace gn
