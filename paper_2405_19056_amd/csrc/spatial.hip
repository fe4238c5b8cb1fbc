// The spatial GlassNet networks (Sec. 3.4): F and B as U-Nets, h and R as
// CNNs whose first layers are 3 x 3 convolutions, on the gfx950 matrix cores
// (bf16 operands, fp32 accumulation).
//
// Reading of the architecture (the paper gives no widths, depths or levels):
//   U-Net (F on [G; s], B on [sigma; tau]): e1 = relu(conv3 x); d = 2 x 2
//     average of e1; m = relu(conv3 d) at half resolution; u = m repeated
//     2 x 2; e2 = relu(conv3 [e1; u]); out = conv1 e2.
//   h(b_i, sigma) = conv1 relu(conv1 relu(conv3 [b_i; sigma])); the pool of
//     Eq. (5) per pixel over the buffers with alpha > 0 there.
//   R = conv1 relu(conv3 relu(conv3 [phi; L_d])) with 3 outputs.
// conv3: 3 x 3, zero padding of one pixel; conv1: 1 x 1; every conv has a
// bias.  Width W (64 or 128) throughout.
//
// Layout.  Activations live in HBM as bf16 [n][H][W][C] (channels innermost,
// C a multiple of 32), so the 8 channels one lane presents to the matrix
// core for one pixel are one 16-byte load.  Every conv is an implicit GEMM,
// Y^T = A X^T: the weights are the A operand (16 output channels per M-tile),
// 16 pixels of one row the B operand, K = (tap, input channel) in 32-deep
// steps; the zero padding is a zero B fragment.  Two inputs can be
// concatenated along the channels, the second optionally at half resolution
// and read through a 2 x 2 nearest upsample (the U-Net's skip join), so the
// concatenation and the upsample are never materialised.
//
// Work split (sp_conv_kernel).  A workgroup of four waves owns a tile of TR
// rows x 16 columns and every output channel.  It stages the tile's inputs and
// a one-pixel halo, all channels, in LDS once (each value is read nine times
// from there, from L2 before), then runs the K loop without a barrier: each
// wave takes half of the output channels of half of the rows, its weight
// fragments straight from L2 into registers several K-steps ahead, its input
// fragments from LDS one step ahead.  Every output is the same sum in the same
// order (tap, then channel block) whatever the tile.
//
// Epilogues, through the LDS the halo has left: bias and ReLU, then a bf16
// store (with the U-Net's 2 x 2 average where that is the next input), an fp32
// store, or the following 1 x 1 convolution (the U-Nets' and R's last ones),
// whose input then never leaves the chip.
//
// h over the buffers, the pool and T's last layer run in one kernel of their
// own (sp_slots_kernel below): the per-buffer activations and the running
// sum stay on the chip.  (The generic table also packs T's layers as
// ordinary convs; only their biases are read from it.)
#include <algorithm>
#include <type_traits>

#include "gn_internal.h"
#include "lds_limit.h"

namespace gn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8, kThreads = kWaves * 64;    // sp_slots_kernel's workgroup

constexpr int kFrag = 1024;                  // one A fragment: 64 lanes x 16 bytes

__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

__device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Input loads go through buffer resources bounded by the input's size: a
// load at an offset past the bound returns zeros (the conv's zero padding),
// so no select on the loaded value holds up the next K-step's loads.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr uint32_t kOutside = 0x80000000u;     // past every bound (inputs stay under 2 GiB)
__device__ __forceinline__ rsrc_t make_rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                           0x00020000);
}
__device__ __forceinline__ u32x4 bld(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

}  // namespace

// One 3 x 3 convolution launch.
struct SpConvArgs {
  const uint8_t *in0;       // bf16 [n][H][W][C0], or null: F's input from the caller's planes
  const uint8_t *in1;       // bf16 [n][H1][W1][C1] (Src: half or full resolution)
  const float *gbuf, *scene;  // planes of F's input or of L_d
  const uint8_t *wfrag;     // A fragments [step][mt][lane] (16 B each)
  const float *bias;        // [MT * 16]
  const uint8_t *wfrag1;    // the following 1 x 1 conv's, its bias
  const float *bias1;
  int n, H, Wd;             // output (= in0) size
  uint8_t *out;             // bf16 [n][H][W][W], or fp32 (E_F32), or the image (E_RGB)
  uint8_t *pool;            // bf16 [n][H/2][W/2][W]: the 2 x 2 average, or null
};

namespace {

// The second source: none, at full resolution, at half resolution through a
// 2 x 2 nearest upsample, or L_d's planes.
enum Src { S_NONE, S_FULL, S_HALF, S_LIGHT };
// ReLU and a bf16 store (and average); an fp32 store; ReLU, then the 1 x 1
// conv to W channels, or to the image.
enum Epi { E_ACT, E_F32, E_CONV1, E_RGB };

constexpr int kConvThreads = 256, kTC = 16, kHW = kTC + 2;   // tile columns, halo columns

// LDS position (bytes) of 16-byte unit u of a pixel with UN units: XORed by
// the pixel so that 16 neighbouring pixels' same unit fills all banks.
template <int UN>
__device__ __forceinline__ uint32_t unit_at(int px, int u) {
  constexpr int kShift = UN >= 16 ? 0 : (UN == 8 ? 1 : 2);
  return (uint32_t)(px * UN + (u ^ ((px >> kShift) & (UN < 16 ? UN - 1 : 15)))) * 16;
}

// A block of bf16 activations [..][C] around (y0, x0), `rows` x `cols` pixels,
// into LDS; pixels outside the frame's H x Wd read zero.
template <int CB, int ROWS, int COLS>
__device__ __forceinline__ void stage_act(uint8_t *dst, const uint8_t *src, int n, int f, int H, int Wd,
                                          int y0, int x0) {
  constexpr int UN = 4 * CB, N = ROWS * COLS * UN, kIt = (N + kConvThreads - 1) / kConvThreads;
  constexpr int kG = kIt < 11 ? kIt : 11;             // loads in flight per thread
  const rsrc_t rs = make_rsrc(src, (uint32_t)((int64_t)n * H * Wd * CB * 64));
#pragma unroll
  for (int i0 = 0; i0 < kIt; i0 += kG) {
    u32x4 v[kG];
#pragma unroll
    for (int j = 0; j < kG; ++j) {
      const int e = min((int)threadIdx.x + (i0 + j) * kConvThreads, N - 1), px = e / UN, u = e % UN;
      const int y = y0 + px / COLS, x = x0 + px % COLS;
      const bool ok = y >= 0 && y < H && x >= 0 && x < Wd;
      if (i0 + j < kIt)
        v[j] = bld(rs, ok ? (uint32_t)((((int64_t)f * H + y) * Wd + x) * (CB * 64) + u * 16) : kOutside);
    }
#pragma unroll
    for (int j = 0; j < kG; ++j) {
      const int e = (int)threadIdx.x + (i0 + j) * kConvThreads, px = e / UN, u = e % UN;
      if (i0 + j < kIt && e < N) *(u32x4 *)(dst + unit_at<UN>(px, u)) = v[j];
    }
  }
}

// The same for 32-channel blocks made from the caller's planes: F's input
// [G 0..13; scene 0..15; 0, 0], or L_d (G 11..13) and zeros.
template <bool LIGHT, int ROWS>
__device__ __forceinline__ void stage_planes(uint8_t *dst, const float *gbuf, const float *scene,
                                             int f, int H, int Wd, int y0, int x0) {
  const int64_t hw = (int64_t)H * Wd;
  for (int px = threadIdx.x; px < ROWS * kHW; px += kConvThreads) {
    const int y = y0 + px / kHW, x = x0 + px % kHW;
    const bool ok = y >= 0 && y < H && x >= 0 && x < Wd;
    float c[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) c[j] = 0.0f;
    if (ok) {
      const float *G = gbuf + (int64_t)f * kNG * hw + (int64_t)y * Wd + x;
      if constexpr (LIGHT) {
#pragma unroll
        for (int j = 0; j < 3; ++j) c[j] = G[(11 + j) * hw];
      } else {
#pragma unroll
        for (int j = 0; j < kNG; ++j) c[j] = G[j * hw];
#pragma unroll
        for (int j = 0; j < kNS; ++j) c[kNG + j] = scene[(int64_t)f * kNS + j];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      *(u32x4 *)(dst + unit_at<4>(px, u)) =
          u32x4{pk_bf16(c[8 * u], c[8 * u + 1]), pk_bf16(c[8 * u + 2], c[8 * u + 3]),
                pk_bf16(c[8 * u + 4], c[8 * u + 5]), pk_bf16(c[8 * u + 6], c[8 * u + 7])};
  }
}

// LDS bytes of a tile: the two sources' halos, or the tile itself afterwards.
template <int MT, int TR, int CB0, int SRC1, int CB1>
struct ConvLds {
  static constexpr int k0 = (TR + 2) * kHW * CB0 * 64;
  static constexpr int k1 = SRC1 == S_NONE   ? 0
                            : SRC1 == S_HALF ? (TR / 2 + 2) * (kTC / 2 + 2) * CB1 * 64
                                             : (TR + 2) * kHW * CB1 * 64;
  static constexpr int kTile = TR * kTC * MT * 32;
  static constexpr int kBytes = k0 + k1 > kTile ? k0 + k1 : kTile;
};

// MT: output channels / 16; CB0, CB1: 32-channel blocks of the sources; PLANES:
// the first source is F's input, made from the planes.
//
// What bounds it: at W = 128 and 8 rows a wave's K-step is 16 MFMAs (256
// cycles) for 4 KiB of LDS reads and 4 KiB of weights, 64 bytes of each per
// cycle and CU: half the LDS rate, the whole of L1's.  Two workgroups share a
// CU (one, in B's first layer at W = 128: 90 KiB of LDS); a 256^2 frame is one
// round of them, so a launch's halo loads and epilogues (about half of its 19 us)
// overlap little.  256^2, W -> W: 19-24 us against 35-40 with inputs read nine
// times through L2; the whole forward (K = 4) 258 us against 470.
template <int MT, int TR, int CB0, int SRC1, int CB1, bool PLANES, int EPI>
__global__ __launch_bounds__(kConvThreads, 2) void sp_conv_kernel(SpConvArgs a) {
  constexpr int MW = MT / 2, NT = TR / 2;               // a wave's tiles
  constexpr int kCbt = CB0 + CB1, kSteps = 9 * kCbt;
  constexpr int kAhead = TR == 8 ? 4 : 6;   // K-steps of weights in flight
  constexpr int kWUn = MT * 2;                          // 16-byte units of an output pixel
  using LD = ConvLds<MT, TR, CB0, SRC1, CB1>;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  uint8_t *L0 = lds, *L1 = lds + LD::k0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, col = lane & 15, wm = wave & 1, wn = wave >> 1;
  const int H = a.H, Wd = a.Wd;
  const int tx_n = (Wd + kTC - 1) / kTC, ty_n = (H + TR - 1) / TR;
  // Workgroups reach the 8 XCDs round-robin: give each XCD a contiguous run
  // of tiles, so that neighbours' halos are mostly in its own L2.
  const int full = gridDim.x & ~7;
  const int tile = (int)blockIdx.x < full ? (blockIdx.x & 7) * (full >> 3) + (blockIdx.x >> 3)
                                          : (int)blockIdx.x;
  const int f = tile / (tx_n * ty_n), rem = tile - f * (tx_n * ty_n);
  const int y0 = rem / tx_n * TR, x0 = rem % tx_n * kTC;

  // weight fragments of step s, this wave's half of the rows
  const rsrc_t rw = make_rsrc(a.wfrag, (uint32_t)(kSteps * MT * kFrag));
  auto load_a = [&](int s, u32x4 (&w)[MW]) {
#pragma unroll
    for (int m = 0; m < MW; ++m)
      w[m] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                           rw, lane * 16, (s * MT + wm * MW + m) * kFrag, 0));
  };
  u32x4 w[kAhead][MW];
#pragma unroll
  for (int s = 0; s < kAhead; ++s) load_a(s, w[s]);

  if constexpr (PLANES) stage_planes<false, TR + 2>(L0, a.gbuf, a.scene, f, H, Wd, y0 - 1, x0 - 1);
  else stage_act<CB0, TR + 2, kHW>(L0, a.in0, a.n, f, H, Wd, y0 - 1, x0 - 1);
  if constexpr (SRC1 == S_FULL) stage_act<CB1, TR + 2, kHW>(L1, a.in1, a.n, f, H, Wd, y0 - 1, x0 - 1);
  if constexpr (SRC1 == S_HALF)
    stage_act<CB1, TR / 2 + 2, kTC / 2 + 2>(L1, a.in1, a.n, f, H / 2, Wd / 2, y0 / 2 - 1, x0 / 2 - 1);
  if constexpr (SRC1 == S_LIGHT)
    stage_planes<true, TR + 2>(L1, a.gbuf, nullptr, f, H, Wd, y0 - 1, x0 - 1);
  __syncthreads();

  // B fragments of step i of tap row dy (column i / kCbt, channel block i % kCbt)
  auto load_b = [&](int dy, int i, u32x4 (&b)[NT]) {
    const int cb = i % kCbt, dx = i / kCbt;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int r = wn * NT + t + dy, c = col + dx;      // halo coordinates
      if (cb < CB0) {
        b[t] = *(const u32x4 *)(L0 + unit_at<4 * CB0>(r * kHW + c, 4 * cb + g));
      } else if constexpr (SRC1 == S_HALF) {
        // full-resolution row y0 - 1 + r is half-resolution row (r + 1) / 2 of the block
        const int h = ((r + 1) >> 1) * (kTC / 2 + 2) + ((c + 1) >> 1);
        b[t] = *(const u32x4 *)(L1 + unit_at<4 * CB1>(h, 4 * (cb - CB0) + g));
      } else if constexpr (SRC1 != S_NONE) {
        b[t] = *(const u32x4 *)(L1 + unit_at<4 * CB1>(r * kHW + c, 4 * (cb - CB0) + g));
      }
    }
  };
  f32x4 acc[NT][MW];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MW; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  // one tap row: kRow steps, straight-line; the rows are a loop where all
  // three would be too much code
  constexpr int kRow = 3 * kCbt;
  u32x4 b[2][NT];
  load_b(0, 0, b[0]);
  auto tap_row = [&](int dy, auto base) {
    constexpr int s0 = base;                     // its first step, as far as the buffers go
#pragma unroll
    for (int i = 0; i < kRow; ++i) {
      const int q = s0 + i;
      if (i + 1 < kRow) load_b(dy, i + 1, b[(q + 1) & 1]);
      else load_b(min(dy + 1, 2), 0, b[(q + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t][m] = mma(w[q % kAhead][m], b[q & 1][t], acc[t][m]);
      __builtin_amdgcn_sched_barrier(0);
      load_a(min(dy * kRow + i + kAhead, kSteps - 1), w[q % kAhead]);   // past the last: re-read
    }
  };
  if constexpr (kSteps <= 45) {
    tap_row(0, std::integral_constant<int, 0>());
    tap_row(1, std::integral_constant<int, kRow>());
    tap_row(2, std::integral_constant<int, 2 * kRow>());
  } else {
    static_assert(kSteps <= 45 || (kRow % kAhead == 0 && kRow % 2 == 0), "buffers repeat every tap row");
#pragma unroll 1
    for (int dy = 0; dy < 3; ++dy) tap_row(dy, std::integral_constant<int, 0>());
  }

  // ---- epilogue: lane (g, col) holds output channels 16 mt + 4 g + j of its pixel
  auto value = [&](const f32x4 (&ac)[MW], const float *bias, int m, bool relu) {
    f32x4 v = ac[m] + *(const f32x4 *)(bias + 16 * (wm * MW + m) + 4 * g);
    if (relu) {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = fmaxf(v[j], 0.0f);
    }
    return v;
  };
  if constexpr (EPI == E_F32) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int y = y0 + wn * NT + t, x = x0 + col;
      if (y >= H || x >= Wd) continue;
      float *o = (float *)a.out + (((int64_t)f * H + y) * Wd + x) * (MT * 16) + 4 * g;
#pragma unroll
      for (int m = 0; m < MW; ++m) *(f32x4 *)(o + 16 * (wm * MW + m)) = value(acc[t], a.bias, m, false);
    }
    return;
  }
  // the tile as bf16 [row][column][channel] in the LDS the halo has left
  auto put = [&](const f32x4 (&ac)[NT][MW], const float *bias, bool relu) {
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int m = 0; m < MW; ++m) {
        const f32x4 v = value(ac[t], bias, m, relu);
        const int px = (wn * NT + t) * kTC + col, u = 2 * (wm * MW + m) + (g >> 1);
        *(uint2 *)(lds + unit_at<kWUn>(px, u) + 8 * (g & 1)) =
            uint2{pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3])};
      }
    __syncthreads();
  };
  put(acc, a.bias, true);
  if constexpr (EPI == E_CONV1) {
    // the 1 x 1 conv on the tile: K-step cb is channel block cb
    const rsrc_t r1 = make_rsrc(a.wfrag1, (uint32_t)(MT / 2 * MT * kFrag));
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int m = 0; m < MW; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int cb = 0; cb < MT / 2; ++cb) {
      u32x4 w1[MW], b1[NT];
#pragma unroll
      for (int m = 0; m < MW; ++m)
        w1[m] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                              r1, lane * 16, (cb * MT + wm * MW + m) * kFrag, 0));
#pragma unroll
      for (int t = 0; t < NT; ++t)
        b1[t] = *(const u32x4 *)(lds + unit_at<kWUn>((wn * NT + t) * kTC + col, 4 * cb + g));
#pragma unroll
      for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t][m] = mma(w1[m], b1[t], acc[t][m]);
    }
    put(acc, a.bias1, false);
  }
  if constexpr (EPI == E_RGB) {
    // one row tile (3 real outputs); the waves share the tile's rows
    const rsrc_t r1 = make_rsrc(a.wfrag1, (uint32_t)(MT / 2 * kFrag));
    u32x4 w1[MT / 2];
#pragma unroll
    for (int cb = 0; cb < MT / 2; ++cb)
      w1[cb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r1, lane * 16, cb * kFrag, 0));
    for (int r = wave; r < TR; r += 4) {
      f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int cb = 0; cb < MT / 2; ++cb)
        y = mma(w1[cb], *(const u32x4 *)(lds + unit_at<kWUn>(r * kTC + col, 4 * cb + g)), y);
      const int yy = y0 + r, x = x0 + col;
      if (g == 0 && yy < H && x < Wd) {
        const int64_t hw = (int64_t)H * Wd, q = (int64_t)yy * Wd + x;
        float *o = (float *)a.out + (int64_t)f * 3 * hw + q;
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c * hw] = y[c] + a.bias1[c];
      }
    }
    return;
  }
  // bf16 store, 16 bytes per lane of consecutive units
  for (int e = threadIdx.x; e < TR * kTC * kWUn; e += kConvThreads) {
    const int px = e / kWUn, u = e % kWUn, y = y0 + px / kTC, x = x0 + px % kTC;
    if (y < H && x < Wd)
      *(u32x4 *)(a.out + (((int64_t)f * H + y) * Wd + x) * (MT * 32) + u * 16) =
          *(const u32x4 *)(lds + unit_at<kWUn>(px, u));
  }
  if (EPI == E_ACT && a.pool) {
    // the 2 x 2 average of the stored values (H and Wd are even, as are the
    // tile's corners), the sum in fp32
    const int H2 = H >> 1, W2 = Wd >> 1;
    for (int e = threadIdx.x; e < TR / 2 * (kTC / 2) * kWUn; e += kConvThreads) {
      const int p2 = e / kWUn, u = e % kWUn, r = p2 / (kTC / 2), c = p2 % (kTC / 2);
      const int y = y0 / 2 + r, x = x0 / 2 + c;
      if (y >= H2 || x >= W2) continue;
      float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const u32x4 v =
            *(const u32x4 *)(lds + unit_at<kWUn>((2 * r + (q >> 1)) * kTC + 2 * c + (q & 1), u));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          s[2 * j] += __uint_as_float(v[j] << 16);
          s[2 * j + 1] += __uint_as_float(v[j] & 0xFFFF0000u);
        }
      }
      *(u32x4 *)(a.pool + (((int64_t)f * H2 + y) * W2 + x) * (MT * 32) + u * 16) =
          u32x4{pk_bf16(0.25f * s[0], 0.25f * s[1]), pk_bf16(0.25f * s[2], 0.25f * s[3]),
                pk_bf16(0.25f * s[4], 0.25f * s[5]), pk_bf16(0.25f * s[6], 0.25f * s[7])};
    }
  }
}

// ---- h over every buffer, the pool and T's last layer, in one kernel ----------
// With sigma's part u = conv3 sigma + c1 computed once, each buffer i needs
//   z1 = relu(conv3_b b_i + u), z2 = relu(A2 z1 + c2), Z += [alpha_i > 0] z2,
// and after the last buffer tau = A3 (Z / max(c, 1)) + [c > 0] c3 (mean; the
// sum: A3 Z + c c3).  A wave owns 16 pixels of one row and every channel; u
// and Z stay in registers across the buffers and z1 feeds h's second layer
// from registers, so the per-buffer activations never leave the chip.
//
// Weights stay in LDS for the whole kernel (persistent workgroups):
//   conv3_b: 5 K-steps; lane group g of step s presents tap 2 s + (g >> 1)
//     (the tenth tap is zero), channels 8 (g & 1) .. + 7 of the buffer
//     (12 real, 16 packed);
//   A2, A3: W / 32 K-steps in register order: element e of lane group g in
//     step s multiplies channel 32 s + 4 g + e (e < 4) or 32 s + 16 + 4 g +
//     e - 4, which is where M-tiles 2 s and 2 s + 1 of the previous layer's
//     accumulators hold them.
struct SpSlotsArgs {
  const uint8_t *frag;      // conv3_b, A2, A3 fragments, contiguous
  const float *bias;        // c2 then c3, 16 MT floats each
  const uint8_t *bpk;       // bf16 [n][k][H][W][16]: each buffer's 12 channels, zero padded
  const float *layers;      // the caller's buffers (alpha)
  const float *u;           // fp32 [n][H][W][16 MT]
  uint8_t *tau;             // bf16 [n][H][W][16 MT]
  int n, H, Wd, k, mean;
};

constexpr int kSlotSteps1 = 5;               // conv3_b K-steps (9 taps x 16 channels)

template <int MT>
__global__ __launch_bounds__(kThreads) void sp_slots_kernel(SpSlotsArgs a) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int W = 16 * MT, KS = MT / 2;
  constexpr int kBytes = (kSlotSteps1 + 2 * KS) * MT * kFrag;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, col = lane & 15;
  // every fragment, then the biases, into LDS once
  for (int off = wave * kFrag; off < kBytes; off += kWaves * kFrag)
    __builtin_amdgcn_global_load_lds((const void *)(a.frag + off + lane * 16),
                                     (__attribute__((address_space(3))) void *)(lds + off), 16, 0, 0);
  float *lbias = (float *)(lds + kBytes);
  if (threadIdx.x < 2 * W) lbias[threadIdx.x] = a.bias[threadIdx.x];
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const uint8_t *F1 = lds, *F2 = lds + kSlotSteps1 * MT * kFrag, *F3 = F2 + KS * MT * kFrag;

  const int H = a.H, Wd = a.Wd, k = a.k;
  const int64_t hw = (int64_t)H * Wd;
  const int segs = (Wd + 15) >> 4;
  const int64_t nseg = (int64_t)a.n * H * segs;
  const int64_t ntiles = (nseg + kWaves - 1) / kWaves;
  // workgroups reach the 8 XCDs round-robin: each XCD takes a contiguous run
  // of tiles (neighbouring rows share its L2)
  const int per = gridDim.x >> 3, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  for (int64_t base = 0; base < ntiles; base += gridDim.x) {
    const int64_t seg = (base + (int64_t)xcd * per + slot) * kWaves + wave;
    if (seg >= nseg) continue;
    const int f = __builtin_amdgcn_readfirstlane((int)(seg / ((int64_t)H * segs)));
    const int rem = (int)(seg - (int64_t)f * H * segs);
    const int y = __builtin_amdgcn_readfirstlane(rem / segs);
    const int x0 = __builtin_amdgcn_readfirstlane((rem - y * segs) * 16);
    const int x = x0 + col;
    const bool xin = x < Wd;
    const int xc = min(x, Wd - 1);
    const int64_t px = ((int64_t)f * H + y) * Wd + xc;

    f32x4 u[MT], Z[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      u[mt] = *(const f32x4 *)(a.u + px * W + 16 * mt + 4 * g);
      Z[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float cnt = 0.0f;
    // buffer i's conv3 inputs (tap 2 s + (g >> 1); outside the frame the
    // offset is past the plane's bound and the load returns zeros) and its
    // alpha; the next buffer's are loaded while this one's MFMAs run
    auto load_slot = [&](int i, u32x4 (&b)[kSlotSteps1], float &al) {
      const int64_t fb = (int64_t)f * k + i;
      al = a.layers[(fb * kNL + kAlpha) * hw + (int64_t)y * Wd + xc];
      const rsrc_t rb = make_rsrc(a.bpk + fb * hw * 32, (uint32_t)(hw * 32));
#pragma unroll
      for (int s = 0; s < kSlotSteps1; ++s) {
        const int tap = 2 * s + (g >> 1);
        const int yy = y + tap / 3 - 1, xx = x + tap % 3 - 1;
        const bool ok = tap < 9 && yy >= 0 && yy < H && xx >= 0 && xx < Wd;
        b[s] = bld(rb, ok ? (uint32_t)(yy * Wd + xx) * 32 + 16 * (g & 1) : kOutside);
      }
    };
    u32x4 b[kSlotSteps1], bn[kSlotSteps1];
    float al = 0.0f, aln = 0.0f;
    if (k > 0) load_slot(0, b, al);
    for (int i = 0; i < k; ++i) {
      if (i + 1 < k) load_slot(i + 1, bn, aln);
      __builtin_amdgcn_sched_barrier(0);
      const bool act = xin && al > 0.0f;
      if (!__builtin_amdgcn_ballot_w64(act)) {          // adds exactly nothing
#pragma unroll
        for (int s = 0; s < kSlotSteps1; ++s) b[s] = bn[s];
        al = aln;
        continue;
      }
      f32x4 acc[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = u[mt];
#pragma unroll
      for (int s = 0; s < kSlotSteps1; ++s)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt] = mma(*(const u32x4 *)(F1 + (s * MT + mt) * kFrag + lane * 16), b[s], acc[mt]);
      // z1 in register order, then h's second layer
      u32x4 zb[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const f32x4 p = acc[2 * s], q = acc[2 * s + 1];
        zb[s] = u32x4{pk_bf16(fmaxf(p[0], 0.f), fmaxf(p[1], 0.f)),
                      pk_bf16(fmaxf(p[2], 0.f), fmaxf(p[3], 0.f)),
                      pk_bf16(fmaxf(q[0], 0.f), fmaxf(q[1], 0.f)),
                      pk_bf16(fmaxf(q[2], 0.f), fmaxf(q[3], 0.f))};
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = *(const f32x4 *)(lbias + 16 * mt + 4 * g);
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt] = mma(*(const u32x4 *)(F2 + (s * MT + mt) * kFrag + lane * 16), zb[s], acc[mt]);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) Z[mt][j] += act ? fmaxf(acc[mt][j], 0.0f) : 0.0f;
      cnt += act ? 1.0f : 0.0f;
#pragma unroll
      for (int s = 0; s < kSlotSteps1; ++s) b[s] = bn[s];
      al = aln;
    }
    // the pool's finish and T's last layer
    const float inv = a.mean ? 1.0f / fmaxf(cnt, 1.0f) : 1.0f;
    const float bs = a.mean ? (cnt > 0.0f ? 1.0f : 0.0f) : cnt;
    u32x4 zb[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const f32x4 p = Z[2 * s] * inv, q = Z[2 * s + 1] * inv;
      zb[s] = u32x4{pk_bf16(p[0], p[1]), pk_bf16(p[2], p[3]), pk_bf16(q[0], q[1]),
                    pk_bf16(q[2], q[3])};
    }
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = *(const f32x4 *)(lbias + W + 16 * mt + 4 * g) * bs;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[mt] = mma(*(const u32x4 *)(F3 + (s * MT + mt) * kFrag + lane * 16), zb[s], acc[mt]);
    if (xin) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const uint2 pk = {pk_bf16(acc[mt][0], acc[mt][1]), pk_bf16(acc[mt][2], acc[mt][3])};
        *(uint2 *)(a.tau + (px * W + 16 * mt + 4 * g) * 2) = pk;
      }
    }
  }
}

// ---- input and weight packing -------------------------------------------------
// Every buffer's 12 planes as bf16 [n][k][H][W][16] (zero channels 12..15):
// one thread per (frame, buffer, pixel).
__global__ void sp_pack_slots_kernel(const float *__restrict__ layers, int64_t total, int hw,
                                     uint8_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int64_t fb = i / hw;                 // frame * k + buffer
  const int q = (int)(i - fb * hw);
  const float *src = layers + fb * kNL * hw + q;
  uint32_t w[8];
  for (int j = 0; j < 8; ++j) {
    const int c = 2 * j;
    w[j] = pk_bf16(c < kNL ? src[(int64_t)c * hw] : 0.0f, c + 1 < kNL ? src[(int64_t)(c + 1) * hw] : 0.0f);
  }
  u32x4 *dst = (u32x4 *)(out + i * 32);
  dst[0] = u32x4{w[0], w[1], w[2], w[3]};
  dst[1] = u32x4{w[4], w[5], w[6], w[7]};
}

// Weight fragments of one conv: element e of fragment (step, mt), lane l,
// position j holds W[16 mt + (l & 15)][ci][tap] for step = tap * cbt + cb and
// concatenated input channel 32 cb + 8 (l >> 4) + j, mapped to the master
// input column (zero for padding channels and rows past cout).
struct SpPackDesc {
  int64_t woff;             // float offset of the weight tensor [cout][cin][k][k]
  int64_t out_off;          // byte offset of the fragments in the packed buffer
  int cout, cin, k;         // master tensor shape
  int col0;                 // first master input column this conv multiplies
  int c0real, c0pad, c1real, c1pad;   // its two sources (channels, padded to 32)
  int mt;                   // M-tiles
};

// Everything in one launch: blockIdx.y selects the conv (15), then the
// fragments of sp_slots_kernel: 15 packs conv3_b (T1's buffer columns, master
// [W][12 + W][3][3]), 16 and 17 A2 and A3 ([W][W]) in register order.  The
// biases (padded to whole M-tiles, zero past cout and for T1's buffer part,
// whose bias T1's sigma part carries) go after the convs' fragments.
constexpr int kPackJobs = 18;
struct SpPackAll {
  SpPackDesc d[15];
  int64_t bias_src[15];     // master float offset of each conv's bias (-1: none)
  int64_t bias_dst[15];     // float offset in the packed bias block
  int64_t bias_block;       // byte offset of the bias block
  int64_t slots_off, t[3];  // sp_slots_kernel's fragments; T's three weight tensors
  int W;
};

// A thread per lane of a fragment: its 8 elements, one 16-byte store.
__global__ __launch_bounds__(256) void sp_pack_all_kernel(const float *__restrict__ master,
                                                          SpPackAll all, uint8_t *__restrict__ packed) {
  const int job = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x, l = i & 63;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  uint8_t *dst;
  if (job < 15) {
    const SpPackDesc &d = all.d[job];
    if (i < 16 * d.mt) {
      const int64_t src = all.bias_src[job];
      ((float *)(packed + all.bias_block))[all.bias_dst[job] + i] =
          src >= 0 && i < d.cout ? master[src + i] : 0.0f;
    }
    const int cbt = (d.c0pad + d.c1pad) >> 5, kk = d.k * d.k;
    if (i >= kk * cbt * d.mt * 64) return;
    const int mt = (i >> 6) % d.mt, step = (i >> 6) / d.mt, tap = step / cbt, cb = step % cbt;
    const int row = 16 * mt + (l & 15);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int cc = 32 * cb + 8 * (l >> 4) + j;         // concatenated padded channel
      int ci = -1;
      if (cc < d.c0pad) {
        if (cc < d.c0real) ci = cc;
      } else if (cc - d.c0pad < d.c1real) {
        ci = d.c0real + (cc - d.c0pad);
      }
      if (row < d.cout && ci >= 0)
        v[j] = master[d.woff + ((int64_t)row * d.cin + d.col0 + ci) * kk + tap];
    }
    dst = packed + d.out_off;
  } else {
    const int W = all.W, MT = W / 16, KS = MT / 2, which = job - 15;
    const int steps = which == 0 ? kSlotSteps1 : KS;
    if (i >= steps * MT * 64) return;
    const int mt = (i >> 6) % MT, s = (i >> 6) / MT, g = l >> 4, row = 16 * mt + (l & 15);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (which == 0) {
        const int tap = 2 * s + (g >> 1), ch = 8 * (g & 1) + j;
        if (tap < 9 && ch < kNL) v[j] = master[all.t[0] + ((int64_t)row * (kNL + W) + ch) * 9 + tap];
      } else {
        const int ch = 32 * s + (j < 4 ? 4 * g + j : 16 + 4 * g + j - 4);
        v[j] = master[all.t[which] + (int64_t)row * W + ch];
      }
    }
    dst = packed + all.slots_off +
          (which == 0 ? 0 : (int64_t)(kSlotSteps1 + (which - 1) * KS) * MT * kFrag);
  }
  *(u32x4 *)(dst + (int64_t)i * 16) = u32x4{pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3]),
                                            pk_bf16(v[4], v[5]), pk_bf16(v[6], v[7])};
}

}  // namespace

// ---------------------------------------------------------------------------
// Host side: the layer sequence.

// The 14 convolutions (and T1's split into its buffer and sigma parts).
enum SpConvId {
  SP_F1, SP_F2, SP_F3, SP_F4, SP_T1B, SP_T1S, SP_T2, SP_T3, SP_B1, SP_B2, SP_B3, SP_B4,
  SP_R1, SP_R2, SP_R3, kSpConvs
};

struct SpLayout {
  int W;
  SpPackDesc d[kSpConvs];
  int64_t bias_off[kSpConvs];      // float offset of each conv's padded bias in the bias block
  int64_t frag_bytes, bias_floats;
  int64_t slots_off, slots_bytes;  // sp_slots_kernel's fragments (after the bias block)
  int64_t t1, t2, t3;              // master offsets of T's three weight tensors
};

static int64_t sp_master_offsets(int W, int64_t woff[14], int64_t boff[14], int cout[14],
                                 int cin[14], int ks[14]) {
  const int spec[14][3] = {{W, kNG + kNS, 3}, {W, W, 3}, {W, 2 * W, 3}, {W, W, 1},
                           {W, kNL + W, 3}, {W, W, 1}, {W, W, 1},
                           {W, 2 * W, 3}, {W, W, 3}, {W, 2 * W, 3}, {W, W, 1},
                           {W, W + 3, 3}, {W, W, 3}, {kNOUT, W, 1}};
  int64_t off = 0;
  for (int i = 0; i < 14; ++i) {
    cout[i] = spec[i][0];
    cin[i] = spec[i][1];
    ks[i] = spec[i][2];
    woff[i] = off;
    off += (int64_t)cout[i] * cin[i] * ks[i] * ks[i];
    boff[i] = off;
    off += cout[i];
  }
  return off;
}

size_t spatial_num_params(int W) {
  if (W != 64 && W != 128) return 0;
  int64_t wo[14], bo[14];
  int co[14], ci[14], k[14];
  return (size_t)sp_master_offsets(W, wo, bo, co, ci, k);
}

static SpLayout sp_layout(int W) {
  int64_t wo[14], bo[14];
  int co[14], ci[14], k[14];
  sp_master_offsets(W, wo, bo, co, ci, k);
  // master tensor index of every conv; (col0, sources) of each
  struct M { int m, col0, c0real, c0pad, c1real, c1pad; };
  const M map[kSpConvs] = {
      {0, 0, kNG + kNS, 32, 0, 0},   {1, 0, W, W, 0, 0},  {2, 0, W, W, W, W}, {3, 0, W, W, 0, 0},
      {4, 0, kNL, 32, 0, 0},         {4, kNL, W, W, 0, 0},                     // T1: b part, sigma part
      {5, 0, W, W, 0, 0},            {6, 0, W, W, 0, 0},
      {7, 0, W, W, W, W},            {8, 0, W, W, 0, 0},  {9, 0, W, W, W, W}, {10, 0, W, W, 0, 0},
      {11, 0, W, W, 3, 32},          {12, 0, W, W, 0, 0}, {13, 0, W, W, 0, 0}};
  SpLayout L;
  L.W = W;
  int64_t fb = 0, bf = 0;
  for (int c = 0; c < kSpConvs; ++c) {
    const M &m = map[c];
    SpPackDesc &d = L.d[c];
    d.woff = wo[m.m];
    d.cout = co[m.m];
    d.cin = ci[m.m];
    d.k = k[m.m];
    d.col0 = m.col0;
    d.c0real = m.c0real;
    d.c0pad = m.c0pad;
    d.c1real = m.c1real;
    d.c1pad = m.c1pad;
    d.mt = (d.cout + 15) / 16;
    d.out_off = fb;
    fb += (int64_t)d.k * d.k * ((d.c0pad + d.c1pad) / 32) * d.mt * kFrag;
    L.bias_off[c] = bf;
    bf += d.mt * 16;
  }
  L.frag_bytes = fb;
  L.bias_floats = bf;
  const int MT = W / 16;
  L.slots_off = (fb + 4 * bf + 1023) / 1024 * 1024;
  L.slots_bytes = (int64_t)(kSlotSteps1 + MT) * MT * kFrag;
  L.t1 = wo[4];
  L.t2 = wo[5];
  L.t3 = wo[6];
  return L;
}

// Master bias offset of conv c (T1's two parts share T1's bias; the sigma
// part carries it, the buffer part adds none).
static int64_t sp_bias_master(int W, int c, bool *zero) {
  int64_t wo[14], bo[14];
  int co[14], ci[14], k[14];
  sp_master_offsets(W, wo, bo, co, ci, k);
  const int m[kSpConvs] = {0, 1, 2, 3, 4, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13};
  *zero = c == SP_T1B;
  return bo[m[c]];
}

size_t spatial_weight_bytes(int W) {
  const SpLayout L = sp_layout(W);
  return (size_t)(L.slots_off + L.slots_bytes);
}

// Device bytes of the activations a call of n frames of H x W with k buffers
// needs.
size_t spatial_workspace_bytes(int W, int n, int H, int Wd, int k) {
  const int64_t px = (int64_t)n * H * Wd, half = px / 4;
  // bf16: e1, sigma, tau, phi, r1 (W ch each), half-res d and m (W ch), the k
  // buffers (16 ch each); fp32: u (W ch); rounding slack
  return (size_t)(2 * (5 * px * W + 2 * half * W + px * 16 * (int64_t)k) + 4 * px * W + 16 * 256);
}

hipError_t spatial_pack(const float *master, int W, uint8_t *packed, hipStream_t s) {
  const SpLayout L = sp_layout(W);
  static_assert(kSpConvs == 15, "SpPackAll holds 15 convolutions");
  SpPackAll all;
  int64_t most = 0;
  for (int c = 0; c < kSpConvs; ++c) {
    all.d[c] = L.d[c];
    bool zero = false;
    const int64_t bo = sp_bias_master(W, c, &zero);
    all.bias_src[c] = zero ? -1 : bo;
    all.bias_dst[c] = L.bias_off[c];
    const SpPackDesc &d = L.d[c];
    most = std::max<int64_t>(most, (int64_t)d.k * d.k * ((d.c0pad + d.c1pad) / 32) * d.mt * 64);
  }
  all.bias_block = L.frag_bytes;
  all.slots_off = L.slots_off;
  all.t[0] = L.t1;
  all.t[1] = L.t2;
  all.t[2] = L.t3;
  all.W = W;
  hipLaunchKernelGGL(sp_pack_all_kernel, dim3((unsigned)((most + 255) / 256), kPackJobs), dim3(256),
                     0, s, master, all, packed);
  return hipGetLastError();
}

template <int MT>
static hipError_t sp_slots_launch(const SpSlotsArgs &a, hipStream_t s) {
  const size_t lds = (size_t)(kSlotSteps1 + MT) * MT * kFrag + 2 * 16 * MT * sizeof(float);
  static LdsLimit limit;
  const hipError_t e = limit.raise((const void *)sp_slots_kernel<MT>, lds);
  if (e != hipSuccess) return e;
  const int64_t nseg = (int64_t)a.n * a.H * ((a.Wd + 15) / 16);
  const int64_t ntiles = (nseg + kWaves - 1) / kWaves;
  // persistent: one workgroup per CU (the weights fill most of its LDS), a
  // multiple of the 8 XCDs
  const unsigned grid = (unsigned)std::min<int64_t>(256, (ntiles + 7) / 8 * 8);
  hipLaunchKernelGGL(sp_slots_kernel<MT>, dim3(grid), dim3(kThreads), lds, s, a);
  return hipGetLastError();
}

template <int MT, int TR, int CB0, int SRC1, int CB1, bool PLANES, int EPI>
static hipError_t sp_launch(const SpConvArgs &a, hipStream_t s) {
  constexpr int lds = ConvLds<MT, TR, CB0, SRC1, CB1>::kBytes;
  static LdsLimit limit;
  const hipError_t e =
      limit.raise((const void *)sp_conv_kernel<MT, TR, CB0, SRC1, CB1, PLANES, EPI>, lds);
  if (e != hipSuccess) return e;
  const int64_t tiles = (int64_t)a.n * ((a.H + TR - 1) / TR) * ((a.Wd + kTC - 1) / kTC);
  hipLaunchKernelGGL((sp_conv_kernel<MT, TR, CB0, SRC1, CB1, PLANES, EPI>), dim3((unsigned)tiles),
                     dim3(kConvThreads), lds, s, a);
  return hipGetLastError();
}

// The rows of a tile: 8 while that leaves a tile for every CU, else 4.  (16 rows
// halve the weight traffic but leave one workgroup and one wave per SIMD to a
// CU, whose halo load and epilogue nothing overlaps: the 256^2 W = 128 convs
// took 20-41 us, with 8 rows 19-37.)
template <int MT, int CB0, int SRC1, int CB1, bool PLANES, int EPI>
static hipError_t sp_conv(const SpConvArgs &a, hipStream_t s) {
  constexpr int kCus = 256;
  const int64_t cols = (int64_t)a.n * ((a.Wd + kTC - 1) / kTC);
  if (cols * ((a.H + 7) / 8) >= kCus) return sp_launch<MT, 8, CB0, SRC1, CB1, PLANES, EPI>(a, s);
  return sp_launch<MT, 4, CB0, SRC1, CB1, PLANES, EPI>(a, s);
}

template <int MT>
static hipError_t spatial_run(const SpLayout &L, const uint8_t *packed, int pool, const float *gbuf,
                              const float *layers, const float *scene, int n, int H, int Wd, int k,
                              float *out, uint8_t *ws, hipStream_t s) {
  constexpr int W = MT * 16, CB = MT / 2;
  const float *bias = (const float *)(packed + L.frag_bytes);
  const int64_t px = (int64_t)n * H * Wd, half = px / 4;
  const int hw = H * Wd;
  // workspace carve-up (see spatial_workspace_bytes)
  uint8_t *p = ws;
  auto take = [&](int64_t bytes) { uint8_t *q = p; p += (bytes + 255) & ~(int64_t)255; return q; };
  uint8_t *e1 = take(px * W * 2), *sig = take(px * W * 2), *tau = take(px * W * 2);
  uint8_t *phi = take(px * W * 2), *r1 = take(px * W * 2);
  uint8_t *dh = take(half * W * 2), *mh = take(half * W * 2);
  uint8_t *bpk = take(px * 16 * 2 * (int64_t)k);
  float *u = (float *)take(px * W * 4);
  hipError_t e = hipSuccess;

  auto args = [&](int c, const uint8_t *in0, const uint8_t *in1, void *o, int Hc, int Wc) {
    SpConvArgs a = {};
    a.in0 = in0;
    a.in1 = in1;
    a.gbuf = gbuf;
    a.scene = scene;
    a.wfrag = packed + L.d[c].out_off;
    a.bias = bias + L.bias_off[c];
    a.n = n;
    a.H = Hc;
    a.Wd = Wc;
    a.out = (uint8_t *)o;
    return a;
  };
  // the following 1 x 1 conv
  auto then = [&](SpConvArgs a, int c) {
    a.wfrag1 = packed + L.d[c].out_off;
    a.bias1 = bias + L.bias_off[c];
    return a;
  };
  auto ok = [&](hipError_t r) { if (e == hipSuccess) e = r; };
  // e1's average d, m = relu(conv3 d) at half resolution, then
  // conv1 relu(conv3 [e1; up m])
  auto unet_tail = [&](int c1st, uint8_t *outp) {
    ok(sp_conv<MT, CB, S_NONE, 0, false, E_ACT>(args(c1st + 1, dh, nullptr, mh, H / 2, Wd / 2), s));
    ok(sp_conv<MT, CB, S_HALF, CB, false, E_CONV1>(then(args(c1st + 2, e1, mh, outp, H, Wd), c1st + 3), s));
  };

  // F: sigma = U-Net([G; s])
  SpConvArgs a = args(SP_F1, nullptr, nullptr, e1, H, Wd);
  a.pool = dh;
  ok(sp_conv<MT, 1, S_NONE, 0, true, E_ACT>(a, s));
  unet_tail(SP_F1, sig);
  // T: u = conv3 sigma (T1's sigma columns) + c1; then, in one kernel, per
  // buffer z1 = relu(conv3 b_i + u), Z += [alpha_i > 0] relu(A2 z1 + c2), and
  // tau = A3 (Z / max(c, 1)) + [c > 0] c3 (mean) or A3 Z + c c3 (sum)
  ok(sp_conv<MT, CB, S_NONE, 0, false, E_F32>(args(SP_T1S, sig, nullptr, u, H, Wd), s));
  if (k > 0) {
    const int64_t tot = px * k;
    hipLaunchKernelGGL(sp_pack_slots_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s,
                       layers, tot, hw, bpk);
  }
  {
    SpSlotsArgs t;
    t.frag = packed + L.slots_off;
    t.bias = bias + L.bias_off[SP_T2];       // c2, then c3 (T3's bias block follows T2's)
    t.bpk = bpk;
    t.layers = layers;
    t.u = u;
    t.tau = tau;
    t.n = n;
    t.H = H;
    t.Wd = Wd;
    t.k = k;
    t.mean = pool == GN_POOL_MEAN ? 1 : 0;
    ok(sp_slots_launch<MT>(t, s));
  }
  // B: phi = U-Net([sigma; tau])
  a = args(SP_B1, sig, tau, e1, H, Wd);
  a.pool = dh;
  ok(sp_conv<MT, CB, S_FULL, CB, false, E_ACT>(a, s));
  unet_tail(SP_B1, phi);
  // R: y = conv1 relu(conv3 relu(conv3 [phi; L_d]))
  ok(sp_conv<MT, CB, S_LIGHT, 1, false, E_ACT>(args(SP_R1, phi, nullptr, r1, H, Wd), s));
  ok(sp_conv<MT, CB, S_NONE, 0, false, E_RGB>(then(args(SP_R2, r1, nullptr, out, H, Wd), SP_R3), s));
  if (e == hipSuccess) e = hipGetLastError();
  return e;
}

hipError_t spatial_forward(const uint8_t *packed, int W, int pool, const float *gbuf,
                           const float *layers, const float *scene, int n, int H, int Wd, int k,
                           float *out, uint8_t *ws, hipStream_t s) {
  const SpLayout L = sp_layout(W);
  return W == 128 ? spatial_run<8>(L, packed, pool, gbuf, layers, scene, n, H, Wd, k, out, ws, s)
                  : spatial_run<4>(L, packed, pool, gbuf, layers, scene, n, H, Wd, k, out, ws, s);
}

}  // namespace gn
