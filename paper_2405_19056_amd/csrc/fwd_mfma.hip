// Fused GlassNet forward on the gfx950 matrix cores (bf16 / fp8 in, fp32 acc).
//
// Formulation.  Every layer is Y^T = A X^T with the weights A as the MFMA
// "A" operand (16 output neurons per M-tile) and 16 pixels per N-tile as the
// "B" operand.  The fp32 accumulator of v_mfma_f32_16x16x32_bf16 leaves lane
// l holding 4 consecutive output rows (4*(l>>4) + r) of pixel l & 15; two
// M-tiles give exactly the 8 values that lane must present as the B operand
// of the next layer's 32-deep K-step.  The next layer's weights are stored
// with their input columns permuted the same way, so activations go from one
// layer to the next by a ReLU and a bf16 convert, without leaving registers.
//
// Work split.  A workgroup of 8 waves owns a tile of 256 pixels (32 per wave,
// two N-tiles; 128 where that leaves half of the CUs idle, n_tiles).  Weights
// are staged into LDS chunk by chunk with direct global->LDS loads,
// double-buffered: while a stage computes, the next stage's chunk streams in.
// The weights of the per-slot network h that run inside the slot loop stay
// resident, at W = 64 all of them.  Grid = number of CUs; each workgroup
// walks tiles with a stride of the grid (tiles may come from a table that
// mixes frames of different sizes and slot counts).
//
// The method (Sec. 3.3-3.4): sigma = F([G; s]); tau = pool_i h(b_i, sigma)
// over slots with alpha_i > 0 (Eq. (5)); phi = B([sigma; tau]);
// y = R([phi; L_d]).  Two exact rewrites of h are used: its first layer's
// sigma part is computed once per pixel (u = W1s sigma + c1), and because its
// last layer is affine the masked pool moves in front of it:
// sum_i m_i (A3 a_i + c3) = A3 (sum_i m_i a_i) + (sum_i m_i) c3.  The running
// sum is fp32 in registers, so memory does not grow with the slot count.
#include "gn_internal.h"
#include "lds_limit.h"
#include "slot_order.h"

namespace gn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef const float __attribute__((address_space(1))) gcfloat;
typedef float __attribute__((address_space(1))) gfloat;
typedef u32x4 __attribute__((address_space(1))) gu32x4;
typedef f32x4 __attribute__((address_space(1))) gf32x4;

constexpr int kWaves = 8;
constexpr int kNT = 2;                // N-tiles of 16 pixels per wave
constexpr int kThreads = kWaves * 64;
static_assert(kWaves * kNT * 16 == kTilePx, "tile = waves x N-tiles x 16 pixels");
constexpr int kFrag = 1024;            // one bf16 A fragment: 64 lanes x 16 B

struct MfmaArgs {
  const uint8_t *packed;
  int64_t stage_off[kMaxStages + 1];
  int64_t res_off, res_bytes, stage_max, bias_off, t2q_off, t2s_off;
  FwdBatch b;
  const FrameDesc *frames;
  const TileRef *tiles;
  int ntiles;
  int tiles_per_frame;
  int pool;
  float sa, inv_sa;                    // fp8 activation scale and its inverse
  uint8_t *sig_scratch;                // per (workgroup, wave): sigma fragments, stage 1 -> 3
  int sig_lds_waves;                   // waves 0 .. n-1 park sigma in LDS instead:
  int sig_tail_waves;                  // the first n - t after the stage buffers, the
                                       // last t in the stage buffers' idle tails
  uint8_t *state;                      // object streaming: per-tile state (modes other than FULL)
  int state_load;                      // 1: the state holds a running sum to continue from
  int dense;                           // 1: the state's layout for few tiles (StreamTile)
  int canon;                           // FULL: pool each pixel's slots in canonical order
  int kpad;                            // bytes per pixel of the LDS slot-order table
  int aslots;                          // slots whose alphas the LDS alpha table holds
  int alpha_alias;                     // 1: the alpha table sits in sigma's parking area
};

// Two floats -> packed bf16 pair (round to nearest even), one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// max(x, 0) in one v_med3_f32 (fmaxf on a matrix-core result would first
// canonicalise its operand, costing a second instruction).
__device__ __forceinline__ float relu1(float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, 3.402823466e+38f); }

__device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 16x16x16 bf16 MFMA: lane group g supplies inputs 4g..4g+3.
__device__ __forceinline__ f32x4 mma16(uint2 a, uint2 b, f32x4 c) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a),
                                                   __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 relu4(f32x4 v) {
  return f32x4{relu1(v.x), relu1(v.y), relu1(v.z), relu1(v.w)};
}

// ReLU of two packed bf16: sign-magnitude values order like signed 16-bit
// integers, so max(x, 0) as int16 zeroes exactly the negative numbers.
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t x) {
  typedef short s16x2 __attribute__((ext_vector_type(2)));
  s16x2 v = __builtin_bit_cast(s16x2, x);
  s16x2 z = {0, 0};
  v = __builtin_elementwise_max(v, z);
  return __builtin_bit_cast(uint32_t, v);
}

// Four floats -> four OCP E4M3 bytes (round to nearest even) of
// min(max(v, 0), 448): ReLU and the clamp to the format's largest finite
// magnitude in one v_med3 each.
__device__ __forceinline__ int relu_pack_fp8x4(f32x4 v) {
  const float M = 448.0f;
  const float x = __builtin_amdgcn_fmed3f(v.x, 0.0f, M), y = __builtin_amdgcn_fmed3f(v.y, 0.0f, M);
  const float z = __builtin_amdgcn_fmed3f(v.z, 0.0f, M), w = __builtin_amdgcn_fmed3f(v.w, 0.0f, M);
  int r = __builtin_amdgcn_cvt_pk_fp8_f32(x, y, 0, false);
  return __builtin_amdgcn_cvt_pk_fp8_f32(z, w, r, true);
}

// 16x16x128 E4M3 x E4M3 -> fp32 on the gfx950 matrix cores, unit block scales.
__device__ __forceinline__ f32x4 mma_fp8(i32x8 a, i32x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
}

// s_waitcnt for at most VM vector-memory and LGKM LDS/scalar operations in
// flight (15: any).  The builtin and not inline assembly, so that the compiler
// knows what has landed and puts no wait of its own before its use.
template <int VM, int LGKM>
__device__ __forceinline__ void wait_cnt() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (LGKM << 8) | ((VM >> 4) << 14));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_vm() { wait_cnt<0, 15>(); }

// The positional-encoding blocks of x (Sec. 3.4) up to block NB - 1: x, then
// sin(2^k pi x) (block 2k + 1) and cos(2^k pi x) (block 2k + 2).  Level 0
// comes from the hardware sine and cosine, which take revolutions: x / 2 is
// reduced exactly to [0, 1) first.  Each further level follows from the one
// before by the double-angle identities (sin 2a = 2 sin a cos a,
// cos 2a = 1 - 2 sin^2 a): a few fp32 roundings per level, far below the
// bf16 rounding the values then get.
template <int NB>
__device__ __forceinline__ void pe_blocks_of(float x, float (&e)[NB]) {
  e[0] = x;
  if constexpr (NB > 1) {
    const float r = __builtin_amdgcn_fractf(x * 0.5f);
    float sn = __builtin_amdgcn_sinf(r), cs = __builtin_amdgcn_cosf(r);
#pragma unroll
    for (int b = 1; b < NB; b += 2) {
      if (b > 1) {
        const float s2 = 2.0f * sn * cs;
        cs = __builtin_fmaf(-2.0f * sn, sn, 1.0f);
        sn = s2;
      }
      e[b] = sn;
      if (b + 1 < NB) e[b + 1] = cs;
    }
  }
}

// Stage boundary that leaves the newest N vector-memory operations in flight:
// N global stores issued after the next stage's LDS fill, whose completion
// nothing in the workgroup waits for.  The fill itself (older) has landed in
// LDS once vmcnt <= N; LDS traffic is drained and every wave has arrived.
template <int N>
__device__ __forceinline__ void stage_sync_after_stores() {
  wait_cnt<N, 0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// Stage boundary: the next stage's copy has landed, every wave has arrived.
__device__ __forceinline__ void stage_sync() { stage_sync_after_stores<0>(); }

// Copy `bytes` (a multiple of 1 KiB) from global to LDS: each wave moves whole
// 1 KiB blocks, lane i writing bytes [16 i, 16 i + 16) of its block.
__device__ __forceinline__ void lds_fill(uint8_t *dst, const uint8_t *src, int64_t bytes,
                                         int wave, int lane) {
  for (int64_t off = (int64_t)wave * kFrag; off < bytes; off += kWaves * kFrag) {
    __builtin_amdgcn_global_load_lds(
        (const void *)(src + off + lane * 16),
        (__attribute__((address_space(3))) void *)(dst + off), 16, 0, 0);
  }
}

// The same for a compile-time size: straight-line copies.
template <int BYTES>
__device__ __forceinline__ void lds_copy(uint8_t *dst, const uint8_t *src, int wave, int lane) {
  constexpr int kBlocks = BYTES / kFrag;
#pragma unroll
  for (int i = 0; i < (kBlocks + kWaves - 1) / kWaves; ++i) {
    const int b = i * kWaves + wave;
    if (kBlocks % kWaves == 0 || i < kBlocks / kWaves || b < kBlocks)
      __builtin_amdgcn_global_load_lds((const void *)(src + (uint32_t)(b * kFrag + lane * 16)),
                                       (__attribute__((address_space(3))) void *)(dst + b * kFrag),
                                       16, 0, 0);
  }
}

__device__ __forceinline__ u32x4 ld_frag(const uint8_t *chunk, int idx, int lane) {
  return *(const u32x4 *)(chunk + (size_t)idx * kFrag + lane * 16);
}

// One A fragment of the 16x16x16 bf16 instruction: 64 lanes x 8 bytes.
__device__ __forceinline__ uint2 ld_frag16(const uint8_t *chunk, int idx, int lane) {
  return *(const uint2 *)(chunk + (size_t)idx * 512 + lane * 8);
}

// One fp8 A fragment of the 16x16x128 instruction: 64 lanes x 32 bytes,
// stored as two 1 KiB halves (bytes 0-15 of every lane, then bytes 16-31),
// so each 16-byte LDS read has consecutive lanes 16 bytes apart (a 32-byte
// lane stride would put two lanes on every bank).
__device__ __forceinline__ i32x8 ld_frag8(const uint8_t *chunk, int idx, int lane) {
  const uint8_t *f = chunk + (size_t)idx * 2 * kFrag + lane * 16;
  const i32x4 lo = *(const i32x4 *)f, hi = *(const i32x4 *)(f + kFrag);
  return i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}

template <int MT_, int NT>
__device__ __forceinline__ void bias_init(f32x4 (&acc)[NT][MT_], const float *bias, int g) {
#pragma unroll
  for (int mt = 0; mt < MT_; ++mt) {
    const f32x4 b = *(const f32x4 *)(bias + 16 * mt + 4 * g);
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t][mt] = b;
  }
}

// Accumulator rows -> next layer's B fragments (M-tiles 2j and 2j+1 make K-step j).
template <int MT_, bool RELU, int NT>
__device__ __forceinline__ void to_frags(const f32x4 (&acc)[NT][MT_], u32x4 (&out)[NT][MT_ / 2]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
#pragma unroll
    for (int mt = 0; mt < MT_; ++mt) {
      const f32x4 v = acc[t][mt];
      uint32_t lo = pk_bf16(v.x, v.y), hi = pk_bf16(v.z, v.w);
      if (RELU) {
        lo = relu_bf16x2(lo);
        hi = relu_bf16x2(hi);
      }
      out[t][mt >> 1][2 * (mt & 1)] = lo;
      out[t][mt >> 1][2 * (mt & 1) + 1] = hi;
    }
  }
}

// One chained layer, an M-tile pair at a time: out[t][p] = pack(act(A in + bias))
// for M-tiles 2p and 2p+1.  The pair's weight fragments are read up front and
// the next pair's are requested before this pair's MFMAs issue, so LDS
// latency overlaps matrix-core work instead of stalling every K-step.
// EARLY: a scheduling barrier keeps the next M-tiles' fragment reads ahead of
// the current M-tiles' MFMAs (left alone, the scheduler sinks each read next
// to its MFMAs and waits for it alone): 3.5-5% of the bf16 frame, 2% of the
// fp8 one, whose kernel spills with it in T3 and B's first layer and there
// leaves the placement to the scheduler.
template <int MT_, int KS_, bool RELU, bool EARLY, int NT>
__device__ __forceinline__ void layer(u32x4 (&out)[NT][MT_ / 2], const uint8_t *chunk,
                                      const u32x4 (&in)[NT][KS_], const float *bias, int g,
                                      int lane) {
  u32x4 wb[2][2][KS_];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int ks = 0; ks < KS_; ++ks) wb[0][h][ks] = ld_frag(chunk, h * KS_ + ks, lane);
#pragma unroll
  for (int p = 0; p < MT_ / 2; ++p) {
    const int cur = p & 1;
    if (p + 1 < MT_ / 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int ks = 0; ks < KS_; ++ks)
          wb[cur ^ 1][h][ks] = ld_frag(chunk, (2 * (p + 1) + h) * KS_ + ks, lane);
    }
    if constexpr (EARLY) __builtin_amdgcn_sched_barrier(0);
    f32x4 acc[NT][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 b = *(const f32x4 *)(bias + 16 * (2 * p + h) + 4 * g);
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t][h] = b;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int ks = 0; ks < KS_; ++ks) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t][h] = mma(wb[cur][h][ks], in[t][ks], acc[t][h]);
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 v = acc[t][h];
        uint32_t lo = pk_bf16(v.x, v.y), hi = pk_bf16(v.z, v.w);
        if (RELU) {
          lo = relu_bf16x2(lo);
          hi = relu_bf16x2(hi);
        }
        out[t][p][2 * h] = lo;
        out[t][p][2 * h + 1] = hi;
      }
    }
  }
}

// acc[t][mt] += A(chunk) . in[t] over the chunk's KS_ K-steps, one M-tile's
// fragments read ahead of its MFMAs and the next M-tile's requested early
// (EARLY as for layer).
template <int MT_, int KS_, bool EARLY, int NT>
__device__ __forceinline__ void mm(f32x4 (&acc)[NT][MT_], const uint8_t *chunk,
                                   const u32x4 (&in)[NT][KS_], int lane) {
  u32x4 wb[2][KS_];
#pragma unroll
  for (int ks = 0; ks < KS_; ++ks) wb[0][ks] = ld_frag(chunk, ks, lane);
#pragma unroll
  for (int mt = 0; mt < MT_; ++mt) {
    const int cur = mt & 1;
    if (mt + 1 < MT_) {
#pragma unroll
      for (int ks = 0; ks < KS_; ++ks) wb[cur ^ 1][ks] = ld_frag(chunk, (mt + 1) * KS_ + ks, lane);
    }
    if constexpr (EARLY) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS_; ++ks)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t][mt] = mma(wb[cur][ks], in[t][ks], acc[t][mt]);
  }
}

// F's encoded input as B fragments: K-step b (of N) is encoding block B0 + b
// of the 8 raw channels the lane holds.
template <int B0, int N, int NT>
__device__ __forceinline__ void enc_frags(const float (&xr)[NT][8], u32x4 (&x)[NT][N]) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float e0[B0 + N], e1[B0 + N];
      pe_blocks_of<B0 + N>(xr[t][2 * q], e0);
      pe_blocks_of<B0 + N>(xr[t][2 * q + 1], e1);
#pragma unroll
      for (int b = 0; b < N; ++b) x[t][b][q] = pk_bf16(e0[B0 + b], e1[B0 + b]);
    }
}

template <int W>
struct Shape {
  static constexpr int MT = W / 16, KS = W / 32;
  static constexpr int kBiasBytes = kNumLayers * W * 4;
};

// Bytes of the resident weights (T1's slot columns, T2 and, in fp8, T2's row
// scales) and of a stage buffer (the largest stage: R's first layer, or half
// of the encoded F1).
template <int W, int PREC, int PE>
struct LdsMap {
  static constexpr int MT = W / 16, KS = W / 32;
  static constexpr int kT1A = (MT * (PE > 0 ? pe_k16_steps(PE) : 1) * 512 + 1023) & ~1023;
  static constexpr int kRes =
      kT1A + (PREC == GN_FP8_T ? MT * 2048 + ((W * 4 + 1023) & ~1023) : MT * KS * kFrag);
  static constexpr int kF1 = PE > 0 ? (pe_blocks(PE) + 1) / 2 : 0;
  static constexpr int kStage = MT * (KS + 1 > kF1 ? KS + 1 : kF1) * kFrag;
  // bytes of stage s (without encoding F1 and F2 share stage 0)
  static constexpr int stage_bytes(int s) {
    const int sq = MT * KS * kFrag, last = kNumStages + stage_shift(PE) - 1;
    if (s == last) return sq + KS * kFrag;                       // R2, R3
    if (s == last - 1) return sq + MT * kFrag;                   // R1
    if (PE == 0) return s == 0 ? MT * kFrag + sq : sq;
    return s == 0 ? kF1 * MT * kFrag : (s == 1 ? (pe_blocks(PE) - kF1) * MT * kFrag : sq);
  }
  // offset of stage s in the packed form; every stage together
  static constexpr int stage_at(int s) { return s == 0 ? 0 : stage_at(s - 1) + stage_bytes(s - 1); }
  static constexpr int kAll = stage_at(kNumStages + stage_shift(PE));
};

// At W = 64 without encoding all of the forward's weights fit in LDS (90 KiB):
// they stay there, and a tile has two barriers instead of eleven.  Its stages
// are 32 matrix instructions a SIMD long, and each had waited for a barrier and
// for L2.  256^2, K = 4: 14.7 -> 13.6 us; 512^2, K = 8: 80.0 -> 75.8 us.
template <int W, int MODE, int PE>
constexpr bool all_resident() { return W == 64 && MODE == FWD_FULL && PE == 0; }

// Object-streaming state of one tile (modes other than FWD_FULL): sigma as bf16 B
// fragments, the running masked sum Z of h's hidden layer as fp32 accumulator rows
// (16-byte lane vectors each), the active-slot count [pixel].
//
// Where there are many tiles, pixel by pixel: sigma [pixel][ks][g], Z [pixel][mt]
// [g].  What bounds the accumulate calls is this state's traffic, and with a
// pixel's values side by side the pixels an object does not cover move none of
// it (512^2, W = 128, half of the pixels covered: 35 us a call, 54 when all of it
// moved).  A pixel whose count is zero has no valid Z: nobody reads it.
//
// Where there are few, at most nine for 16 CUs (dense), 16 pixels at a time: sigma
// [16 pixels][ks][g][pixel], Z [16 pixels][mt][g][pixel], all of it moved.  A call
// is then one chain of latencies, shorter by the wait for the alphas, and an
// instruction's lanes read 1 KiB in one piece instead of 64 bytes from each of
// 16 pixels.  A frame of 8 objects, one a call: 64^2 88 -> 78 us, 128^2 93 -> 86,
// 176^2 102 -> 100; 192^2 105 either way; 224^2 114 -> 123.
template <int W>
struct StreamTile {
  static constexpr int64_t kSig = (int64_t)kTilePx * W * 2;
  static constexpr int64_t kZ = (int64_t)kTilePx * W * 4;
  static constexpr int64_t kCnt = (int64_t)kTilePx * 4;
  static constexpr int64_t kBytes = kSig + kZ + kCnt;
};

// The state is reached through a buffer resource of the tile's size: a lane
// whose offset lies outside it loads zeros and stores nothing.
constexpr int kOutside = 0x40000000;

// (off: the lane's first vector; at: the uniform offset of the one meant)
__device__ __forceinline__ u32x4 state_load16(__amdgpu_buffer_rsrc_t r, int off, int at) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, at, 0));
}

__device__ __forceinline__ void state_store16(__amdgpu_buffer_rsrc_t r, int off, int at, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, off, at, 0);
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <class T>
__device__ __forceinline__ T *uniform(T *p) {
  const uint64_t v = (uint64_t)p;
  return (T *)((uint64_t)(uint32_t)uniform((int)(v >> 32)) << 32 | (uint32_t)uniform((int)v));
}

// MODE selects the part of the path one launch runs: FWD_FULL the whole
// forward; FWD_BEGIN stages 0-1 (sigma into the state); FWD_ACC stage 2 (the
// slot loop, continuing the state's running sum); FWD_FINISH stages 3-9 from
// the state.
//
// PE > 0: F's and h's inputs are positionally encoded with PE levels; F1 then
// runs over two stages of its own (stage indices below), and h's first layer
// takes pe_k16_steps(PE) 16-deep K-steps per slot.
// NT: N-tiles of 16 pixels per wave (n_tiles below).
template <int W, int PREC, int MODE, int PE, int NT>
__global__ __launch_bounds__(kThreads) void fwd_mfma_kernel(MfmaArgs a) {
  constexpr int kNT = NT, kTilePx = kWaves * NT * 16;
  constexpr int MT = Shape<W>::MT, KS = Shape<W>::KS;
  constexpr int kShift = stage_shift(PE);
  // stage of each weight group (F1 and F2 share stage 0 without encoding)
  constexpr int sF1 = 0, sF1B = 1, sF2 = kShift, sF3 = 1 + kShift, sT1S = 2 + kShift,
                sT3 = 3 + kShift, sB1S = 4 + kShift, sB1T = 5 + kShift, sB2 = 6 + kShift,
                sB3 = 7 + kShift, sR1 = 8 + kShift, sR2 = 9 + kShift;
  constexpr int kE = pe_blocks(PE);                   // encoding blocks
  constexpr int kF1A = PE > 0 ? (kE + 1) / 2 : 1;     // F1's blocks in stage sF1
  constexpr int kF1B = kE - kF1A;                     // and in stage sF1B
  constexpr int kNK16 = PE > 0 ? pe_k16_steps(PE) : 1;   // h layer 1's K=16 steps
  constexpr bool kSlots = MODE == FWD_FULL || MODE == FWD_ACC;     // runs the slot loop
  constexpr bool kTrunk = MODE == FWD_FULL || MODE == FWD_BEGIN;   // runs F
  constexpr bool kHead = MODE == FWD_FULL || MODE == FWD_FINISH;   // runs T3, B, R
  const int wave = threadIdx.x >> 6;

  // LDS: the resident weights, the biases and the two stage buffers are arrays
  // of their own (the compiler makes an LDS read wait for every direct
  // global->LDS copy in flight that may write the array it reads: with one
  // array for all, each stage began by waiting for the copy of the next one),
  // then [slot order | alphas | sigma] of a size the launch decides.
  using LM = LdsMap<W, PREC, PE>;
  __shared__ __attribute__((aligned(1024))) uint8_t L_res[LM::kRes];
  __shared__ __attribute__((aligned(1024))) float L_bias[kNumLayers * W];
  constexpr bool kAllRes = all_resident<W, MODE, PE>();
  __shared__ __attribute__((aligned(1024))) uint8_t L_stage0[kAllRes ? LM::kAll : LM::kStage];
  __shared__ __attribute__((aligned(1024))) uint8_t L_stage1[kAllRes ? 16 : LM::kStage];
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int res_bytes = LM::kRes, stage_max = LM::kStage;
  // slot-order table: for each pixel of the tile, its slots' indices in
  // canonical order (kpad bytes per pixel, a multiple of 4), and the tile's
  // alphas [slot][pixel] that the order is computed from (aslots slots)
  // (in sigma's LDS parking area, free until F's last layer ends, when that
  // area holds at least the table)
  uint8_t *L_perm = lds;
  float *L_alpha = (float *)(L_perm + (size_t)kTilePx * a.kpad);
  uint8_t *L_sig =
      L_perm + (size_t)kTilePx * a.kpad + (a.alpha_alias ? 0 : (size_t)kTilePx * 4 * a.aslots);
  // FWD_FINISH runs an odd number of stages per tile, so its buffer parity
  // flips from one tile to the next (par); every other mode keeps par = 0.
  int par = 0;
  auto stage_buf = [&](int s) -> uint8_t * {
    if constexpr (kAllRes) return L_stage0 + LM::stage_at(s);
    return ((s + par) & 1) ? L_stage1 : L_stage0;
  };
  // the boundary between two stages of a tile
  auto next_stage = [&]() {
    if constexpr (!kAllRes) stage_sync();
  };
  // resident weights of the slot loop and all biases, once per workgroup
  const int lane0 = threadIdx.x & 63;
#define FILL0(s) lds_copy<LM::stage_bytes(s)>(stage_buf(s), a.packed + a.stage_off[s], wave, lane0)
  // bf16: [T1A | T2 (bf16)]; fp8: [T1A | T2 (fp8, 2 KiB fragments) | T2 row scales]
  constexpr bool kFp8 = PREC == GN_FP8_T;
  // fragment reads held ahead of their MFMAs (layer, mm): everywhere in bf16;
  // in fp8 everywhere but T3 and B's first layer (it spills there)
  constexpr bool kEarly = true, kEarlyT3B1 = !kFp8;
  constexpr int kT1ABytes = LM::kT1A;   // K=16 fragments of 512 B
  if constexpr (kSlots) {
    if (kFp8) {
      constexpr int64_t t1a = kT1ABytes;
      lds_fill(L_res, a.packed + a.res_off, t1a, wave, lane0);
      lds_fill(L_res + t1a, a.packed + a.t2q_off, res_bytes - t1a, wave, lane0);
    } else {
      lds_fill(L_res, a.packed + a.res_off, res_bytes, wave, lane0);
    }
  }
  lds_fill((uint8_t *)L_bias, a.packed + a.bias_off, Shape<W>::kBiasBytes, wave, lane0);
  if ((int)blockIdx.x < a.ntiles) {
    // FULL streams every stage; BEGIN (without encoding) and ACC keep their
    // few stages resident for the whole launch; BEGIN with encoding streams
    // its four stages per tile; FINISH starts its pipeline at T3's stage.
    if constexpr (kAllRes) lds_copy<LM::kAll>(L_stage0, a.packed, wave, lane0);
    else if constexpr (MODE == FWD_FULL) FILL0(sF1);
    if constexpr (MODE == FWD_BEGIN) {
      FILL0(sF1);
      if constexpr (PE == 0) FILL0(sF3);
    }
    if constexpr (MODE == FWD_ACC) FILL0(sT1S);
    if constexpr (MODE == FWD_FINISH) FILL0(sT3);
  }
  wait_vm();
  __syncthreads();

  const uint8_t *T1A = L_res;
  const uint8_t *T2 = L_res + kT1ABytes;                           // bf16 form
  float *T2scale = (float *)(L_res + kT1ABytes + MT * 2 * kFrag);  // fp8 form
  if (kFp8 && kSlots) {
    // dequantisation factor s of the fp8 layer (weight row scale x activation
    // scale), and that layer's bias divided by it: the slot loop sums
    // relu(acc + c2 / s) = relu(s acc + c2) / s (s > 0) and the pool
    // multiplies by s once
    if ((int)threadIdx.x < W) {
      const float sc = T2scale[threadIdx.x] * a.sa;
      T2scale[threadIdx.x] = sc;
      L_bias[L_T2 * W + threadIdx.x] /= sc;
    }
    __syncthreads();
  }
  const float *bF1 = L_bias + L_F1 * W, *bF2 = L_bias + L_F2 * W, *bF3 = L_bias + L_F3 * W;
  const float *bT1 = L_bias + L_T1 * W, *bT2 = L_bias + L_T2 * W, *bT3 = L_bias + L_T3 * W;
  const float *bB1 = L_bias + L_B1 * W, *bB2 = L_bias + L_B2 * W, *bB3 = L_bias + L_B3 * W;
  const float *bR1 = L_bias + L_R1 * W, *bR2 = L_bias + L_R2 * W, *bR3 = L_bias + L_R3 * W;
  const int64_t f1_bytes = (int64_t)MT * kFrag;          // F1 precedes F2 in stage 0
  const int64_t r1p_bytes = (int64_t)MT * KS * kFrag;    // R1P precedes R1L in stage 8
  const int64_t r2_bytes = (int64_t)MT * KS * kFrag;     // R2 precedes R3 in stage 9

  // ---- tile -> frame pointers, first pixel
  // Frame pointers in the global address space: loads and stores through
  // them are global (vector-memory counter only).  Through generic pointers
  // they would be flat operations, which also count against the LDS counter,
  // so every wait for an LDS fragment would also wait for the HBM loads in
  // flight (the prefetched slot inputs among them).
  struct TileInfo {
    gcfloat *G, *L, *S;
    gfloat *O;
    int hw, K, q0;
  };
  auto resolve = [&](int tile) {
    TileInfo ti;
    if (a.tiles) {
      // (the tables come through vector loads: without the move to scalar
      // registers every later load would first check whether they have landed)
      const TileRef tr = a.tiles[tile];
      const FrameDesc fd = a.frames[uniform(tr.frame)];
      ti.G = (gcfloat *)uniform(fd.g); ti.L = (gcfloat *)uniform(fd.L);
      ti.S = (gcfloat *)uniform(fd.s); ti.O = (gfloat *)uniform(fd.out);
      ti.hw = uniform(fd.hw); ti.K = uniform(fd.k);
      ti.q0 = uniform(tr.q0);
    } else {
      const int f = tile / a.tiles_per_frame;
      ti.hw = a.b.hw;
      ti.K = a.b.k;
      ti.q0 = (tile - f * a.tiles_per_frame) * kTilePx;
      ti.G = (gcfloat *)(a.b.gbuf + (size_t)f * kNG * ti.hw);
      ti.L = (gcfloat *)(a.b.layers + (size_t)f * ti.K * kNL * ti.hw);
      ti.S = (gcfloat *)(a.b.scene + (size_t)f * kNS);
      ti.O = (gfloat *)(a.b.out + (size_t)f * kNOUT * ti.hw);
    }
    return ti;
  };
  // F's input (G-buffer planes 0..13, scene 0..15, zero pad) of a tile: lane
  // group g holds columns 8g..8g+7 of its pixel.  Loaded one tile ahead, from
  // selected addresses: with a branch per kind of column every load waited for
  // the one before it (FWD_BEGIN at 512^2: 40 us, now 27).
  auto load_x = [&](const TileInfo &ti, int ln, float (&xr)[kNT][8]) {
    const int gg = ln >> 4, cc = ln & 15;
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      const int q = ti.q0 + wave * (kNT * 16) + t * 16 + cc;
      const int qq = q < ti.hw ? q : ti.hw - 1;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int c = 8 * gg + j;
        uint64_t p = (uint64_t)(c < kNG ? ti.G + ((size_t)c * ti.hw + qq)
                                        : ti.S + min(c - kNG, kNS - 1));
        asm volatile("" : "+v"(p));     // (else the compiler makes the branches again)
        xr[t][j] = *(gcfloat *)p;
      }
    }
  };
  // zeroes the pad columns where the values are used
  auto pad_x = [&](int ln, float (&xr)[kNT][8]) {
#pragma unroll
    for (int t = 0; t < kNT; ++t)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (24 + j >= kNG + kNS) xr[t][j] = (ln >> 4) == 3 ? 0.0f : xr[t][j];
  };
  // Canonical slot order (FULL mode, if the handle asks for it): each
  // pixel's slots are pooled in an order that depends only on their records,
  // so the rounding of the running sum cannot depend on the order the caller
  // passed them in.  With up to kFastK slots the tile's alphas are copied to
  // LDS during F's last layer and ranked at the start of the slot stage.
  constexpr int kFastK = 8;
  // this lane's pieces of a tile's streaming state
  using ST = StreamTile<W>;
  auto st_rsrc = [&](int tile) {
    return __builtin_amdgcn_make_buffer_rsrc(a.state + (size_t)tile * ST::kBytes, (short)0,
                                             (int)ST::kBytes, 0x00020000);
  };
  auto st_px = [&](int ln, int t) { return wave * (kNT * 16) + t * 16 + (ln & 15); };
  const bool dense = MODE != FWD_FULL && a.dense;
  const int st_next = dense ? kFrag : 64;            // from a lane's vector to its next
  auto st_lane = [&](int ln, int t, int px_bytes) {
    return (wave * kNT + t) * 16 * px_bytes + (ln & 15) * (dense ? 16 : px_bytes) +
           (ln >> 4) * (dense ? 256 : 16);
  };
  auto st_sig = [&](int ln, int t) { return st_lane(ln, t, W * 2); };
  auto st_z = [&](int ln, int t) { return (int)ST::kSig + st_lane(ln, t, W * 4); };
  auto st_cnt = [&](int ln, int t) { return (int)(ST::kSig + ST::kZ) + st_px(ln, t) * 4; };
  auto load_cnt = [&](int tile, int ln, float (&c)[kNT]) {
    const auto r = st_rsrc(tile);
#pragma unroll
    for (int t = 0; t < kNT; ++t)
      c[t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                           r, a.state_load ? st_cnt(ln, t) : kOutside, 0, 0));
  };
  // ACC: the largest alpha of a tile's pixels over the call's objects (NaN
  // counts as inactive, as in the slot loop); loaded one tile ahead, as the
  // counts are.
  auto load_alpha = [&](const TileInfo &ti, int ln, float (&al)[kNT]) {
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      const int q = min(ti.q0 + st_px(ln, t), ti.hw - 1);
      al[t] = ti.L[(size_t)kAlpha * ti.hw + q];
      for (int j = 1; j < ti.K; ++j)
        al[t] = fmaxf(al[t], ti.L[((size_t)j * kNL + kAlpha) * ti.hw + q]);
    }
  };
  // FINISH: the running sum of the pixels that have one (dense: of all)
  auto load_z = [&](int tile, int ln, const float (&c)[kNT], f32x4 (&z)[kNT][MT]) {
    const auto r = st_rsrc(tile);
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      const int off = (dense ? a.state_load != 0 : c[t] > 0.0f) ? st_z(ln, t) : kOutside;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        z[t][mt] = __builtin_bit_cast(f32x4, state_load16(r, off, mt * st_next));
    }
  };
  float xr[kNT][8];
  float nal[kNT], ncnt[kNT];   // ACC: load_alpha's values; ACC, FINISH: the counts
  f32x4 nz[kNT][MT];           // FINISH: the next tile's running sum
  TileInfo nti;
  if ((int)blockIdx.x < a.ntiles) {
    nti = resolve(blockIdx.x);
    if constexpr (kTrunk) load_x(nti, lane0, xr);
    if constexpr (MODE == FWD_ACC)
      if (!dense) load_alpha(nti, lane0, nal);
    if constexpr (MODE == FWD_ACC || MODE == FWD_FINISH) load_cnt(blockIdx.x, lane0, ncnt);
    if constexpr (MODE == FWD_FINISH) load_z(blockIdx.x, lane0, ncnt, nz);
  }

  for (int tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x) {
    const bool has_next = tile + (int)gridDim.x < a.ntiles;
    // Opaque per-tile copies of the lane id and the packed-weight base keep
    // the compiler from hoisting every derived address (staging sources of
    // all stages, channel masks) out of the tile loop and holding them in
    // registers for its whole length.
    int lane = threadIdx.x & 63;
    const uint8_t *packed = a.packed;
    asm volatile("" : "+v"(lane), "+s"(packed));
    const int g = lane >> 4, col = lane & 15;
#define FILL(s) \
  if constexpr (!kAllRes) \
  lds_copy<LM::stage_bytes(s)>(stage_buf(s), packed + a.stage_off[s], wave, lane)
    // ---- the tile's frame (resolved one tile ahead)
    const TileInfo ti = nti;
    gcfloat *Gp = ti.G, *Lp = ti.L;
    gfloat *Op = ti.O;
    const int hw = ti.hw, K = ti.K, q0 = ti.q0;
    int qc[kNT];
    bool valid[kNT];
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      const int q = q0 + wave * (kNT * 16) + t * 16 + col;
      valid[t] = q < hw;
      qc[t] = valid[t] ? q : hw - 1;          // tail lanes recompute a real pixel
    }
    u32x4 sig[kNT][KS];   // sigma: from F (FULL, BEGIN) or from the state (ACC)
    f32x4 Z[kNT][MT];     // running masked sum of h's hidden layer, and
    float cnt[kNT];       // the number of active slots it holds
    bool touched[kNT];    // ACC: an object of this call covers the pixel
    if constexpr (MODE == FWD_ACC) {
      bool any = false;
#pragma unroll
      for (int t = 0; t < kNT; ++t) {
        touched[t] = dense || nal[t] > 0.0f;
        cnt[t] = ncnt[t];
        any = any || touched[t];
      }
      if (has_next) {
        nti = resolve(tile + gridDim.x);
        if (!dense) load_alpha(nti, lane, nal);
        load_cnt(tile + gridDim.x, lane, ncnt);
      }
      // no pixel of this wave's part takes part: only a first call's counts
      // are left to write
      if (!dense && __builtin_amdgcn_ballot_w64(any) == 0) {
        if (!a.state_load && g == 0) {
          const auto sr = st_rsrc(tile);
#pragma unroll
          for (int t = 0; t < kNT; ++t)
            __builtin_amdgcn_raw_buffer_store_b32(0u, sr, st_cnt(lane, t), 0, 0);
        }
        continue;
      }
    }

    // FULL: sigma is needed again only by B's first layer: park it in this wave's
    // scratch instead of holding 32 registers through the slot loop
    // (LDS left free by the weights holds it for the first sig_lds_waves
    // waves; the others use a per-wave slot in HBM)
    constexpr int kSigBytes = kNT * KS * kFrag;
    // Both stage buffers hold only stages 1-4's fragments (stage_max bytes or
    // fewer) while sigma is parked, so their tails serve the last waves.
    const bool sig_in_lds = wave < a.sig_lds_waves;
    const int nfree = a.sig_lds_waves - a.sig_tail_waves;
    uint8_t *sig_lds = wave < nfree ? L_sig + (size_t)wave * kSigBytes
                                    : ((wave - nfree) & 1 ? L_stage1 : L_stage0) + stage_max -
                                          (size_t)(1 + (wave - nfree) / 2) * kSigBytes;
    uint8_t *sig_slot = a.sig_scratch + ((size_t)blockIdx.x * kWaves + wave) * kSigBytes;

    // The tile's alphas, slot by slot, into the LDS alpha table (canonical
    // order with up to kFastK slots): 64-pixel blocks, lane i copying pixel i
    // of its block (clamped to the frame).  Issued with F's second layer and
    // ranked before its last.
    const bool canon_fast = MODE == FWD_FULL && a.canon && K > 1 && K <= kFastK;
    auto copy_alphas = [&]() {
      constexpr int kBlk = kTilePx / 64;
      for (int b = wave; b < kBlk * K; b += kWaves) {
        const int j = b / kBlk, p0 = b % kBlk * 64;
        const int q = min(q0 + p0 + lane, hw - 1);
        __builtin_amdgcn_global_load_lds(
            (const void *)(Lp + ((size_t)j * kNL + kAlpha) * hw + q),
            (__attribute__((address_space(3))) void *)(L_alpha + j * kTilePx + p0), 4, 0, 0);
      }
    };

    // BEGIN: the next tile's F input, requested ahead of this tile's stores
    // (loads issued behind stores wait for them)
    auto next_x = [&]() {
      if (!has_next) return;
      nti = resolve(tile + gridDim.x);
      load_x(nti, lane, xr);
    };

    if constexpr (kTrunk) {
      u32x4 h2[kNT][KS];
      if constexpr (PE == 0) {
        // ================= stage 0: F layers 1-2 =================
        // (xr is read before the copies are issued: waiting for it behind them
        // would wait for them too)
        u32x4 x[kNT][1];
        pad_x(lane, xr);
#pragma unroll
        for (int t = 0; t < kNT; ++t)
          x[t][0] = u32x4{pk_bf16(xr[t][0], xr[t][1]), pk_bf16(xr[t][2], xr[t][3]),
                          pk_bf16(xr[t][4], xr[t][5]), pk_bf16(xr[t][6], xr[t][7])};
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MODE == FWD_FULL) FILL(sF3);
        if constexpr (MODE == FWD_BEGIN) next_x();
        if (canon_fast) copy_alphas();
        {
          const uint8_t *S = stage_buf(sF1);
          u32x4 h1[kNT][KS];
          layer<MT, 1, true, kEarly>(h1, S, x, bF1, g, lane);
          layer<MT, KS, true, kEarly>(h2, S + f1_bytes, h1, bF2, g, lane);
        }
        if constexpr (MODE == FWD_FULL) {
          stage_sync();
        }
      } else {
        // ====== stages 0-1: F layer 1 on the encoded input; stage 2: F layer 2 ======
        pad_x(lane, xr);
        __builtin_amdgcn_sched_barrier(0);
        FILL(sF1B);
        f32x4 acc[kNT][MT];
        bias_init(acc, bF1, g);
        {
          u32x4 x[kNT][kF1A];
          enc_frags<0, kF1A>(xr, x);
          mm<MT, kF1A, kEarly>(acc, stage_buf(sF1), x, lane);
        }
        stage_sync();
        FILL(sF2);
        u32x4 h1[kNT][KS];
        {
          u32x4 x[kNT][kF1B];
          enc_frags<kF1A, kF1B>(xr, x);
          mm<MT, kF1B, kEarly>(acc, stage_buf(sF1B), x, lane);
          to_frags<MT, true>(acc, h1);
        }
        stage_sync();
        FILL(sF3);
        if (canon_fast) copy_alphas();
        layer<MT, KS, true, kEarly>(h2, stage_buf(sF2), h1, bF2, g, lane);
        stage_sync();
      }

      // ================= F layer 3 -> sigma =================
      if constexpr (MODE == FWD_FULL) FILL(sT1S);
      // Canonical order of each pixel's slots, into this wave's part of the
      // LDS table (byte r of a pixel's entry: its slot of rank r).  Keys: the
      // bits of alpha for active slots, 0xFFFFFF00 + j for an inactive slot j
      // (above every active key, distinct), 0xFFFFFFFF past K.  With up to
      // kFastK slots each lane ranks its lane group's slots g and g + 4 from the
      // alphas in LDS (they landed by the last barrier); two active slots of
      // equal alpha (and more than kFastK slots) take the full comparison of
      // slot_order.h.  (All reads are unconditional: one behind a branch on K
      // is waited for before the next.)
      if (MODE == FWD_FULL && a.canon && K > 1) {
        uint8_t *perm_px[kNT];
#pragma unroll
        for (int t = 0; t < kNT; ++t)
          perm_px[t] = L_perm + (size_t)(wave * (kNT * 16) + t * 16 + col) * a.kpad;
        if (K <= kFastK) {
          float alk[kNT][kFastK];
#pragma unroll
          for (int t = 0; t < kNT; ++t)
#pragma unroll
            for (int j = 0; j < kFastK; ++j)
              alk[t][j] = L_alpha[min(j, K - 1) * kTilePx + wave * (kNT * 16) + t * 16 + col];
          unsigned slow = 0;
#pragma unroll
          for (int t = 0; t < kNT; ++t) {
            uint32_t key[kFastK];
#pragma unroll
            for (int j = 0; j < kFastK; ++j)
              key[j] = j >= K ? 0xFFFFFFFFu
                              : (alk[t][j] > 0.0f ? __float_as_uint(alk[t][j]) : 0xFFFFFF00u + j);
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
              const int i = g + 4 * sl;
              uint32_t ki = key[4 * sl];
#pragma unroll
              for (int jj = 1; jj < 4; ++jj) ki = g == jj ? key[4 * sl + jj] : ki;
              int lt = 0, le = 0;
#pragma unroll
              for (int j = 0; j < kFastK; ++j) {
                lt += key[j] < ki ? 1 : 0;
                le += key[j] <= ki ? 1 : 0;
              }
              if (i < K) {
                if (le == lt + 1)
                  perm_px[t][lt] = ki >= 0xFFFFFF00u ? (uint8_t)0xFF : (uint8_t)i;
                else
                  slow |= 1u << (2 * t + sl);
              }
            }
          }
          if (__builtin_amdgcn_ballot_w64(slow != 0)) {
#pragma unroll
            for (int t = 0; t < kNT; ++t)
#pragma unroll
              for (int sl = 0; sl < 2; ++sl)
                if (slow & (1u << (2 * t + sl)))
                  perm_px[t][slot_rank(Lp + qc[t], (size_t)hw, K, g + 4 * sl)] =
                      slot_active(Lp + qc[t], hw, g + 4 * sl) ? (uint8_t)(g + 4 * sl) : (uint8_t)0xFF;
          }
        } else {
#pragma unroll
          for (int t = 0; t < kNT; ++t)
            for (int i = g; i < K; i += 4)
              perm_px[t][slot_rank(Lp + qc[t], (size_t)hw, K, i)] =
                  slot_active(Lp + qc[t], hw, i) ? (uint8_t)i : (uint8_t)0xFF;
        }
        // the wave reads the table back in its own slot loop (LDS operations of
        // one wave complete in order)
      }
      // the alpha table shares sigma's parking area: every wave has read it
      // before any wave parks sigma there
      if (canon_fast && a.alpha_alias) __syncthreads();
      if constexpr (MODE == FWD_BEGIN && PE > 0) {
        if (has_next) FILL(sF1);      // the next tile's first stage
        next_x();
      }
      layer<MT, KS, false, kEarly>(sig, stage_buf(sF3), h2, bF3, g, lane);
      if constexpr (MODE == FWD_BEGIN) {
        // sigma goes to the streaming state
        const auto sr = st_rsrc(tile);
#pragma unroll
        for (int t = 0; t < kNT; ++t)
#pragma unroll
          for (int k = 0; k < KS; ++k) state_store16(sr, st_sig(lane, t), k * st_next, sig[t][k]);
        if constexpr (PE > 0) {
          // the next tile's first stage has landed; this stage's buffer is free
          next_stage();
        }
      } else {
        if (sig_in_lds) {
#pragma unroll
          for (int t = 0; t < kNT; ++t)
#pragma unroll
            for (int k = 0; k < KS; ++k) *(u32x4 *)(sig_lds + (t * KS + k) * kFrag + lane * 16) = sig[t][k];
        } else {
#pragma unroll
          for (int t = 0; t < kNT; ++t)
#pragma unroll
            for (int k = 0; k < KS; ++k) *(u32x4 *)(sig_slot + (t * KS + k) * kFrag + lane * 16) = sig[t][k];
        }
        // the kNT x KS stores above stay in flight; the same wave reads them back
        // in stage 3, after stage 2's full wait
        if constexpr (!kAllRes) {
          if (sig_in_lds)
            stage_sync_after_stores<0>();
          else
            stage_sync_after_stores<kNT * KS>();
        }
      }
    }

    if constexpr (kSlots) {
      // ================= stage 2: u = W1s sigma + c1, then the slot loop =======
      if constexpr (MODE == FWD_FULL) FILL(sT3);
      if constexpr (MODE == FWD_ACC) {
        // sigma, and the running sum that earlier calls left
        const auto sr = st_rsrc(tile);
#pragma unroll
        for (int t = 0; t < kNT; ++t) {
          const int off = touched[t] ? st_sig(lane, t) : kOutside;
#pragma unroll
          for (int k = 0; k < KS; ++k) sig[t][k] = state_load16(sr, off, k * st_next);
        }
#pragma unroll
        for (int t = 0; t < kNT; ++t) {
          const bool has = dense ? a.state_load != 0 : touched[t] && cnt[t] > 0.0f;
          const int off = has ? st_z(lane, t) : kOutside;
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            Z[t][mt] = __builtin_bit_cast(f32x4, state_load16(sr, off, mt * st_next));
        }
      }
      {
        // the slot-order table of this tile (written above): the lane's pixel
        // of N-tile t has its entry at byte pofs + 16 t kpad
        const bool canon = MODE == FWD_FULL && a.canon && K > 1;
        const uint32_t pofs = (uint32_t)(wave * (kNT * 16) + col) * a.kpad;
        // Slot inputs: lane group g < 3 carries planes 4g..4g+3 of its pixel (the
        // K=16 operand of h's first layer; with encoding, lane group g carries
        // planes 3g..3g+2 and their encodings); the next slot's planes are
        // loaded one slot ahead so their latency overlaps the current slot's work.
        constexpr int kRaw = PE > 0 ? 3 : 4;
        float nxt[kNT][kRaw];
        // Iteration i takes each pixel's slot of rank i (canonical order) or
        // slot i (input order).  In canonical order the inactive slots come
        // last and their table bytes are 0xFF: such a pixel loads nothing and
        // presents zeros (alpha 0: its term is masked out exactly), so half the
        // loads of the workloads' slot stage never reach the memory system.
        auto load_slot = [&](int i) {
          uint32_t qs[kNT];      // element offsets (frames of the MFMA path stay below 2^32)
          bool act[kNT];
#pragma unroll
          for (int t = 0; t < kNT; ++t) {
            const int si = canon ? (int)L_perm[pofs + t * 16 * a.kpad + i] : i;
            act[t] = MODE == FWD_ACC ? touched[t] : si != 0xFF;
            qs[t] = (uint32_t)si * (uint32_t)(kNL * hw) + (uint32_t)qc[t];
            asm volatile("" : "+v"(qs[t]));   // per-slot addresses stay in the loop body
          }
#pragma unroll
          for (int t = 0; t < kNT; ++t)
#pragma unroll
            for (int j = 0; j < kRaw; ++j) {
              if constexpr (PE > 0)
                nxt[t][j] = act[t] ? Lp[(size_t)(3 * g + j) * hw + qs[t]] : 0.0f;
              else
                nxt[t][j] = g < 3 && act[t] ? Lp[(size_t)(4 * g + j) * hw + qs[t]] : 0.0f;
            }
        };
        if (K > 0) load_slot(0);
        // u = W1s sigma + c1 in fp32 accumulator layout: the C operand of h's
        // first layer for every slot
        f32x4 u[kNT][MT];
        bias_init(u, bT1, g);
        mm<MT, KS, kEarly>(u, stage_buf(sT1S), sig, lane);

        if constexpr (kFp8) {
          // fp8: h's first layer runs in units of the activation scale (its
          // inputs b_i and u are divided by it), so its output quantises directly
#pragma unroll
          for (int t = 0; t < kNT; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) u[t][mt] *= a.inv_sa;
        }
        if constexpr (MODE == FWD_FULL) {
#pragma unroll
          for (int t = 0; t < kNT; ++t) {
            cnt[t] = 0.0f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) Z[t][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        }
        for (int i = 0; i < K; ++i) {
          float cur[kNT][kRaw];
#pragma unroll
          for (int t = 0; t < kNT; ++t)
#pragma unroll
            for (int j = 0; j < kRaw; ++j) cur[t][j] = nxt[t][j];
          if (i + 1 < K) load_slot(i + 1);
          // A slot in which no pixel of this wave takes part adds exactly zero
          // to the running sum and the count: skip its two layers.  The lanes
          // that loaded alpha decide (lane group 2 position 1, or with
          // encoding lane group 3 position 0).
          bool any = false;
#pragma unroll
          for (int t = 0; t < kNT; ++t)
            any = any || (PE > 0 ? (g == 3 && cur[t][0] > 0.0f) : (g == 2 && cur[t][1] > 0.0f));
          if (__builtin_amdgcn_ballot_w64(any) == 0) continue;
          uint2 bi[kNT][kNK16];
          float m[kNT];
#pragma unroll
          for (int t = 0; t < kNT; ++t) {
            if constexpr (PE > 0) {
              // value v = 4 s + j of the lane group's list: block v / 3 of raw
              // plane 3 g + v % 3 (zero past the last block)
              float enc[3][kE];
#pragma unroll
              for (int c = 0; c < 3; ++c) pe_blocks_of<kE>(cur[t][c], enc[c]);
              float e[4 * kNK16];
#pragma unroll
              for (int v = 0; v < 4 * kNK16; ++v) {
                const float x = v / 3 < kE ? enc[v % 3][v / 3] : 0.0f;
                e[v] = kFp8 ? x * a.inv_sa : x;
              }
#pragma unroll
              for (int st = 0; st < kNK16; ++st)
                bi[t][st] = uint2{pk_bf16(e[4 * st], e[4 * st + 1]),
                                  pk_bf16(e[4 * st + 2], e[4 * st + 3])};
              // alpha (plane 9) sits in lane group 3 at position 0: broadcast it
              const float al = __int_as_float(
                  __builtin_amdgcn_ds_bpermute((col + 48) * 4, __float_as_int(cur[t][0])));
              m[t] = al > 0.0f ? 1.0f : 0.0f;
            } else {
              if constexpr (kFp8)
                bi[t][0] = uint2{pk_bf16(cur[t][0] * a.inv_sa, cur[t][1] * a.inv_sa),
                                 pk_bf16(cur[t][2] * a.inv_sa, cur[t][3] * a.inv_sa)};
              else
                bi[t][0] = uint2{pk_bf16(cur[t][0], cur[t][1]), pk_bf16(cur[t][2], cur[t][3])};
              // alpha (plane 9) sits in lane group 2 at position 1: broadcast it
              const float al = __int_as_float(
                  __builtin_amdgcn_ds_bpermute((col + 32) * 4, __float_as_int(cur[t][1])));
              m[t] = al > 0.0f ? 1.0f : 0.0f;
            }
          }
          if constexpr (kFp8) {
          // h layer 1 (bf16 MFMA, in activation-scale units), quantised to
          // E4M3: lane byte 4*mt + r holds row 16*mt + 4*g + r, the order the
          // fp8 weights of layer 2 were packed in.
          i32x8 zq[kNT];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            if constexpr (PE > 0) {
              f32x4 acc1[kNT];
#pragma unroll
              for (int t = 0; t < kNT; ++t) acc1[t] = u[t][mt];
#pragma unroll
              for (int st = 0; st < kNK16; ++st) {
                const uint2 w = ld_frag16(T1A, mt * kNK16 + st, lane);
#pragma unroll
                for (int t = 0; t < kNT; ++t) acc1[t] = mma16(w, bi[t][st], acc1[t]);
              }
#pragma unroll
              for (int t = 0; t < kNT; ++t) zq[t][mt] = relu_pack_fp8x4(acc1[t]);
            } else {
              const uint2 w = ld_frag16(T1A, mt, lane);
#pragma unroll
              for (int t = 0; t < kNT; ++t)
                zq[t][mt] = relu_pack_fp8x4(mma16(w, bi[t][0], u[t][mt]));
            }
          }
          __builtin_amdgcn_s_setprio(1);   // as for the bf16 layer 2 below
          // h layer 2 on the fp8 matrix cores (K = 128 in one instruction),
          // the running sum kept in units of the dequantisation factor s
          // (applied at the pool); each M-tile's fragment is requested one
          // M-tile ahead of its MFMAs.
          i32x8 wn = ld_frag8(T2, 0, lane);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const i32x8 w = wn;
            if (mt + 1 < MT) wn = ld_frag8(T2, mt + 1, lane);
            const f32x4 b = *(const f32x4 *)(bT2 + 16 * mt + 4 * g);     // c2 / s
#pragma unroll
            for (int t = 0; t < kNT; ++t) {
              const f32x4 r = relu4(mma_fp8(w, zq[t], b));
              Z[t][mt].x = fmaf(m[t], r.x, Z[t][mt].x);
              Z[t][mt].y = fmaf(m[t], r.y, Z[t][mt].y);
              Z[t][mt].z = fmaf(m[t], r.z, Z[t][mt].z);
              Z[t][mt].w = fmaf(m[t], r.w, Z[t][mt].w);
            }
          }
          } else {
          // h layer 1: z1 = relu(W1b b_i + u)
          u32x4 z1[kNT][KS];
#pragma unroll
          for (int p = 0; p < KS; ++p) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              f32x4 acc1[kNT];
              if constexpr (PE > 0) {
#pragma unroll
                for (int t = 0; t < kNT; ++t) acc1[t] = u[t][2 * p + h];
#pragma unroll
                for (int st = 0; st < kNK16; ++st) {
                  const uint2 w = ld_frag16(T1A, (2 * p + h) * kNK16 + st, lane);
#pragma unroll
                  for (int t = 0; t < kNT; ++t) acc1[t] = mma16(w, bi[t][st], acc1[t]);
                }
              } else {
                const uint2 w = ld_frag16(T1A, 2 * p + h, lane);
#pragma unroll
                for (int t = 0; t < kNT; ++t) acc1[t] = mma16(w, bi[t][0], u[t][2 * p + h]);
              }
#pragma unroll
              for (int t = 0; t < kNT; ++t) {
                const f32x4 v = acc1[t];
                z1[t][p][2 * h] = relu_bf16x2(pk_bf16(v.x, v.y));
                z1[t][p][2 * h + 1] = relu_bf16x2(pk_bf16(v.z, v.w));
              }
            }
          }
          // h layer 2 at raised wave priority: of the two waves that share a
          // SIMD, the one in this layer issues first, which offsets the pair
          // so that one's matrix-core work overlaps the other's layer 1 and
          // LDS reads (1-1.5% of the 512^2 K = 8 frame in bf16, ~1% in fp8;
          // issuing the next M-tile's MFMAs before each M-tile's relu and
          // running sum was slower in both forms).
          __builtin_amdgcn_s_setprio(1);
          // h layer 2 and the masked running sum: Z += m * relu(A2 z1 + c2).
          // The fragments stream one K-step ahead of the MFMAs that use them.
          u32x4 wnext = ld_frag(T2, 0, lane);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const f32x4 b = *(const f32x4 *)(bT2 + 16 * mt + 4 * g);
            f32x4 acc[kNT];
#pragma unroll
            for (int t = 0; t < kNT; ++t) acc[t] = b;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
              const u32x4 w = wnext;
              if (mt * KS + ks + 1 < MT * KS) wnext = ld_frag(T2, mt * KS + ks + 1, lane);
#pragma unroll
              for (int t = 0; t < kNT; ++t) acc[t] = mma(w, z1[t][ks], acc[t]);
            }
#pragma unroll
            for (int t = 0; t < kNT; ++t) {
              const f32x4 r = relu4(acc[t]);    // one v_med3 each
              Z[t][mt].x = fmaf(m[t], r.x, Z[t][mt].x);
              Z[t][mt].y = fmaf(m[t], r.y, Z[t][mt].y);
              Z[t][mt].z = fmaf(m[t], r.z, Z[t][mt].z);
              Z[t][mt].w = fmaf(m[t], r.w, Z[t][mt].w);
            }
          }
          }
#pragma unroll
          for (int t = 0; t < kNT; ++t) cnt[t] += m[t];
          __builtin_amdgcn_s_setprio(0);
        }
      }
      if constexpr (MODE == FWD_ACC) {
        const auto sr = st_rsrc(tile);
#pragma unroll
        for (int t = 0; t < kNT; ++t) {
          // (Z is zero in pixels that stay without objects, and left unwritten)
          const int off = touched[t] ? st_z(lane, t) : kOutside;
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            state_store16(sr, off, mt * st_next, __builtin_bit_cast(u32x4, Z[t][mt]));
          __builtin_amdgcn_raw_buffer_store_b32(
              __builtin_bit_cast(uint32_t, cnt[t]), sr,
              g == 0 && (touched[t] || !a.state_load) ? st_cnt(lane, t) : kOutside, 0, 0);
        }
      } else {
        next_stage();
      }
    }

    if constexpr (kHead) {
      // ================= stage 3: pool and h layer 3 -> tau =================
      u32x4 sig2[kNT][KS];
      if constexpr (MODE == FWD_FINISH) {
        // the pool state (requested a tile ahead) and sigma come from the
        // streaming state
        const auto sr = st_rsrc(tile);
#pragma unroll
        for (int t = 0; t < kNT; ++t) {
          cnt[t] = ncnt[t];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) Z[t][mt] = nz[t][mt];
#pragma unroll
          for (int k = 0; k < KS; ++k) sig2[t][k] = state_load16(sr, st_sig(lane, t), k * st_next);
        }
      } else if (sig_in_lds) {
#pragma unroll
        for (int t = 0; t < kNT; ++t)
#pragma unroll
          for (int k = 0; k < KS; ++k)
            sig2[t][k] = *(const u32x4 *)(sig_lds + (t * KS + k) * kFrag + lane * 16);
      } else {
#pragma unroll
        for (int t = 0; t < kNT; ++t)
#pragma unroll
          for (int k = 0; k < KS; ++k)
            sig2[t][k] = *(gu32x4 *)(sig_slot + (t * KS + k) * kFrag + lane * 16);
      }
      __builtin_amdgcn_sched_barrier(0);
      FILL(sB1S);
      u32x4 tau[kNT][KS];
      {
        // fp8: the running sum is in units of the dequantisation factor s
        // (weight row scale x activation scale) of the slot loop's fp8 layer
        f32x4 s8[MT];
        if constexpr (kFp8) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            if constexpr (MODE == FWD_FULL)
              s8[mt] = *(const f32x4 *)(T2scale + 16 * mt + 4 * g);
            else
              s8[mt] = *(const f32x4 *)((const float *)(a.packed + a.t2s_off) + 16 * mt + 4 * g) *
                       a.sa;
          }
        }
        u32x4 zs[kNT][KS];
        f32x4 acc[kNT][MT];
#pragma unroll
        for (int t = 0; t < kNT; ++t) {
          const bool mean = a.pool == GN_POOL_MEAN;
          const float inv = mean ? 1.0f / fmaxf(cnt[t], 1.0f) : 1.0f;
          const float bs = mean ? (cnt[t] > 0.0f ? 1.0f : 0.0f) : cnt[t];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const f32x4 v = kFp8 ? (Z[t][mt] * s8[mt]) * inv : Z[t][mt] * inv;
            zs[t][mt >> 1][2 * (mt & 1)] = pk_bf16(v.x, v.y);
            zs[t][mt >> 1][2 * (mt & 1) + 1] = pk_bf16(v.z, v.w);
            acc[t][mt] = *(const f32x4 *)(bT3 + 16 * mt + 4 * g) * bs;
          }
        }
        mm<MT, KS, kEarlyT3B1>(acc, stage_buf(sT3), zs, lane);
        to_frags<MT, false>(acc, tau);
      }
      next_stage();

      // ================= stages 4-5: B layer 1 on [sigma; tau] =================
      FILL(sB1T);
      f32x4 accB[kNT][MT];
      bias_init(accB, bB1, g);
      mm<MT, KS, kEarlyT3B1>(accB, stage_buf(sB1S), sig2, lane);
      next_stage();

      FILL(sB2);
      u32x4 hb[kNT][KS];
      mm<MT, KS, kEarlyT3B1>(accB, stage_buf(sB1T), tau, lane);
      to_frags<MT, true>(accB, hb);
      next_stage();

      // ================= stage 6: B layer 2 =================
      FILL(sB3);
      // L_d for R's first layer (stage 8), requested two stages early
      float ldr[kNT][3];
#pragma unroll
      for (int t = 0; t < kNT; ++t)
#pragma unroll
        for (int c = 0; c < 3; ++c) ldr[t][c] = g == 0 ? Gp[(size_t)(11 + c) * hw + qc[t]] : 0.0f;
      {
        u32x4 hb2[kNT][KS];
        layer<MT, KS, true, kEarly>(hb2, stage_buf(sB2), hb, bB2, g, lane);
#pragma unroll
        for (int t = 0; t < kNT; ++t)
#pragma unroll
          for (int k = 0; k < KS; ++k) hb[t][k] = hb2[t][k];
      }
      next_stage();

      // ================= stage 7: B layer 3 -> phi =================
      FILL(sR1);
      u32x4 phi[kNT][KS];
      layer<MT, KS, false, kEarly>(phi, stage_buf(sB3), hb, bB3, g, lane);
      next_stage();

      // ================= stage 8: R layer 1 on [phi; L_d] =================
      FILL(sR2);
      if constexpr (MODE == FWD_FINISH) {
        if (has_next) load_cnt(tile + gridDim.x, lane, ncnt);
      }
      u32x4 hr[kNT][KS];
      {
        u32x4 ld[kNT][1];
#pragma unroll
        for (int t = 0; t < kNT; ++t)
          ld[t][0] = u32x4{pk_bf16(ldr[t][0], ldr[t][1]), pk_bf16(ldr[t][2], 0.0f), 0u, 0u};
        f32x4 acc[kNT][MT];
        bias_init(acc, bR1, g);
        mm<MT, KS, kEarly>(acc, stage_buf(sR1), phi, lane);
        mm<MT, 1, kEarly>(acc, stage_buf(sR1) + r1p_bytes, ld, lane);
        to_frags<MT, true>(acc, hr);
      }
      next_stage();

      // ================= stage 9: R layers 2-3 -> radiance =================
      if (has_next) {
        // (the tile's frame first: reading its table behind the copies would
        // wait for them)
        if constexpr (MODE == FWD_FULL) {
          nti = resolve(tile + gridDim.x);
          __builtin_amdgcn_sched_barrier(0);
          FILL(sF1);
          load_x(nti, lane, xr);
        } else {
          // the next tile's T3 stage goes to the buffer this tile's R1 stage used
          lds_copy<LM::stage_bytes(sT3)>(((sT3 + (par ^ 1)) & 1) ? L_stage1 : L_stage0,
                                         packed + a.stage_off[sT3], wave, lane);
          nti = resolve(tile + gridDim.x);
          load_z(tile + gridDim.x, lane, ncnt, nz);
        }
      }
      {
        u32x4 hr2[kNT][KS];
        layer<MT, KS, true, kEarly>(hr2, stage_buf(sR2), hr, bR2, g, lane);
        f32x4 y[kNT][1];
        bias_init(y, bR3, g);
        mm<1, KS, kEarly>(y, stage_buf(sR2) + r2_bytes, hr2, lane);
        // Lane group 0 holds rows 0..2.  Tail lanes store the value of pixel
        // hw - 1 they recomputed (bitwise the same as that pixel's own lane),
        // so exactly 3 kNT store instructions issue, with a non-empty mask.
#pragma unroll
        for (int t = 0; t < kNT; ++t) {
          if (g == 0) {
            Op[qc[t]] = y[t][0].x;
            Op[(size_t)hw + qc[t]] = y[t][0].y;
            Op[(size_t)2 * hw + qc[t]] = y[t][0].z;
          }
        }
      }
      stage_sync_after_stores<3 * kNT>();
      if constexpr (MODE == FWD_FINISH) par ^= 1;
    }
  }
#undef FILL0
#undef FILL
}

// ---- weight packing ---------------------------------------------------------
struct PackArgs {
  const float *master;
  uint8_t *packed;
  ChunkDesc chunk[kNumChunks];
  LayerOff lo[kNumLayers];
  int W;
  int64_t bias_off;
};

__device__ __forceinline__ int chain_col(int ks, int g, int j) {
  return 32 * ks + (j < 4 ? 4 * g + j : 16 + 4 * g + (j - 4));
}

// One thread per lane of a fragment (8 elements, 4 in the K = 16 chunks), one
// store; blockIdx.y: the chunk, then the biases.
__global__ __launch_bounds__(256) void pack_bf16_kernel(PackArgs p) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.y == kNumChunks) {
    const int l = e / p.W, o = e % p.W;
    if (l < kNumLayers)
      ((float *)(p.packed + p.bias_off))[e] = o < p.lo[l].out ? p.master[p.lo[l].b + o] : 0.0f;
    return;
  }
  const ChunkDesc d = p.chunk[blockIdx.y];
  const bool half = d.kmap == KMAP_MEM16 || d.kmap == KMAP_PE16;
  if (e >= d.mt * d.ks * 64) return;
  const int lane = e & 63, fragi = e >> 6;
  const int mt = fragi / d.ks, ks = fragi - mt * d.ks;
  const int row = 16 * mt + (lane & 15);
  const int g = lane >> 4;
  const LayerOff lo = p.lo[d.layer];
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    int k;
    if (d.kmap == KMAP_ENC) {
      const int c = 8 * g + j;
      k = c < d.raw ? (d.ks0 + ks) * d.raw + c : d.ncols;
    } else if (d.kmap == KMAP_PE16) {
      const int q = 4 * ks + j, blk = q / 3;
      k = blk < d.nblocks ? blk * d.raw + 3 * g + q % 3 : d.ncols;
    } else {
      k = d.kmap == KMAP_MEM     ? 32 * ks + 8 * g + j
          : d.kmap == KMAP_MEM16 ? 16 * ks + 4 * g + j
                                 : chain_col(ks, g, j);
    }
    const bool in = row < d.nrows && k < d.ncols && (j < 4 || !half);
    v[j] = in ? p.master[lo.w + (int64_t)row * lo.in + d.col0 + k] : 0.0f;
  }
  const uint2 a = {pk_bf16(v[0], v[1]), pk_bf16(v[2], v[3])};
  if (half)
    ((uint2 *)(p.packed + d.offset))[e] = a;
  else
    ((u32x4 *)(p.packed + d.offset))[e] = u32x4{a.x, a.y, pk_bf16(v[4], v[5]), pk_bf16(v[6], v[7])};
}

// fp8 copy of h's second layer (the layer that runs once per slot): per output
// row n a scale s_n = max_k |A2[n][k]| / 448 and bytes E4M3(A2[n][k] / s_n),
// stored as MT fragments of 64 lanes x 32 bytes.  Lane 16 g + (n & 15) of
// fragment n >> 4 holds, at byte 4 q + r, input k = 16 q + 4 g + r; a
// fragment keeps bytes 0-15 of every lane in its first KiB and bytes 16-31
// in its second (ld_frag8).
// One block per output row, one thread per input.
__global__ void pack_fp8_t2_kernel(PackArgs p, uint8_t *q8, float *scale) {
  __shared__ float red[256];
  const int n = blockIdx.x, k = threadIdx.x, W = p.W;
  const LayerOff lo = p.lo[L_T2];
  const float v = k < W ? p.master[lo.w + (int64_t)n * W + k] : 0.0f;
  red[k] = fabsf(v);
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (k < w) red[k] = fmaxf(red[k], red[k + w]);
    __syncthreads();
  }
  const float s = red[0] > 0.0f ? red[0] / 448.0f : 1.0f;
  if (k == 0) scale[n] = s;
  if (k >= W) return;
  const float x = fminf(fmaxf(v / s, -448.0f), 448.0f);
  const uint8_t b = (uint8_t)(__builtin_amdgcn_cvt_pk_fp8_f32(x, 0.0f, 0, false) & 0xff);
  const int g = (k & 15) >> 2, j = 4 * (k >> 4) + (k & 3);
  const int lane = 16 * g + (n & 15);
  q8[(size_t)(n >> 4) * 2048 + (j >> 4) * 1024 + lane * 16 + (j & 15)] = b;
}

}  // namespace

size_t mfma_sig_scratch_bytes(int W, int grid) {
  return (size_t)grid * kWaves * kNT * (W / 32) * kFrag;
}

hipError_t launch_pack_weights(const float *master, uint8_t *packed, const PackedLayout &pl,
                               int precision, hipStream_t stream) {
  PackArgs p;
  p.master = master;
  p.packed = packed;
  for (int c = 0; c < kNumChunks; ++c) p.chunk[c] = pl.chunk[c];
  layer_offsets(pl.W, pl.pe, p.lo);
  p.W = pl.W;
  p.bias_off = pl.bias_off;
  int most = kNumLayers * pl.W;
  for (int c = 0; c < kNumChunks; ++c) most = std::max(most, pl.chunk[c].mt * pl.chunk[c].ks * 64);
  hipLaunchKernelGGL(pack_bf16_kernel, dim3((unsigned)((most + 255) / 256), kNumChunks + 1),
                     dim3(256), 0, stream, p);
  if (precision == GN_FP8_T)
    hipLaunchKernelGGL(pack_fp8_t2_kernel, dim3(pl.W), dim3(pl.W), 0, stream, p,
                       packed + pl.t2q_off, (float *)(packed + pl.t2scale_off));
  return hipGetLastError();
}

// Resident LDS bytes of the slot loop's weights for a precision.
static int64_t resident_bytes(const PackedLayout &pl, int precision) {
  const int MT = pl.W / 16;
  if (precision == GN_FP8_T)
    return (((int64_t)MT * pl.chunk[C_T1A].ks * 512 + 1023) & ~(int64_t)1023) +
           (pl.t2scale_off - pl.t2q_off) + (pl.total_bytes - pl.t2scale_off);
  return pl.resident_bytes;
}

// order_bytes: the canonical order's LDS tables (order and alphas) per tile.
// all: every stage has a place of its own (all_resident).
static size_t mfma_base_lds_bytes(const PackedLayout &pl, int precision, int order_bytes, bool all) {
  int64_t stage_max = 0;
  for (int s = 0; s < pl.nstages; ++s)
    stage_max = std::max<int64_t>(stage_max, pl.stage_off[s + 1] - pl.stage_off[s]);
  return (size_t)(resident_bytes(pl, precision) + (int64_t)kNumLayers * pl.W * 4 +
                  (int64_t)order_bytes + (all ? pl.stage_off[pl.nstages] + 16 : 2 * stage_max));
}

// Waves whose sigma fits in the LDS the weights leave free (160 KiB per CU),
// and how many of them sit in the stage buffers' tails: from F3's stage to
// B1S's (stages 1-4, shifted by two with encoded inputs) buffer 1 holds the
// first and third of them, buffer 0 the second and fourth.
static void mfma_sig_lds(const PackedLayout &pl, int precision, int order_bytes, bool all,
                         int nt, int *nlds, int *ntail) {
  constexpr size_t kLdsMax = 160 * 1024;
  const size_t per_wave = (size_t)nt * (pl.W / 32) * kFrag;
  const size_t base = mfma_base_lds_bytes(pl, precision, order_bytes, all);
  int64_t stage_max = 0;
  for (int s = 0; s < pl.nstages; ++s)
    stage_max = std::max<int64_t>(stage_max, pl.stage_off[s + 1] - pl.stage_off[s]);
  const int sh = stage_shift(pl.pe);
  auto size = [&](int s) { return pl.stage_off[sh + s + 1] - pl.stage_off[sh + s]; };
  const int64_t tail1 = stage_max - std::max(size(1), size(3));
  const int64_t tail0 = stage_max - std::max(size(2), size(4));
  const int free_waves = base >= kLdsMax ? 0 : (int)((kLdsMax - base) / per_wave);
  int t = 0;
  // tails are used alternately (buffer 0, buffer 1, buffer 0, ...)
  for (int64_t used0 = 0, used1 = 0; !all; ++t) {
    int64_t &u = (t & 1) ? used1 : used0;
    const int64_t cap = (t & 1) ? tail1 : tail0;
    if (u + (int64_t)per_wave > cap) break;
    u += per_wave;
  }
  const int n = std::min(kWaves, free_waves + t);
  *ntail = std::max(0, n - free_waves);
  *nlds = n;
}

// LDS past the arrays that the kernel declares: the order's tables and sigma of
// the waves that have no tail.
static size_t mfma_dynamic_lds(const PackedLayout &pl, int order_bytes, int nt, int nlds, int ntail) {
  return order_bytes + (size_t)(nlds - ntail) * nt * (pl.W / 32) * kFrag;
}

template <int W, int PREC, int MODE, int PE, int NT>
static hipError_t launch_one(const MfmaArgs &a, int grid, size_t lds, hipStream_t stream) {
  using LM = LdsMap<W, PREC, PE>;
  constexpr size_t fixed = LM::kRes + Shape<W>::kBiasBytes +
                           (all_resident<W, MODE, PE>() ? LM::kAll + 16 : 2 * LM::kStage);
  if (a.res_bytes != LM::kRes || a.stage_max != LM::kStage || lds + fixed > 160 * 1024)
    return hipErrorInvalidValue;
  static LdsLimit limit;
  const hipError_t e = limit.raise((const void *)fwd_mfma_kernel<W, PREC, MODE, PE, NT>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((fwd_mfma_kernel<W, PREC, MODE, PE, NT>), dim3(grid), dim3(kThreads), lds,
                     stream, a);
  return hipGetLastError();
}

// N-tiles per wave.  Two: every weight fragment read from LDS then serves two
// matrix instructions.  One, half a tile per workgroup, in whole forwards of a
// batch whose 256-pixel tiles leave half of the CUs idle: W = 128, K = 4, 128^2
// 28.4 -> 18.5 us, 128 x 256 28.5 -> 19.4; at 192^2 half tiles need a second
// round, 34.4 us against 28.5.  (In the begin and accumulate calls, two
// workgroups of half tiles to a CU took 30 and 49 us at 512^2 against 27 and 35.)
static int n_tiles(int mode, bool batch, int ntiles, int grid) {
  return mode == FWD_FULL && batch && 2 * ntiles <= grid ? 1 : 2;
}

template <int W, int PREC, int PE>
static hipError_t launch_mode(int mode, int nt, const MfmaArgs &a, int grid, size_t lds,
                              hipStream_t stream) {
  switch (mode) {
    case FWD_FULL:
      return nt == 1 ? launch_one<W, PREC, FWD_FULL, PE, 1>(a, grid, lds, stream)
                     : launch_one<W, PREC, FWD_FULL, PE, 2>(a, grid, lds, stream);
    case FWD_BEGIN: return launch_one<W, PREC, FWD_BEGIN, PE, 2>(a, grid, lds, stream);
    case FWD_ACC: return launch_one<W, PREC, FWD_ACC, PE, 2>(a, grid, lds, stream);
    case FWD_FINISH: return launch_one<W, PREC, FWD_FINISH, PE, 2>(a, grid, lds, stream);
  }
  return hipErrorInvalidValue;
}

template <int W, int PREC>
static hipError_t launch_pe(int pe, int mode, int nt, const MfmaArgs &a, int grid, size_t lds,
                            hipStream_t stream) {
  switch (pe) {
    case 0: return launch_mode<W, PREC, 0>(mode, nt, a, grid, lds, stream);
    case 1: return launch_mode<W, PREC, 1>(mode, nt, a, grid, lds, stream);
    case 2: return launch_mode<W, PREC, 2>(mode, nt, a, grid, lds, stream);
    case 3: return launch_mode<W, PREC, 3>(mode, nt, a, grid, lds, stream);
    case 4: return launch_mode<W, PREC, 4>(mode, nt, a, grid, lds, stream);
  }
  return hipErrorInvalidValue;
}

size_t stream_state_tile_bytes(int W) {
  return W == 64 ? (size_t)StreamTile<64>::kBytes : (size_t)StreamTile<128>::kBytes;
}

static hipError_t launch_impl(int W, int precision, int pool, const uint8_t *packed,
                              const PackedLayout &pl, const FwdBatch *batch,
                              const FrameDesc *frames, const TileRef *tiles, int ntiles,
                              float fp8_act_scale, int grid, uint8_t *sig_scratch, int mode,
                              uint8_t *state, int state_load, int slot_kmax,
                              hipStream_t stream) {
  MfmaArgs a;
  a.sig_scratch = sig_scratch;
  a.state = state;
  a.state_load = state_load;
  a.dense = mode != FWD_FULL && 16 * ntiles <= 9 * grid;
  // canonical order: a table of slot_kmax bytes per pixel, rounded up to 4
  a.canon = slot_kmax > 1 ? 1 : 0;
  a.kpad = a.canon ? (slot_kmax + 3) / 4 * 4 : 0;
  a.aslots = a.canon ? std::min(slot_kmax, 8) : 0;
  // the alpha table goes into sigma's parking area when that area holds it,
  // else into LDS of its own
  const int nt = n_tiles(mode, batch != nullptr, ntiles, grid), tile_px = kWaves * nt * 16;
  int order_bytes = tile_px * a.kpad;
  const bool all = W == 64 && mode == FWD_FULL && pl.pe == 0;     // all_resident
  mfma_sig_lds(pl, precision, order_bytes, all, nt, &a.sig_lds_waves, &a.sig_tail_waves);
  const int alpha_bytes = tile_px * 4 * a.aslots;
  a.alpha_alias = (a.sig_lds_waves - a.sig_tail_waves) * nt * (W / 32) * kFrag >= alpha_bytes;
  if (!a.alpha_alias) {
    order_bytes += alpha_bytes;
    mfma_sig_lds(pl, precision, order_bytes, all, nt, &a.sig_lds_waves, &a.sig_tail_waves);
  }
  a.packed = packed;
  for (int s = 0; s <= kMaxStages; ++s) a.stage_off[s] = s <= pl.nstages ? pl.stage_off[s] : 0;
  a.res_off = pl.resident_off;
  a.res_bytes = resident_bytes(pl, precision);
  a.stage_max = 0;
  for (int s = 0; s < pl.nstages; ++s)
    a.stage_max = std::max(a.stage_max, pl.stage_off[s + 1] - pl.stage_off[s]);
  a.bias_off = pl.bias_off;
  a.t2q_off = pl.t2q_off;
  a.t2s_off = pl.t2scale_off;
  if (batch) {
    a.b = *batch;
    a.tiles_per_frame = (batch->hw + tile_px - 1) / tile_px;
    ntiles = batch->n * a.tiles_per_frame;
  } else {
    a.b = FwdBatch{};
    a.tiles_per_frame = 1;
  }
  a.frames = frames;
  a.tiles = tiles;
  a.ntiles = ntiles;
  a.pool = pool;
  a.sa = fp8_act_scale;
  a.inv_sa = 1.0f / fp8_act_scale;
  if (ntiles <= 0) return hipSuccess;
  grid = std::max(1, std::min(grid, ntiles));   // the scratch holds `grid` workgroups
  if (all && a.sig_lds_waves < kWaves) return hipErrorInvalidValue;
  const size_t lds =
      mfma_dynamic_lds(pl, order_bytes, nt, a.sig_lds_waves, a.sig_tail_waves);
  if (precision == GN_BF16) {
    if (W == 64) return launch_pe<64, GN_BF16>(pl.pe, mode, nt, a, grid, lds, stream);
    if (W == 128) return launch_pe<128, GN_BF16>(pl.pe, mode, nt, a, grid, lds, stream);
  }
  if (precision == GN_FP8_T && W == 128)
    return launch_pe<128, GN_FP8_T>(pl.pe, mode, nt, a, grid, lds, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_fwd_mfma(int W, int precision, int pool, const uint8_t *packed,
                           const PackedLayout &pl, const FwdBatch *batch,
                           const FrameDesc *frames, const TileRef *tiles, int ntiles,
                           float fp8_act_scale, int grid, uint8_t *sig_scratch,
                           int slot_kmax, hipStream_t stream) {
  return launch_impl(W, precision, pool, packed, pl, batch, frames, tiles, ntiles, fp8_act_scale,
                     grid, sig_scratch, FWD_FULL, nullptr, 0, slot_kmax, stream);
}

hipError_t launch_fwd_stream(int W, int precision, int pool, const uint8_t *packed,
                             const PackedLayout &pl, const FwdBatch &batch, float fp8_act_scale,
                             int grid, int mode, uint8_t *state, int state_load,
                             hipStream_t stream) {
  if (mode == FWD_FULL || !state) return hipErrorInvalidValue;
  const int tpf = (batch.hw + kTilePx - 1) / kTilePx;
  return launch_impl(W, precision, pool, packed, pl, &batch, nullptr, nullptr, batch.n * tpf,
                     fp8_act_scale, grid, nullptr, mode, state, state_load, 0, stream);
}

}  // namespace gn
