// Shared by the fp32 per-pixel kernels (fwd_fp32.hip, bwd_fp32.hip): fp32
// arithmetic on the bf16 matrix cores, encoding, the slots' order, and the
// sequence in which weight stages are streamed.
#pragma once

#include "gn_internal.h"
#include "slot_order.h"

namespace gn {
namespace f32 {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

__device__ __forceinline__ f32x4 relu4(f32x4 v) {
  return f32x4{fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
}

// fp32 operands of the bf16 matrix cores: x = hi + mid + lo in bf16, each the
// rounding of what the ones before leave (24 bits: exact but for the last
// bits of the smallest magnitudes).  A product takes the six partial products
// down to 2^-16 of the first; the three left out are below 2^-25 of it, under
// fp32's own rounding.  Six 16-cycle instructions replace eight 32-cycle ones.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Split {
  u32x4 hi, mid, lo;
};

__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xFFFF0000u); }

// An infinite x is (bf16's largest, 2^120, infinity) with its sign: of its
// partial products only lo's with the other operand's hi is infinite, and it has
// the product's sign.  (As hi, infinity would also meet the other operand's mid
// and lo, which may have the other sign or be zero: NaN, which a ReLU turns into
// zero.)  hi's product with mid stays finite for other operands up to 256.  A NaN
// x is one in lo.
template <bool HI>
__device__ __forceinline__ float part(float x) {
  constexpr float kMost = HI ? 0x1.fep127f : 0x1p120f;
  return __builtin_amdgcn_fmed3f(x, -kMost, kMost);
}

// WIDE: any values; else none that watch() would find.
template <bool WIDE = true>
__device__ __forceinline__ Split split8(const float (&x)[8]) {
  Split s;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = x[2 * i], b = x[2 * i + 1];
    const uint32_t h = WIDE ? pk_bf16(part<true>(a), part<true>(b)) : pk_bf16(a, b);
    const float ra = a - bf16_lo(h), rb = b - bf16_hi(h);
    const uint32_t m = WIDE ? pk_bf16(part<false>(ra), part<false>(rb)) : pk_bf16(ra, rb);
    s.hi[i] = h;
    s.mid[i] = m;
    s.lo[i] = pk_bf16(ra - bf16_lo(m), rb - bf16_hi(m));
  }
  return s;
}

// Whether values need the WIDE split, for many of them together (one operation
// a value against the clamps' two): the running sum of 4 x stays finite unless
// some are infinite, NaN or beyond 2^126, or add up to that.
__device__ __forceinline__ float watch(float x, float sum) { return fmaf(x, 4.0f, sum); }
__device__ __forceinline__ bool found(float sum) { return !(fabsf(sum) < __builtin_inff()); }

__device__ __forceinline__ f32x4 mma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// c + a b, the small partial products first.
__device__ __forceinline__ f32x4 mma_split(const Split &a, const Split &b, f32x4 c) {
  c = mma_bf16(a.lo, b.hi, c);
  c = mma_bf16(a.hi, b.lo, c);
  c = mma_bf16(a.mid, b.mid, c);
  c = mma_bf16(a.mid, b.hi, c);
  c = mma_bf16(a.hi, b.mid, c);
  return mma_bf16(a.hi, b.hi, c);
}

// The sign with which the i-th of many addends is computed (and undone): by
// the parity of i's bits (the Thue-Morse sequence).  What is left of the bf16
// instruction's one-sided rounding then cancels in a sum over them; unlike by
// the parity of i, also where all that matters sits at every second, fourth,
// ... place.
__device__ __forceinline__ float sign_of(uint32_t i) { return __popc(i) & 1 ? -1.0f : 1.0f; }

// Positional-encoding block b of x (Sec. 3.4): x for b = 0, then
// sin(2^k pi x) for b = 2k + 1 and cos(2^k pi x) for b = 2k + 2 (sinpi and
// cospi reduce the argument exactly; the scaling by 2^k is exact).
__device__ __forceinline__ float pe_value(float x, int b) {
  if (b == 0) return x;
  const float t = x * (float)(1 << ((b - 1) >> 1));
  return (b & 1) ? sinpif(t) : cospif(t);
}

// Writes a pixel's canonical slot order (slot_order.h) to order[rank] from its
// alphas: lane group g ranks slots g and g + 4 of up to kFastK.  Keys: the
// bits of alpha for active slots, above them the inactive ones by index; equal
// alphas take the full comparison.
constexpr int kFastK = 8;
__device__ __forceinline__ void rank_slots(const float (&al)[kFastK], const float *L, int hw, int k,
                                           int g, uint8_t *order) {
  uint32_t key[kFastK];
#pragma unroll
  for (int j = 0; j < kFastK; ++j)
    key[j] = j >= k ? 0xFFFFFFFFu : (al[j] > 0.0f ? __float_as_uint(al[j]) : 0xFFFFFF00u + j);
#pragma unroll
  for (int h = 0; h < kFastK; h += 4) {
    const uint32_t ki = g < 2 ? (g == 0 ? key[h] : key[h + 1]) : (g == 2 ? key[h + 2] : key[h + 3]);
    int lt = 0, le = 0;
#pragma unroll
    for (int j = 0; j < kFastK; ++j) {
      lt += key[j] < ki ? 1 : 0;
      le += key[j] <= ki ? 1 : 0;
    }
    const int i = h + g;
    if (i < k) order[le == lt + 1 ? lt : slot_rank(L, (size_t)hw, k, i)] = (uint8_t)i;
  }
}

// The stages one tile consumes: [pre0, pre1), then [loop0, loop1) k times,
// then [post0, post1) if post; the next tile starts over.  None is empty.
struct Program {
  int32_t pre0, pre1, loop0, loop1, post0, post1, k, post;
};

// Weights are loaded through a buffer resource: one lane offset, the stage's
// a scalar.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void *base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, -1, 0x00020000);
}

// The next stage of a program (wave-uniform, without branches: it is inlined
// into every stage, and the code has to fit the instruction cache).
struct Sequence {
  Program pg;
  int pos, end, range;   // the stage to load next, in which range of the program
  __device__ __forceinline__ void start(const Program &p) {
    pg = p;
    pos = p.pre0;
    end = p.pre1;
    range = 0;
  }
  __device__ __forceinline__ int next() {
    const int at = pos++;
    const bool turn = pos == end;
    const int r = range == pg.k + pg.post ? 0 : range + 1;
    const bool loop = r <= pg.k;
    range = turn ? r : range;
    pos = turn ? (r == 0 ? pg.pre0 : (loop ? pg.loop0 : pg.post0)) : pos;
    end = turn ? (r == 0 ? pg.pre1 : (loop ? pg.loop1 : pg.post1)) : end;
    return at;
  }
};

constexpr int kRing = 3;     // stage buffers in LDS

// The weights of the kernels with split operands.  Packed as the three parts'
// fragments (64 lanes x 16 bytes) in the order the kernel consumes them, they
// stream through LDS in 24 KiB stages (a K-step at W = 128, two at 64) by way of
// registers, in a ring of three buffers with one barrier in the middle of each
// stage: past it every wave is done with the stage before, whose buffer then
// takes the stage after the next one, and the next stage's first fragments are
// read before this one ends.
constexpr int kSplitFrags = 24, kSplitStage = kSplitFrags * 1024;

// FRESH: a map sets the accumulators instead of adding to them, and a K-step's
// products are summed by themselves and then added by the vector unit.  The bf16
// instruction rounds its sums towards minus infinity: in one chain each of the six
// partial products shifts the whole sum down by a fraction of its ulp, here only
// the K-step's own sum.
template <int MT, int WAVES, bool FRESH>
struct SplitPipe {
  static constexpr int kThreads = WAVES * 64;
  static constexpr int kHold = kSplitStage / 16 / kThreads;
  static constexpr int kSteps = kSplitFrags / (3 * MT);    // K-steps per stage
  static constexpr int KS = MT / 2;                        // K-steps of a W-wide map
  rsrc_t base;
  uint8_t *lds;          // kRing stage buffers
  Sequence seq;          // of the stages to load
  int cur;               // buffer of the stage being consumed
  u32x4 hold[kHold];     // the stage two ahead of it
  u32x4 w[2][6];         // two row tiles' three parts; w[0]: the first of the stage to consume

  __device__ __forceinline__ void load() {
    const uint32_t at = (uint32_t)seq.next() * kSplitStage;
#pragma unroll
    for (int i = 0; i < kHold; ++i)
      hold[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                              base, threadIdx.x * 16, at + i * kThreads * 16, 0));
  }
  __device__ __forceinline__ void store(int buf) {
    u32x4 *dst = (u32x4 *)(lds + buf * kSplitStage) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < kHold; ++i) dst[i * kThreads] = hold[i];
  }
  __device__ __forceinline__ void start(const uint8_t *b, uint8_t *l, const Program &p) {
    base = make_rsrc(b);
    lds = l;
    seq.start(p);
    cur = 0;
    load();
    store(0);
    load();
    store(1);
    load();
    __syncthreads();
    fetch(w[0], 0, 0);
  }
  // Six fragments of a buffer: two row tiles of a K-step.
  __device__ __forceinline__ void fetch(u32x4 (&d)[6], int buf, int group) {
    const u32x4 *s = (const u32x4 *)(lds + buf * kSplitStage) + (threadIdx.x & 63) + group * 384;
#pragma unroll
    for (int m = 0; m < 6; ++m) d[m] = s[m * 64];
  }
  __device__ __forceinline__ int after(int buf) const { return buf == kRing - 1 ? 0 : buf + 1; }
  // The middle of a stage.  Only LDS traffic is drained: the loads and stores
  // in flight stay so.
  __device__ __forceinline__ void middle() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    store(cur == 0 ? kRing - 1 : cur - 1);
    load();
    __builtin_amdgcn_sched_barrier(0);
  }

  // One stage: K-steps s0 .. of a map; step s0 + i is used while s0 + i <
  // steps.  x(i) gives its inputs.  Two row tiles' fragments are read ahead of
  // the twelve MFMAs of the two before (a scheduling barrier keeps them there).
  template <class X>
  __device__ __forceinline__ void stage(f32x4 (&acc)[MT], int s0, int steps, X x) {
    constexpr int kPer = MT / 2;                 // tile pairs per K-step
    f32x4 late[2];                               // FRESH: the sums of the pair before
    // adds them while the next pair's MFMAs run (pinned: left to itself the
    // compiler keeps all sums and adds them at the map's end)
    auto add = [&](int i) {
      if (s0 + i / kPer >= steps) return;
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        f32x4 &c = acc[2 * (i % kPer) + m];
        c = s0 + i / kPer > 0 ? c + late[m] : late[m];
        asm volatile("" : "+v"(c));
      }
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m0 = 2 * (i % kPer);
      if (i == 2) middle();
      if (i < 3) fetch(w[(i + 1) & 1], cur, i + 1);
      else fetch(w[0], after(cur), 0);
      __builtin_amdgcn_sched_barrier(0);
      f32x4 sum[2];
      if (s0 + i / kPer < steps) {
        const Split &b = x(i / kPer);
        const u32x4(&a)[6] = w[i & 1];
#pragma unroll
        for (int m = 0; m < 2; ++m) sum[m] = FRESH ? zero4() : acc[m0 + m];
        // small partial products first, the two tiles in turn
#pragma unroll
        for (int p = 0; p < 6; ++p) {
          constexpr int kA[6] = {2, 0, 1, 1, 0, 0}, kB[6] = {0, 2, 1, 0, 1, 0};
          const u32x4 bv = kB[p] == 0 ? b.hi : (kB[p] == 1 ? b.mid : b.lo);
#pragma unroll
          for (int m = 0; m < 2; ++m) sum[m] = mma_bf16(a[3 * m + kA[p]], bv, sum[m]);
        }
        if constexpr (!FRESH) {
#pragma unroll
          for (int m = 0; m < 2; ++m) acc[m0 + m] = sum[m];
        }
      }
      if constexpr (FRESH) {
        if (i > 0) add(i - 1);
#pragma unroll
        for (int m = 0; m < 2; ++m) late[m] = sum[m];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (FRESH) add(3);
    cur = after(cur);
  }
  // A map over W inputs, in[s] K-step s.
  __device__ __forceinline__ void chain(f32x4 (&acc)[MT], const Split (&in)[KS]) {
#pragma unroll
    for (int st = 0; st < KS / kSteps; ++st)
      stage(acc, st * kSteps, KS, [&](int i) -> const Split & { return in[st * kSteps + i]; });
  }
  // A map of `steps` K-steps whose inputs x(s) computes.
  template <class X>
  __device__ __forceinline__ void gather(f32x4 (&acc)[MT], int steps, X x) {
    for (int s0 = 0; s0 < steps; s0 += kSteps) {
      Split v[kSteps];
#pragma unroll
      for (int i = 0; i < kSteps; ++i)
        if (s0 + i < steps) v[i] = x(s0 + i);
      stage(acc, s0, steps, [&](int i) -> const Split & { return v[i]; });
    }
  }
  // A map of one row tile over W inputs: KS K-steps of three fragments.
  __device__ __forceinline__ f32x4 tail(const Split (&in)[KS]) {
    f32x4 acc = zero4();
    if (KS > 2) fetch(w[1], cur, 1);
    middle();
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const u32x4 *a = &w[s >> 1][3 * (s & 1)];
      acc = mma_split(Split{a[0], a[1], a[2]}, in[s], acc);
    }
    cur = after(cur);
    fetch(w[0], cur, 0);
    return acc;
  }
};

}  // namespace f32
}  // namespace gn
