// Shared core of the fp32 per-pixel kernels (fwd_fp32.hip, bwd_fp32.hip): the
// networks' linear maps on v_mfma_f32_16x16x4f32, chained in registers.
//
// Formulation.  A wave owns 16 pixels.  Every map is D = A X with a 16-row
// tile of A (weights) as the row operand and the 16 pixels as the columns.
// K-step s of the instruction takes inputs 4s .. 4s+3: lane group g (lane >>
// 4) presents input 4s + g of its pixel (lane & 15).  The accumulator leaves
// lane group g with tile rows 4g + r (r = 0..3), so the rows of A are stored
// permuted: row 4g + r of tile mt is neuron 16 mt + 4r + g.  Register r of
// tile mt is then neuron 4 (4 mt + r) + g, exactly what lane group g presents
// in K-step 4 mt + r of the next map: activations go from map to map without
// any cross-lane move, and every sum runs over its inputs in natural order.
//
// Weights.  They stream through LDS as a sequence of 16 KiB stages of
// fragments (64 lanes x 16 bytes: four K-steps of one row tile), in the order
// the kernel consumes them, through a ring of three buffers with one barrier
// in the middle of each stage: past it every wave is done with the stage
// before, whose buffer then takes the stage after the next one, and the next
// stage's first fragments are read before this one ends, so no wave starts a
// stage by waiting for LDS.  The stages go through registers rather than by
// direct global->LDS copies: the compiler makes every LDS read wait for the
// direct copies in flight, which would put a memory latency into every stage.
#pragma once

#include "gn_internal.h"

namespace gn {
namespace f32 {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256, kWaves = 4;
constexpr int kTile = kWaves * 16;         // pixels per workgroup tile
constexpr int kStageFrags = 16;
constexpr int kStageBytes = kStageFrags * 1024;

// The linear maps of the forward and of the backward (the transposes), each
// list in the order its kernel consumes them.
enum Op {
  O_F1, O_F2, O_F3, O_T1S, O_T1A, O_T2, O_T3, O_B1S, O_B1T, O_B2, O_B3, O_R1P, O_R1L, O_R2, O_R3,
  kNumOps
};
enum BwdOp {
  O_R3T, O_R2T, O_R1T, O_B3T, O_B2T, O_B1ST, O_B1TT, O_T3T, O_T2T, O_T1ST, O_F3T, O_F2T, kNumBwdOps
};

// Map o multiplies A (M x K): A[m][k] = W[m][col0 + k] of a layer, or
// W[k][col0 + m] (trans).
struct OpDesc {
  int64_t woff;      // float offset of the layer's matrix in the master vector
  int32_t ld;        // the layer's input count (master row length)
  int32_t col0, M, K, trans;
  int32_t mt, kq;    // 16-row tiles, 16-deep K groups
  int32_t stage0, nstages;
};

struct OpTable {
  OpDesc op[kNumOps];
  int32_t nops, stages;            // stages of every map together
  LayerOff lo[kNumLayers];
  int32_t W, pe;
};

void make_ops(int W, int pe, OpTable *t);
void make_bwd_ops(int W, int pe, OpTable *t);
// The packed form: the stages, then the 12 biases (W floats each, in the
// position order below; R3's 3 in natural order).
inline size_t packed_bytes(const OpTable &t) {
  return (size_t)t.stages * kStageBytes + sizeof(float) * kNumLayers * t.W;
}
hipError_t launch_pack(const float *master, const OpTable &t, uint8_t *packed, hipStream_t s);

// What the backward keeps of a slab of np pixels (a multiple of kTile, the
// tail repeating the last pixel): blocks [pixel][width] in position order.
// The slots' blocks follow each other slot by slot ([slot][pixel][width]).
struct Planes {
  int64_t p0, np;            // first pixel of the slab; its padded length
  float *x;                  // F's encoded input, nx wide
  float *a1, *a2, *sig, *zs, *tau, *d1, *d2, *phi, *g1, *g2;
  float *z1, *bi;            // per slot: h's first activation; its encoded input, nb wide
  float *inv, *bs;           // per pixel: 1 / max(c, 1) (mean) or 1; T3's bias scale
  uint32_t *mask;            // [kMasks + 2 k][np / 16][64]: ReLU signs, bit 4 mt + r
  // the deltas of the maps' outputs (dsig: sigma's; dz: Z's; dz1 per slot)
  float *dg2, *dg1, *dphi, *dd2, *dd1, *dtau, *dsig, *dz, *du, *da2, *da1, *dz1, *dy;
  int32_t nx, nb;
};
// Mask layers; then per slot z1's and z2's, the latter of active slots only.
enum { K_A1, K_A2, K_D1, K_D2, K_G1, K_G2, kMasks };
constexpr int kDyWidth = 16;

// Position p of a W-row block (16 mt + 4 g + r) holds this neuron.
__host__ __device__ inline int neuron_at(int p) {
  return (p & ~15) + 4 * (p & 3) + ((p >> 2) & 3);
}

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

// An infinite x keeps its infinite hi: what is left of it (inf - inf) becomes
// a finite value instead of a NaN.
__device__ __forceinline__ float left_of(float x, float h) {
  return __builtin_amdgcn_fmed3f(x - h, -6.7e35f, 6.7e35f);
}

__device__ __forceinline__ Split split8(const float (&x)[8]) {
  Split s;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = x[2 * i], b = x[2 * i + 1];
    const uint32_t h = pk_bf16(a, b);
    const float ra = left_of(a, bf16_lo(h)), rb = left_of(b, bf16_hi(h));
    const uint32_t m = pk_bf16(ra, rb);
    s.hi[i] = h;
    s.mid[i] = m;
    s.lo[i] = pk_bf16(ra - bf16_lo(m), rb - bf16_hi(m));
  }
  return s;
}

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

// Positional-encoding block b of x (Sec. 3.4): x for b = 0, then
// sin(2^k pi x) for b = 2k + 1 and cos(2^k pi x) for b = 2k + 2 (sinpi and
// cospi reduce the argument exactly; the scaling by 2^k is exact).
__device__ __forceinline__ float pe_value(float x, int b) {
  if (b == 0) return x;
  const float t = x * (float)(1 << ((b - 1) >> 1));
  return (b & 1) ? sinpif(t) : cospif(t);
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

constexpr int kRing = 3;

template <int MT>
struct Pipe {
  static constexpr int kQ = kStageFrags / MT;    // K groups per stage of a full map
  rsrc_t base;
  uint8_t *lds;          // kRing stage buffers
  Program pg;
  int pos, end, range;   // the stage to load next, in which range of the program
  int cur;               // buffer of the stage being consumed
  f32x4 hold[4];         // the stage two ahead of it
  f32x4 w[2][4];         // fragments; w[0]: the first of the stage to consume

  // The next stage of the program (wave-uniform, without branches: it is
  // inlined into every stage, and the code has to fit the instruction cache).
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
  __device__ __forceinline__ void load() {
    const uint32_t at = (uint32_t)next() * kStageBytes;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      hold[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                              base, threadIdx.x * 16, at + i * kThreads * 16, 0));
  }
  __device__ __forceinline__ void store(int buf) {
    f32x4 *dst = (f32x4 *)(lds + buf * kStageBytes) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[i * kThreads] = hold[i];
  }
  __device__ __forceinline__ void start(const uint8_t *b, uint8_t *l, const Program &p) {
    base = make_rsrc(b);
    lds = l;
    pg = p;
    pos = p.pre0;
    end = p.pre1;
    range = 0;
    cur = 0;
    load();
    store(0);
    load();
    store(1);
    load();
    __syncthreads();
    fetch(w[0], 0, 0);
  }
  // Four fragments of a buffer.
  __device__ __forceinline__ void fetch(f32x4 (&d)[4], int buf, int group) {
    const f32x4 *s = (const f32x4 *)(lds + buf * kStageBytes) + (threadIdx.x & 63) + group * 256;
#pragma unroll
    for (int m = 0; m < 4; ++m) d[m] = s[m * 64];
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

  // One stage: K groups q0 .. of a map of MT row tiles; group q0 + i is used
  // while q0 + i < kq.  x(q) gives the four K-steps' inputs.  Four fragments
  // are read ahead of the sixteen MFMAs of the four before (a scheduling
  // barrier keeps them there).
  template <class X>
  __device__ __forceinline__ void stage(f32x4 (&acc)[MT], int q0, int kq, X x) {
    f32x4 xv = zero4();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      constexpr int kPer = MT / 4;               // fragment groups per K group
      const int q = q0 + i / kPer, m0 = 4 * (i % kPer);
      if (i == 2) middle();
      if (i < 3) fetch(w[(i + 1) & 1], cur, i + 1);
      else fetch(w[0], after(cur), 0);
      __builtin_amdgcn_sched_barrier(0);
      if (q < kq) {
        if (i % kPer == 0) xv = x(i / kPer);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int m = 0; m < 4; ++m)
            acc[m0 + m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i & 1][m][j], xv[j], acc[m0 + m],
                                                                0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    cur = after(cur);
  }
  // A map over W inputs held in registers, in[q] K group q.
  __device__ __forceinline__ void chain(f32x4 (&acc)[MT], const f32x4 (&in)[MT]) {
#pragma unroll
    for (int st = 0; st < MT / kQ; ++st)
      stage(acc, st * kQ, MT, [&](int i) { return in[st * kQ + i]; });
  }
  // A map over kq K groups whose inputs x(q) computes.
  template <class X>
  __device__ __forceinline__ void gather(f32x4 (&acc)[MT], int kq, X x) {
    for (int q0 = 0; q0 < kq; q0 += kQ) stage(acc, q0, kq, [&](int i) { return x(q0 + i); });
  }
  // A map of one row tile over W inputs in registers.
  __device__ __forceinline__ f32x4 tail(const f32x4 (&in)[MT]) {
    f32x4 acc = zero4();
    if (MT > 4) fetch(w[1], cur, 1);
    middle();
#pragma unroll
    for (int q = 0; q < MT; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q >> 2][q & 3][j], in[q][j], acc, 0, 0, 0);
    cur = after(cur);
    fetch(w[0], cur, 0);
    return acc;
  }
};

}  // namespace f32
}  // namespace gn
