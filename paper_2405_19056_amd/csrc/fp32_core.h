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
// the kernel consumes them, double-buffered: while stage s computes, stage
// s + 1 is written to LDS from registers and stage s + 2 is loaded into them.
// Through registers rather than by direct global->LDS copies: the compiler
// makes every LDS read wait for the direct copies in flight, which would put
// a memory latency into every stage.
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

// Positional-encoding block b of x (Sec. 3.4): x for b = 0, then
// sin(2^k pi x) for b = 2k + 1 and cos(2^k pi x) for b = 2k + 2 (sinpi and
// cospi reduce the argument exactly; the scaling by 2^k is exact).
__device__ __forceinline__ float pe_value(float x, int b) {
  if (b == 0) return x;
  const float t = x * (float)(1 << ((b - 1) >> 1));
  return (b & 1) ? sinpif(t) : cospif(t);
}

// The stages one tile consumes: [pre0, pre1), then [loop0, loop1) k times,
// then [post0, post1); the next tile starts over.
struct Program {
  int32_t pre0, pre1, loop0, loop1, post0, post1, k;
};

template <int MT>
struct Pipe {
  static constexpr int kQ = kStageFrags / MT;    // K groups per stage of a full map
  const uint8_t *base;
  uint8_t *lds;          // two stage buffers
  Program pg;
  int phase, pos, slot;  // the stage to load next
  int par;               // buffer of the stage to consume next
  f32x4 hold[4];         // the stage after it

  // The next stage of the program (wave-uniform).
  __device__ __forceinline__ int next() {
    for (;;) {
      if (phase == 0) {
        if (pos < pg.pre1) break;
        phase = 1;
        slot = 0;
        pos = pg.loop0;
      }
      if (phase == 1) {
        if (pos < pg.loop1 && slot < pg.k) break;
        if (slot + 1 < pg.k && pg.loop0 < pg.loop1) {
          ++slot;
          pos = pg.loop0;
          break;
        }
        phase = 2;
        pos = pg.post0;
      }
      if (pos < pg.post1) break;
      phase = 0;
      pos = pg.pre0;
    }
    return pos++;
  }
  __device__ __forceinline__ void load() {
    const f32x4 *src = (const f32x4 *)(base + (size_t)next() * kStageBytes) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) hold[i] = src[i * kThreads];
  }
  __device__ __forceinline__ void store(int buf) {
    f32x4 *dst = (f32x4 *)(lds + buf * kStageBytes) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[i * kThreads] = hold[i];
  }
  __device__ __forceinline__ void start(const uint8_t *b, uint8_t *l, const Program &p) {
    base = b;
    lds = l;
    pg = p;
    phase = 0;
    pos = p.pre0;
    slot = 0;
    par = 0;
    load();
    store(0);
    load();
  }
  // The fragments of the next stage.  Every wave has written its part of it
  // and is done with the stage before, whose buffer takes the one after.
  // (Only LDS traffic is drained: the loads and stores in flight stay so.)
  __device__ __forceinline__ const f32x4 *begin() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    store(par ^ 1);
    load();
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 *s = (const f32x4 *)(lds + par * kStageBytes) + (threadIdx.x & 63);
    par ^= 1;
    return s;
  }

  // One stage: K groups q0 .. of a map of MT row tiles; group q0 + i is used
  // while q0 + i < kq.  x(q) gives the four K-steps' inputs.  Four fragments
  // are read ahead of the sixteen MFMAs of the four before (a scheduling
  // barrier keeps them there).
  template <class X>
  __device__ __forceinline__ void stage(f32x4 (&acc)[MT], int q0, int kq, X x) {
    const f32x4 *s = begin();
    f32x4 w[2][4], xv = zero4();
#pragma unroll
    for (int m = 0; m < 4; ++m) w[0][m] = s[m * 64];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      constexpr int kPer = MT / 4;               // fragment groups per K group
      const int q = q0 + i / kPer, m0 = 4 * (i % kPer);
      if (i < 3) {
#pragma unroll
        for (int m = 0; m < 4; ++m) w[(i + 1) & 1][m] = s[(4 * (i + 1) + m) * 64];
      }
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
    const f32x4 *s = begin();
    f32x4 acc = zero4();
#pragma unroll
    for (int q = 0; q < MT; ++q) {
      const f32x4 w = s[q * 64];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j], in[q][j], acc, 0, 0, 0);
    }
    return acc;
  }
};

}  // namespace f32
}  // namespace gn
