// The fp32 backward: dL/dw of F, T, B and R for a given dL/dy (Sec. 3.5
// trains the four networks jointly, end to end).
//
// Per slab of pixels:
//   1. recompute: the forward on v_mfma_f32_16x16x4f32, every activation a
//      weight gradient needs written as it passes, and the sign of every ReLU
//      as one bit.  It stays on the fp32 instruction, each sum over its
//      inputs in natural order: a pre-activation within a rounding of zero
//      takes the branch it has always taken, whatever the forward's form.
//      (The FP8 calibration is the same kernel up to h's first layer: its
//      scale decides every fp8 rounding of a handle.)
//   2. deltas: one kernel chains the transposed maps in registers from dL/dy
//      to F's first layer, the slots in between: dz2 = [z2 > 0] m_i dZ is a
//      selection of dZ's registers, dz1 = [z1 > 0] W_T2^T dz2, du = sum dz1.
//      The ReLU derivatives are the stored bits; the arithmetic is fp32 on the
//      bf16 matrix cores (operands split in three).
//   3. weight gradients: sum_p delta_p a_p^T of every layer on the matrix
//      cores, each pixel block read once per product.
// Then one fixed-order reduction of the workgroups' partial sums into grad_w
// (deterministic, no atomics).
//
// Slabs bound the workspace (most_plane_bytes): it does not grow with the number
// of slots past four; their activations are recomputed for a slab at a time.
//
// Formulation of the recompute (the deltas' weights: SplitPipe of fp32_core.h).
// A wave owns 16 pixels.  Every map is D = A X with a 16-row
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
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "fp32_core.h"
#include "gn_api_state.h"
#include "lds_limit.h"

namespace gn {

struct BwdWorkspace {
  uint8_t *mem = nullptr;       // a slab's planes, then the packed weights and the partials
  size_t bytes = 0;
};

namespace f32 {

constexpr int kThreads = 256, kWaves = 4;
constexpr int kTile = kWaves * 16;         // pixels per workgroup tile
constexpr int kStageFrags = 16;
constexpr int kStageBytes = kStageFrags * 1024;

// The linear maps of the forward and of the backward (the transposes), each
// list in the order its kernel consumes them.
enum Op {
  O_F1, O_F2, O_F3, O_T1S, O_T1A, O_T2, O_T3, O_B1S, O_B1T, O_B2, O_B3, O_R1P, O_R1L, O_R2,
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
  int32_t col0, M, K;
  int32_t mt, kq;    // 16-row tiles, K groups (16 deep; the backward's 32)
  int32_t stage0, nstages;
};

struct OpTable {
  OpDesc op[kNumOps];
  int32_t nops, stages;            // stages of every map together
  int32_t stage_bytes;
  LayerOff lo[kNumLayers];
  int32_t W, pe;
};

// The packed form: the stages, then the 12 biases (W floats each, in the
// position order below).
static size_t packed_bytes(const OpTable &t) {
  return ((size_t)t.stages * t.stage_bytes + sizeof(float) * kNumLayers * t.W + 1023) / 1024 * 1024;
}

// What the backward keeps of a slab of np pixels (a multiple of 2 kTile, the
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

struct OpSpec { int op; Layer l; int col0, M, K; };

static void fill_table(int W, int pe, const OpSpec *s, int n, int trans, OpTable *t) {
  layer_offsets(W, pe, t->lo);
  t->W = W;
  t->pe = pe;
  t->nops = n;
  // the forward's maps as fp32 fragments, the backward's split in three
  t->stage_bytes = trans ? kSplitStage : kStageBytes;
  int stage = 0;
  for (int i = 0; i < n; ++i) {
    OpDesc &d = t->op[s[i].op];
    d.woff = t->lo[s[i].l].w;
    d.ld = t->lo[s[i].l].in;
    d.col0 = s[i].col0;
    d.M = s[i].M;
    d.K = s[i].K;
    d.mt = (d.M + 15) / 16;
    d.kq = trans ? (d.K + 31) / 32 : (d.K + 15) / 16;
    d.stage0 = stage;
    d.nstages = (d.kq * d.mt * (trans ? 3 : 1) * 1024 + t->stage_bytes - 1) / t->stage_bytes;
    stage += d.nstages;
  }
  t->stages = stage;
}

static void make_ops(int W, int pe, OpTable *t) {
  const int nx = (kNG + kNS) * pe_blocks(pe), nb = kNL * pe_blocks(pe);
  const OpSpec s[kNumOps] = {
      {O_F1, L_F1, 0, W, nx},  {O_F2, L_F2, 0, W, W},   {O_F3, L_F3, 0, W, W},
      {O_T1S, L_T1, nb, W, W}, {O_T1A, L_T1, 0, W, nb}, {O_T2, L_T2, 0, W, W},
      {O_T3, L_T3, 0, W, W},   {O_B1S, L_B1, 0, W, W},  {O_B1T, L_B1, W, W, W},
      {O_B2, L_B2, 0, W, W},   {O_B3, L_B3, 0, W, W},   {O_R1P, L_R1, 0, W, W},
      {O_R1L, L_R1, W, W, 3},  {O_R2, L_R2, 0, W, W}};
  fill_table(W, pe, s, kNumOps, 0, t);
}

static void make_bwd_ops(int W, int pe, OpTable *t) {
  const int nb = kNL * pe_blocks(pe);
  const OpSpec s[kNumBwdOps] = {
      {O_R3T, L_R3, 0, W, kNOUT}, {O_R2T, L_R2, 0, W, W},  {O_R1T, L_R1, 0, W, W},
      {O_B3T, L_B3, 0, W, W},     {O_B2T, L_B2, 0, W, W},  {O_B1ST, L_B1, 0, W, W},
      {O_B1TT, L_B1, W, W, W},    {O_T3T, L_T3, 0, W, W},  {O_T2T, L_T2, 0, W, W},
      {O_T1ST, L_T1, nb, W, W},   {O_F3T, L_F3, 0, W, W},  {O_F2T, L_F2, 0, W, W}};
  fill_table(W, pe, s, kNumBwdOps, 1, t);
}

// One thread per 16 bytes of a fragment, then the biases; blockIdx.y selects
// the forward's or the backward's maps.  Fragment f of a forward's map is K
// group f / mt of row tile f % mt; element j of lane l is A[row (l & 15)][16 q
// + 4 j + (l >> 4)], zero outside M x K.  The backward's: a thread per lane of
// a K group's row tile (its three parts); element e of lane group g is input
// 32 q + 16 (e / 4) + 4 (e % 4) + g, what it holds in element e of the map
// before (R3's three: input g in element 0).
struct PackArgs {
  OpTable t[2];
  uint8_t *packed[2];
};
__global__ __launch_bounds__(kThreads) void f32_pack_kernel(const float *__restrict__ master,
                                                            PackArgs a) {
  const OpTable &t = a.t[blockIdx.y];
  uint8_t *packed = a.packed[blockIdx.y];
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (blockIdx.y == 1) {
    const int n = e >> 6, lane = e & 63, g = lane >> 4, i = lane & 15;
    if (n >= t.stages * (kSplitFrags / 3)) return;
    int o = 0;
    while (o + 1 < t.nops && n / (kSplitFrags / 3) >= t.op[o + 1].stage0) ++o;
    const OpDesc d = t.op[o];
    const int f = n - d.stage0 * (kSplitFrags / 3), q = f / d.mt;
    const int m = 16 * (f % d.mt) + 4 * (i & 3) + (i >> 2);   // rows in position order
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = d.K < 16 ? (j == 0 ? g : d.K) : 32 * q + 16 * (j >> 2) + 4 * (j & 3) + g;
      x[j] = q < d.kq && m < d.M && k < d.K ? master[d.woff + (int64_t)k * d.ld + d.col0 + m] : 0.0f;
    }
    const Split s = split8(x);
    u32x4 *dst = (u32x4 *)packed + (size_t)n * 3 * 64 + lane;
    dst[0] = s.hi;
    dst[64] = s.mid;
    dst[128] = s.lo;
    return;
  }
  const int total = t.stages * kStageFrags * 64;
  if (e >= total) {
    const int b = e - total, l = b / t.W, p = b % t.W;
    if (l < kNumLayers)
      ((float *)(packed + (size_t)t.stages * kStageBytes))[b] =
          neuron_at(p) < t.lo[l].out ? master[t.lo[l].b + neuron_at(p)] : 0.0f;
    return;
  }
  const int stage = e / (kStageFrags * 64);
  int o = 0;
  while (o + 1 < t.nops && stage >= t.op[o + 1].stage0) ++o;
  const OpDesc d = t.op[o];
  const int f = (e >> 6) - d.stage0 * kStageFrags, lane = e & 63;
  const int q = f / d.mt, mt = f % d.mt, i = lane & 15;
  const int m = 16 * mt + 4 * (i & 3) + (i >> 2);       // rows in position order
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = 16 * q + 4 * j + (lane >> 4);
    if (m < d.M && k < d.K)
      v[j] = master[d.woff + (int64_t)m * d.ld + d.col0 + k];
  }
  ((f32x4 *)packed)[e] = v;
}

template <int MT>
struct Pipe {
  static constexpr int kQ = kStageFrags / MT;    // K groups per stage of a full map
  rsrc_t base;
  uint8_t *lds;          // kRing stage buffers
  Sequence seq;          // of the stages to load
  int cur;               // buffer of the stage being consumed
  f32x4 hold[4];         // the stage two ahead of it
  f32x4 w[2][4];         // fragments; w[0]: the first of the stage to consume

  __device__ __forceinline__ void load() {
    const uint32_t at = (uint32_t)seq.next() * kStageBytes;
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
};

// ---- the recompute ------------------------------------------------------------------
struct SaveArgs {
  const uint8_t *packed;
  int32_t bias_stage;        // the biases follow this many stages
  Program pg;
  const float *gbuf, *layers, *scene;
  int32_t hw, k, mean, pe, kpad;
  int32_t canon;             // pool in canonical order
  int32_t kq_x, kq_b;        // K groups of F1 and of T1's slot columns
  int64_t npx;
  Planes pl;
  unsigned *amax;            // calibration: float bits of the largest z1
};

// CAL: the FP8 calibration, which keeps no block and ends after h's first
// layer of every slot.  ENC: with positional encoding (a form of its own: the sine and cosine's code
// and registers stay out of the plain one).
template <int W, bool ENC, bool CAL>
__global__ __launch_bounds__(kThreads, 2) void f32_save_kernel(SaveArgs a) {
  constexpr int MT = W / 16;
  // LDS: the stage ring | biases | slot order per pixel
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  float *l_bias = (float *)(lds + kRing * kStageBytes);
  uint8_t *l_order = (uint8_t *)(l_bias + kNumLayers * W);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  {
    const float *b = (const float *)(a.packed + (size_t)a.bias_stage * kStageBytes);
    for (int i = threadIdx.x; i < kNumLayers * W; i += kThreads) l_bias[i] = b[i];
  }
  Pipe<MT> pipe;
  pipe.start(a.packed, lds, a.pg);       // ends with a barrier
  const int hw = a.hw, nblk = ENC ? pe_blocks(a.pe) : 1;
  const int64_t ntiles = a.pl.np / kTile;
  float amax = 0.0f;

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    // Opaque per-tile copies of the lane's place keep the compiler from holding
    // every address derived from them in registers across the tile loop.
    int g = lane >> 4, col = lane & 15;
    asm volatile("" : "+v"(g), "+v"(col));
    const int64_t pl = tile * kTile + wave * 16 + col;         // pixel of the slab
    const int64_t pc = std::min<int64_t>(a.pl.p0 + pl, a.npx - 1);   // tail: a real pixel again
    const int f = (int)(pc / hw), q = (int)(pc - (int64_t)f * hw);
    const float *G = a.gbuf + (size_t)f * kNG * hw + q;
    const float *L = a.layers + (size_t)f * a.k * kNL * hw + q;
    const float *S = a.scene + (size_t)f * kNS;
    uint8_t *order = l_order + (wave * 16 + col) * a.kpad;
    auto bias = [&](int layer, int mt) { return *(const f32x4 *)(l_bias + layer * W + 16 * mt + 4 * g); };
    // in = act(acc + bias)
    auto next = [&](f32x4 (&in)[MT], f32x4 (&acc)[MT], int layer, bool relu) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const f32x4 v = acc[mt] + bias(layer, mt);
        in[mt] = relu ? relu4(v) : v;
        acc[mt] = zero4();
      }
    };
    // a block of W values per pixel (32-bit offsets from a uniform base: the
    // caller bounds a slab's blocks), the signs of a ReLU's outputs
    const uint32_t at = (uint32_t)pl * (W * 4) + 16 * g;
    auto save = [&](float *plane, const f32x4 (&v)[MT]) {
      if constexpr (CAL) return;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) *(f32x4 *)((char *)plane + at + 64 * mt) = v[mt];
    };
    auto signs = [&](int layer, const f32x4 (&v)[MT], bool keep) {
      if constexpr (CAL) return;
      uint32_t b = 0;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int r = 0; r < 4; ++r) b |= v[mt][r] > 0.0f ? 1u << (4 * mt + r) : 0u;
        asm volatile("" : "+v"(b));
      }
      uint32_t *words = a.pl.mask + (int64_t)layer * (a.pl.np / 16) * 64;
      words[(uint32_t)(tile * kThreads) + threadIdx.x] = keep ? b : 0u;
    };
    auto keep = [&](float *plane, int layer, const f32x4 (&v)[MT]) {
      save(plane, v);
      signs(layer, v, true);
    };
    f32x4 in[MT], acc[MT], u[MT], Z[MT], xr[2];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = zero4();
    if constexpr (!ENC) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = 4 * i + g;
        xr[i >> 2][i & 3] = c < kNG ? G[(size_t)c * hw] : (c < kNG + kNS ? S[c - kNG] : 0.0f);
      }
    }
    if (a.canon) {                      // read back by the same wave
      if (a.k <= kFastK) {
        float al[kFastK];
#pragma unroll
        for (int j = 0; j < kFastK; ++j)
          al[j] = j < a.k ? L[((size_t)j * kNL + kAlpha) * hw] : 0.0f;
        rank_slots(al, L, hw, a.k, g, order);
      } else {
        for (int i = g; i < a.k; i += 4) order[slot_rank(L, (size_t)hw, a.k, i)] = (uint8_t)i;
      }
    }
    // A slot's raw channels g, 4 + g, 8 + g (the inputs of K-steps 0..2 of
    // every encoding block: 12 channels, three steps) and its alpha.
    auto load = [&](int i, float (&r)[3], float &alpha) {
      const int slot = a.canon ? (int)order[i] : i;
      const float *Li = L + (size_t)slot * kNL * hw;
#pragma unroll
      for (int j = 0; j < 3; ++j) r[j] = Li[(size_t)(4 * j + g) * hw];
      alpha = Li[(size_t)kAlpha * hw];
    };
    float raw[3] = {0.f, 0.f, 0.f}, al = 0.0f;
    if (a.k > 0) load(0, raw, al);

    // F on the (encoded) [G; s]: input k is channel k % 30 of block k / 30
    pipe.gather(acc, ENC ? a.kq_x : 2, [&](int qq) {
      f32x4 x;
      if constexpr (!ENC) {
        x = qq == 0 ? xr[0] : xr[1];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = 16 * qq + 4 * j + g, b = k / (kNG + kNS), c = k - b * (kNG + kNS);
          const float v = c < kNG ? G[(size_t)c * hw] : S[c - kNG];
          x[j] = b < nblk ? pe_value(v, b) : 0.0f;
        }
      }
      if constexpr (!CAL) *(f32x4 *)(a.pl.x + (uint32_t)pl * a.pl.nx + 16 * qq + 4 * g) = x;
      return x;
    });
    next(in, acc, L_F1, true);
    if constexpr (ENC && !CAL)                           // the block's padding
      for (int i = a.kq_x; i < a.pl.nx / 16; ++i)
        *(f32x4 *)(a.pl.x + (uint32_t)pl * a.pl.nx + 16 * i + 4 * g) = zero4();
    keep(a.pl.a1, K_A1, in);
    pipe.chain(acc, in);
    next(in, acc, L_F2, true);
    keep(a.pl.a2, K_A2, in);
    pipe.chain(acc, in);
    next(in, acc, L_F3, false);                          // sigma
    save(a.pl.sig, in);
    // u = W_T1,sigma sigma + b_T1 (the sigma-hoist)
    pipe.chain(acc, in);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      u[mt] = acc[mt] + bias(L_T1, mt);
      acc[mt] = zero4();
      Z[mt] = zero4();
    }
    // per slot: z1 = relu(W_T1,b b_i + u), Z += m_i relu(W_T2 z1 + b_T2)
    float cnt = 0.0f;
    for (int i = 0; i < a.k; ++i) {
      float rn[3] = {0.f, 0.f, 0.f}, an = 0.0f;
      if (i + 1 < a.k) load(i + 1, rn, an);
      const float m = al > 0.0f ? 1.0f : 0.0f;
      float *bi = a.pl.bi + i * a.pl.np * a.pl.nb;
      pipe.gather(acc, ENC ? a.kq_b : 1, [&](int qq) {
        f32x4 x = {raw[0], raw[1], raw[2], 0.0f};
        if constexpr (ENC) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int s = 4 * qq + j, b = s / 3, c = s - 3 * b;
            const float r = c == 0 ? raw[0] : (c == 1 ? raw[1] : raw[2]);
            x[j] = b < nblk ? pe_value(r, b) : 0.0f;
          }
        }
        if constexpr (!CAL) *(f32x4 *)(bi + (uint32_t)pl * a.pl.nb + 16 * qq + 4 * g) = x;
        return x;
      });
      if constexpr (ENC && !CAL)                         // the block's padding
        for (int j = a.kq_b; j < a.pl.nb / 16; ++j)
          *(f32x4 *)(bi + (uint32_t)pl * a.pl.nb + 16 * j + 4 * g) = zero4();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        in[mt] = relu4(acc[mt] + u[mt]);
        acc[mt] = zero4();
      }
      if constexpr (CAL) {
        if (a.pl.p0 + pl < a.npx)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            amax = fmaxf(amax, fmaxf(fmaxf(in[mt][0], in[mt][1]), fmaxf(in[mt][2], in[mt][3])));
      } else {
        keep(a.pl.z1 + (int64_t)i * a.pl.np * W, kMasks + 2 * i, in);
        pipe.chain(acc, in);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = acc[mt] + bias(L_T2, mt);
        signs(kMasks + 2 * i + 1, acc, al > 0.0f);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          Z[mt] += relu4(acc[mt]) * m;
          acc[mt] = zero4();
        }
        cnt += m;
      }
#pragma unroll
      for (int j = 0; j < 3; ++j) raw[j] = rn[j];
      al = an;
    }
    if constexpr (CAL) continue;
    // the pool, T3 (tau), B on [sigma; tau], R on [phi; L_d]
    const float ld = g < 3 ? G[(size_t)(11 + g) * hw] : 0.0f;
    const float inv = a.mean ? 1.0f / fmaxf(cnt, 1.0f) : 1.0f;
    const float bs = a.mean ? (cnt > 0.0f ? 1.0f : 0.0f) : cnt;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) in[mt] = Z[mt] * inv;
    save(a.pl.zs, in);
    if (g == 0) {
      a.pl.inv[pl] = inv;
      a.pl.bs[pl] = bs;
    }
    pipe.chain(acc, in);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const f32x4 b = bias(L_T3, mt);
#pragma unroll
      for (int r = 0; r < 4; ++r) in[mt][r] = fmaf(b[r], bs, acc[mt][r]);
      acc[mt] = zero4();
    }
    save(a.pl.tau, in);
    {
      f32x4 s[MT];                                       // sigma, back from its block
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) s[mt] = *(const f32x4 *)((const char *)a.pl.sig + at + 64 * mt);
      pipe.chain(acc, s);
    }
    pipe.chain(acc, in);
    next(in, acc, L_B1, true);
    keep(a.pl.d1, K_D1, in);
    pipe.chain(acc, in);
    next(in, acc, L_B2, true);
    keep(a.pl.d2, K_D2, in);
    pipe.chain(acc, in);
    next(in, acc, L_B3, false);                          // phi
    save(a.pl.phi, in);
    pipe.chain(acc, in);
    pipe.gather(acc, 1, [&](int) { return f32x4{ld, 0.f, 0.f, 0.f}; });
    next(in, acc, L_R1, true);
    keep(a.pl.g1, K_G1, in);
    pipe.chain(acc, in);
    next(in, acc, L_R2, true);
    keep(a.pl.g2, K_G2, in);
  }
  if constexpr (CAL) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) amax = fmaxf(amax, __shfl_xor(amax, d));
    if (lane == 0) atomicMax(a.amax, __float_as_uint(amax));   // non-negative: bit order
  }
}

// ---- deltas ---------------------------------------------------------------------
struct DeltaArgs {
  const uint8_t *packed;
  Program pg;
  Planes pl;
  const float *dy;           // the caller's dL/dy [n][3][hw]
  int32_t hw, k;
  int64_t npx;
};

// A wave owns 16 pixels, a workgroup WAVES * 16.  The maps run on split operands
// (fp32_core.h); sigma's delta waits in LDS while the slots run.  The bf16
// instruction rounds its sums towards minus infinity, which a sum over many
// pixels would collect (1e-5 of a gradient over 2^18 pixels with random dy): so
// each K-step is summed by itself (SplitPipe's FRESH), and a pixel's deltas are
// computed with the sign of its place (sign_of).
//
// What bounds it: HBM and the matrix cores in turn.  16 x 128^2, K = 4, W = 128:
// 2.0 GB of deltas written (390 us at the copy rate) and 340 us of matrix-core
// work take 855 us (837 with the K-steps in one chain, whose gradient is 2 to
// 15 times further from 64 bits); on the fp32 instruction, with 900 us of such
// work, 1132.
template <int W, int WAVES>
__global__ __launch_bounds__(WAVES * 64, WAVES / 4) void f32_delta_kernel(DeltaArgs a) {
  constexpr int MT = W / 16, KS = W / 32, kPx = WAVES * 16;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int wave = threadIdx.x >> 6;
  f32x4 *l_dsig = (f32x4 *)(lds + kRing * kSplitStage) + wave * MT * 64 + (threadIdx.x & 63);
  SplitPipe<MT, WAVES, true> pipe;
  pipe.start(a.packed, lds, a.pg);
  const int64_t ntiles = a.pl.np / kPx;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    int g = (threadIdx.x & 63) >> 4, col = threadIdx.x & 15;
    asm volatile("" : "+v"(g), "+v"(col));      // per-tile copies, as in the forward
    const int64_t pl = tile * kPx + wave * 16 + col, p = a.pl.p0 + pl;
    const uint32_t at = (uint32_t)pl * (W * 4) + 16 * g;
    const float sign = sign_of((uint32_t)p);
    f32x4 acc[MT];
    Split in[KS];
    auto signs = [&](int layer) {
      const uint32_t *words = a.pl.mask + (int64_t)layer * (a.pl.np / 16) * 64;
      return words[(uint32_t)(tile * (WAVES * 64)) + threadIdx.x];
    };
    // v to its plane; v, split, to the next map
    auto put = [&](float *plane, const f32x4 (&v)[MT]) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) *(f32x4 *)((char *)plane + at + 64 * mt) = sign * v[mt];
    };
    auto feed = [&](const f32x4 (&v)[MT]) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = v[2 * s + (j >> 2)][j & 3];
        in[s] = split8(x);
      }
    };
    // v where the bits say so
    auto mask = [&](f32x4 (&v)[MT], uint32_t bits) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[mt][r] = bits & (1u << (4 * mt + r)) ? v[mt][r] : 0.0f;
    };
    // dL/dy of the pixel: lane group g < 3 channel g (padding pixels: zero, so
    // every delta of theirs is zero)
    float dy = 0.0f;
    if (g < 3 && p < a.npx) {
      const int64_t f = p / a.hw;
      dy = a.dy[(f * kNOUT + g) * a.hw + (p - f * a.hw)];
    }
    *(f32x4 *)(a.pl.dy + (uint32_t)pl * kDyWidth + 4 * g) = f32x4{dy, 0.f, 0.f, 0.f};
    dy *= sign;
    uint32_t bits = signs(K_G2), nbits = signs(K_G1);
    pipe.gather(acc, 1, [&](int) {
      const float x[8] = {dy, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      return split8(x);
    });
    auto next = [&](float *plane) {            // the accumulators are this plane's delta
      put(plane, acc);
      feed(acc);
    };
    mask(acc, bits);
    next(a.pl.dg2);
    bits = signs(K_D2);
    pipe.chain(acc, in);
    mask(acc, nbits);
    next(a.pl.dg1);
    pipe.chain(acc, in);
    next(a.pl.dphi);
    nbits = signs(K_D1);
    pipe.chain(acc, in);
    mask(acc, bits);
    next(a.pl.dd2);
    const float inv = a.pl.inv[(uint32_t)pl];
    pipe.chain(acc, in);
    mask(acc, nbits);
    next(a.pl.dd1);
    pipe.chain(acc, in);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) l_dsig[mt * 64] = acc[mt];
    pipe.chain(acc, in);
    next(a.pl.dtau);
    pipe.chain(acc, in);
    f32x4 dz[MT], du[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      dz[mt] = acc[mt] * inv;                   // dZ = W_T3^T dtau / max(c, 1)
      du[mt] = zero4();
    }
    put(a.pl.dz, dz);
    uint32_t b2 = 0, b1 = 0;
    if (a.k > 0) {
      b1 = signs(kMasks);
      b2 = signs(kMasks + 1);
    }
    for (int i = 0; i < a.k; ++i) {
      uint32_t n1 = 0, n2 = 0;
      if (i + 1 < a.k) {
        n1 = signs(kMasks + 2 * i + 2);
        n2 = signs(kMasks + 2 * i + 3);
      }
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          x[j] = b2 & (1u << (8 * s + j)) ? dz[2 * s + (j >> 2)][j & 3] : 0.0f;
        in[s] = split8(x);
      }
      pipe.chain(acc, in);
      mask(acc, b1);
      put(a.pl.dz1 + (int64_t)i * a.pl.np * W, acc);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) du[mt] += acc[mt];
      b1 = n1;
      b2 = n2;
    }
    put(a.pl.du, du);
    feed(du);
    bits = signs(K_A2);
    nbits = signs(K_A1);
    pipe.chain(acc, in);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] += l_dsig[mt * 64];
    next(a.pl.dsig);
    pipe.chain(acc, in);
    mask(acc, bits);
    next(a.pl.da2);
    pipe.chain(acc, in);
    mask(acc, nbits);
    put(a.pl.da1, acc);
  }
}

// ---- weight gradients -------------------------------------------------------------
// One product sum_p D[p] A[p]^T over a slab's pixels (and its slots): D a
// block W wide, A 16 MI columns of a block lda wide.
struct DwJob {
  const float *D, *A;
  const uint32_t *mask;      // D taken where the bits say so (dz2 = selected dZ), or null
  const float *wgt;          // per-pixel weight of D in its sums (T3's bias scale), or null
  int64_t dslot, aslot, mslot;   // slot strides (elements)
  int32_t lda, slots;
};
constexpr int kMaxJobs = 20;
// The products of one shape, and the split of their steps (kStep pixels each)
// over the workgroups: workgroup w takes steps [w per, (w + 1) per) of the
// jobs laid end to end and writes one partial per job it meets, the w-th plus
// the job's number.
struct DwArgs {
  DwJob job[kMaxJobs];
  int32_t njobs, per, accumulate;
  int64_t np, steps;         // pixels; steps per slot (the first slab's)
  float *part;
};
constexpr int kStep = 32;
// A partial: the product [W][16 MI], D's column sums (W), A's (16 MI).
constexpr int part_floats(int W, int MI) { return W * 16 * MI + W + 16 * MI; }

// Four waves split the W x 16 MI tile: 2 x 2 for a square one, by rows for a
// narrow one.  Each 32-pixel step of both blocks is loaded to registers while
// the step before computes, then written to LDS; row p of a block keeps its
// 16-byte unit c at c ^ swz(p), so that the four pixels that the lane groups
// read fall into distinct banks.  A step is one 32-deep group of the bf16 matrix
// cores on operands split in three (fp32_core.h), summed by itself before it is
// added, a workgroup's with the sign of its place, as the deltas are.  The plain
// split is used, and the values are watched as they are stored: a segment with
// one that it does not take is run again with the wide one (16 x 128^2, K = 4,
// W = 128, the square products' launch: 983 us with the wide split throughout,
// 910 as it is; 890 with the K-steps in one chain).
template <int W, int MI>
__global__ __launch_bounds__(kThreads, 2) void f32_dw_kernel(DwArgs a) {
  constexpr int MO = W / 16;
  constexpr bool kSquare = MI >= 4;
  constexpr int WR = kSquare ? 2 : 4, WC = 4 / WR;           // wave grid
  constexpr int TO = MO / WR, TI = MI / WC;                   // tiles per wave
  constexpr int DU = W / 4, AU = 4 * MI;                      // 16-byte units per pixel
  constexpr int ND = kStep * DU / kThreads;                   // units per thread
  constexpr int NA = (kStep * AU + kThreads - 1) / kThreads;
  __shared__ f32x4 ld[2][kStep * DU], la[2][kStep * AU];
  __shared__ float lw[2][kStep];
  __shared__ int l_wide;             // some value of the segment needs the wide split
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l = lane & 15;
  const int wr = wave / WC, wc = wave % WC;
  const float sign = sign_of(blockIdx.x);
  auto dswz = [](int p) { return 4 * (p & 3); };
  auto aswz = [](int p) { return MI >= 4 ? 4 * (p & 3) : (MI == 2 ? 4 * ((p >> 1) & 1) : 0); };

  int64_t step = (int64_t)blockIdx.x * a.per, end = step + a.per, first = 0;
  for (int j = 0; j < a.njobs; ++j) {
    const DwJob &job = a.job[j];
    const int64_t jend = first + job.slots * a.steps;
    // (a short last slab ends its jobs early: its partials are complete)
    const int64_t s0 = std::max(step, first) - first;
    const int64_t s1 = std::min(std::min(end, jend) - first, job.slots * (a.np / kStep));
    first = jend;
    if (s0 >= s1) continue;
    f32x4 hd[ND], ha[NA];
    uint32_t hm[ND];
    float hw = 1.0f;
    auto load = [&](int64_t s) {
      s = std::min(s, s1 - 1);
      // pixels first, a pixel block's slots in turn (dZ, the same for all of
      // them, then comes from L2)
      const int64_t ps = s / job.slots, slot = s - ps * job.slots, px = ps * kStep;
      const float *D = job.D + slot * job.dslot + px * W;
      const float *A = job.A + slot * job.aslot + px * job.lda;
#pragma unroll
      for (int i = 0; i < ND; ++i) hd[i] = ((const f32x4 *)D)[tid + i * kThreads];
      if (job.mask) {
        const uint32_t *M = job.mask + slot * job.mslot + px * 4;   // 64 words per 16 pixels
#pragma unroll
        for (int i = 0; i < ND; ++i) {
          const int e = tid + i * kThreads, p = e / DU, u = e % DU;
          hm[i] = M[(p >> 4) * 64 + (u & 3) * 16 + (p & 15)] >> (4 * (u >> 2));
        }
      }
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const int e = std::min(tid + i * kThreads, kStep * AU - 1);
        ha[i] = *(const f32x4 *)(A + (e / AU) * job.lda + 4 * (e % AU));
      }
      if (job.wgt && tid < kStep) hw = job.wgt[px + tid];
    };
    auto store = [&](int b) {
      float sum = 0.0f;
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        const int e = tid + i * kThreads, p = e / DU, u = e % DU;
        f32x4 v = hd[i];
        if (job.mask) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = hm[i] & (1u << r) ? v[r] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) sum = watch(v[r], sum);
        ld[b][p * DU + (u ^ dswz(p))] = v;
      }
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const int e = tid + i * kThreads, p = e / AU, u = e % AU;
#pragma unroll
        for (int r = 0; r < 4; ++r) sum = watch(ha[i][r], sum);
        if (kStep * AU % kThreads == 0 || e < kStep * AU)
          la[b][p * AU + (u ^ aswz(p))] = sign * ha[i];
      }
      if (tid < kStep) lw[b][tid] = hw;
      if (found(sum)) l_wide = 1;
    };
    f32x4 acc[TO][TI];
    float dsum[TO], asum[TI];
    auto segment = [&](auto wide) {
      constexpr bool kWide = decltype(wide)::value;
#pragma unroll
      for (int o = 0; o < TO; ++o) {
        dsum[o] = 0.0f;
#pragma unroll
        for (int i = 0; i < TI; ++i) acc[o][i] = zero4();
      }
#pragma unroll
      for (int i = 0; i < TI; ++i) asum[i] = 0.0f;
      // both buffers are free: every wave is past the last run's reads
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      load(s0);
      store(0);
      load(s0 + 1);
      for (int64_t s = s0; s < s1; ++s) {
        const int b = (int)(s - s0) & 1;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        store(b ^ 1);
        load(s + 2);
        __builtin_amdgcn_sched_barrier(0);
        const float *D = (const float *)ld[b], *A = (const float *)la[b];
        // a lane's eight pixels of a row: 4 t + g (dswz(p) = 4 g for each)
        float w8[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) w8[t] = lw[b][4 * t + g];
        Split d[TO];
#pragma unroll
        for (int o = 0; o < TO; ++o) {
          float v[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const int p = 4 * t + g;
            v[t] = D[p * W + ((4 * (wr * TO + o)) ^ dswz(p)) * 4 + l];
            if (wc == 0) dsum[o] = fmaf(v[t], w8[t], dsum[o]);
          }
          d[o] = split8<kWide>(v);
        }
#pragma unroll
        for (int i = 0; i < TI; ++i) {
          float v[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const int p = 4 * t + g;
            v[t] = A[p * 16 * MI + ((4 * (wc * TI + i)) ^ aswz(p)) * 4 + l];
            if (!kSquare) asum[i] += v[t];
          }
          const Split x = split8<kWide>(v);
#pragma unroll
          for (int o = 0; o < TO; ++o) acc[o][i] += mma_split(d[o], x, zero4());
        }
      }
    };
    // Set back before the run's first barrier: no wave sets it before that, and
    // where it is set, every wave has read it before the second run's first.
    if (tid == 0) l_wide = 0;
    segment(std::false_type());
    // again from the start where a value asks for it
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (__builtin_amdgcn_readfirstlane(l_wide)) segment(std::true_type());
    float *P = a.part + (size_t)(blockIdx.x + j) * part_floats(W, MI);
    auto put = [&](float *dst, float v) { *dst = a.accumulate ? *dst + v : v; };
#pragma unroll
    for (int o = 0; o < TO; ++o)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          put(P + (16 * (wr * TO + o) + 4 * g + r) * 16 * MI + 16 * (wc * TI + i) + l,
              sign * acc[o][i][r]);
#pragma unroll
    for (int o = 0; o < TO; ++o) {
      dsum[o] += __shfl_xor(dsum[o], 16);
      dsum[o] += __shfl_xor(dsum[o], 32);
      if (wc == 0 && g == 0) put(P + W * 16 * MI + 16 * (wr * TO + o) + l, dsum[o]);
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      asum[i] += __shfl_xor(asum[i], 16);
      asum[i] += __shfl_xor(asum[i], 32);
      if (wr == 0 && g == 0) put(P + W * 16 * MI + W + 16 * (wc * TI + i) + l, sign * asum[i]);
    }
  }
}

// ---- reduction into grad_w ----------------------------------------------------------
// Where a product lands: grad_w[w + o so + i si] for row o (a neuron) and
// input i in [i0, i1) of the block (less ibase); D's column sums are the bias
// gradient of layer bias, A's that of R's last layer (asum).
struct RedJob {
  const float *part;         // the first of its partials
  int32_t count, floats;     // partials, their stride
  int32_t cols;              // 16 MI
  int32_t acol;              // first column of the block
  int64_t w;
  int32_t so, si, i0, i1, ibase;
  int64_t bias, asum;        // float offsets in grad_w, or -1
};
constexpr int kMaxRed = 24;
struct RedArgs {
  RedJob job[kMaxRed];
  float *gw;
  int32_t W;
};

// A workgroup owns 16 float4 columns of a product: its thread group c sums
// partials c, c + 16, ... in order, then group 0 adds the 16 sums in order.
// (A thread per column and a plain loop over up to 150 partials is one chain
// of memory latencies: 115 us against 33 at 16 x 128^2, K = 4, W = 128.)
__global__ __launch_bounds__(kThreads) void f32_reduce_kernel(RedArgs a) {
  __shared__ f32x4 red[16][16];
  const RedJob &j = a.job[blockIdx.y];
  const int W = a.W, v = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int e = (blockIdx.x * 16 + v) * 4;
  f32x4 s = zero4();
  if (e < j.floats)
    for (int c = grp; c < j.count; c += 16) s += *(const f32x4 *)(j.part + (size_t)c * j.floats + e);
  red[grp][v] = s;
  __syncthreads();
  if (grp != 0 || e >= j.floats) return;
  for (int c = 1; c < 16; ++c) s += red[c][v];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int x = e + t;
    if (x < W * j.cols) {
      const int o = neuron_at(x / j.cols), i = neuron_at(j.acol + x % j.cols);
      if (i >= j.i0 && i < j.i1) a.gw[j.w + (int64_t)o * j.so + (int64_t)(i - j.ibase) * j.si] = s[t];
    } else if (x < W * j.cols + W) {
      if (j.bias >= 0) a.gw[j.bias + neuron_at(x - W * j.cols)] = s[t];
    } else if (j.asum >= 0) {
      const int i = neuron_at(x - W * j.cols - W);
      if (i < kNOUT) a.gw[j.asum + i] = s[t];
    }
  }
}

// ---- host ---------------------------------------------------------------------------
static inline int64_t rup(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Widths of the encoded inputs' blocks: 32 and 16 without encoding, else
// whole W-wide products.
static int x_width(int W, int pe) { return pe == 0 ? 32 : (int)rup((kNG + kNS) * pe_blocks(pe), W); }
static int b_width(int W, int pe) { return pe == 0 ? 16 : (int)rup(kNL * pe_blocks(pe), W); }

// Floats a slab keeps per pixel (its planes, signs and scalars).
static int64_t px_floats(int W, int pe, int k) {
  return x_width(W, pe) + 21 * (int64_t)W + kDyWidth + 2 + 4 * (kMasks + 2 * k) +
         (int64_t)k * (2 * W + b_width(W, pe));
}

// The most bytes that a call's planes take: what its pixels, or kSlabLeast of
// them, need with four slots, and never more than kSlabBytes.  A call of more
// slots runs in more slabs instead (16 x 128^2, W = 128, K = 8: two), so that
// the workspace does not grow with their number.  kSlabLeast: that many pixels
// are one round of the recompute's workgroups; smaller slabs would leave CUs
// idle (128^2, W = 128, K = 8: 512 us in one slab, 749 in two).
constexpr size_t kSlabBytes = (size_t)16 << 30;
constexpr int64_t kSlabStep = 2 * kTile, kSlabLeast = 32768;
static int64_t most_plane_bytes(int W, int pe, int64_t npx) {
  return std::min((int64_t)kSlabBytes, (int64_t)sizeof(float) * px_floats(W, pe, 4) *
                                           std::max(rup(npx, kSlabStep), kSlabLeast));
}
// A slab's pixels: slabs of equal length (the last may be shorter).
static int64_t slab_px(int W, int pe, int k, int64_t npx) {
  const int64_t fit = most_plane_bytes(W, pe, npx) / ((int64_t)sizeof(float) * px_floats(W, pe, k));
  const int64_t most = fit / kSlabStep * kSlabStep, slabs = (npx + most - 1) / most;
  return rup((npx + slabs - 1) / slabs, kSlabStep);
}

static Planes carve(float *mem, int W, int pe, int k, int64_t np) {
  Planes p{};
  p.np = np;
  p.nx = x_width(W, pe);
  p.nb = b_width(W, pe);
  auto take = [&](int64_t width) { float *q = mem; mem += width * np; return q; };
  p.x = take(p.nx);
  for (float **q : {&p.a1, &p.a2, &p.sig, &p.zs, &p.tau, &p.d1, &p.d2, &p.phi, &p.g1, &p.g2, &p.dg2,
                    &p.dg1, &p.dphi, &p.dd2, &p.dd1, &p.dtau, &p.dsig, &p.dz, &p.du, &p.da2, &p.da1})
    *q = take(W);
  p.dy = take(kDyWidth);
  p.inv = take(1);
  p.bs = take(1);
  p.mask = (uint32_t *)take(4 * (kMasks + 2 * k));
  p.z1 = take((int64_t)k * W);
  p.dz1 = take((int64_t)k * W);
  p.bi = take((int64_t)k * p.nb);
  return p;
}

// The products of one shape over a slab, and where they land.
struct DwGroup {
  int MI;                    // 16-column tiles of A
  DwArgs a;
  RedJob red[kMaxJobs];
  int grid;
  int64_t total;
};

class Gradient {
 public:
  Gradient(int W, int pe, int k, int num_cus) : W_(W), k_(k), cus_(num_cus) {
    layer_offsets(W, pe, lo_);
    pe_ = pe;
    for (int i = 0; i < 3; ++i) memset(&g_[i], 0, sizeof g_[i]);
    g_[0].MI = W / 16;
    g_[1].MI = 1;
    g_[2].MI = 2;
    jobs(Planes{});
  }
  // As many workgroups as the CUs hold (LDS: two of 64 KB, four of the smaller
  // ones).
  static int64_t group_cap(int W, int MI, int cus) { return (int64_t)cus * (W == 128 && MI >= 4 ? 2 : 4); }
  // The floats of all partials, whatever the call.
  static size_t part_room(int W, int cus) {
    size_t floats = 0;
    for (int MI : {W / 16, 1, 2}) floats += (size_t)(group_cap(W, MI, cus) + kMaxJobs) * part_floats(W, MI);
    return floats;
  }
  // Splits the groups' steps over workgroups for slabs of np pixels.
  void split(int64_t np) {
    size_t floats = 0;
    for (DwGroup &g : g_) {
      g.a.steps = np / kStep;
      g.total = 0;
      for (int j = 0; j < g.a.njobs; ++j) g.total += g.a.job[j].slots * g.a.steps;
      // at least 4 steps each (a partial costs about as much traffic as two)
      const int64_t cap = group_cap(W_, g.MI, cus_);
      g.a.per = (int32_t)std::max<int64_t>((g.total + cap - 1) / cap, 4);
      g.grid = (int)((g.total + g.a.per - 1) / g.a.per);
      g.a.part = (float *)nullptr + floats;                  // an offset, until bind()
      floats += (size_t)(cap + kMaxJobs) * part_floats(W_, g.MI);
    }
  }
  void bind(float *part) {
    for (DwGroup &g : g_) g.a.part = part + (g.a.part - (float *)nullptr);
  }
  hipError_t accumulate(const Planes &p, bool first, hipStream_t s) {
    jobs(p);
    for (DwGroup &g : g_) {
      g.a.np = p.np;
      g.a.accumulate = first ? 0 : 1;
      if (g.grid == 0) continue;
#define GO(W, MI) hipLaunchKernelGGL((f32_dw_kernel<W, MI>), dim3(g.grid), dim3(kThreads), 0, s, g.a)
      if (W_ == 128) {
        if (g.MI == 8) GO(128, 8); else if (g.MI == 1) GO(128, 1); else GO(128, 2);
      } else {
        if (g.MI == 4) GO(64, 4); else if (g.MI == 1) GO(64, 1); else GO(64, 2);
      }
#undef GO
    }
    return hipGetLastError();
  }
  hipError_t reduce(float *gw, hipStream_t s) {
    RedArgs r;
    r.gw = gw;
    r.W = W_;
    int n = 0, most = 0;
    for (DwGroup &g : g_) {
      int64_t first = 0;
      for (int j = 0; j < g.a.njobs; ++j) {
        RedJob &d = r.job[n++] = g.red[j];
        const int64_t end = first + g.a.job[j].slots * g.a.steps;
        d.floats = part_floats(W_, g.MI);
        d.cols = 16 * g.MI;
        d.count = end > first ? (int)((end - 1) / g.a.per - first / g.a.per + 1) : 0;
        d.part = g.a.part + (size_t)(first / g.a.per + j) * d.floats;
        most = std::max(most, d.floats);
        first = end;
      }
    }
    hipLaunchKernelGGL(f32_reduce_kernel, dim3((most / 4 + 15) / 16, n),
                       dim3(kThreads), 0, s, r);
    return hipGetLastError();
  }

 private:
  // Adds a product to a group (its split and partials stay as they are).
  void add(int grp, DwJob job, RedJob red) {
    DwGroup &g = g_[grp];
    g.red[g.a.njobs] = red;
    g.a.job[g.a.njobs++] = job;
  }
  void jobs(const Planes &p) {
    const int W = W_;
    for (DwGroup &g : g_) g.a.njobs = 0;
    auto mat = [&](const float *D, const float *A, Layer l, int col0, bool bias,
                   const float *wgt = nullptr) {
      add(0, DwJob{D, A, nullptr, wgt, 0, 0, 0, W, 1},
          RedJob{nullptr, 0, 0, 0, 0, lo_[l].w + col0, lo_[l].in, 1, 0, W, 0, bias ? lo_[l].b : -1, -1});
    };
    const int nb = kNL * pe_blocks(pe_), nx = (kNG + kNS) * pe_blocks(pe_);
    // h's second layer over every slot: dz2 is dZ where z2 > 0 and alpha > 0
    add(0, DwJob{p.dz, p.z1, p.mask + (int64_t)(kMasks + 1) * (p.np / 16) * 64, nullptr, 0, p.np * W,
                 2 * (p.np / 16) * 64, W, k_},
        RedJob{nullptr, 0, 0, 0, 0, lo_[L_T2].w, W, 1, 0, W, 0, lo_[L_T2].b, -1});
    mat(p.dg2, p.g1, L_R2, 0, true);
    mat(p.dg1, p.phi, L_R1, 0, true);
    mat(p.dphi, p.d2, L_B3, 0, true);
    mat(p.dd2, p.d1, L_B2, 0, true);
    mat(p.dd1, p.sig, L_B1, 0, true);
    mat(p.dd1, p.tau, L_B1, W, false);
    mat(p.dtau, p.zs, L_T3, 0, true, p.bs);
    mat(p.du, p.sig, L_T1, nb, false);
    mat(p.dsig, p.a2, L_F3, 0, true);
    mat(p.da2, p.a1, L_F2, 0, true);
    // R1's L_d columns: G-buffer channels 11..13, in F's input block
    add(2, DwJob{p.dg1, p.x, nullptr, nullptr, 0, 0, 0, x_width(W, pe_), 1},
        RedJob{nullptr, 0, 0, 0, 0, lo_[L_R1].w + W, W + 3, 1, 11, 14, 11, -1, -1});
    // R3, transposed: rows are its inputs, columns its outputs
    add(1, DwJob{p.g2, p.dy, nullptr, nullptr, 0, 0, 0, kDyWidth, 1},
        RedJob{nullptr, 0, 0, 0, 0, lo_[L_R3].w, 1, W, 0, kNOUT, 0, -1, lo_[L_R3].b});
    // F1 and h's slot columns: narrow without encoding, W columns at a time with it
    const int xw = pe_ == 0 ? 32 : W, bw = pe_ == 0 ? 16 : W;
    for (int c = 0; c < x_width(W, pe_); c += xw)
      add(pe_ == 0 ? 2 : 0, DwJob{p.da1, p.x + c, nullptr, nullptr, 0, 0, 0, x_width(W, pe_), 1},
          RedJob{nullptr, 0, 0, 0, c, lo_[L_F1].w, nx, 1, 0, nx, 0, c == 0 ? lo_[L_F1].b : -1, -1});
    for (int c = 0; c < b_width(W, pe_); c += bw)
      add(pe_ == 0 ? 1 : 0,
          DwJob{p.dz1, p.bi + c, nullptr, nullptr, p.np * W, p.np * b_width(W, pe_), 0, b_width(W, pe_), k_},
          RedJob{nullptr, 0, 0, 0, c, lo_[L_T1].w, nb + W, 1, 0, nb, 0, c == 0 ? lo_[L_T1].b : -1, -1});
  }

  int W_, pe_, k_, cus_;
  LayerOff lo_[kNumLayers];
  DwGroup g_[3];             // W x W, W x 16, W x 32
};

template <int W, bool ENC, bool CAL>
static hipError_t launch_save_form(const SaveArgs &a, int num_cus, hipStream_t s) {
  const size_t lds = kRing * kStageBytes + sizeof(float) * kNumLayers * W + (size_t)kTile * a.kpad;
  static LdsLimit limit;
  const hipError_t e = limit.raise((const void *)f32_save_kernel<W, ENC, CAL>, lds);
  if (e != hipSuccess) return e;
  const unsigned grid = (unsigned)std::min<int64_t>(a.pl.np / kTile, 2 * num_cus);
  hipLaunchKernelGGL((f32_save_kernel<W, ENC, CAL>), dim3(grid), dim3(kThreads), lds, s, a);
  return hipGetLastError();
}

template <bool CAL>
static hipError_t launch_save(int W, const SaveArgs &a, int num_cus, hipStream_t s) {
  if (W == 128)
    return a.pe > 0 ? launch_save_form<128, true, CAL>(a, num_cus, s)
                    : launch_save_form<128, false, CAL>(a, num_cus, s);
  return a.pe > 0 ? launch_save_form<64, true, CAL>(a, num_cus, s)
                  : launch_save_form<64, false, CAL>(a, num_cus, s);
}

// Packs the maps of up to two tables.
static hipError_t launch_pack(const float *master, const PackArgs &p, int tables, hipStream_t s) {
  int64_t n = 0;
  for (int i = 0; i < tables; ++i)
    n = std::max<int64_t>(n, (int64_t)p.t[i].stages * (i ? kSplitFrags / 3 : kStageFrags) * 64 +
                                 (i ? 0 : kNumLayers * p.t[i].W));
  hipLaunchKernelGGL(f32_pack_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads), tables),
                     dim3(kThreads), 0, s, master, p);
  return hipGetLastError();
}

// The recompute's arguments of a frame (but for its slab), packed weights of
// table t; cal: up to h's first layer.
static SaveArgs save_args(gn_handle *h, const gn_frame *frame, const OpTable &t, const uint8_t *packed,
                          bool cal) {
  SaveArgs a{};
  a.packed = packed;
  a.bias_stage = t.stages;
  const int slots = t.op[O_T1A].stage0, head = t.op[O_T3].stage0;
  a.pg = cal ? Program{0, slots, slots, t.op[O_T2].stage0, 0, 0, frame->k, 0}
             : Program{0, slots, slots, head, head, t.stages, frame->k, 1};
  a.gbuf = frame->gbuf;
  a.layers = frame->layers;
  a.scene = frame->scene;
  a.hw = frame->h * frame->w;
  a.k = frame->k;
  a.mean = h->cfg.pool == GN_POOL_MEAN ? 1 : 0;
  a.pe = h->pl.pe;
  a.canon = !cal && gn_slot_kmax(h) > 1 && frame->k > 1 ? 1 : 0;
  a.kpad = a.canon ? (frame->k + 3) & ~3 : 0;
  a.kq_x = t.op[O_F1].kq;
  a.kq_b = t.op[O_T1A].kq;
  a.npx = (int64_t)frame->n * frame->h * frame->w;
  return a;
}

template <int W, int WAVES>
static hipError_t launch_delta_form(const DeltaArgs &a, int num_cus, hipStream_t s) {
  constexpr int lds = kRing * kSplitStage + WAVES * (W / 16) * 1024;
  static LdsLimit limit;
  const hipError_t e = limit.raise((const void *)f32_delta_kernel<W, WAVES>, lds);
  if (e != hipSuccess) return e;
  const unsigned grid = (unsigned)std::min<int64_t>(a.pl.np / (WAVES * 16), num_cus);
  hipLaunchKernelGGL((f32_delta_kernel<W, WAVES>), dim3(grid), dim3(WAVES * 64), lds, s, a);
  return hipGetLastError();
}

// Four waves (64 pixels) a workgroup where eight would leave CUs idle, as in
// the fp32 forward.
template <int W>
static hipError_t launch_delta(const DeltaArgs &a, int num_cus, hipStream_t s) {
  return a.pl.np <= (int64_t)num_cus * kTile ? launch_delta_form<W, 4>(a, num_cus, s)
                                             : launch_delta_form<W, 8>(a, num_cus, s);
}

}  // namespace f32
}  // namespace gn

using namespace gn;

void gn_bwd_free(gn_handle *h) {
  if (!h->bwd) return;
  (void)hipFree(h->bwd->mem);
  delete h->bwd;
  h->bwd = nullptr;
}

size_t gn_bwd_bytes(gn_handle *h) { return h->bwd ? h->bwd->bytes : 0; }

static gn_status backward(gn_handle *h, const gn_frame *frame, const float *dy, float *grad_w,
                          hipStream_t s) {
  const int W = h->W, pe = h->pl.pe, k = frame->k;
  const int64_t npx = (int64_t)frame->n * frame->h * frame->w;
  if (f32::rup(npx, 4096) > gn_f32_max_px)
    return gn_set_error(GN_E_INVAL, "more than 3 * 2^20 pixels in one call");
  f32::PackArgs pk;
  f32::make_ops(W, pe, &pk.t[0]);
  f32::make_bwd_ops(W, pe, &pk.t[1]);
  const f32::OpTable &tf = pk.t[0], &tb = pk.t[1];
  const int64_t np = f32::slab_px(W, pe, k, npx);
  f32::Gradient grad(W, pe, k, h->num_cus);
  grad.split(np);
  const size_t planes = f32::rup(np * f32::px_floats(W, pe, k) * (int64_t)sizeof(float), 1024);
  const size_t need = planes + f32::packed_bytes(tf) + f32::packed_bytes(tb) +
                      sizeof(float) * f32::Gradient::part_room(W, h->num_cus);
  if (!h->bwd) h->bwd = new BwdWorkspace();
  BwdWorkspace *ws = h->bwd;
  hipError_t e = hipSuccess;
  if (need > ws->bytes) {
    // a grown workspace replaces the old one once the device's earlier work is done
    (void)hipFree(ws->mem);
    ws->mem = nullptr;
    ws->bytes = 0;
    e = hipMalloc((void **)&ws->mem, need);
    if (e == hipSuccess) ws->bytes = need;
  }
  if (e != hipSuccess) {
    gn_bwd_free(h);
    return gn_check_device(h, e, "backward workspace");
  }
  pk.packed[0] = ws->mem + planes;
  pk.packed[1] = pk.packed[0] + f32::packed_bytes(tf);
  grad.bind((float *)(pk.packed[1] + f32::packed_bytes(tb)));
  e = f32::launch_pack(h->d_master, pk, 2, s);
  f32::SaveArgs a = f32::save_args(h, frame, tf, pk.packed[0], false);
  f32::DeltaArgs d{};
  d.packed = pk.packed[1];
  d.pg = f32::Program{0, tb.op[f32::O_T2T].stage0, tb.op[f32::O_T2T].stage0, tb.op[f32::O_T1ST].stage0,
                      tb.op[f32::O_T1ST].stage0, tb.stages, k, 1};
  d.dy = dy;
  d.hw = a.hw;
  d.k = k;
  d.npx = npx;
  const int cus = h->num_cus;
  for (int64_t p0 = 0; p0 < npx && e == hipSuccess; p0 += np) {
    f32::Planes pl = f32::carve((float *)ws->mem, W, pe, k, std::min(np, f32::rup(npx - p0, 2 * f32::kTile)));
    pl.p0 = p0;
    a.pl = d.pl = pl;
    e = f32::launch_save<false>(W, a, cus, s);
    if (e == hipSuccess)
      e = W == 128 ? f32::launch_delta<128>(d, cus, s) : f32::launch_delta<64>(d, cus, s);
    if (e == hipSuccess) e = grad.accumulate(pl, p0 == 0, s);
  }
  if (e == hipSuccess) e = grad.reduce(grad_w, s);
  return gn_check_device(h, e, "backward launch");
}

// The largest first-layer activation of h over every slot of every pixel, as
// float bits in *amax (device).  The packed weights it needs live for the call.
gn_status gn_f32_calibrate(gn_handle *h, const gn_frame *frame, unsigned *amax, hipStream_t s) {
  const int64_t npx = (int64_t)frame->n * frame->h * frame->w;
  if (f32::rup(npx, 4096) > gn_f32_max_px)
    return gn_set_error(GN_E_INVAL, "more than 3 * 2^20 pixels in one call");
  f32::PackArgs pk{};
  f32::make_ops(h->W, h->pl.pe, &pk.t[0]);
  hipError_t e = hipMalloc((void **)&pk.packed[0], f32::packed_bytes(pk.t[0]));
  if (e != hipSuccess) return gn_check_device(h, e, "calibration");
  e = f32::launch_pack(h->d_master, pk, 1, s);
  f32::SaveArgs a = f32::save_args(h, frame, pk.t[0], pk.packed[0], true);
  a.pl.np = f32::rup(npx, f32::kTile);
  a.amax = amax;
  if (e == hipSuccess) e = f32::launch_save<true>(h->W, a, h->num_cus, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(pk.packed[0]);
  return gn_check_device(h, e, "calibration");
}

extern "C" gn_status glassnet_backward(gn_handle *h, const gn_frame *frame,
                                       const float *grad_out, float *grad_w, void *hip_stream) {
  if (!h) return gn_set_error(GN_E_INVAL, "handle is NULL");
  if (h->poisoned) return gn_set_error(GN_E_DEVICE, "handle poisoned by an earlier device error");
  if (!grad_out || !grad_w || ((uintptr_t)grad_out & 3) || ((uintptr_t)grad_w & 3))
    return gn_set_error(GN_E_INVAL, "grad_out and grad_w must be non-NULL, 4-byte aligned");
  gn_status st = gn_validate_frame(h, frame, nullptr);
  if (st != GN_OK) return st;
  int prev = -1;
  (void)hipGetDevice(&prev);
  if (hipSetDevice(h->device) != hipSuccess) return gn_set_error(GN_E_DEVICE, "hipSetDevice failed");
  st = backward(h, frame, grad_out, grad_w, (hipStream_t)hip_stream);
  if (prev >= 0) (void)hipSetDevice(prev);
  return st;
}
