// The fp32 forward: the whole per-pixel network (Sec. 3.3-3.4) in one kernel,
// every activation in registers, fp32 arithmetic on the bf16 matrix cores
// (fp32_core.h: operands split in three, six partial products).  The same
// kernel, cut at compile time, serves the FP32 form's object streaming.
//
// Formulation.  Every map is D = A X with a 16-row tile of A (weights) as the
// row operand and 16 pixels, one wave's, as the columns of
// v_mfma_f32_16x16x32_bf16.  The accumulator leaves lane group g (lane >> 4)
// with rows 4g + r of pixel lane & 15; two row tiles hold the eight values
// that lane presents in a 32-deep K-step of the next map, whose weight
// columns are packed in that order, so activations go from map to map by a
// ReLU and a split inside the lane.
//
// Weights: SplitPipe of fp32_core.h.
//
// Work split.  One workgroup of eight waves per CU takes tiles of 128 pixels
// (four waves and 64 where 128 would leave CUs idle).  Per pixel and wave the
// live state is u, the running sum Z, one map's split inputs and accumulators:
// 144 registers at W = 128; sigma waits in LDS for B's first layer.  The
// slots are pooled in an fp32 running sum in canonical order (slot_order.h),
// or in input order.
//
// What bounds it: the matrix cores and the LDS alike.  16 pixels per fragment
// read make 3 KiB of LDS traffic per six 16-cycle instructions, 128 bytes per
// cycle from a CU's four SIMDs, the rate measured for the LDS.
#include <algorithm>

#include "fp32_core.h"
#include "gn_api_state.h"
#include "lds_limit.h"

namespace gn {
namespace f32 {

// The linear maps in the order the kernel consumes them.
enum Op {
  O_F1, O_F2, O_F3, O_T1S, O_T1A, O_T2, O_T3, O_B1S, O_B1T, O_B2, O_B3, O_R1P, O_R1L, O_R2, O_R3,
  kNumOps
};
// Which input element e of lane group g presents in K-step s: a previous map's
// row (CHAIN); input 32 s + 8 g + e (MEM); value v = 8 s + e of the group's
// list, raw channel 3 g + v % 3 of encoding block v / 3 (SLOT); input g in
// element 0 (LIGHT).
enum Order { CHAIN, MEM, SLOT, LIGHT };

struct OpDesc {
  int64_t woff;      // float offset of the layer's matrix in the master vector
  int32_t ld;        // the layer's input count (master row length)
  int32_t col0, M, K, order;
  int32_t mt, steps; // 16-row tiles, 32-deep K-steps
  int32_t stage0;
};

struct OpTable {
  OpDesc op[kNumOps];
  int32_t stages;
  LayerOff lo[kNumLayers];
  int32_t W, pe;
};

static void make_ops(int W, int pe, OpTable *t) {
  const int blocks = pe_blocks(pe), nx = (kNG + kNS) * blocks, nb = kNL * blocks;
  layer_offsets(W, pe, t->lo);
  t->W = W;
  t->pe = pe;
  const int xs = (nx + 31) / 32, bs = (3 * blocks + 7) / 8, ws = W / 32;
  struct S { Op o; Layer l; int col0, M, K, order, steps; };
  const S s[kNumOps] = {
      {O_F1, L_F1, 0, W, nx, MEM, xs},    {O_F2, L_F2, 0, W, W, CHAIN, ws},
      {O_F3, L_F3, 0, W, W, CHAIN, ws},   {O_T1S, L_T1, nb, W, W, CHAIN, ws},
      {O_T1A, L_T1, 0, W, nb, SLOT, bs},  {O_T2, L_T2, 0, W, W, CHAIN, ws},
      {O_T3, L_T3, 0, W, W, CHAIN, ws},   {O_B1S, L_B1, 0, W, W, CHAIN, ws},
      {O_B1T, L_B1, W, W, W, CHAIN, ws},  {O_B2, L_B2, 0, W, W, CHAIN, ws},
      {O_B3, L_B3, 0, W, W, CHAIN, ws},   {O_R1P, L_R1, 0, W, W, CHAIN, ws},
      {O_R1L, L_R1, W, W, 3, LIGHT, 1},   {O_R2, L_R2, 0, W, W, CHAIN, ws},
      {O_R3, L_R3, 0, kNOUT, W, CHAIN, ws}};
  int stage = 0;
  for (int i = 0; i < kNumOps; ++i) {
    OpDesc &d = t->op[s[i].o];
    d.woff = t->lo[s[i].l].w;
    d.ld = t->lo[s[i].l].in;
    d.col0 = s[i].col0;
    d.M = s[i].M;
    d.K = s[i].K;
    d.order = s[i].order;
    d.steps = s[i].steps;
    d.mt = (d.M + 15) / 16;
    d.stage0 = stage;
    stage += (d.steps * d.mt * 3 + kSplitFrags - 1) / kSplitFrags;
  }
  t->stages = stage;
}

// The stages, then the 12 biases (W floats each).
static size_t packed_bytes(const OpTable &t) {
  return (size_t)t.stages * kSplitStage + sizeof(float) * kNumLayers * t.W;
}

// One thread per lane of a K-step's row tile (its three parts), then the
// biases.  Row i of tile mt is output 16 mt + i.
__global__ __launch_bounds__(256) void f32_split_pack_kernel(const float *__restrict__ master,
                                                             OpTable t, uint8_t *__restrict__ packed) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int total = t.stages * (kSplitFrags / 3) * 64;
  if (e >= total) {
    const int b = e - total, l = b / t.W, o = b % t.W;
    if (l < kNumLayers)
      ((float *)(packed + (size_t)t.stages * kSplitStage))[b] =
          o < t.lo[l].out ? master[t.lo[l].b + o] : 0.0f;
    return;
  }
  const int stage = e / (kSplitFrags / 3 * 64);
  int o = 0;
  while (o + 1 < kNumOps && stage >= t.op[o + 1].stage0) ++o;
  const OpDesc d = t.op[o];
  const int n = (e >> 6) - d.stage0 * (kSplitFrags / 3), lane = e & 63, g = lane >> 4;
  const int step = n / d.mt, m = 16 * (n % d.mt) + (lane & 15);
  float x[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    int k = -1;
    if (step < d.steps) {
      const int v = 8 * step + j;
      if (d.order == CHAIN) k = 32 * step + 16 * (j >> 2) + 4 * g + (j & 3);
      else if (d.order == MEM) k = 32 * step + 8 * g + j;
      else if (d.order == SLOT) k = v / 3 * kNL + 3 * g + v % 3;
      else k = j == 0 ? g : -1;
    }
    x[j] = m < d.M && k >= 0 && k < d.K ? master[d.woff + (int64_t)m * d.ld + d.col0 + k] : 0.0f;
  }
  const Split s = split8(x);
  u32x4 *dst = (u32x4 *)packed + (size_t)(e >> 6) * 3 * 64 + lane;
  dst[0] = s.hi;
  dst[64] = s.mid;
  dst[128] = s.lo;
}

struct FwdArgs {
  const uint8_t *packed;
  int32_t bias_stage;        // the biases follow this many stages
  Program pg;
  const float *gbuf, *layers, *scene;
  float *out;
  int32_t hw, k, mean, pe, kpad;
  int32_t canon;             // pool in canonical order
  int32_t steps_x, steps_b;  // K-steps of F1 and of T1's slot columns
  int64_t npx;
  // object streaming: sigma and the running sum [pixel][W], the active count
  // [pixel]
  float *sig, *z, *cnt;
  int32_t fresh;             // the state holds no sum yet
};

enum Mode { M_FULL, M_BEGIN, M_ACC, M_FINISH };

// ENC: with positional encoding (a form of its own: the sine and cosine's code
// and registers stay out of the plain one).
template <int W, int MODE, bool ENC, int WAVES>
__global__ __launch_bounds__(WAVES * 64, WAVES / 4) void f32_forward_kernel(FwdArgs a) {
  constexpr int MT = W / 16, KS = W / 32, kTile = WAVES * 16;
  constexpr bool kTrunk = MODE == M_FULL || MODE == M_BEGIN;
  constexpr bool kSlots = MODE == M_FULL || MODE == M_ACC;
  constexpr bool kHead = MODE == M_FULL || MODE == M_FINISH;
  // LDS: the stage ring | biases | sigma per wave | slot order per pixel
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  float *l_bias = (float *)(lds + kRing * kSplitStage);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  f32x4 *l_sig = (f32x4 *)(l_bias + kNumLayers * W) + wave * MT * 64 + lane;
  uint8_t *l_order = (uint8_t *)(l_bias + kNumLayers * W) + (kHead ? WAVES * MT * 1024 : 0);
  {
    const float *b = (const float *)(a.packed + (size_t)a.bias_stage * kSplitStage);
    for (int i = threadIdx.x; i < kNumLayers * W; i += WAVES * 64) l_bias[i] = b[i];
  }
  SplitPipe<MT, WAVES, false> pipe;
  pipe.start(a.packed, lds, a.pg);       // ends with a barrier
  const int hw = a.hw, nblk = ENC ? pe_blocks(a.pe) : 1;
  const int64_t ntiles = (a.npx + kTile - 1) / kTile;

  // A lane's pixel of a tile (tail lanes recompute a real pixel), and the
  // first loads it waits for: the inputs of F1 (without encoding) and the
  // alphas its slots are ranked by (up to kFastK slots).  FULL issues them a
  // tile ahead, in the head, where u and Z have left their registers.
  constexpr bool kAhead = MODE == M_FULL;
  struct Pixel {
    int64_t p;
    int f, q;
    bool valid;
  };
  auto locate = [&](int64_t tile, int col) {
    Pixel x;
    x.p = tile * kTile + wave * 16 + col;
    x.valid = x.p < a.npx;
    const int64_t pc = x.valid ? x.p : a.npx - 1;
    x.f = (int)(pc / hw);
    x.q = (int)(pc - (int64_t)x.f * hw);
    return x;
  };
  const bool fast = kSlots && a.canon && a.k <= kFastK;
  auto first_loads = [&](const Pixel &x, int g, float (&xr)[8], float (&al)[kFastK]) {
    if constexpr (kTrunk && !ENC) {
      const float *G = a.gbuf + (size_t)x.f * kNG * hw + x.q, *S = a.scene + (size_t)x.f * kNS;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int c = 8 * g + j;
        xr[j] = c < kNG ? G[(size_t)c * hw] : (c < kNG + kNS ? S[c - kNG] : 0.0f);
      }
    }
    if (fast) {
      const float *L = a.layers + (size_t)x.f * a.k * kNL * hw + x.q;
#pragma unroll
      for (int j = 0; j < kFastK; ++j) al[j] = j < a.k ? L[((size_t)j * kNL + kAlpha) * hw] : 0.0f;
    }
  };
  Pixel nx = locate(blockIdx.x, lane & 15);
  float xr[8], alk[kFastK];
  if constexpr (kAhead) first_loads(nx, lane >> 4, xr, alk);

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    // Opaque per-tile copies of the lane's place keep the compiler from holding
    // every address derived from them in registers across the tile loop.
    int g = lane >> 4, col = lane & 15;
    asm volatile("" : "+v"(g), "+v"(col));
    const Pixel px = kAhead ? nx : locate(tile, col);
    if constexpr (!kAhead) first_loads(px, g, xr, alk);
    const int64_t p = px.p;
    const bool valid = px.valid;
    const int64_t pc = valid ? p : a.npx - 1;
    const int f = px.f, q = px.q;
    const float *G = a.gbuf + (size_t)f * kNG * hw + q;
    const float *L = a.layers + (size_t)f * a.k * kNL * hw + q;
    const float *S = a.scene + (size_t)f * kNS;
    uint8_t *order = l_order + (wave * 16 + col) * a.kpad;
    f32x4 acc[MT], u[MT], Z[MT];
    Split in[KS];
    auto bias = [&](int layer) {           // the accumulators start at the bias
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = *(const f32x4 *)(l_bias + layer * W + 16 * mt + 4 * g);
    };
    // the next map's inputs from values in accumulator order
    auto put = [&](const f32x4 (&v)[MT], bool relu) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const f32x4 x = relu ? relu4(v[2 * s]) : v[2 * s], y = relu ? relu4(v[2 * s + 1]) : v[2 * s + 1];
        const float e[8] = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
        in[s] = split8(e);
      }
    };
    if (kSlots && a.canon) {               // read back by the same wave
      if (fast) rank_slots(alk, L, hw, a.k, g, order);
      else
        for (int i = g; i < a.k; i += 4) order[slot_rank(L, (size_t)hw, a.k, i)] = (uint8_t)i;
    }
    // A slot's raw channels 3g .. 3g + 2 and its alpha.
    auto load = [&](int i, float (&r)[3], float &alpha) {
      const int slot = a.canon ? (int)order[i] : i;
      const float *Li = L + (size_t)slot * kNL * hw;
#pragma unroll
      for (int j = 0; j < 3; ++j) r[j] = Li[(size_t)(3 * g + j) * hw];
      alpha = Li[(size_t)kAlpha * hw];
    };
    float raw[3] = {0.f, 0.f, 0.f}, al = 0.0f;
    if (kSlots && a.k > 0) load(0, raw, al);

    if constexpr (kTrunk) {
      // F on the (encoded) [G; s]: input k is channel k % 30 of block k / 30
      bias(L_F1);
      pipe.gather(acc, ENC ? a.steps_x : 1, [&](int s) {
        if constexpr (!ENC) return split8(xr);
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int k = 32 * s + 8 * g + j, b = k / (kNG + kNS), c = k - b * (kNG + kNS);
          const float v = c < kNG ? G[(size_t)c * hw] : S[c - kNG];
          x[j] = b < nblk ? pe_value(v, b) : 0.0f;
        }
        return split8(x);
      });
      put(acc, true);
      bias(L_F2);
      pipe.chain(acc, in);
      put(acc, true);
      bias(L_F3);
      pipe.chain(acc, in);                         // sigma
    }
    if constexpr (MODE == M_BEGIN) {
      if (valid)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) *(f32x4 *)(a.sig + p * W + 16 * mt + 4 * g) = acc[mt];
      continue;
    }
    if constexpr (MODE == M_ACC || MODE == M_FINISH) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = *(const f32x4 *)(a.sig + pc * W + 16 * mt + 4 * g);
    }
    if constexpr (kHead) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) l_sig[mt * 64] = acc[mt];
    }
    float cnt = 0.0f;
    if constexpr (kSlots) {
      // u = W_T1,sigma sigma + b_T1 (the sigma-hoist)
      put(acc, false);
      bias(L_T1);
      pipe.chain(acc, in);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        u[mt] = acc[mt];
        Z[mt] = MODE == M_ACC && !a.fresh ? *(const f32x4 *)(a.z + pc * W + 16 * mt + 4 * g) : zero4();
      }
      // per slot: z1 = relu(W_T1,b b_i + u), Z += m_i relu(W_T2 z1 + b_T2)
      for (int i = 0; i < a.k; ++i) {
        float rn[3] = {0.f, 0.f, 0.f}, an = 0.0f;
        if (i + 1 < a.k) load(i + 1, rn, an);
        const float m = al > 0.0f ? 1.0f : 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = u[mt];
        pipe.gather(acc, ENC ? a.steps_b : 1, [&](int s) {
          float x[8] = {raw[0], raw[1], raw[2], 0.f, 0.f, 0.f, 0.f, 0.f};
          if constexpr (ENC) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int v = 8 * s + j, b = v / 3, c = v - 3 * b;
              const float r = c == 0 ? raw[0] : (c == 1 ? raw[1] : raw[2]);
              x[j] = b < nblk ? pe_value(r, b) : 0.0f;
            }
          }
          return split8(x);
        });
        put(acc, true);
        bias(L_T2);
        pipe.chain(acc, in);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) Z[mt] += relu4(acc[mt]) * m;
        cnt += m;
#pragma unroll
        for (int j = 0; j < 3; ++j) raw[j] = rn[j];
        al = an;
      }
    }
    if constexpr (MODE == M_ACC) {
      if (valid) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) *(f32x4 *)(a.z + p * W + 16 * mt + 4 * g) = Z[mt];
        if (g == 0) a.cnt[p] = a.fresh ? cnt : a.cnt[p] + cnt;
      }
    }
    if constexpr (MODE == M_FINISH) {
      cnt = a.fresh ? 0.0f : a.cnt[pc];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        Z[mt] = a.fresh ? zero4() : *(const f32x4 *)(a.z + pc * W + 16 * mt + 4 * g);
    }
    if constexpr (kHead) {
      const float ld = g < 3 ? G[(size_t)(11 + g) * hw] : 0.0f;
      if constexpr (kAhead) {
        nx = locate(std::min<int64_t>(tile + gridDim.x, ntiles - 1), col);
        first_loads(nx, g, xr, alk);
      }
      // the pool, T3 (tau), B on [sigma; tau], R on [phi; L_d]
      const float inv = a.mean ? 1.0f / fmaxf(cnt, 1.0f) : 1.0f;
      const float bs = a.mean ? (cnt > 0.0f ? 1.0f : 0.0f) : cnt;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) Z[mt] = Z[mt] * inv;
      put(Z, false);
      bias(L_T3);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = acc[mt] * bs;
      pipe.chain(acc, in);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        Z[mt] = acc[mt];                           // tau
        acc[mt] = l_sig[mt * 64];
      }
      put(acc, false);
      bias(L_B1);
      pipe.chain(acc, in);
      put(Z, false);
      pipe.chain(acc, in);
      put(acc, true);
      bias(L_B2);
      pipe.chain(acc, in);
      put(acc, true);
      bias(L_B3);
      pipe.chain(acc, in);
      put(acc, false);                             // phi
      bias(L_R1);
      pipe.chain(acc, in);
      pipe.gather(acc, 1, [&](int) {
        const float x[8] = {ld, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        return split8(x);
      });
      put(acc, true);
      bias(L_R2);
      pipe.chain(acc, in);
      put(acc, true);
      const f32x4 y = pipe.tail(in);
      if (valid && g == 0) {
        float *o = a.out + (size_t)f * kNOUT * hw + q;
#pragma unroll
        for (int c = 0; c < kNOUT; ++c) o[(size_t)c * hw] = y[c] + l_bias[L_R3 * W + c];
      }
    }
  }
}

template <int W, int MODE, bool ENC, int WAVES>
static hipError_t launch_waves(const FwdArgs &a, int num_cus, hipStream_t s) {
  constexpr bool kHead = MODE == M_FULL || MODE == M_FINISH;
  const size_t lds = kRing * kSplitStage + sizeof(float) * kNumLayers * W +
                     (kHead ? (size_t)WAVES * (W / 16) * 1024 : 0) + (size_t)WAVES * 16 * a.kpad;
  static LdsLimit limit;
  const hipError_t e = limit.raise((const void *)f32_forward_kernel<W, MODE, ENC, WAVES>, lds);
  if (e != hipSuccess) return e;
  const int64_t ntiles = (a.npx + WAVES * 16 - 1) / (WAVES * 16);
  const unsigned grid = (unsigned)std::min<int64_t>(ntiles, num_cus);    // persistent
  hipLaunchKernelGGL((f32_forward_kernel<W, MODE, ENC, WAVES>), dim3(grid), dim3(WAVES * 64), lds, s,
                     a);
  return hipGetLastError();
}

// Four waves where that many tiles still leave no CU without one: a frame of
// few tiles then spreads over twice the CUs (64^2, W = 64: FULL only).
template <int W, int MODE, bool ENC>
static hipError_t launch_mode(const FwdArgs &a, int num_cus, hipStream_t s) {
  if constexpr (MODE == M_FULL)
    if ((a.npx + 63) / 64 <= num_cus) return launch_waves<W, MODE, ENC, 4>(a, num_cus, s);
  return launch_waves<W, MODE, ENC, 8>(a, num_cus, s);
}

template <int MODE, bool ENC>
static hipError_t launch_width(int W, const FwdArgs &a, int num_cus, hipStream_t s) {
  return W == 128 ? launch_mode<128, MODE, ENC>(a, num_cus, s)
                  : launch_mode<64, MODE, ENC>(a, num_cus, s);
}

static hipError_t launch(int W, int mode, const FwdArgs &a, int num_cus, hipStream_t s) {
#define GO(M) \
  (a.pe > 0 ? launch_width<M, true>(W, a, num_cus, s) : launch_width<M, false>(W, a, num_cus, s))
  switch (mode) {
    case M_FULL: return GO(M_FULL);
    case M_BEGIN: return GO(M_BEGIN);
    case M_ACC: return GO(M_ACC);
    case M_FINISH: return launch_width<M_FINISH, false>(W, a, num_cus, s);   // reads no encoded input
  }
#undef GO
  return hipErrorInvalidValue;
}

}  // namespace f32
}  // namespace gn

using namespace gn;

size_t gn_f32_packed_bytes(int W, int pe) {
  f32::OpTable t;
  f32::make_ops(W, pe, &t);
  return f32::packed_bytes(t);
}

hipError_t gn_f32_pack(gn_handle *h, hipStream_t s) {
  f32::OpTable t;
  f32::make_ops(h->W, h->pl.pe, &t);
  const int n = t.stages * (f32::kSplitFrags / 3) * 64 + kNumLayers * t.W;
  hipLaunchKernelGGL(f32::f32_split_pack_kernel, dim3((n + 255) / 256), dim3(256), 0, s, h->d_master,
                     t, h->d_f32);
  return hipGetLastError();
}

static gn_status f32_run(gn_handle *h, const gn_frame *fr, int mode, f32::FwdArgs &a, bool canonical,
                         const char *what, hipStream_t s) {
  const int64_t npx = (int64_t)fr->n * fr->h * fr->w;
  if ((npx + 4095) / 4096 * 4096 > gn_f32_max_px)
    return gn_set_error(GN_E_INVAL, "more than 3 * 2^20 pixels in one call");
  f32::OpTable t;
  f32::make_ops(h->W, h->pl.pe, &t);
  auto first = [&](f32::Op o) { return t.op[o].stage0; };
  const bool trunk = mode == f32::M_FULL || mode == f32::M_BEGIN;
  const bool slots = mode == f32::M_FULL || mode == f32::M_ACC;
  const bool head = mode == f32::M_FULL || mode == f32::M_FINISH;
  const int k = slots ? fr->k : 0;
  // (an ACC call starts with T1's sigma part, a FINISH call with T3)
  a.pg.pre0 = trunk ? first(f32::O_F1) : first(slots ? f32::O_T1S : f32::O_T3);
  a.pg.pre1 = slots ? first(f32::O_T1A) : (trunk ? first(f32::O_T1S) : t.stages);
  a.pg.loop0 = first(f32::O_T1A);
  a.pg.loop1 = first(f32::O_T3);
  a.pg.post0 = first(f32::O_T3);
  a.pg.post1 = t.stages;
  a.pg.k = k;
  a.pg.post = slots && head ? 1 : 0;
  a.packed = h->d_f32;
  a.bias_stage = t.stages;
  a.gbuf = fr->gbuf;
  a.layers = fr->layers;
  a.scene = fr->scene;
  a.hw = fr->h * fr->w;
  a.k = k;
  a.mean = h->cfg.pool == GN_POOL_MEAN ? 1 : 0;
  a.pe = h->pl.pe;
  a.canon = canonical && gn_slot_kmax(h) > 1 && k > 1 ? 1 : 0;
  a.kpad = a.canon ? (k + 3) & ~3 : 0;
  a.steps_x = t.op[f32::O_F1].steps;
  a.steps_b = t.op[f32::O_T1A].steps;
  a.npx = npx;
  return gn_check_device(h, f32::launch(h->W, mode, a, h->num_cus, s), what);
}

gn_status gn_f32_forward(gn_handle *h, const gn_frame *frame, float *out, hipStream_t s) {
  f32::FwdArgs a{};
  a.out = out;
  return f32_run(h, frame, f32::M_FULL, a, true, "fp32 forward", s);
}

// Object streaming of GN_FP32 handles: the state holds sigma and the running
// sum Z ([pixel][W] each) and the active count per pixel.  accumulate adds the
// call's slots in call order, continuing the state's sum; the arithmetic and
// its order are the input-order forward's.
size_t gn_f32_stream_bytes(int W, int64_t npx) {
  return sizeof(float) * (size_t)(2 * W + 1) * (size_t)npx;
}

gn_status gn_f32_stream(gn_handle *h, const gn_frame *frame, int mode, float *state, int fresh,
                        float *out, hipStream_t s) {
  const int64_t npx = (int64_t)frame->n * frame->h * frame->w;
  f32::FwdArgs a{};
  a.sig = state;
  a.z = state + (size_t)h->W * npx;
  a.cnt = state + (size_t)2 * h->W * npx;
  a.fresh = fresh;
  a.out = out;
  const int m = mode == FWD_BEGIN ? f32::M_BEGIN : (mode == FWD_ACC ? f32::M_ACC : f32::M_FINISH);
  return f32_run(h, frame, m, a, false, "fp32 stream", s);
}
