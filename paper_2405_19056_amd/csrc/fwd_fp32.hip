// The fp32 forward: the whole per-pixel network (Sec. 3.3-3.4) in one kernel
// on the fp32 matrix cores, every activation in registers (fp32_core.h).  The
// same kernel, cut at compile time, serves the FP32 form's object streaming,
// the FP8 calibration and the backward's recompute (SAVE: every activation
// and ReLU sign the backward needs is written as it passes).
//
// A workgroup of four waves takes tiles of 64 pixels (16 per wave), two
// workgroups per CU: their stage barriers are independent, so one's epilogues
// and gathers run under the other's matrix work.  Per pixel and wave the live
// state is u, the running sum Z, one map's inputs and accumulators: 128
// registers at W = 128; sigma waits in LDS for B's first layer.  The slots are
// pooled in an fp32 running sum in canonical order (slot_order.h), or in
// input order.
//
// What bounds it: the matrix cores.  16x16x4 fp32 takes 32 cycles per SIMD for
// 2,048 FLOP, and a fragment of 256 bytes per instruction keeps the LDS at an
// eighth of its rate.
#include <algorithm>

#include "fp32_core.h"
#include "gn_api_state.h"
#include "slot_order.h"

namespace gn {
namespace f32 {

struct OpSpec { int op; Layer l; int col0, M, K; };

static void fill_table(int W, int pe, const OpSpec *s, int n, int trans, OpTable *t) {
  layer_offsets(W, pe, t->lo);
  t->W = W;
  t->pe = pe;
  t->nops = n;
  int stage = 0;
  for (int i = 0; i < n; ++i) {
    OpDesc &d = t->op[s[i].op];
    d.woff = t->lo[s[i].l].w;
    d.ld = t->lo[s[i].l].in;
    d.col0 = s[i].col0;
    d.M = s[i].M;
    d.K = s[i].K;
    d.trans = trans;
    d.mt = (d.M + 15) / 16;
    d.kq = (d.K + 15) / 16;
    d.stage0 = stage;
    d.nstages = (d.kq * d.mt + kStageFrags - 1) / kStageFrags;
    stage += d.nstages;
  }
  t->stages = stage;
}

void make_ops(int W, int pe, OpTable *t) {
  const int nx = (kNG + kNS) * pe_blocks(pe), nb = kNL * pe_blocks(pe);
  const OpSpec s[kNumOps] = {
      {O_F1, L_F1, 0, W, nx},  {O_F2, L_F2, 0, W, W},   {O_F3, L_F3, 0, W, W},
      {O_T1S, L_T1, nb, W, W}, {O_T1A, L_T1, 0, W, nb}, {O_T2, L_T2, 0, W, W},
      {O_T3, L_T3, 0, W, W},   {O_B1S, L_B1, 0, W, W},  {O_B1T, L_B1, W, W, W},
      {O_B2, L_B2, 0, W, W},   {O_B3, L_B3, 0, W, W},   {O_R1P, L_R1, 0, W, W},
      {O_R1L, L_R1, W, W, 3},  {O_R2, L_R2, 0, W, W},   {O_R3, L_R3, 0, kNOUT, W}};
  fill_table(W, pe, s, kNumOps, 0, t);
}

void make_bwd_ops(int W, int pe, OpTable *t) {
  const int nb = kNL * pe_blocks(pe);
  const OpSpec s[kNumBwdOps] = {
      {O_R3T, L_R3, 0, W, kNOUT}, {O_R2T, L_R2, 0, W, W},  {O_R1T, L_R1, 0, W, W},
      {O_B3T, L_B3, 0, W, W},     {O_B2T, L_B2, 0, W, W},  {O_B1ST, L_B1, 0, W, W},
      {O_B1TT, L_B1, W, W, W},    {O_T3T, L_T3, 0, W, W},  {O_T2T, L_T2, 0, W, W},
      {O_T1ST, L_T1, nb, W, W},   {O_F3T, L_F3, 0, W, W},  {O_F2T, L_F2, 0, W, W}};
  fill_table(W, pe, s, kNumBwdOps, 1, t);
}

// One thread per 16 bytes of a fragment; then the biases.  Fragment f of a
// map is K group f / mt of row tile f % mt; element j of lane l is
// A[row (l & 15)][16 q + 4 j + (l >> 4)], zero outside M x K.
__global__ __launch_bounds__(kThreads) void f32_pack_kernel(const float *__restrict__ master,
                                                            OpTable t, uint8_t *__restrict__ packed) {
  const int e = blockIdx.x * kThreads + threadIdx.x;
  const int total = t.stages * kStageFrags * 64;
  if (e >= total) {
    const int b = e - total, l = b / t.W, p = b % t.W;
    if (l < kNumLayers) {
      const int o = l == L_R3 ? p : neuron_at(p);
      ((float *)(packed + (size_t)t.stages * kStageBytes))[b] =
          o < t.lo[l].out ? master[t.lo[l].b + o] : 0.0f;
    }
    return;
  }
  const int stage = e / (kStageFrags * 64);
  int o = 0;
  while (o + 1 < t.nops && stage >= t.op[o + 1].stage0) ++o;
  const OpDesc d = t.op[o];
  const int f = (e >> 6) - d.stage0 * kStageFrags, lane = e & 63;
  const int q = f / d.mt, mt = f % d.mt, i = lane & 15;
  // one row tile (R3): rows in natural order; else in position order
  const int m = d.mt == 1 ? i : 16 * mt + 4 * (i & 3) + (i >> 2);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = 16 * q + 4 * j + (lane >> 4);
    if (m < d.M && k < d.K)
      v[j] = d.trans ? master[d.woff + (int64_t)k * d.ld + d.col0 + m]
                     : master[d.woff + (int64_t)m * d.ld + d.col0 + k];
  }
  ((f32x4 *)packed)[e] = v;
}

hipError_t launch_pack(const float *master, const OpTable &t, uint8_t *packed, hipStream_t s) {
  const int n = t.stages * kStageFrags * 64 + kNumLayers * t.W;
  hipLaunchKernelGGL(f32_pack_kernel, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, s,
                     master, t, packed);
  return hipGetLastError();
}

struct FwdArgs {
  const uint8_t *packed;
  int32_t bias_stage;        // the biases follow this many stages
  Program pg;
  const float *gbuf, *layers, *scene;
  float *out;
  int32_t hw, k, mean, pe, kpad;
  int32_t canon;             // pool in canonical order
  int32_t kq_x, kq_b;        // K groups of F1 and of T1's slot columns
  int64_t npx;
  // object streaming: sigma and the running sum [pixel][W] (positions), the
  // active count [pixel]
  float *sig, *z, *cnt;
  int32_t fresh;             // the state holds no sum yet
  unsigned *amax;            // calibration: float bits of the largest z1
  Planes pl;                 // SAVE: what the backward keeps of the slab
};

enum Mode { M_FULL, M_BEGIN, M_ACC, M_FINISH, M_CAL, M_SAVE };

// ENC: with positional encoding (a form of its own: the sine and cosine's code
// and registers stay out of the plain one).
template <int W, int MODE, bool ENC>
__global__ __launch_bounds__(kThreads, W == 128 || MODE == M_SAVE ? 2 : 3) void
f32_forward_kernel(FwdArgs a) {
  constexpr int MT = W / 16;
  constexpr bool kSave = MODE == M_SAVE;
  constexpr bool kTrunk = MODE == M_FULL || MODE == M_BEGIN || MODE == M_CAL || kSave;
  constexpr bool kSlots = MODE == M_FULL || MODE == M_ACC || MODE == M_CAL || kSave;
  constexpr bool kHead = MODE == M_FULL || MODE == M_FINISH || kSave;
  // LDS: the stage ring | biases | sigma per wave | slot order per pixel.
  // At W = 128 two workgroups leave room for six of sigma's eight row tiles;
  // the last two stay in registers.  (SAVE reads it back from its plane.)
  constexpr int kSigLds = MT < 6 ? MT : 6;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  float *l_bias = (float *)(lds + kRing * kStageBytes);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  f32x4 *l_sig = (f32x4 *)(l_bias + kNumLayers * W) + wave * kSigLds * 64 + lane;
  uint8_t *l_order = (uint8_t *)(l_bias + kNumLayers * W) + (kHead && !kSave ? kWaves * kSigLds * 1024 : 0);
  {
    const float *b = (const float *)(a.packed + (size_t)a.bias_stage * kStageBytes);
    for (int i = threadIdx.x; i < kNumLayers * W; i += kThreads) l_bias[i] = b[i];
  }
  Pipe<MT> pipe;
  pipe.start(a.packed, lds, a.pg);       // ends with a barrier
  const int hw = a.hw, nblk = ENC ? pe_blocks(a.pe) : 1;
  const int64_t ntiles = kSave ? a.pl.np / kTile : (a.npx + kTile - 1) / kTile;
  float amax = 0.0f;

  // A lane's pixel of a tile (tail lanes recompute a real pixel), and the
  // first loads it waits for: the inputs of F1 (without encoding) and the
  // alphas its slots are ranked by (up to kFastK slots).  FULL and SAVE issue
  // them a tile ahead, in the head, where u and Z have left their registers.
  constexpr bool kAhead = kTrunk && kHead && !kSave;
  constexpr int kFastK = 8;
  struct Pixel {
    int64_t p;
    int f, q;
    bool valid;
  };
  auto locate = [&](int64_t tile, int col) {
    Pixel x;
    x.p = (kSave ? a.pl.p0 : 0) + tile * kTile + wave * 16 + col;
    x.valid = x.p < a.npx;
    const int64_t pc = x.valid ? x.p : a.npx - 1;
    x.f = (int)(pc / hw);
    x.q = (int)(pc - (int64_t)x.f * hw);
    return x;
  };
  const bool fast = kSlots && a.canon && a.k <= kFastK;
  auto first_loads = [&](const Pixel &x, int g, f32x4 (&xr)[2], float (&al)[kFastK]) {
    if constexpr (kTrunk && !ENC) {
      const float *G = a.gbuf + (size_t)x.f * kNG * hw + x.q, *S = a.scene + (size_t)x.f * kNS;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = 4 * i + g;
        xr[i >> 2][i & 3] =
            c < kNG ? G[(size_t)c * hw] : (c < kNG + kNS ? S[c - kNG] : 0.0f);
      }
    }
    if (fast) {
      const float *L = a.layers + (size_t)x.f * a.k * kNL * hw + x.q;
#pragma unroll
      for (int j = 0; j < kFastK; ++j) al[j] = j < a.k ? L[((size_t)j * kNL + kAlpha) * hw] : 0.0f;
    }
  };
  Pixel nx = locate(blockIdx.x, lane & 15);
  f32x4 xr[2];
  float alk[kFastK];
  if constexpr (kAhead) first_loads(nx, lane >> 4, xr, alk);

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    // Opaque per-tile copies of the lane's place keep the compiler from holding
    // every address derived from them in registers across the tile loop.
    int g = lane >> 4, col = lane & 15;
    asm volatile("" : "+v"(g), "+v"(col));
    const Pixel px = kAhead ? nx : locate(tile, col);
    if constexpr (!kAhead) first_loads(px, g, xr, alk);
    const int64_t pl = tile * kTile + wave * 16 + col, p = px.p;      // pl: pixel of a SAVE's slab
    const bool valid = px.valid;
    const int64_t pc = valid ? p : a.npx - 1;
    const int f = px.f, q = px.q;
    uint8_t *l_perm = l_order + (wave * 16 + col) * a.kpad;
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
    // SAVE: a block of W values per pixel, the signs of a ReLU's outputs
    // (32-bit offsets from a uniform base: the caller bounds a slab's blocks)
    const uint32_t at = (uint32_t)pl * (W * 4) + 16 * g;
    auto save = [&](float *plane, const f32x4 (&v)[MT]) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) *(f32x4 *)((char *)plane + at + 64 * mt) = v[mt];
    };
    auto signs = [&](int layer, const f32x4 (&v)[MT], bool keep) {
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
    const float *G = a.gbuf + (size_t)f * kNG * hw + q;
    const float *L = a.layers + (size_t)f * a.k * kNL * hw + q;
    const float *S = a.scene + (size_t)f * kNS;
    f32x4 in[MT], acc[MT], u[MT], Z[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = zero4();

    // The pixel's slots in canonical order: lane group g ranks slots g, g + 4,
    // ... (read back by the same wave).  Keys: the bits of alpha for active
    // slots, above them the inactive ones by index; equal alphas (and more
    // than kFastK slots) take the full comparison.
    if (kSlots && a.canon) {
      if (fast) {
        uint32_t key[kFastK];
#pragma unroll
        for (int j = 0; j < kFastK; ++j)
          key[j] = j >= a.k ? 0xFFFFFFFFu
                            : (alk[j] > 0.0f ? __float_as_uint(alk[j]) : 0xFFFFFF00u + j);
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
          if (i < a.k) l_perm[le == lt + 1 ? lt : slot_rank(L, (size_t)hw, a.k, i)] = (uint8_t)i;
        }
      } else {
        for (int i = g; i < a.k; i += 4) l_perm[slot_rank(L, (size_t)hw, a.k, i)] = (uint8_t)i;
      }
    }
    // A slot's raw channels g, 4 + g, 8 + g and its alpha.
    auto load = [&](int i, float (&r)[3], float &alpha) {
      const int slot = a.canon ? (int)l_perm[i] : i;
      const float *Li = L + (size_t)slot * kNL * hw;
#pragma unroll
      for (int j = 0; j < 3; ++j) r[j] = Li[(size_t)(4 * j + g) * hw];
      alpha = Li[(size_t)kAlpha * hw];
    };
    float raw[3] = {0.f, 0.f, 0.f}, al = 0.0f;
    if (kSlots && a.k > 0) load(0, raw, al);

    if constexpr (kTrunk) {
      // F on the (encoded) [G; s]: input k is channel k % 30 of block k / 30
      pipe.gather(acc, ENC ? a.kq_x : 2, [&](int qq) {
        f32x4 x;
        if constexpr (!ENC) {
          x = qq == 0 ? xr[0] : xr[1];
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int k = 16 * qq + 4 * j + g, b = k / (kNG + kNS), c = k - b * (kNG + kNS);
            const float raw = c < kNG ? G[(size_t)c * hw] : S[c - kNG];
            x[j] = b < nblk ? pe_value(raw, b) : 0.0f;
          }
        }
        if constexpr (kSave) *(f32x4 *)(a.pl.x + (uint32_t)pl * a.pl.nx + 16 * qq + 4 * g) = x;
        return x;
      });
      next(in, acc, L_F1, true);
      if constexpr (kSave) {
        if constexpr (ENC)                                   // the block's padding
          for (int i = a.kq_x; i < a.pl.nx / 16; ++i)
            *(f32x4 *)(a.pl.x + (uint32_t)pl * a.pl.nx + 16 * i + 4 * g) = zero4();
        save(a.pl.a1, in);
        signs(K_A1, in, true);
      }
      pipe.chain(acc, in);
      next(in, acc, L_F2, true);
      if constexpr (kSave) {
        save(a.pl.a2, in);
        signs(K_A2, in, true);
      }
      pipe.chain(acc, in);
      next(in, acc, L_F3, false);                  // sigma
      if constexpr (kSave) save(a.pl.sig, in);
    }
    if constexpr (MODE == M_BEGIN) {
      if (valid)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) *(f32x4 *)(a.sig + p * W + 16 * mt + 4 * g) = in[mt];
      continue;
    }
    if constexpr (MODE == M_ACC || MODE == M_FINISH) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) in[mt] = *(const f32x4 *)(a.sig + pc * W + 16 * mt + 4 * g);
    }
    f32x4 sig[MT - kSigLds + 1];
    if constexpr (kHead && !kSave) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        if (mt < kSigLds) l_sig[mt * 64] = in[mt];
        else sig[mt - kSigLds] = in[mt];
    }
    float cnt = 0.0f;
    if constexpr (kSlots) {
      // u = W_T1,sigma sigma + b_T1 (the sigma-hoist)
      pipe.chain(acc, in);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        u[mt] = acc[mt] + bias(L_T1, mt);
        acc[mt] = zero4();
        Z[mt] = MODE == M_ACC && !a.fresh ? *(const f32x4 *)(a.z + pc * W + 16 * mt + 4 * g) : zero4();
      }
      // per slot: z1 = relu(W_T1,b b_i + u), Z += m_i relu(W_T2 z1 + b_T2).
      // Lane group g's raw channels are the inputs of K-steps 0..2 of every
      // encoding block (12 channels, three steps).
      for (int i = 0; i < a.k; ++i) {
        float rn[3] = {0.f, 0.f, 0.f}, an = 0.0f;
        if (i + 1 < a.k) load(i + 1, rn, an);
        const float m = al > 0.0f ? 1.0f : 0.0f;
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
          if constexpr (kSave)
            *(f32x4 *)(a.pl.bi + i * a.pl.np * a.pl.nb + (uint32_t)pl * a.pl.nb + 16 * qq + 4 * g) = x;
          return x;
        });
        if constexpr (kSave && ENC)                          // the block's padding
          for (int j = a.kq_b; j < a.pl.nb / 16; ++j)
            *(f32x4 *)(a.pl.bi + i * a.pl.np * a.pl.nb + (uint32_t)pl * a.pl.nb + 16 * j + 4 * g) =
                zero4();
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          in[mt] = relu4(acc[mt] + u[mt]);
          acc[mt] = zero4();
        }
        if constexpr (MODE == M_CAL) {
          if (valid)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              amax = fmaxf(amax, fmaxf(fmaxf(in[mt][0], in[mt][1]), fmaxf(in[mt][2], in[mt][3])));
        } else {
          if constexpr (kSave) {
            save(a.pl.z1 + (int64_t)i * a.pl.np * W, in);
            signs(kMasks + 2 * i, in, true);
          }
          pipe.chain(acc, in);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt] = acc[mt] + bias(L_T2, mt);
          if constexpr (kSave) signs(kMasks + 2 * i + 1, acc, al > 0.0f);
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
      for (int mt = 0; mt < MT; ++mt) in[mt] = Z[mt] * inv;
      if constexpr (kSave) {
        save(a.pl.zs, in);
        if (g == 0) {
          a.pl.inv[pl] = inv;
          a.pl.bs[pl] = bs;
        }
      }
      pipe.chain(acc, in);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const f32x4 b = bias(L_T3, mt);
#pragma unroll
        for (int r = 0; r < 4; ++r) in[mt][r] = fmaf(b[r], bs, acc[mt][r]);
        acc[mt] = zero4();
      }
      if constexpr (kSave) save(a.pl.tau, in);
      {
        f32x4 s[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          s[mt] = kSave ? *(const f32x4 *)((const char *)a.pl.sig + at + 64 * mt)
                        : (mt < kSigLds ? l_sig[mt * 64] : sig[mt - kSigLds]);
        pipe.chain(acc, s);
      }
      pipe.chain(acc, in);
      next(in, acc, L_B1, true);
      if constexpr (kSave) {
        save(a.pl.d1, in);
        signs(K_D1, in, true);
      }
      pipe.chain(acc, in);
      next(in, acc, L_B2, true);
      if constexpr (kSave) {
        save(a.pl.d2, in);
        signs(K_D2, in, true);
      }
      pipe.chain(acc, in);
      next(in, acc, L_B3, false);                  // phi
      if constexpr (kSave) save(a.pl.phi, in);
      pipe.chain(acc, in);
      pipe.gather(acc, 1, [&](int) { return f32x4{ld, 0.f, 0.f, 0.f}; });
      next(in, acc, L_R1, true);
      if constexpr (kSave) {
        save(a.pl.g1, in);
        signs(K_G1, in, true);
      }
      pipe.chain(acc, in);
      next(in, acc, L_R2, true);
      if constexpr (kSave) {
        save(a.pl.g2, in);
        signs(K_G2, in, true);
      } else {
        const f32x4 y = pipe.tail(in);
        if (valid && g == 0) {
          float *o = a.out + (size_t)f * kNOUT * hw + q;
#pragma unroll
          for (int c = 0; c < kNOUT; ++c) o[(size_t)c * hw] = y[c] + l_bias[L_R3 * W + c];
        }
      }
    }
  }
  if constexpr (MODE == M_CAL) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) amax = fmaxf(amax, __shfl_xor(amax, d));
    if (lane == 0) atomicMax(a.amax, __float_as_uint(amax));   // non-negative: bit order
  }
}

template <int W, int MODE, bool ENC>
static hipError_t launch_mode(const FwdArgs &a, int num_cus, hipStream_t s) {
  constexpr bool kSig = MODE == M_FULL || MODE == M_FINISH;
  const size_t lds = kRing * kStageBytes + sizeof(float) * kNumLayers * W +
                     (kSig ? (size_t)kWaves * std::min(W / 16, 6) * 1024 : 0) + (size_t)kTile * a.kpad;
  static const hipError_t attr =     // per process; the attribute is per function
      hipFuncSetAttribute((const void *)f32_forward_kernel<W, MODE, ENC>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, 84 * 1024);
  if (attr != hipSuccess) return attr;
  const int64_t ntiles = MODE == M_SAVE ? a.pl.np / kTile : (a.npx + kTile - 1) / kTile;
  // persistent: two workgroups per CU at W = 128, three at 64 (registers)
  const unsigned grid = (unsigned)std::min<int64_t>(ntiles, (W == 128 ? 2 : 3) * num_cus);
  hipLaunchKernelGGL((f32_forward_kernel<W, MODE, ENC>), dim3(grid), dim3(kThreads), lds, s, a);
  return hipGetLastError();
}

static hipError_t launch(int W, int mode, const FwdArgs &a, int num_cus, hipStream_t s) {
#define GO(M)                                                                          \
  (a.pe > 0 ? (W == 128 ? launch_mode<128, M, true>(a, num_cus, s)                     \
                        : launch_mode<64, M, true>(a, num_cus, s))                     \
            : (W == 128 ? launch_mode<128, M, false>(a, num_cus, s)                    \
                        : launch_mode<64, M, false>(a, num_cus, s)))
  switch (mode) {
    case M_FULL: return GO(M_FULL);
    case M_BEGIN: return GO(M_BEGIN);
    case M_ACC: return GO(M_ACC);
    case M_FINISH: return GO(M_FINISH);
    case M_CAL: return GO(M_CAL);
    case M_SAVE: return GO(M_SAVE);
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
  return f32::launch_pack(h->d_master, t, h->d_f32, s);
}

// The handle's packed fp32 weights: GN_FP32 handles pack them with every
// upload; the others hold none until a calibration or a backward asks, and
// pack per call.
static gn_status f32_weights(gn_handle *h, hipStream_t s) {
  if (h->cfg.precision == GN_FP32) return GN_OK;
  hipError_t e = hipSuccess;
  if (!h->d_f32) {
    const size_t bytes = gn_f32_packed_bytes(h->W, h->pl.pe);
    e = hipMalloc((void **)&h->d_f32, bytes);
    if (e == hipSuccess) h->bytes_held += bytes; else h->d_f32 = nullptr;
  }
  if (e == hipSuccess) e = gn_f32_pack(h, s);
  return gn_check_device(h, e, "fp32 weight packing");
}

static gn_status f32_run(gn_handle *h, const gn_frame *fr, int mode, f32::FwdArgs &a, bool canonical,
                         const char *what, hipStream_t s) {
  const int64_t npx = (int64_t)fr->n * fr->h * fr->w;
  if ((npx + 4095) / 4096 * 4096 > gn_f32_max_px)
    return gn_set_error(GN_E_INVAL, "more than 3 * 2^20 pixels in one call");
  // (a backward of several slabs packs once)
  const gn_status st = mode == f32::M_SAVE && a.pl.p0 > 0 ? GN_OK : f32_weights(h, s);
  if (st != GN_OK) return st;
  f32::OpTable t;
  f32::make_ops(h->W, h->pl.pe, &t);
  auto first = [&](f32::Op o) { return t.op[o].stage0; };
  const bool keep = mode == f32::M_SAVE;
  const bool trunk = mode == f32::M_FULL || mode == f32::M_BEGIN || mode == f32::M_CAL || keep;
  const bool slots = mode == f32::M_FULL || mode == f32::M_ACC || mode == f32::M_CAL || keep;
  const bool head = mode == f32::M_FULL || mode == f32::M_FINISH || keep;
  // (an ACC call starts with T1's sigma part, a FINISH call with T3)
  const int k = slots ? fr->k : 0;
  a.pg.pre0 = trunk ? first(f32::O_F1) : first(slots ? f32::O_T1S : f32::O_T3);
  a.pg.pre1 = slots ? first(f32::O_T1A) : (trunk ? first(f32::O_T1S) : t.stages);
  a.pg.loop0 = first(f32::O_T1A);
  a.pg.loop1 = first(mode == f32::M_CAL ? f32::O_T2 : f32::O_T3);
  a.pg.post0 = first(f32::O_T3);
  a.pg.post1 = keep ? first(f32::O_R3) : t.stages;
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
  a.canon = canonical && gn_slot_kmax(h) > 1 && fr->k > 1 ? 1 : 0;
  a.kpad = a.canon ? (fr->k + 3) & ~3 : 0;
  a.kq_x = t.op[f32::O_F1].kq;
  a.kq_b = t.op[f32::O_T1A].kq;
  a.npx = npx;
  return gn_check_device(h, f32::launch(h->W, mode, a, h->num_cus, s), what);
}

gn_status gn_f32_forward(gn_handle *h, const gn_frame *frame, float *out, hipStream_t s) {
  f32::FwdArgs a{};
  a.out = out;
  return f32_run(h, frame, f32::M_FULL, a, true, "fp32 forward", s);
}

gn_status gn_f32_calibrate(gn_handle *h, const gn_frame *frame, unsigned *amax, hipStream_t s) {
  f32::FwdArgs a{};
  a.amax = amax;
  return f32_run(h, frame, f32::M_CAL, a, false, "calibration", s);
}

// The backward's recompute of one slab.
gn_status gn_f32_save(gn_handle *h, const gn_frame *frame, const f32::Planes &pl, hipStream_t s) {
  f32::FwdArgs a{};
  a.pl = pl;
  return f32_run(h, frame, f32::M_SAVE, a, true, "backward recompute", s);
}

// Object streaming of GN_FP32 handles: the state holds sigma and the running
// sum Z ([pixel][W] each, in position order) and the active count per pixel.
// accumulate adds the call's slots in call order, continuing the state's sum;
// the arithmetic and its order are the input-order forward's.
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
