// The fp32 backward: dL/dw of F, T, B and R for a given dL/dy (Sec. 3.5
// trains the four networks jointly, end to end).
//
// Per slab of pixels:
//   1. recompute (fwd_fp32.hip, SAVE): every activation a weight gradient
//      needs, and the sign of every ReLU as one bit.
//   2. deltas: one kernel chains the transposed maps in registers from dL/dy
//      to F's first layer (fp32_core.h), the slots in between: dz2 = [z2 > 0]
//      m_i dZ is a selection of dZ's registers, dz1 = [z1 > 0] W_T2^T dz2,
//      du = sum dz1.  The ReLU derivatives are the stored bits.
//   3. weight gradients: sum_p delta_p a_p^T of every layer on the matrix
//      cores, each pixel block read once per product.
// Then one fixed-order reduction of the workgroups' partial sums into grad_w
// (deterministic, no atomics).
//
// Slabs bound the workspace: a slab's blocks take at most kSlabBytes.
#include <string.h>

#include <algorithm>

#include "fp32_core.h"
#include "gn_api_state.h"

namespace gn {

struct BwdWorkspace {
  uint8_t *mem = nullptr;       // a slab's planes, then the packed weights and the partials
  size_t bytes = 0;
};

namespace f32 {

constexpr size_t kSlabBytes = (size_t)16 << 30;

// ---- deltas ---------------------------------------------------------------------
struct DeltaArgs {
  const uint8_t *packed;
  Program pg;
  Planes pl;
  const float *dy;           // the caller's dL/dy [n][3][hw]
  int32_t hw, k;
  int64_t npx;
};

template <int W>
__global__ __launch_bounds__(kThreads, 2) void f32_delta_kernel(DeltaArgs a) {
  constexpr int MT = W / 16;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int wave = threadIdx.x >> 6;
  Pipe<MT> pipe;
  pipe.start(a.packed, lds, a.pg);
  const int64_t ntiles = a.pl.np / kTile;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    int g = (threadIdx.x & 63) >> 4, col = threadIdx.x & 15;
    asm volatile("" : "+v"(g), "+v"(col));      // per-tile copies, as in the forward
    const int64_t pl = tile * kTile + wave * 16 + col, p = a.pl.p0 + pl;
    const uint32_t at = (uint32_t)pl * (W * 4) + 16 * g;
    f32x4 in[MT], acc[MT];
    auto save = [&](float *plane, const f32x4 (&v)[MT]) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) *(f32x4 *)((char *)plane + at + 64 * mt) = v[mt];
    };
    auto signs = [&](int layer) {
      const uint32_t *words = a.pl.mask + (int64_t)layer * (a.pl.np / 16) * 64;
      return words[(uint32_t)(tile * kThreads) + threadIdx.x];
    };
    // out = the accumulators where the bits say so
    auto masked = [&](f32x4 (&out)[MT], uint32_t bits) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          out[mt][r] = bits & (1u << (4 * mt + r)) ? acc[mt][r] : 0.0f;
          acc[mt][r] = 0.0f;
        }
    };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = zero4();
    // dL/dy of the pixel: lane group g < 3 channel g (padding pixels: zero, so
    // every delta of theirs is zero)
    float dy = 0.0f;
    if (g < 3 && p < a.npx) {
      const int64_t f = p / a.hw;
      dy = a.dy[(f * kNOUT + g) * a.hw + (p - f * a.hw)];
    }
    *(f32x4 *)(a.pl.dy + (uint32_t)pl * kDyWidth + 4 * g) = f32x4{dy, 0.f, 0.f, 0.f};
    uint32_t bits = signs(K_G2), nbits = signs(K_G1);
    pipe.gather(acc, 1, [&](int) { return f32x4{dy, 0.f, 0.f, 0.f}; });
    masked(in, bits);
    save(a.pl.dg2, in);
    bits = signs(K_D2);
    pipe.chain(acc, in);
    masked(in, nbits);
    save(a.pl.dg1, in);
    pipe.chain(acc, in);
    masked(in, ~0u);
    save(a.pl.dphi, in);
    nbits = signs(K_D1);
    pipe.chain(acc, in);
    masked(in, bits);
    save(a.pl.dd2, in);
    const float inv = a.pl.inv[(uint32_t)pl];
    pipe.chain(acc, in);
    masked(in, nbits);
    save(a.pl.dd1, in);
    f32x4 dsig[MT], dz[MT], du[MT];
    pipe.chain(acc, in);
    masked(dsig, ~0u);
    pipe.chain(acc, in);
    masked(in, ~0u);                            // dtau
    save(a.pl.dtau, in);
    pipe.chain(acc, in);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      dz[mt] = acc[mt] * inv;                   // dZ = W_T3^T dtau / max(c, 1)
      acc[mt] = zero4();
      du[mt] = zero4();
    }
    save(a.pl.dz, dz);
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
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) in[mt][r] = b2 & (1u << (4 * mt + r)) ? dz[mt][r] : 0.0f;
      pipe.chain(acc, in);
      masked(in, b1);
      save(a.pl.dz1 + (int64_t)i * a.pl.np * W, in);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) du[mt] += in[mt];
      b1 = n1;
      b2 = n2;
    }
    save(a.pl.du, du);
    bits = signs(K_A2);
    nbits = signs(K_A1);
    pipe.chain(acc, du);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      in[mt] = acc[mt] + dsig[mt];
      acc[mt] = zero4();
    }
    save(a.pl.dsig, in);
    pipe.chain(acc, in);
    masked(in, bits);
    save(a.pl.da2, in);
    pipe.chain(acc, in);
    masked(in, nbits);
    save(a.pl.da1, in);
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
// cores on operands split in three (fp32_core.h).
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
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l = lane & 15;
  const int wr = wave / WC, wc = wave % WC;
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
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        const int e = tid + i * kThreads, p = e / DU, u = e % DU;
        f32x4 v = hd[i];
        if (job.mask) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = hm[i] & (1u << r) ? v[r] : 0.0f;
        }
        ld[b][p * DU + (u ^ dswz(p))] = v;
      }
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const int e = tid + i * kThreads, p = e / AU, u = e % AU;
        if (kStep * AU % kThreads == 0 || e < kStep * AU)
          la[b][p * AU + (u ^ aswz(p))] = ha[i];
      }
      if (tid < kStep) lw[b][tid] = hw;
    };
    f32x4 acc[TO][TI];
    float dsum[TO], asum[TI];
#pragma unroll
    for (int o = 0; o < TO; ++o) {
      dsum[o] = 0.0f;
#pragma unroll
      for (int i = 0; i < TI; ++i) acc[o][i] = zero4();
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) asum[i] = 0.0f;
    // both buffers are free: every wave is past the last segment's reads
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
        d[o] = split8(v);
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
        const Split x = split8(v);
#pragma unroll
        for (int o = 0; o < TO; ++o) acc[o][i] = mma_split(d[o], x, acc[o][i]);
      }
    }
    float *P = a.part + (size_t)(blockIdx.x + j) * part_floats(W, MI);
    auto put = [&](float *dst, float v) { *dst = a.accumulate ? *dst + v : v; };
#pragma unroll
    for (int o = 0; o < TO; ++o)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          put(P + (16 * (wr * TO + o) + 4 * g + r) * 16 * MI + 16 * (wc * TI + i) + l, acc[o][i][r]);
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
      if (wr == 0 && g == 0) put(P + W * 16 * MI + W + 16 * (wc * TI + i) + l, asum[i]);
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
// of memory latencies: 115 us against 14 at 16 x 128^2, K = 4, W = 128.)
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
  // Splits the groups' steps over workgroups for slabs of np pixels; returns
  // the floats of all partials.
  size_t split(int64_t np) {
    size_t floats = 0;
    for (DwGroup &g : g_) {
      g.a.steps = np / kStep;
      g.total = 0;
      for (int j = 0; j < g.a.njobs; ++j) g.total += g.a.job[j].slots * g.a.steps;
      // as many workgroups as the CUs hold (LDS: two of 64 KB, four of the
      // smaller ones), each with at least 4 steps (a partial costs about as
      // much traffic as two)
      const int64_t cap = (int64_t)cus_ * (W_ == 128 && g.MI >= 4 ? 2 : 4);
      g.a.per = (int32_t)std::max<int64_t>((g.total + cap - 1) / cap, 4);
      g.grid = (int)((g.total + g.a.per - 1) / g.a.per);
      g.a.part = (float *)nullptr + floats;                  // an offset, until bind()
      floats += (size_t)(g.grid + g.a.njobs) * part_floats(W_, g.MI);
    }
    return floats;
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

template <int W>
static hipError_t launch_delta(const DeltaArgs &a, int num_cus, hipStream_t s) {
  const unsigned grid = (unsigned)std::min<int64_t>(a.pl.np / kTile, 2 * num_cus);
  hipLaunchKernelGGL(f32_delta_kernel<W>, dim3(grid), dim3(kThreads), kRing * kStageBytes, s, a);
  return hipGetLastError();
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
  f32::OpTable t;
  f32::make_bwd_ops(W, pe, &t);
  // slabs of equal length (the last may be shorter) within the workspace bound
  const int64_t per_px = f32::px_floats(W, pe, k) * (int64_t)sizeof(float);
  const int64_t most = (int64_t)(f32::kSlabBytes / per_px), slabs = (npx + most - 1) / most;
  const int64_t np = f32::rup((npx + slabs - 1) / slabs, f32::kTile);
  f32::Gradient grad(W, pe, k, h->num_cus);
  const size_t part = grad.split(np) * sizeof(float);
  const size_t planes = f32::rup(np * per_px, 1024), packed = f32::rup(f32::packed_bytes(t), 1024);
  const size_t need = planes + packed + part;
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
  uint8_t *frag = ws->mem + planes;
  grad.bind((float *)(frag + packed));
  e = f32::launch_pack(h->d_master, t, frag, s);
  for (int64_t p0 = 0; p0 < npx && e == hipSuccess; p0 += np) {
    f32::Planes pl = f32::carve((float *)ws->mem, W, pe, k, std::min(np, f32::rup(npx - p0, f32::kTile)));
    pl.p0 = p0;
    const gn_status st = gn_f32_save(h, frame, pl, s);
    if (st != GN_OK) return st;
    f32::DeltaArgs d{};
    d.packed = frag;
    d.pg = f32::Program{0, t.op[f32::O_T2T].stage0, t.op[f32::O_T2T].stage0, t.op[f32::O_T1ST].stage0,
                        t.op[f32::O_T1ST].stage0, t.stages, k, 1};
    d.pl = pl;
    d.dy = dy;
    d.hw = frame->h * frame->w;
    d.k = k;
    d.npx = npx;
    e = W == 128 ? f32::launch_delta<128>(d, h->num_cus, s) : f32::launch_delta<64>(d, h->num_cus, s);
    if (e == hipSuccess) e = grad.accumulate(pl, p0 == 0, s);
  }
  if (e == hipSuccess) e = grad.reduce(grad_w, s);
  return gn_check_device(h, e, "backward launch");
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
