// Expert execution of fp32 layers (the fp32 counterpart of ffn.hip): the
// SwiGLU FFN of every work item and of the shared expert's pieces.
//
// Both products run on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32
// operands, products and sums, like a chain of fused multiply-adds).  The
// weights are reduction-major (w13[e][h][u], w2[e][i][j]), so one 16-lane row
// of a wave reads U consecutive output units per lane of one reduction index
// (U = 4: 256 contiguous bytes) and the four 16-lane rows four indices; lane
// (q, c) thereby holds the matrix operand of units u0 + U*c .. + U-1 at
// reduction index 16*g + 4*q + i for i = 0..3 (four loads), and the token
// operand of the same four indices is one 16-byte load of its token's
// values.  The order in which a matrix instruction sums its indices does not
// matter as long as both operands agree, so neither is rearranged.
//
// What bounds it: the weight stream at few tokens, the fp32 matrix rate
// (a sixteenth of bf16's) at many.  A workgroup covers 16*U units and at most
// 32 rows of an item (its other rows are further workgroups: at this rate a
// second pass costs more than reading the weights again from a cache); its
// four waves split the reduction (summed in wave order through LDS, so
// results do not depend on scheduling) and keep two bursts of weights in
// flight each.  Measured on two blocks of 32 tokens over 32 experts (hidden
// 1024, intermediate 512 + shared 512, top-4, token routing; 207 MB), whole
// layer: 513 us with scalar-FMA kernels of eight tokens per pass, 137 with
// these at U = 4 and passes in a loop (the U = 4 gate/up spilled), 100 at
// U = 2, 80 with the passes spread over workgroups.  fp32 rounding only: the
// distance from float64 is that of the scalar kernels (4.8e-7 of the output).
#include <algorithm>
#include <type_traits>

#include "dmoe_common.h"
#include "ffn_dev.h"

namespace dmoe {
namespace {

using fdev::decode_item;
using fdev::Group;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kPassRows = 32;  // rows of an item per workgroup (two token tiles)
constexpr int kGroup = 16;  // reduction indices of one group: four per 16-lane row
constexpr int kBurst = 2;  // groups loaded together; two such bursts are in flight

struct F32Params {
  const float* xk;  // activations, chunk-major [H/4][T][4]
  const float* xr;  // the same row-major [T][H], or nullptr
  const float *w13, *w2, *ws13, *ws2;
  const int *n_work, *work, *row_token, *row_slot;
  int T, H, E, I, I_s, k, Tk, max_work, ldh;
  int base;         // first unit (output feature) of the launch (size_t offsets only; 8 bytes more of arguments cost 0.2 us)
  float* hbuf;      // SwiGLU activations [Tk (+ T)][ldh]
  float* slot_out;  // [T][k][H]
  float* shared_out;
};

// Units and output features past a row's end pass 2^31 only in the widest layers.
template <typename Off>
using Unit = std::conditional_t<(sizeof(Off) > 4), unsigned, int>;

// One burst of a wave's operands: NM weight matrices (gate and up, or down
// alone), NT tiles of 16 tokens.
template <int U, int NM, int NT>
struct Burst {
  float a[kBurst][4][NM][U];
  f32x4 b[kBurst][NT];
};

template <int U, bool kStream>
__device__ __forceinline__ void ld_units(const float* p, float (&v)[U]) {
  if constexpr (U > 1) {
    typedef float vec __attribute__((ext_vector_type(U)));
    const vec* pv = reinterpret_cast<const vec*>(p);
    const vec x = kStream ? __builtin_nontemporal_load(pv) : *pv;
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = x[u];
  } else {
    static_assert(U == 1, "units per lane");
    v[0] = kStream ? __builtin_nontemporal_load(p) : *p;
  }
}

template <int U, int NM, int NT>
__device__ __forceinline__ void mma_group(const float (&a)[4][NM][U], const f32x4 (&b)[NT], f32x4 (&acc)[NM][U][NT]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
          acc[m][u][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][m][u], b[ct][i], acc[m][u][ct], 0, 0, 0);
}

// acc += W . B over the reduction groups g0 .. g1-1 of a reduction of length
// K.  W[m]: matrix m, row stride ldw; lo: this lane's offset in it, index 4*q
// at its units.
// pb[ct]: token tile ct's values at index 4*q; bstep elements to the next
// group; kVecB: its four values are one aligned 16-byte load.  Groups past
// the end of a burst reload the last one (straight-line loads) and are not
// used; a last group that K does not fill is loaded element by element, with
// zeros past K in both operands.
template <int U, int NM, int NT, bool kStream, bool kVecB, typename Off>
__device__ __forceinline__ void wave_dot_f32(const float* const (&W)[NM], Off lo, size_t ldw, const float* const (&pb)[NT],
                                             int bstep, int K, int g0, int g1, int q, f32x4 (&acc)[NM][U][NT]) {
  const int nfull = K / kGroup;
  const int ge = min(g1, nfull);
  Burst<U, NM, NT> r[2];
  auto load = [&](Burst<U, NM, NT>& d, int g) {
#pragma unroll
    for (int s = 0; s < kBurst; ++s) {
      const int gs = min(g + s, ge - 1);
      const size_t row = static_cast<size_t>(gs) * kGroup;
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) {
        const float* p = pb[ct] + static_cast<size_t>(gs) * bstep;
        if constexpr (kVecB)
          d.b[s][ct] = *reinterpret_cast<const f32x4*>(p);
        else
#pragma unroll
          for (int i = 0; i < 4; ++i) d.b[s][ct][i] = p[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < NM; ++m) ld_units<U, kStream>(W[m] + (row + i) * ldw + lo, d.a[s][i][m]);
    }
  };
  auto mma = [&](const Burst<U, NM, NT>& d, int g) {
#pragma unroll
    for (int s = 0; s < kBurst; ++s)
      if (g + s < ge) mma_group<U, NM, NT>(d.a[s], d.b[s], acc);  // uniform
  };
  if (g0 < ge) {
    load(r[0], g0);
    for (int g = g0; g < ge; g += 2 * kBurst) {
      load(r[1], g + kBurst);
      __builtin_amdgcn_sched_barrier(0);
      mma(r[0], g);
      __builtin_amdgcn_sched_barrier(0);
      load(r[0], g + 2 * kBurst);
      __builtin_amdgcn_sched_barrier(0);
      mma(r[1], g + kBurst);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (K % kGroup && g0 <= nfull && nfull < g1) {  // uniform: the wave that owns the partial group
    float a[4][NM][U];
    f32x4 b[NT];
    const size_t row = static_cast<size_t>(nfull) * kGroup;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = static_cast<int>(row) + 4 * q + i < K;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
#pragma unroll
        for (int u = 0; u < U; ++u) a[i][m][u] = in ? (W[m] + (row + i) * ldw)[lo + u] : 0.f;
      }
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) b[ct][i] = in ? pb[ct][static_cast<size_t>(nfull) * bstep + i] : 0.f;
    }
    mma_group<U, NM, NT>(a, b, acc);
  }
}

// Sum the four waves' partial tiles into wave 0's registers (wave order).
template <int U, int NM, int NT>
__device__ __forceinline__ void reduce_waves_f32(f32x4 (&acc)[NM][U][NT], f32x4* red, int wave, int lane) {
  constexpr int kTiles = NM * U * NT;
  if (wave > 0) {
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) red[((wave - 1) * kTiles + (m * U + u) * NT + ct) * kWave + lane] = acc[m][u][ct];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
          for (int w = 0; w < kWaves - 1; ++w) acc[m][u][ct] += red[(w * kTiles + (m * U + u) * NT + ct) * kWave + lane];
  }
}

template <int U, int NM, int NT>
__device__ __forceinline__ void zero_f32(f32x4 (&acc)[NM][U][NT]) {
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) acc[m][u][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// One pass of the gate/up kernel: 16*NT rows of the item from row p0.
template <int U, int NT, bool kStream, typename Off>
__device__ __forceinline__ void gateup_pass(const F32Params& p, const Group& g, int Iw, Unit<Off> u0, int p0, f32x4* red) {
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const float* W = g.expert >= 0 ? p.w13 + static_cast<size_t>(g.expert) * 2 * p.I * p.H : p.ws13;
  const size_t ldw = 2 * static_cast<size_t>(Iw);
  const int uc = min<Unit<Off>>(u0 + U * c, Iw - U);  // units past the last: the last ones again, not stored
  const float* const pw[2] = {W, W + Iw};
  const Off lo = 4 * q * static_cast<Off>(ldw) + uc;
  const float* pb[NT];
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    const int col = min(p0 + ct * 16 + c, g.n - 1);
    const int tok = g.tok ? g.tok[col] : g.t0 + col;
    pb[ct] = p.xr ? p.xr + static_cast<size_t>(tok) * p.H + 4 * q : p.xk + (static_cast<size_t>(q) * p.T + tok) * 4;
  }
  const int ng = (p.H + kGroup - 1) / kGroup, per = (ng + kWaves - 1) / kWaves;
  f32x4 acc[2][U][NT];
  zero_f32(acc);
  wave_dot_f32<U, 2, NT, kStream, true, Off>(pw, lo, ldw, pb, p.xr ? kGroup : kGroup * p.T, p.H, wave * per, min(ng, (wave + 1) * per), q, acc);
  reduce_waves_f32(acc, red, wave, lane);
  if (wave == 0) {
    // accumulator r of lane (q, c): units u0 + U*(4q + r) + u of row p0 + 16ct + c
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
      const int col = p0 + ct * 16 + c;
      if (col >= g.n) continue;
      float* dst = p.hbuf + static_cast<size_t>(g.r0 + col) * p.ldh;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const Unit<Off> u1 = u0 + U * (4 * q + r);
        float h[U];
#pragma unroll
        for (int u = 0; u < U; ++u) h[u] = silu_f32(acc[0][u][ct][r]) * acc[1][u][ct][r];
        if (u1 < static_cast<Unit<Off>>(Iw)) {  // I % U == 0: the U units lie wholly in or past the row
          if constexpr (U > 1) {
            typedef float vec __attribute__((ext_vector_type(U)));
            vec v;
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = h[u];
            *reinterpret_cast<vec*>(dst + u1) = v;
          } else {
            dst[u1] = h[0];
          }
        }
      }
    }
  }
}

// f(token tiles of the pass, non-temporal weight loads).  An item of several
// passes is read by as many workgroups, whose later ones can find its weights
// in a cache: plain loads, also in a launch that streams.  Token routing,
// us per layer, layers in rotation: two blocks of 32 tokens over 128 experts
// (hidden 768, intermediate 384) 110.0 -> 108.4, Zipf-biased 70.0 -> 67.2,
// four of 48 93.6 -> 88.1.  (The passes of an item adjacent in the grid, as in
// the bf16 kernels, measured 110 -> 195: rows that hold no work between the
// others.)
template <bool kStream, typename F>
__device__ __forceinline__ void by_rows(const Group& g, int p0, F f) {
  constexpr std::integral_constant<int, 1> one;
  constexpr std::integral_constant<int, 2> two;
  if (kStream && g.n <= kPassRows) {
    if (g.n > 16)
      f(two, std::bool_constant<kStream>{});
    else
      f(one, std::bool_constant<kStream>{});
  } else if (g.n - p0 > 16) {
    f(two, std::false_type{});
  } else {
    f(one, std::false_type{});
  }
}

// grid (ceil(ldh / (16 U)), items, passes): units 16*U*bx .. of rows 32*bz ..
// of item y.  I % U == 0 and I_s % U == 0 (aligned loads and stores).
template <int U, bool kStream, typename Off>
__global__ __launch_bounds__(kThreads, 2) void ffn_gateup_f32_kernel(F32Params p) {
  __shared__ f32x4 red[(kWaves - 1) * 2 * U * 2 * kWave];
  Group g;
  if (!decode_item(blockIdx.y, 0, p.max_work, p.n_work, p.work, p.row_token, p.T, p.Tk, p.E, g)) return;
  const int Iw = g.expert >= 0 ? p.I : p.I_s;
  const Unit<Off> u0 = (sizeof(Off) > 4 ? p.base : 0) + blockIdx.x * 16 * U;
  if (u0 >= static_cast<Unit<Off>>(Iw)) return;
  const int p0 = blockIdx.z * kPassRows;
  if (p0 >= g.n) return;
  by_rows<kStream>(g, p0, [&](auto nt, auto stream) {
    gateup_pass<U, decltype(nt)::value, decltype(stream)::value, Off>(p, g, Iw, u0, p0, red);
  });
}

template <int U, int NT, bool kStream, bool kVecB, typename Off>
__device__ __forceinline__ void down_pass(const F32Params& p, const Group& g, int Kd, Unit<Off> j0, int p0, f32x4* red) {
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int H = p.H;
  const float* W = g.expert >= 0 ? p.w2 + static_cast<size_t>(g.expert) * H * p.I : p.ws2;
  const int jc = min<Unit<Off>>(j0 + U * c, H - U);
  const float* const pw[1] = {W};
  const Off lo = 4 * q * static_cast<Off>(H) + jc;
  const float* pb[NT];
#pragma unroll
  for (int ct = 0; ct < NT; ++ct)
    pb[ct] = p.hbuf + static_cast<size_t>(g.r0 + min(p0 + ct * 16 + c, g.n - 1)) * p.ldh + 4 * q;
  const int ng = (Kd + kGroup - 1) / kGroup, per = (ng + kWaves - 1) / kWaves;
  f32x4 acc[1][U][NT];
  zero_f32(acc);
  wave_dot_f32<U, 1, NT, kStream, kVecB, Off>(pw, lo, H, pb, kGroup, Kd, wave * per, min(ng, (wave + 1) * per), q, acc);
  reduce_waves_f32(acc, red, wave, lane);
  if (wave == 0) {
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
      const int col = p0 + ct * 16 + c;
      if (col >= g.n) continue;
      const int row = g.r0 + col;
      float* dst = g.tok ? p.slot_out + (static_cast<size_t>(p.row_token[row]) * p.k + p.row_slot[row]) * H
                         : p.shared_out + static_cast<size_t>(g.t0 + col) * H;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const Unit<Off> j1 = j0 + U * (4 * q + r);
        if constexpr (U == 4) {
          if (j1 < static_cast<Unit<Off>>(H))
            *reinterpret_cast<f32x4*>(dst + j1) =
                f32x4{acc[0][0][ct][r], acc[0][1][ct][r], acc[0][2][ct][r], acc[0][3][ct][r]};  // H % 4 == 0
        } else {
          if (j1 < static_cast<Unit<Off>>(H)) dst[j1] = acc[0][0][ct][r];
        }
      }
    }
  }
}

// grid (ceil(H / (16 U)), items, passes): output features 16*U*bx .. of item y.
// kVecB: rows of the activations are 16-byte aligned (ldh % 4 == 0).
template <int U, bool kStream, bool kVecB, typename Off>
__global__ __launch_bounds__(kThreads, 2) void ffn_down_f32_kernel(F32Params p) {
  __shared__ f32x4 red[(kWaves - 1) * U * 2 * kWave];
  Group g;
  if (!decode_item(blockIdx.y, 0, p.max_work, p.n_work, p.work, p.row_token, p.T, p.Tk, p.E, g)) return;
  const int Kd = g.expert >= 0 ? p.I : p.I_s;
  const Unit<Off> j0 = (sizeof(Off) > 4 ? p.base : 0) + blockIdx.x * 16 * U;
  const int p0 = blockIdx.z * kPassRows;
  if (p0 >= g.n) return;
  by_rows<kStream>(g, p0, [&](auto nt, auto stream) {
    down_pass<U, decltype(nt)::value, decltype(stream)::value, kVecB, Off>(p, g, Kd, j0, p0, red);
  });
}

// Units per lane: gate/up 2 (two matrices; at 4 the operands leave one burst
// in flight, 80 -> 86 us on the layer above), down 4; launches of fewer than
// kFillGroups workgroups (one per CU) take 1, four times the workgroups (a
// tiny layer of hidden 256, intermediate 128, 8 tokens: gate/up 4.8 us).
constexpr int kWideGu = 2, kWideDn = 4;
constexpr long kFillGroups = 256;
// Workgroups in a grid's x dimension (a grid has fewer than 2^32 threads in
// each): wider layers take several launches.
constexpr int kMaxGridX = 1 << 23;

}  // namespace

hipError_t launch_ffn_f32(const FfnArgs& a, int ldh, int items, hipStream_t s) {
  F32Params p{static_cast<const float*>(a.x), static_cast<const float*>(a.xr), static_cast<const float*>(a.w13), static_cast<const float*>(a.w2),
              static_cast<const float*>(a.ws13), static_cast<const float*>(a.ws2), a.sched.n_work, a.sched.work,
              a.sched.row_token, a.sched.row_slot, a.T, a.H, a.E, a.I, a.I_s, a.k, a.T * a.k, a.max_work, ldh, 0,
              static_cast<float*>(a.workspace), static_cast<float*>(a.slot_out), a.shared_out};
  // Items of few rows read their weights once per launch: non-temporal loads
  // (by_rows), where the weights of all items, an upper bound of what is read,
  // exceed 128 MiB.  Layers in rotation, so that weights come from HBM, us per
  // layer, plain / non-temporal loads throughout: the layer at the top of
  // the file, token routing (207 MB at most) 85.4 / 81.5, one block of 8 tokens 70.4 / 66.7;
  // smaller launches mostly the other way: block routing (57 MB) 65.6 / 73.4,
  // one block of 8 (31 MB) 34.6 / 37.1, a layer of hidden 768 and intermediate 384 50.0
  // / 59.3, of hidden 256 20.4 / 21.4; but token routing over many experts
  // (117 MB at most) 49.0 / 46.0, and 30.8 / 32.5 when few are popular.
  const long rows = static_cast<long>(a.T) * std::max(a.k, 1);
  const size_t weights = static_cast<size_t>(items) * 3 * a.H * ldh * sizeof(float);
  const bool stream = rows <= 32L * items && weights > (size_t{128} << 20);
  // A lane's weight offset, 12 rows and a row's units at most, in 32 bits unless
  // the layer is wider than any (three blocks of 32 tokens over 72 experts,
  // hidden 360, intermediate 376: 60.8 us per layer against 62.7 with 64 bits).
  // Such a layer may also need more than one launch.
  const bool big = 13 * std::max(2 * static_cast<long>(ldh), static_cast<long>(a.H)) > (1L << 32) - 1 ||
                   std::max(ldh, a.H) > 16 * kMaxGridX;
  const bool wide_ok = a.I % kWideGu == 0 && a.I_s % kWideGu == 0;  // aligned loads and stores
  const bool wide = wide_ok && (static_cast<long>(ldh) + 16 * kWideGu - 1) / (16 * kWideGu) * items >= kFillGroups;
  // an item holds each token at most once
  const int passes = (std::min(a.T, DMOE_WORK_ROWS) + kPassRows - 1) / kPassRows;
  const int gu = wide ? 16 * kWideGu : 16;  // units per gate/up workgroup
  hipError_t err = hipSuccess;
  const int gx_gu = static_cast<int>((static_cast<long>(ldh) + gu - 1) / gu);
  for (int x = 0; x < gx_gu && err == hipSuccess; x += kMaxGridX) {
    p.base = x * gu;
    const dim3 grid(std::min(gx_gu - x, kMaxGridX), items, passes);
#define DMOE_GATEUP_F32(U_, S_, B_, OFF_)                                    \
  if (wide == (U_ == kWideGu) && (stream && !big) == S_ && big == B_)        \
    ffn_gateup_f32_kernel<U_, S_, OFF_><<<grid, kThreads, 0, s>>>(p);
    DMOE_GATEUP_F32(kWideGu, true, false, uint32_t)
    DMOE_GATEUP_F32(kWideGu, false, false, uint32_t)
    DMOE_GATEUP_F32(1, true, false, uint32_t)
    DMOE_GATEUP_F32(1, false, false, uint32_t)
    DMOE_GATEUP_F32(kWideGu, false, true, size_t)
    DMOE_GATEUP_F32(1, false, true, size_t)
#undef DMOE_GATEUP_F32
    err = hipGetLastError();
  }
  const bool vec_b = ldh % 4 == 0;
  const bool wide_dn = (static_cast<long>(a.H) + 16 * kWideDn - 1) / (16 * kWideDn) * items >= kFillGroups;
  const int du = wide_dn ? 16 * kWideDn : 16;
  const int gx_dn = static_cast<int>((static_cast<long>(a.H) + du - 1) / du);
  for (int x = 0; x < gx_dn && err == hipSuccess; x += kMaxGridX) {
    p.base = x * du;
    const dim3 grid(std::min(gx_dn - x, kMaxGridX), items, passes);
#define DMOE_DOWN_F32(U_, S_, V_, B_, OFF_)                                                          \
  if (wide_dn == (U_ == kWideDn) && (stream && !big) == S_ && vec_b == V_ && big == B_)              \
    ffn_down_f32_kernel<U_, S_, V_, OFF_><<<grid, kThreads, 0, s>>>(p);
    DMOE_DOWN_F32(kWideDn, true, true, false, uint32_t)
    DMOE_DOWN_F32(kWideDn, false, true, false, uint32_t)
    DMOE_DOWN_F32(1, true, true, false, uint32_t)
    DMOE_DOWN_F32(1, false, true, false, uint32_t)
    DMOE_DOWN_F32(kWideDn, true, false, false, uint32_t)
    DMOE_DOWN_F32(kWideDn, false, false, false, uint32_t)
    DMOE_DOWN_F32(1, true, false, false, uint32_t)
    DMOE_DOWN_F32(1, false, false, false, uint32_t)
    DMOE_DOWN_F32(kWideDn, false, true, true, size_t)
    DMOE_DOWN_F32(1, false, true, true, size_t)
    DMOE_DOWN_F32(kWideDn, false, false, true, size_t)
    DMOE_DOWN_F32(1, false, false, true, size_t)
#undef DMOE_DOWN_F32
    err = hipGetLastError();
  }
  return err;
}

}  // namespace dmoe
