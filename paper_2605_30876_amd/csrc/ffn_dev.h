// Wave-level helpers of the bf16 expert FFN kernels: packed weight tiles as
// the matrix-core A operand, chunk-major token rows as the B operand, bursts
// of K-steps with double-buffered token chunks, and the fixed-order sum of
// the four waves' partial tiles.  Internal; shared by ffn.hip and layer.hip.
#pragma once

#include "dmoe_common.h"

namespace dmoe {
namespace fdev {

struct Group {
  int r0;          // first row of the item in the row space (h buffer row)
  int n;           // rows (tokens) in the item
  int expert;      // routed expert id, or -1 for the shared expert
  const int* tok;  // token of each row (routed), or nullptr: row c is token t0 + c
  int t0;
  int piece;       // index of the item among its expert's items (0, 1, ...)
};

// Grid row y: the schedule's max_work items, then the shared expert's pieces
// (kSharedFirst: the pieces first).  One memory round trip: the item count
// and the item are loaded together (the index stays inside the work array;
// an item past n_work is loaded but not used).  An item naming an expert
// outside [0, E) is skipped, so no schedule can steer a weight read outside
// the expert arrays.
template <bool kSharedFirst = false>
__device__ __forceinline__ bool decode_item(int y, int shared_items, int max_work, const int* n_work,
                                            const int* work, const int* row_token, int T, int Tk, int E, Group& g) {
  const int w = kSharedFirst ? y - shared_items : y;
  if (kSharedFirst ? w >= 0 : w < max_work) {
    const int nw = *n_work;
    const int4 it = reinterpret_cast<const int4*>(work)[w];
    g.expert = it.x;
    g.r0 = it.y;
    g.n = (w < nw && static_cast<unsigned>(it.x) < static_cast<unsigned>(E)) ? it.z : 0;
    g.tok = row_token + it.y;
    g.t0 = 0;
    g.piece = it.w;
  } else {
    const int c = kSharedFirst ? y : y - max_work;
    g.expert = -1;
    g.piece = c;
    g.t0 = c * DMOE_WORK_ROWS;
    g.r0 = Tk + g.t0;
    g.n = min(DMOE_WORK_ROWS, T - g.t0);
    g.tok = nullptr;
  }
  return g.n > 0;
}

constexpr int kFrag = 512;  // bf16 elements of one packed 16 x 32 weight tile (1 KiB)

// Operands of one wave for up to KMAX K-steps (32 each) of its K-slice.
// A: RT 16-row weight tiles, all steps issued at once; B: NT 16-column token
// tiles in chunks of BC steps, double-buffered when a burst has more than one
// chunk.  Each B fragment feeds RT matrix instructions.
template <int NT, int KMAX, int BC, int RT = 1>
struct WaveOps {
  static constexpr int kChunks = KMAX / BC;
  bf16x8 a[RT][KMAX];
  bf16x8 b[kChunks > 1 ? 2 : 1][BC][NT];
};

// A: packed tiles, step s of tile r at pa + r*tstride + s*kFrag (one
// contiguous burst per tile).  kStream: non-temporal loads, for weights no
// other workgroup of the launch reads again.
template <bool kStream, int NT, int KMAX, int BC, int RT>
__device__ __forceinline__ void issue_a(WaveOps<NT, KMAX, BC, RT>& w, const bf16_t* pa, size_t tstride, int ns) {
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int s = 0; s < KMAX; ++s)
      if (s < ns)
        w.a[r][s] = kStream ? ld_bf16x8_stream(pa + r * tstride + s * kFrag) : ld_bf16x8(pa + r * tstride + s * kFrag);
}

// B: chunk-major rows, step s at pb[ct] + s*bstep.
template <int BUF, int NT, int KMAX, int BC, int RT>
__device__ __forceinline__ void issue_b(WaveOps<NT, KMAX, BC, RT>& w, const bf16_t* const* pb, int bstep, int chunk,
                                        int ns) {
#pragma unroll
  for (int s = 0; s < BC; ++s)
    if (chunk * BC + s < ns)
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) w.b[BUF][s][ct] = ld_bf16x8(pb[ct] + (chunk * BC + s) * bstep);
}

template <int C, int NT, int KMAX, int BC, int RT>
__device__ __forceinline__ void mma_chunk(WaveOps<NT, KMAX, BC, RT>& w, const bf16_t* const* pb, int bstep, int ns,
                                          f32x4 (&acc)[RT][NT]) {
  constexpr int NCH = KMAX / BC;
  if constexpr (C < NCH) {
    if (C * BC < ns) {
      if constexpr (C + 1 < NCH) issue_b<(C + 1) & 1>(w, pb, bstep, C + 1, ns);
      __builtin_amdgcn_sched_barrier(0);  // keep the next chunk's loads where they are
#pragma unroll
      for (int s = 0; s < BC; ++s)
        if (C * BC + s < ns)
#pragma unroll
          for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int r = 0; r < RT; ++r)
              acc[r][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.a[r][C * BC + s], w.b[C & 1][s][ct], acc[r][ct],
                                                                   0, 0, 0);
      mma_chunk<C + 1>(w, pb, bstep, ns, acc);
    }
  }
}

// acc[ct] += A . B_ct^T over this wave's `steps` K-steps, in bursts of KMAX
// steps: token chunk 0, the weight burst, then the remaining token chunks.
// With a_held (the slice is one burst, steps <= KMAX, already in w.a from
// the previous pass over the same weights) the weights are not loaded again.
// kStream: the weights are loaded non-temporally (see issue_a).
template <bool kStream, int NT, int KMAX, int BC, int RT>
__device__ __forceinline__ void wave_dot(WaveOps<NT, KMAX, BC, RT>& w, const bf16_t* pa, size_t tstride,
                                         const bf16_t* const* pb, int bstep, int steps, f32x4 (&acc)[RT][NT],
                                         bool a_held) {
  for (int sc = 0; sc < steps; sc += KMAX) {
    const int ns = min(KMAX, steps - sc);
    const bf16_t* pbs[NT];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) pbs[ct] = pb[ct] + sc * bstep;
    issue_b<0>(w, pbs, bstep, 0, ns);
    if (!a_held) issue_a<kStream>(w, pa + sc * kFrag, tstride, ns);
    __builtin_amdgcn_sched_barrier(0);
    mma_chunk<0>(w, pbs, bstep, ns, acc);
  }
}

// wave_dot for one full burst (KMAX steps, straight-line: the compiler's wait
// counts are exact) with three token chunk buffers: chunks
// and their weights are issued alternately, so that a chunk's tokens return
// with its weights.  (With two buffers, chunk C + 1 is issued once chunk C - 1
// is done: after the weights have arrived, the last chunks each wait for a
// round trip of their own.)
template <int NT, int KMAX, int BC, int RT>
struct WaveOps3 {
  static constexpr int kChunks = KMAX / BC;
  static_assert(kChunks == 4, "four chunks");
  bf16x8 a[RT][KMAX];
  bf16x8 b[3][BC][NT];
};

// Token chunk C of a full burst into its buffer: step s of tile ct at pb +
// s*bstep + lb[ct] (pb uniform over the wave: the loads take a scalar base and
// a 32-bit lane offset, which leaves the registers to the operands).
template <int C, int NT, int KMAX, int BC, int RT>
__device__ __forceinline__ void issue_b3(WaveOps3<NT, KMAX, BC, RT>& w, const bf16_t* pb, const uint32_t (&lb)[NT],
                                         int bstep) {
#pragma unroll
  for (int s = 0; s < BC; ++s)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) w.b[C % 3][s][ct] = ld_bf16x8(pb + (C * BC + s) * bstep + lb[ct]);
}

// pa is uniform too, la the lane's offset.
template <bool kStream, int NT, int KMAX, int BC, int RT>
__device__ __forceinline__ void wave_dot_burst(WaveOps3<NT, KMAX, BC, RT>& w, const bf16_t* pa, uint32_t la, size_t tstride,
                                               const bf16_t* pb, const uint32_t (&lb)[NT], int bstep, f32x4 (&acc)[RT][NT]) {
  auto ld_a = [&](int chunk) {
#pragma unroll
    for (int s = chunk * BC; s < (chunk + 1) * BC; ++s)
#pragma unroll
        for (int r = 0; r < RT; ++r)
          w.a[r][s] = kStream ? ld_bf16x8_stream(pa + r * tstride + s * kFrag + la) : ld_bf16x8(pa + r * tstride + s * kFrag + la);
  };
  auto mma = [&](int chunk, int buf) {
#pragma unroll
    for (int s = 0; s < BC; ++s)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
          for (int r = 0; r < RT; ++r)
            acc[r][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.a[r][chunk * BC + s], w.b[buf][s][ct], acc[r][ct], 0,
                                                                 0, 0);
  };
  issue_b3<0>(w, pb, lb, bstep);
  ld_a(0);
  __builtin_amdgcn_sched_barrier(0);
  issue_b3<1>(w, pb, lb, bstep);
  ld_a(1);
  __builtin_amdgcn_sched_barrier(0);
  issue_b3<2>(w, pb, lb, bstep);
  ld_a(2);
  ld_a(3);
  __builtin_amdgcn_sched_barrier(0);
  mma(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  issue_b3<3>(w, pb, lb, bstep);
  __builtin_amdgcn_sched_barrier(0);
  mma(1, 1);
  mma(2, 2);
  mma(3, 0);
}

// The same for a burst of K steps whose operands all fit in registers.
template <bool kStream, int K, int NT, int RT>
__device__ __forceinline__ void wave_dot_short(const bf16_t* pa, uint32_t la, size_t tstride, const bf16_t* pb,
                                               const uint32_t (&lb)[NT], int bstep, f32x4 (&acc)[RT][NT]) {
  bf16x8 a[RT][K], b[K][NT];
#pragma unroll
  for (int s = 0; s < K; ++s) {
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) b[s][ct] = ld_bf16x8(pb + s * bstep + lb[ct]);
#pragma unroll
    for (int r = 0; r < RT; ++r)
      a[r][s] = kStream ? ld_bf16x8_stream(pa + r * tstride + s * kFrag + la)
                        : ld_bf16x8(pa + r * tstride + s * kFrag + la);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < K; ++s)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int r = 0; r < RT; ++r)
        acc[r][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r][s], b[s][ct], acc[r][ct], 0, 0, 0);
}

// Sum the four waves' partial tiles into wave 0's registers (wave order).
template <int RT, int NT>
__device__ __forceinline__ void reduce_waves(f32x4 (&acc)[RT][NT], f32x4 (*red)[RT][NT][kWave], int wave,
                                             int lane) {
  if (wave > 0) {
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) red[wave - 1][r][ct][lane] = acc[r][ct];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int ct = 0; ct < NT; ++ct)
#pragma unroll
        for (int ww = 0; ww < 3; ++ww) acc[r][ct] += red[ww][r][ct][lane];
  }
}

template <int RT, int NT>
__device__ __forceinline__ void zero(f32x4 (&acc)[RT][NT]) {
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) acc[r][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
}

}  // namespace fdev
}  // namespace dmoe
