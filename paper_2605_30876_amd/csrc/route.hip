// The routing stage of one forward: router scores (Sec. 4.2), expert
// selection (block routing, Sec. 4.2 aggregation and Alg. 1 with a coreset
// of size k; or the token-level baseline), combine weights and the
// unique-expert schedule.
//
// A decode step routes few tokens; its routing kernels are bound by memory
// round trips (each kernel boundary adds a write, a cache flush and a re-read
// from another XCD), not by arithmetic.  Blocks of up to 8 to 64 tokens
// (route_block_fits) run everything after the router in one workgroup each
// with a single round trip: all partial logits are loaded at once, then softmax
// rows (into LDS), block sums, top-k and combine weights run on chip, and for
// a forward of one block the schedule too.  (Token routing has T rows to select; spread
// over T/4 workgroups it is faster, so it runs the softmax and each token's
// selection in one launch of T/4 workgroups, then the schedule.)  The
// arithmetic is that of
// the separate kernels (same device routines, same summation orders), so the
// results are bit-identical to dmoe_router_logits +
// dmoe_block_aggregate_topk / dmoe_token_topk + dmoe_build_expert_schedule.
// Larger forwards chain those kernels.
#include "route_dev.h"

namespace dmoe {
namespace {

constexpr int kThreads = dev::kSchedThreads;  // the schedule's workgroup size
constexpr int kWaves = kThreads / kWave;
// The largest block that gains (64 tokens over 256 experts: 68 KB), with
// headroom for static LDS.  (The registers leave one workgroup per CU either
// way.)
constexpr size_t kMaxLdsBytes = 76 * 1024;

// LDS words of the block kernel (4-byte words; rows padded to a multiple of 4
// floats for 128-bit reads).
struct FusedLayout {
  int Es;  // padded row stride
  size_t sb, sel, selv, bufv, bufi, sched, total;
};

__host__ __device__ inline FusedLayout fused_layout(int T, int E, int k) {
  FusedLayout L;
  L.Es = (E + 3) & ~3;
  L.sb = static_cast<size_t>(T) * L.Es;  // P [T][Es]
  L.sel = L.sb + L.Es;                   // S [Es]
  L.selv = L.sel + (k + 1);              // sel [k+1]
  L.bufv = L.selv + (k + 1);             // selv [k+1]
  L.bufi = L.bufv + (k + 1);             // top-k gather
  L.sched = L.bufi + (k + 1);
  L.total = L.sched + kWave;             // closed-form schedule scratch
  return L;
}

constexpr int kWBatch = 8;  // selected probabilities of a token loaded together

// Routes one block of T tokens.  kPerBlock: workgroup b routes block b of a
// forward of T_all tokens (the partial planes have T_all rows), and the
// schedule is left to a launch of its own; otherwise the block is the forward
// and the kernel writes the (closed-form) schedule too.  Several small blocks
// in one workgroup, with the general schedule built there as well, measured
// slower than a workgroup each and a schedule launch even for two: five blocks
// of 24 tokens over 48 experts 54.9 -> 47.8 us per layer, three 43.9 -> 40.1,
// two 36.6 -> 35.5.
template <int NQ, bool kPerBlock>
__global__ __launch_bounds__(kThreads) void route_small_kernel(
    const float* part, int S, const float* __restrict__ bias, int T, int E, int k,
    float* probs, float* __restrict__ logits, float* __restrict__ block_scores,
    int32_t* __restrict__ experts, float* __restrict__ cw, float* __restrict__ gap,
    dmoe_schedule sched, int T_all) {
  extern __shared__ float lds[];
  __shared__ dev::BlockTopkLds tk;
  if (kPerBlock) {
    const size_t b = blockIdx.x;
    part += b * T * E;
    probs += b * T * E;
    if (logits) logits += b * T * E;
    if (block_scores) block_scores += b * E;
    experts += b * k;
    cw += b * T * k;
    if (gap) gap += b;
  }
  const FusedLayout L = fused_layout(T, E, k);
  const int Es = L.Es;
  float* P = lds;
  float* Sb = lds + L.sb;
  int* sel = reinterpret_cast<int*>(lds + L.sel);
  float* selv = lds + L.selv;
  const int tid = threadIdx.x, wave = tid >> 6;

  // 1. router softmax: wave w owns rows w, w + 8, ...; a batch of RB rows
  //    has all of its partial loads in flight together, then each row is
  //    reduced in registers into probs and P.  (part may alias probs: a row
  //    is read only by the wave that writes it, before it writes it.)
  {
    constexpr int RB = 4 / NQ;
    const size_t plane = static_cast<size_t>(T_all) * E;
    for (int t0 = wave; t0 < T; t0 += kWaves * RB) {
      dev::RowPartials<NQ> r[RB];
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int t = t0 + u * kWaves;
        if (t < T) dev::load_row<NQ>(part, plane, S, bias, E, t, r[u]);
      }
      bool live[RB];
      float* out[RB];
      float* prow[RB];
      float* lo[RB];
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int t = min(t0 + u * kWaves, T - 1);
        live[u] = t0 + u * kWaves < T;
        out[u] = probs + static_cast<size_t>(t) * E;
        prow[u] = P + static_cast<size_t>(t) * Es;
        lo[u] = logits ? logits + static_cast<size_t>(t) * E : nullptr;
      }
      dev::softmax_loaded<NQ, RB>(r, live, S, bias != nullptr, E, out, prow, lo);
    }
  }
  __syncthreads();

  // 2. selection: the block mean in token order, then sel[0..rounds) in
  //    (score desc, id asc) order
  const int rounds = k < E ? k + 1 : k;
  const float n_tok = static_cast<float>(T);
  for (int e = tid; e < E; e += kThreads) {
    const float* pe = P + e;
    float acc = 0.f;
#pragma unroll 8
    for (int t = 0; t < T; ++t) acc += pe[static_cast<size_t>(t) * Es];  // token order
    const float v = acc / n_tok;
    Sb[e] = v;
    if (block_scores) block_scores[e] = v;
  }
  __syncthreads();
  // All threads select when the group maxima bound the candidates (at least
  // `rounds` groups of 16) or every expert as a candidate is cheap; otherwise
  // one wave's radix search (112 experts, top-8: 8.2 us for the kernel
  // against 9.6; 256 experts, top-8, the other way round: 9.9 against 9.0).
  if (dev::block_topk_fits(E, rounds) && (E >= 16 * rounds || E <= 64))
    dev::block_topk_small(Sb, E, rounds, sel, selv, tk);
  else if (wave == 0)
    dev::wave_topk_radix_n<4 * NQ>(Sb, E, rounds, sel, selv, lds + L.bufv, reinterpret_cast<int*>(lds + L.bufi));
  __syncthreads();

  // 3. expert list, gap, and every token's weights renormalised over the
  //    selection (summed in slot order)
  if (tid < k) experts[tid] = sel[tid];
  if (gap && tid == 0) gap[0] = k < E ? selv[k - 1] - selv[k] : INFINITY;
  // one thread per (token, slot); each sums its token's k values in slot order
  for (int i = tid; i < T * k; i += kThreads) {
    const int t = i / k, j = i - t * k;
    const float* prow = P + static_cast<size_t>(t) * Es;
    float denom = 0.f;
    for (int j0 = 0; j0 < k; j0 += kWBatch) {
      float v[kWBatch];
#pragma unroll
      for (int u = 0; u < kWBatch; ++u)
        if (j0 + u < k) v[u] = prow[sel[j0 + u]];
#pragma unroll
      for (int u = 0; u < kWBatch; ++u)
        if (j0 + u < k) denom += v[u];
    }
    cw[i] = prow[sel[j]] / denom;
  }
  if (kPerBlock) return;

  // 4. the closed-form schedule of one block
  dev::schedule_one_group(sel, T, k, reinterpret_cast<int*>(lds + L.sched), sched);
}

}  // namespace

// One workgroup per block when a block's rows fit in LDS and it is faster than
// separate softmax and block top-k launches, which spread the rows over the
// chip: its eight waves take the rows four at a time, so it pays by the row,
// and more for rows that are not 16-byte aligned (scalar loads), above all of
// several partial planes (bf16 routers; fp32 ones have one).  Routing of blocks
// over E experts (bf16, hidden 512 to 2048, top-8), us, one workgroup / separate:
//   aligned, E = 256: 2 x 32 15.9 / 18.2, 2 x 64 19.0 / 19.9, 64 x 64 25.7 / 30.6,
//     2 x 96 22.6 / 22.0; E = 192: 2 x 48 19.5 / 19.5, 24 x 64 26.0 / 27.2; E = 128:
//     2 x 32 17.3 / 17.9, 2 x 48 19.9 / 19.0, 8 x 128 31.3 / 25.2
//   not aligned, E = 219: 8 x 16 17.8 / 18.7, 8 x 24 20.8 / 19.7, 8 x 64 31.1 / 21.9
//   one block, where separate launches also schedule in one of their own:
//     E = 128: 48 17.1 / 18.6, 64 18.5 / 18.9, 96 23.1 / 21.1; not aligned, E = 101:
//     32 15.8 / 17.1, 64 21.5 / 19.0; E = 219: 32 19.1 / 18.6; E = 301: 16 17.7 /
//     20.9, 32 24.5 / 21.8
//   fp32 (hidden 256), aligned, E = 128: 8 x 48 21.1 / 21.4, 8 x 64 22.0 / 22.0, 8 x 96
//     29.1 / 27.8; not aligned, E = 161: 8 x 40 21.5 / 22.3, 2 x 64 21.6 / 21.2; E =
//     219: 8 x 64 27.2 / 26.6, one block of 64 19.1 / 20.8, of 96 23.4 / 23.1
static bool route_block_fits(dmoe_dtype dt, int G, int gs, int E, int k) {
  if (E > dev::kRegSoftmaxMaxE || k > dev::kMaxK) return false;
  if (fused_layout(gs, E, k).total * sizeof(float) > kMaxLdsBytes) return false;
  if (dt == DMOE_F32) return gs <= (E % 4 && G > 1 ? 40 : 64);
  if (E % 4) return gs * (E > 256 ? 2 : 1) <= (G == 1 ? 32 : 16);
  return gs <= (G == 1 || E >= 192 ? 64 : 32);
}

// Alg. 1 with the Top-P coreset: the router, every token's own top-k (with
// the softmax in one launch when the router's partial logits allow it), the
// coreset of each block, each token's top-k inside it, then the token-level
// schedule.
static hipError_t launch_route_topp(const RouteArgs& a, dmoe_dtype dt, hipStream_t s) {
  hipError_t err;
  bool own_done = false;
  if (softmax_token_topk_fits(a.E)) {
    float* part = nullptr;
    int S = 1;
    err = launch_router_partials(a.x, a.w, dt, a.T, a.H, a.E, a.probs, a.x_chunked, a.workspace, a.ws_bytes, s,
                                 &part, &S);
    if (err != hipSuccess) return err;
    err = launch_softmax_token_topk(part, S, a.bias, a.T, a.E, a.k, a.probs, a.logits, a.experts, a.combine_w,
                                    nullptr, s, true);  // the selected probabilities, for the coreset
    own_done = true;
  } else {
    err = launch_router(a.x, a.w, a.bias, dt, a.T, a.H, a.E, a.logits, a.probs, a.x_chunked, a.workspace,
                        a.ws_bytes, s);
  }
  if (err != hipSuccess) return err;
  err = launch_block_topp(a.probs, a.T / a.gs, a.gs, a.E, a.k, a.top_p, a.min_coreset, a.block_scores, a.coreset,
                          a.coreset_size, a.experts, a.combine_w, a.gap, s, own_done);
  if (err != hipSuccess) return err;
  return launch_schedule(a.experts, a.T, 1, a.k, a.E, a.sched, s);
}

hipError_t launch_route(const RouteArgs& a, dmoe_dtype dt, hipStream_t s) {
  if (a.topp) return launch_route_topp(a, dt, s);
  const int G = a.block ? a.T / a.gs : a.T;
  if (a.block && route_block_fits(dt, G, a.gs, a.E, a.k)) {
    float* part = nullptr;
    int S = 1;
    hipError_t err = launch_router_partials(a.x, a.w, dt, a.T, a.H, a.E, a.probs, a.x_chunked, a.workspace,
                                            a.ws_bytes, s, &part, &S);
    if (err != hipSuccess) return err;
    const size_t lds = fused_layout(a.gs, a.E, a.k).total * sizeof(float);
#define DMOE_ROUTE_BLOCK(NQ_, PER_)                                                                               \
  route_small_kernel<NQ_, PER_><<<G, kThreads, lds, s>>>(part, S, a.bias, a.gs, a.E, a.k, a.probs, a.logits,      \
                                                         a.block_scores, a.experts, a.combine_w, a.gap, a.sched, a.T)
    if (G == 1) {
      if (a.E <= 256)
        DMOE_ROUTE_BLOCK(1, false);
      else
        DMOE_ROUTE_BLOCK(2, false);
      return hipGetLastError();
    }
    if (a.E <= 256)
      DMOE_ROUTE_BLOCK(1, true);
    else
      DMOE_ROUTE_BLOCK(2, true);
#undef DMOE_ROUTE_BLOCK
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    return launch_schedule(a.experts, G, a.gs, a.k, a.E, a.sched, s);
  }
  hipError_t err;
  if (!a.block && softmax_token_topk_fits(a.E)) {
    // token routing: the softmax and each token's selection in one launch
    float* part = nullptr;
    int S = 1;
    err = launch_router_partials(a.x, a.w, dt, a.T, a.H, a.E, a.probs, a.x_chunked, a.workspace, a.ws_bytes, s,
                                 &part, &S);
    if (err != hipSuccess) return err;
    err = launch_softmax_token_topk(part, S, a.bias, a.T, a.E, a.k, a.probs, a.logits, a.experts, a.combine_w,
                                    a.gap, s);
    if (err != hipSuccess) return err;
    return launch_schedule(a.experts, G, 1, a.k, a.E, a.sched, s);
  }
  err = launch_router(a.x, a.w, a.bias, dt, a.T, a.H, a.E, a.logits, a.probs, a.x_chunked, a.workspace,
                      a.ws_bytes, s);
  if (err != hipSuccess) return err;
  if (a.block)
    err = launch_block_topk(a.probs, G, a.gs, a.E, a.k, a.block_scores, a.experts, a.combine_w, a.gap, s);
  else
    err = launch_token_topk(a.probs, a.T, a.E, a.k, a.experts, a.combine_w, a.gap, s);
  if (err != hipSuccess) return err;
  return launch_schedule(a.experts, G, a.block ? a.gs : 1, a.k, a.E, a.sched, s);
}

}  // namespace dmoe
