// Expert execution: the SwiGLU FFN of every unique expert of the forward over
// the rows that selected it, plus the always-on shared expert over all tokens.
//
//   h    = silu(Wg x) * (Wu x)        gate/up kernel -> h rows (workspace)
//   out  = Wd h                       down kernel    -> slot_out[t][j] / shared_out[t]
//
// Work items: max_work grid rows for the schedule's work items (up to
// DMOE_WORK_ROWS rows of one routed expert; rows past n_work exit at once)
// and rows for the shared expert's T tokens cut into pieces of
// DMOE_WORK_ROWS.  One-tile launches (schedules of many small items, whose
// max_work bound is loose) put the shared pieces first so that the rows that
// exit at once are dispatched last; the others put them last (measured
// faster for block-routed decode steps).  A decode workgroup owns one or two
// 16-row weight tiles of one item, streams them from HBM and applies them to
// the item's rows (tokens); a tile workgroup owns 64 or 128 weight rows and
// up to 128 tokens.  Each selected expert's weights are read from memory once per forward
// per piece of its rows.
//
// bf16 path (matrix cores, v_mfma_f32_16x16x32_bf16, fp32 accumulation):
//  * A operand = weight rows, B operand = token rows, C = [weight row][token].
//  * A gate/up tile interleaves the gate and up rows of 8 intermediate units,
//    so a lane's four accumulators are (g_i, g_i+1, u_i, u_i+1) of one token
//    and SwiGLU is applied in registers.
//  * Tiles of 16 weight rows give many small workgroups: a burst of weight
//    reads spread over several workgroups per CU keeps every HBM channel busy
//    and the CUs evenly loaded (32-row tiles left a third of the bandwidth
//    unused on small forwards).
//  * The four waves of a workgroup split the reduction dimension in quarters.
//    Each wave issues all of its weight loads at once (one burst per up to
//    KMAX 32-wide K steps), with the token operand double-buffered in chunks
//    behind it; partial tiles are summed in wave order through LDS, so
//    results do not depend on scheduling.
//  * Operand layouts are chosen so that consecutive lanes read consecutive
//    memory: weights are pre-packed in fragment order (a wave's load of one
//    16 x 32 tile is 1 KiB contiguous, its burst a contiguous run), and token
//    rows (x, and the h rows between the two kernels) are chunk-major
//    [K/8][rows][8], so 16 consecutive rows read 256 contiguous bytes per
//    8-element chunk.  Lane (q, c) of a K-step holds chunk 4*step + q of its
//    row in both operands, which is all the matrix instruction needs.
//    Scattered token rows (token-level routing) may instead be read from the
//    row-major x, one 64-byte piece per token and K-step (tile_gathered).
// fp32 layers: ffn_f32.hip.
#include <algorithm>
#include <type_traits>

#include "dmoe_common.h"
#include "ffn_dev.h"

namespace dmoe {
namespace {

constexpr int kThreads = 256;

using fdev::decode_item;
using fdev::Group;
// ---- bf16 kernels ----------------------------------------------------------

// Which copy of x serves a token tile's B loads better.  Lane (q, c) of
// each 16-lane row holds the token of column c (ascending within an item).
// Per K-step the chunk-major copy touches 4 * D8 cache lines (D8: distinct
// groups of 8 consecutive tokens among the 16; one group per line and chunk),
// the row-major copy D lines (D: distinct tokens, one 64-byte piece each).
// Tiles of fewer than 4 distinct tokens stay chunk-major (measured slightly
// faster there: 32-token decode steps under token routing).  Wave-uniform.
__device__ __forceinline__ bool tile_gathered(int tok) {
  // token of lane c - 1 in the same row (lane c = 0 sees its own)
  const int prev = __builtin_amdgcn_update_dpp(tok, tok, 0x111, 0xF, 0xF, false);  // row_shr:1
  const uint32_t new_tok = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(tok != prev)) & 0xFFFFu;
  const uint32_t new_grp = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64((tok >> 3) != (prev >> 3))) & 0xFFFFu;
  const int d = 1 + __builtin_popcount(new_tok), d8 = 1 + __builtin_popcount(new_grp);
  return d >= 4 && d < 4 * d8;
}

struct FfnParams {
  const bf16_t* xk;    // activations, chunk-major [H/8][T][8]
  const bf16_t* xr;    // the same row-major [T][H] (gathered rows read it), or nullptr
  const bf16_t* w13;   // routed gate/up, fragment-packed
  const bf16_t* w2;    // routed down, fragment-packed
  const bf16_t* ws13;  // shared gate/up, fragment-packed
  const bf16_t* ws2;   // shared down, fragment-packed
  const int* n_work;
  const int* work;
  const int* row_token;
  const int* row_slot;
  int T, H, E, I, I_s, k, Tk, R, max_work;  // R: rows of the h buffer
  int shared_items;                        // grid rows of the shared expert's pieces (0: none)
  bf16_t* hk;                              // SwiGLU activations, chunk-major [ldh/8][R][8]
  void* slot_out;                          // [T][k][H], float32 or scaled half (slot_f16s)
  float* shared_out;
  int slot_f16s;
  int adjacent;  // passes of an item: grid dimension y, the items z (else the other way round)
};

// Four consecutive outputs j0 .. j0+3 of schedule row r (token row_token[r],
// slot row_slot[r]) into the slot outputs, float32 or scaled half with the
// exponent e of their 16-feature group (written by the group's lane j0 % 16
// == 0).
__device__ __forceinline__ void store_slot(const FfnParams& p, int r, int j0, const f32x4& v, int e) {
  const size_t row = static_cast<size_t>(p.row_token[r]) * p.k + p.row_slot[r];
  if (p.slot_f16s) {
    uint16_t* hv = static_cast<uint16_t*>(p.slot_out);
    *reinterpret_cast<uint2*>(hv + row * p.H + j0) = f16s_encode(v, e);
    if ((j0 & 15) == 0) {
      int8_t* ev = reinterpret_cast<int8_t*>(hv + static_cast<size_t>(p.T) * p.k * p.H);
      ev[row * (p.H >> 4) + (j0 >> 4)] = static_cast<int8_t>(e);
    }
  } else {
    *reinterpret_cast<f32x4*>(static_cast<float*>(p.slot_out) + row * p.H + j0) = v;
  }
}

// The shared exponent of the 16-feature group a lane's outputs belong to
// (scaled-half slot outputs only; 0 otherwise).  All 64 lanes call it.
__device__ __forceinline__ int slot_exponent(const FfnParams& p, const f32x4& v) {
  return p.slot_f16s ? f16s_exponent(f16s_group_max(v)) : 0;
}

using namespace fdev;  // the wave-level operand helpers of ffn_dev.h

// One gate/up workgroup's rows [pz, pend) of the item: packed tiles it ..
// it + RT - 1 over them.  Wave w reduces over hidden chunks
// [w*H/32, (w+1)*H/32) (K-steps [w*H/128, (w+1)*H/128)).
template <bool kStream, int NT, int KMAX, int BC, int RT>
__device__ __forceinline__ void gateup_rows(const FfnParams& p, const Group& g, int it, int pz, int pend,
                                            f32x4 (*red)[RT][NT][kWave]) {
  const int H = p.H;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int q = lane >> 4, c = lane & 15;
  const int ksteps = H >> 5, steps = ksteps >> 2;
  const bf16_t* W = g.expert >= 0 ? p.w13 + static_cast<size_t>(g.expert) * 2 * p.I * H : p.ws13;
  const bf16_t* pa = W + (static_cast<size_t>(it) * ksteps + wave * steps) * kFrag + lane * 8;
  const size_t tstride = static_cast<size_t>(ksteps) * kFrag;  // next packed tile
  const int bstep = 32 * p.T;  // 4 chunks of T tokens per K-step
  const int chunk0 = wave * steps * 4 + q;
  WaveOps<NT, KMAX, BC, RT> w;  // a one-burst weight slice stays here across passes
  // At two token tiles (items of whole blocks) a one-burst slice is loaded
  // before the token rows are known: the weights wait only for the work
  // item, not for its row list and then x.  With one token tile (many small
  // items) the token fragments going first measured faster.
  bool a_held = false;
  if constexpr (NT == 2) {
    if (steps <= KMAX) {
      issue_a<kStream>(w, pa, tstride, steps);
      a_held = true;
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  for (int p0 = pz; p0 < pend; p0 += 16 * NT) {
    const bf16_t* pb[NT];
    int tok[NT];
    bool gathered = false;
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
      const int col = min(p0 + ct * 16 + c, g.n - 1);
      tok[ct] = g.tok ? g.tok[col] : g.t0 + col;
      if (p.xr && g.tok) gathered |= tile_gathered(tok[ct]);
    }
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
      pb[ct] = gathered ? p.xr + static_cast<size_t>(tok[ct]) * H + chunk0 * 8
                        : p.xk + (static_cast<size_t>(chunk0) * p.T + tok[ct]) * 8;
    f32x4 acc[RT][NT];
    zero(acc);
    wave_dot<kStream>(w, pa, tstride, pb, gathered ? 32 : bstep, steps, acc, a_held || (p0 > pz && steps <= KMAX));
    reduce_waves(acc, red, wave, lane);
    if (wave == 0) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
          const int col = p0 + ct * 16 + c;
          if (col < g.n) {
            // accumulators: (g_i, g_i+1, u_i, u_i+1) with i = 8*(it + r) + 2q
            const f32x4 v = acc[r][ct];
            const uint32_t h0 = f32_to_bf16(silu_f32(v[0]) * v[2]);
            const uint32_t h1 = f32_to_bf16(silu_f32(v[1]) * v[3]);
            bf16_t* dst = p.hk + (static_cast<size_t>(it + r) * p.R + g.r0 + col) * 8 + 2 * q;
            *reinterpret_cast<uint32_t*>(dst) = h0 | (h1 << 16);
          }
        }
    }
    __syncthreads();  // red is reused by the next pass
  }
}

// A workgroup takes all passes of its item, over weights that one burst keeps
// in registers, or (kSplit: two and four token tiles) one pass of 16*NT rows:
// these launches are small, and the passes of an item of many rows, the
// shared expert's above all, were their long pole (five blocks of 24 tokens
// over 48 experts 50.6 -> 47.8 us per layer).  The passes' workgroups load an
// item's weights plainly when there are several, so that the later ones find
// them in a cache.  They come one grid layer after the other, or (adjacent)
// one after the other for each item, tiles a multiple of 8, so that the
// passes of a tile meet in one XCD's L2: launch_decode's callers choose.
// (Both load types in one body spilled: 128 B a lane, two blocks of 32 tokens
// 61.8 us against 52.6.)
// Packed gate/up tile `it` = 8 intermediate units.
template <int NT, int KMAX, int BC, int MINW, bool kSharedFirst, int RT, bool kSplit>
__global__ __launch_bounds__(kThreads, MINW) void ffn_gateup_bf16_kernel(FfnParams p) {
  Group g;
  if (!decode_item<kSharedFirst>(kSplit && p.adjacent ? blockIdx.z : blockIdx.y, p.shared_items, p.max_work, p.n_work, p.work, p.row_token, p.T,
                                 p.Tk, p.E, g))
    return;
  const int Iw = g.expert >= 0 ? p.I : p.I_s;
  const int it = blockIdx.x * RT;  // first of the RT packed tiles (Iw / 8 is a multiple of 16)
  if (it * 8 >= Iw) return;
  __shared__ f32x4 red[3][RT][NT][kWave];
  if constexpr (!kSplit) {
    gateup_rows<true, NT, KMAX, BC, RT>(p, g, it, 0, g.n, red);
  } else {
    const int pz = (p.adjacent ? blockIdx.y : blockIdx.z) * 16 * NT;
    if (pz >= g.n) return;
    if (g.n > 16 * NT)
      gateup_rows<false, NT, KMAX, BC, RT>(p, g, it, pz, min(g.n, pz + 16 * NT), red);
    else
      gateup_rows<true, NT, KMAX, BC, RT>(p, g, it, 0, g.n, red);
  }
}

// The same for the down projection: packed tiles jt .. jt + RT - 1, tile `jt`
// = 16 output features.
template <bool kStream, int NT, int KMAX, int BC, int RT>
__device__ __forceinline__ void down_rows(const FfnParams& p, const Group& g, int jt, int pz, int pend,
                                          f32x4 (*red)[RT][NT][kWave]) {
  const int Kd = g.expert >= 0 ? p.I : p.I_s;
  const int H = p.H;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int q = lane >> 4, c = lane & 15;
  const int ksteps = Kd >> 5, steps = ksteps >> 2;
  const bf16_t* W = g.expert >= 0 ? p.w2 + static_cast<size_t>(g.expert) * H * p.I : p.ws2;
  const bf16_t* pa = W + (static_cast<size_t>(jt) * ksteps + wave * steps) * kFrag + lane * 8;
  const size_t tstride = static_cast<size_t>(ksteps) * kFrag;  // next packed tile
  const int bstep = 32 * p.R;
  const int chunk0 = wave * steps * 4 + q;

  WaveOps<NT, KMAX, BC, RT> w;  // a one-burst weight slice stays here across passes
  for (int p0 = pz; p0 < pend; p0 += 16 * NT) {
    const bf16_t* pb[NT];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
      const int col = min(p0 + ct * 16 + c, g.n - 1);
      pb[ct] = p.hk + (static_cast<size_t>(chunk0) * p.R + g.r0 + col) * 8;
    }
    f32x4 acc[RT][NT];
    zero(acc);
    wave_dot<kStream>(w, pa, tstride, pb, bstep, steps, acc, p0 > pz && steps <= KMAX);
    reduce_waves(acc, red, wave, lane);
    if (wave == 0) {
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) {
        const int col = p0 + ct * 16 + c;
        int ex[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) ex[r] = g.tok ? slot_exponent(p, acc[r][ct]) : 0;  // whole wave
        if (col < g.n) {
          if (g.tok) {
#pragma unroll
            for (int r = 0; r < RT; ++r) store_slot(p, g.r0 + col, (jt + r) * 16 + 4 * q, acc[r][ct], ex[r]);
          } else {
            float* dst = p.shared_out + static_cast<size_t>(g.t0 + col) * H;
#pragma unroll
            for (int r = 0; r < RT; ++r) *reinterpret_cast<f32x4*>(dst + (jt + r) * 16 + 4 * q) = acc[r][ct];
          }
        }
      }
    }
    __syncthreads();
  }
}

template <int NT, int KMAX, int BC, int MINW, bool kSharedFirst, int RT, bool kSplit>
__global__ __launch_bounds__(kThreads, MINW) void ffn_down_bf16_kernel(FfnParams p) {
  Group g;
  if (!decode_item<kSharedFirst>(kSplit && p.adjacent ? blockIdx.z : blockIdx.y, p.shared_items, p.max_work, p.n_work, p.work, p.row_token, p.T,
                                 p.Tk, p.E, g))
    return;
  const int jt = blockIdx.x * RT;  // first of the RT packed tiles (H / 16 is a multiple of 8)
  if (jt * 16 >= p.H) return;
  __shared__ f32x4 red[3][RT][NT][kWave];
  if constexpr (!kSplit) {
    down_rows<true, NT, KMAX, BC, RT>(p, g, jt, 0, g.n, red);
  } else {
    const int pz = (p.adjacent ? blockIdx.y : blockIdx.z) * 16 * NT;
    if (pz >= g.n) return;
    if (g.n > 16 * NT)
      down_rows<false, NT, KMAX, BC, RT>(p, g, jt, pz, min(g.n, pz + 16 * NT), red);
    else
      down_rows<true, NT, KMAX, BC, RT>(p, g, jt, 0, g.n, red);
  }
}

// Workgroups are dispatched to the 8 XCDs round-robin by linear id, and each
// XCD has its own L2.  The 1-D grid of gx * items8 workgroups (gx row blocks
// per item, items8: the grid rows rounded up to a multiple of 8) is mapped
// onto the schedule's live items (the first n_work, then the shared
// expert's) so that each item's row blocks run on S XCDs: its token rows
// enter S L2 caches.  Schedules of many live items (>= 256: thousands of
// tokens, whose token rows per XCD copy cost about as much traffic as the
// weights) take S = 1; the others S = 8 (every XCD shares every item's
// work, the most even load; measured faster for 16 blocks of 32 tokens and
// for the Zipf-biased large layer).  With S = 1, XCD x runs a contiguous
// run of ceil(live / 8) items, one item (all its row blocks) after the
// other: the items of one expert are adjacent in the schedule, so its pieces
// run back to back on one XCD and share that L2's copy of its weights.  With
// S > 1, XCD x of group x / S runs row blocks x % S, x % S + S, ... of the
// group's items (an expert's pieces again meet on the XCDs of each row
// block).
__device__ __forceinline__ bool map_item(const FfnParams& p, int gx, int& item, int& rb) {
  const int nw = min(*p.n_work, p.max_work);
  const int live = nw + p.shared_items;
  const int S = min(live >= 256 ? 1 : 8, gx & -gx);  // a power of two dividing gx
  const int x = blockIdx.x & 7, slot = blockIdx.x >> 3;
  int j;
  if (S == 1) {
    const int q = (live + 7) >> 3, i = slot / gx;  // q items per XCD
    rb = slot % gx;
    if (i >= q) return false;
    j = x * q + i;
  } else {
    const int per = gx / S;  // row blocks of an item on each of its XCDs
    j = (slot / per) * (8 / S) + x / S;
    rb = x % S + S * (slot % per);
  }
  if (j >= live) return false;
  item = j < nw ? j : p.max_work + (j - nw);
  return true;
}

// ---- tile kernels: many tokens per work item --------------------------------
//
// A workgroup of kWaves waves covers kWaves * kRowTiles 16-row weight tiles
// (wave w: packed tiles kRowTiles * (kWaves*bx + w) + m, m < kRowTiles, over the whole
// reduction) x up to 128 tokens of one work item (8 token tiles).  The
// reduction runs in stages of kSteps K-steps.  A stage's token fragments go
// from global memory straight into LDS (no registers), two stages ahead into a ring of
// three stage buffers that all waves read, each fragment read once per wave
// and applied to the wave's kRowTiles weight tiles; each wave streams its own
// weight tiles into registers, two stages ahead as well.  One wait count and
// one barrier end a stage: everything but the loads issued in this stage has
// arrived.  Accumulation order (K ascending) and the epilogues match the
// decode kernels.
//
// What bounds it: what a CU can have in flight to L2 and HBM.  Counters at 64
// blocks of 64 tokens (hidden 2048, 256 experts of intermediate 512; wide
// gate/up 226 us, down 147): 27 and 21 % of the dense bf16 peak, 1.18 and 0.55 GB
// read from the fabric (5.2 and 3.8 TB/s), waves waiting for loads or barriers
// 48 and 50 % of their cycles, for an issue slot 41 and 36 %; reading the
// LDS fragments one, two or three tiles ahead measured the same.  Token
// fragments two stages ahead without registers, instead of one stage ahead
// through registers: that layer 508 -> 490 us, 16 x 32 tokens 173 -> 164,
// the Zipf-biased hidden-4096 layer 188 -> 182.  Scaled-half outputs stored
// as whole rows (below): 490 -> 441, 164 -> 159, 182 -> 173.
constexpr int kTileTok = 8;       // token tiles per workgroup (128 tokens)
static_assert(kTileTok * 16 == DMOE_WORK_ROWS, "a tile workgroup covers one work item's rows");

// One stage's token fragments, each in the lane order of the matrix operand.
template <int kSteps>
using TokStage = bf16x8[kSteps][kTileTok][kWave];  // 8 KiB per step

// LDS of a tile workgroup.  The three stage buffers are separate arrays so
// that the compiler can tell the one being read from those being loaded: it
// would otherwise wait for every load into LDS before each fragment read.
template <int kWaves, int kSteps>
struct TileLds {
  TokStage<kSteps>&s0, &s1, &s2;
  int* dst;     // [DMOE_WORK_ROWS] slot row of each row of the item (down projection)
  int8_t* exps; // [DMOE_WORK_ROWS][2 * kWaves] exponents of the output tiles
};

// Wait until at most N vector-memory operations of this wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// 16 bytes per lane from global memory straight into LDS at dst + 16*lane
// (dst uniform over the wave).
__device__ __forceinline__ void dma16(const bf16_t* src, bf16x8* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

// The workgroup's work once its item is known (kStream: weights loaded
// non-temporally; kCt: token tiles the code covers, at least the item's).
template <bool kGateUp, int kRowTiles, int kWaves, int kSteps, bool kStream, int kCt>
__device__ __forceinline__ void tile_body(const FfnParams& p, const Group& g, int bx,
                                          const TileLds<kWaves, kSteps>& lds) {
  constexpr int kTileRows = kWaves * kRowTiles;  // weight tiles per workgroup
  // token fragments of a stage (tile, K-step) a wave loads
  constexpr int kFrags = kSteps * kCt, kFragWave = (kFrags + kWaves - 1) / kWaves;
  using Stage = TokStage<kSteps>;
  const int H = p.H;
  const int Iw = g.expert >= 0 ? p.I : p.I_s;
  const int Kd = kGateUp ? H : Iw;                    // reduction length
  const int tiles = kGateUp ? Iw / 8 : H / 16;        // packed 16-row tiles of the matrix (a multiple of 8)
  if (bx * kTileRows >= tiles) return;  // uniform: past the matrix
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int uw = __builtin_amdgcn_readfirstlane(wave);
  // a wave past the matrix repeats the last tiles and stores nothing
  const bool wave_live = (bx * kWaves + uw) * kRowTiles < tiles;
  const int tile0 = min((bx * kWaves + wave) * kRowTiles, tiles - kRowTiles);
  const int ksteps = Kd >> 5;                         // multiple of 4
  const bf16_t* W;
  if (kGateUp)
    W = g.expert >= 0 ? p.w13 + static_cast<size_t>(g.expert) * 2 * p.I * H : p.ws13;
  else
    W = g.expert >= 0 ? p.w2 + static_cast<size_t>(g.expert) * H * p.I : p.ws2;
  const bf16_t* pa = W + static_cast<size_t>(tile0) * ksteps * kFrag + lane * 8;
  const size_t tstride = static_cast<size_t>(ksteps) * kFrag;  // next packed tile

  // Token-fragment producer: fragment f = step * kCt + tile of a stage is
  // loaded by wave f % kWaves.  Tiles past the item's last token load its
  // last row again (straight-line code; those fragments are never stored).
  const int q = lane >> 4, c = lane & 15;
  const int rows_b = kGateUp ? p.T : p.R;  // rows of the chunk-major source
  const bf16_t* src = kGateUp ? p.xk : p.hk;
  const bf16_t* pb[kFragWave];
  int row[kFragWave];
  bool gathered = false;
#pragma unroll
  for (int i = 0; i < kFragWave; ++i) {
    const int col = min((uw + kWaves * i) % kCt * 16 + c, g.n - 1);
    if (kGateUp) {
      row[i] = g.tok ? g.tok[col] : g.t0 + col;
      if (p.xr && g.tok) gathered |= tile_gathered(row[i]);
    } else {
      row[i] = g.r0 + col;
    }
  }
  const int bstep = gathered ? 32 : 32 * rows_b;
#pragma unroll
  for (int i = 0; i < kFragWave; ++i)
    pb[i] = (gathered ? p.xr + static_cast<size_t>(row[i]) * H + q * 8
                      : src + (static_cast<size_t>(q) * rows_b + row[i]) * 8) +
            (uw + kWaves * i) / kCt * bstep;
  if (!kGateUp && g.tok && static_cast<int>(threadIdx.x) < g.n)  // read in the epilogue
    lds.dst[threadIdx.x] = p.row_token[g.r0 + threadIdx.x] * p.k + p.row_slot[g.r0 + threadIdx.x];

  f32x4 acc[kRowTiles][kCt];
#pragma unroll
  for (int m = 0; m < kRowTiles; ++m)
#pragma unroll
    for (int ct = 0; ct < kCt; ++ct) acc[m][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 a_reg[3][kSteps][kRowTiles];
  const int nstages = ksteps / kSteps;  // at least two

  auto load_a = [&](int st, bf16x8 (&a)[kSteps][kRowTiles]) {
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
#pragma unroll
      for (int m = 0; m < kRowTiles; ++m)
        a[s][m] = kStream ? ld_bf16x8_stream(pa + m * tstride + (st * kSteps + s) * kFrag)
                          : ld_bf16x8(pa + m * tstride + (st * kSteps + s) * kFrag);
  };
  auto load_b = [&](int st, Stage& d) {
#pragma unroll
    for (int i = 0; i < kFragWave; ++i) {
      const int f = uw + kWaves * i;
      if (kFrags % kWaves == 0 || f < kFrags) dma16(pb[i] + st * kSteps * bstep, &d[f / kCt][f % kCt][0]);
    }
  };
  // Memory operations of one stage's loads.  (Where kWaves does not divide
  // kFrags, a wave loads one fragment of a stage or none; a wave without one
  // has nothing in LDS to wait for.)
  constexpr int kIssued = kFragWave + kSteps * kRowTiles;

  load_b(0, lds.s0);
  load_a(0, a_reg[0]);
  __builtin_amdgcn_sched_barrier(0);
  load_b(1, lds.s1);
  load_a(1, a_reg[1]);
  __builtin_amdgcn_sched_barrier(0);
  wait_vm<kIssued>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  // stage st uses ring slot and LDS buffer R = st % 3 (compile-time indexes:
  // three stages per trip).  The buffer it refills was last read in stage
  // st - 1, before the barrier that ended it.  A stage of the loop (kFull)
  // loads stage st + 2 and waits for all but those loads, whatever their
  // order: stage st + 1 has arrived.  The one or two stages after the loop
  // load nothing; the first waits for everything, the last for nothing.
  enum { kFull, kDrain, kLast };
  auto run_stage = [&](auto slot, auto kind, int st, Stage& cur, Stage& fill) {
    constexpr int R = decltype(slot)::value, kKind = decltype(kind)::value;
    if constexpr (kKind == kFull) {
      const int nx = min(st + 2, nstages - 1);  // past the end: the last stage again, never used
      load_b(nx, fill);
      load_a(nx, a_reg[(R + 2) % 3]);
    }
    __builtin_amdgcn_sched_barrier(0);
    // token tile by token tile: the next tile's fragments are read from LDS
    // while this tile's matrix instructions run
    bf16x8 b[2][kSteps];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) b[0][s] = cur[s][0][lane];
#pragma unroll
    for (int ct = 0; ct < kCt; ++ct) {
      if (ct + 1 < kCt) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s) b[(ct + 1) & 1][s] = cur[s][ct + 1][lane];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < kSteps; ++s)
#pragma unroll
        for (int m = 0; m < kRowTiles; ++m)
          acc[m][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_reg[R][s][m], b[ct & 1][s], acc[m][ct], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kKind == kLast) return;
    wait_vm<kKind == kFull ? kIssued : 0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::integral_constant<int, 0> r0;
  constexpr std::integral_constant<int, 1> r1;
  constexpr std::integral_constant<int, 2> r2;
  constexpr std::integral_constant<int, kFull> full;
  constexpr std::integral_constant<int, kDrain> drain;
  constexpr std::integral_constant<int, kLast> last;
  int st = 0;
  for (; st + 3 <= nstages; st += 3) {
    run_stage(r0, full, st, lds.s0, lds.s2);
    run_stage(r1, full, st + 1, lds.s1, lds.s0);
    run_stage(r2, full, st + 2, lds.s2, lds.s1);
  }
  if (st < nstages) run_stage(r0, drain, st, lds.s0, lds.s2);
  if (st + 1 < nstages) run_stage(r1, last, st + 1, lds.s1, lds.s0);
  wait_vm<0>();  // the loads into LDS end before the buffers are reused or the workgroup ends

  if constexpr (kGateUp) {
    if (!wave_live) return;
#pragma unroll
    for (int m = 0; m < kRowTiles; ++m)
#pragma unroll
      for (int ct = 0; ct < kCt; ++ct) {
        const int col = ct * 16 + c;
        if (col >= g.n) continue;
        // accumulators: (g_i, g_i+1, u_i, u_i+1) with i = 8*tile + 2q
        const f32x4 v = acc[m][ct];
        const uint32_t h0 = f32_to_bf16(silu_f32(v[0]) * v[2]);
        const uint32_t h1 = f32_to_bf16(silu_f32(v[1]) * v[3]);
        bf16_t* dst = p.hk + (static_cast<size_t>(tile0 + m) * p.R + g.r0 + col) * 8 + 2 * q;
        *reinterpret_cast<uint32_t*>(dst) = h0 | (h1 << 16);
      }
    return;
  }
  if (!g.tok) {
    if (!wave_live) return;
#pragma unroll
    for (int m = 0; m < kRowTiles; ++m)
#pragma unroll
      for (int ct = 0; ct < kCt; ++ct) {
        const int col = ct * 16 + c;
        if (col < g.n)
          *reinterpret_cast<f32x4*>(p.shared_out + static_cast<size_t>(g.t0 + col) * H + (tile0 + m) * 16 + 4 * q) =
              acc[m][ct];
      }
    return;
  }
  if (!p.slot_f16s) {
    __syncthreads();  // lds.dst
    if (!wave_live) return;
#pragma unroll
    for (int m = 0; m < kRowTiles; ++m)
#pragma unroll
      for (int ct = 0; ct < kCt; ++ct) {
        const int col = ct * 16 + c;
        if (col < g.n)
          *reinterpret_cast<f32x4*>(static_cast<float*>(p.slot_out) + static_cast<size_t>(lds.dst[col]) * H +
                                    (tile0 + m) * 16 + 4 * q) = acc[m][ct];
      }
    return;
  }
  // Scaled-half slot outputs go through LDS: a lane holds eight bytes of a
  // row, and storing those directly makes four 32-byte write requests per
  // row and tile pair where whole rows of the workgroup's features make two
  // or four of 128 bytes (they were almost half of the kernel's L2 requests).
  // A token tile is 16 rows of kRowBytes; 16-byte unit u of row c sits at u ^ c (no bank
  // conflicts either way).  Rounds of kRound token tiles, as many as the
  // three stage buffers hold.
  constexpr int kRowBytes = kTileRows * 32;
  constexpr int kPerBuf = static_cast<int>(sizeof(Stage)) / (16 * kRowBytes), kRound = 3 * kPerBuf;
  static_assert(kPerBuf >= 1, "a stage buffer holds a token tile's outputs");
  uint16_t* hv = static_cast<uint16_t*>(p.slot_out);
  int8_t* ev = reinterpret_cast<int8_t*>(hv + static_cast<size_t>(p.T) * p.k * H);
  constexpr int kUnits = kRowBytes / 16;                    // 16-byte units of a row
  constexpr int kRowsPass = kWaves * kWave / kUnits;        // rows the workgroup stores together
  const int units = min(kUnits, (tiles - bx * kTileRows) * 2);  // units of this workgroup's live tiles
#pragma unroll
  for (int c0 = 0; c0 < kCt; c0 += kRound) {
    __syncthreads();  // the last stage (or round) has been read
#pragma unroll
    for (int ct = c0; ct < kCt && ct < c0 + kRound; ++ct) {
      Stage& buf = (ct - c0) / kPerBuf == 0 ? lds.s0 : (ct - c0) / kPerBuf == 1 ? lds.s1 : lds.s2;
      char* base = reinterpret_cast<char*>(&buf) + (ct - c0) % kPerBuf * 16 * kRowBytes;
#pragma unroll
      for (int m = 0; m < kRowTiles; ++m) {
        const int e = slot_exponent(p, acc[m][ct]);  // whole wave
        const int u = (wave * kRowTiles + m) * 2 + (q >> 1);
        *reinterpret_cast<uint2*>(base + c * kRowBytes + ((u ^ c) * 16 + (q & 1) * 8)) = f16s_encode(acc[m][ct], e);
        if (q == 0) lds.exps[(ct * 16 + c) * kTileRows + wave * kRowTiles + m] = static_cast<int8_t>(e);
      }
    }
    __syncthreads();
#pragma unroll
    for (int ct = c0; ct < kCt && ct < c0 + kRound; ++ct) {
      Stage& buf = (ct - c0) / kPerBuf == 0 ? lds.s0 : (ct - c0) / kPerBuf == 1 ? lds.s1 : lds.s2;
      const char* base = reinterpret_cast<const char*>(&buf) + (ct - c0) % kPerBuf * 16 * kRowBytes;
#pragma unroll
      for (int r0 = 0; r0 < 16; r0 += kRowsPass) {
        const int r = r0 + static_cast<int>(threadIdx.x) / kUnits, u = threadIdx.x % kUnits;
        const int col = ct * 16 + r;
        if (r < 16 && col < g.n && u < units)
          *reinterpret_cast<uint4*>(hv + static_cast<size_t>(lds.dst[col]) * H + bx * kTileRows * 16 + u * 8) =
              *reinterpret_cast<const uint4*>(base + r * kRowBytes + (u ^ r) * 16);
      }
    }
  }
  if (static_cast<int>(threadIdx.x) < g.n) {  // 8 or 16 exponents of the row
    const size_t d = static_cast<size_t>(lds.dst[threadIdx.x]) * (H >> 4) + bx * kTileRows;
    const uint2* es = reinterpret_cast<const uint2*>(lds.exps + threadIdx.x * kTileRows);
#pragma unroll
    for (int i = 0; i < kTileRows / 8; ++i)
      if (i * 16 < units) reinterpret_cast<uint2*>(ev + d)[i] = es[i];
  }
}

// The code of the smallest even number of token tiles that holds the item.
template <bool kGateUp, int kRowTiles, int kWaves, int kSteps, bool kStream>
__device__ __forceinline__ void tile_tokens(const FfnParams& p, const Group& g, int bx,
                                            const TileLds<kWaves, kSteps>& lds) {
  if (g.n > 96)
    tile_body<kGateUp, kRowTiles, kWaves, kSteps, kStream, 8>(p, g, bx, lds);
  else if (g.n > 64)
    tile_body<kGateUp, kRowTiles, kWaves, kSteps, kStream, 6>(p, g, bx, lds);
  else if (g.n > 32)
    tile_body<kGateUp, kRowTiles, kWaves, kSteps, kStream, 4>(p, g, bx, lds);
  else
    tile_body<kGateUp, kRowTiles, kWaves, kSteps, kStream, 2>(p, g, bx, lds);
}

template <bool kGateUp, int kRowTiles, int kWaves, int kSteps, int kMinWaves>
__global__ __launch_bounds__(kWaves * kWave, kMinWaves) void ffn_tile_bf16_kernel(FfnParams p, int gx) {
  int item, bx;
  if (!map_item(p, gx, item, bx)) return;
  Group g;
  if (!decode_item(item, p.shared_items, p.max_work, p.n_work, p.work, p.row_token, p.T, p.Tk, p.E, g)) return;
  __shared__ TokStage<kSteps> s0, s1, s2;
  __shared__ int dst[kGateUp ? 1 : DMOE_WORK_ROWS];
  __shared__ __align__(16) int8_t exps[kGateUp ? 16 : DMOE_WORK_ROWS * kWaves * kRowTiles];
  const TileLds<kWaves, kSteps> lds{s0, s1, s2, dst, exps};
  // An expert whose rows are one item is the only reader of its weights in
  // the launch (each row block reads its own rows once): they are streamed
  // non-temporally, which measured faster.  The items of an expert with more
  // rows read the same weights one after the other, through the L2 of the
  // XCD they share (non-temporal loads there measured slower).
  bool single;
  if (g.expert >= 0) {
    const int nw = min(*p.n_work, p.max_work);
    single = g.piece == 0 && !(item + 1 < nw && reinterpret_cast<const int4*>(p.work)[item + 1].x == g.expert);
  } else {
    single = p.T <= DMOE_WORK_ROWS;
  }
  if (single)
    tile_tokens<kGateUp, kRowTiles, kWaves, kSteps, true>(p, g, bx, lds);
  else
    tile_tokens<kGateUp, kRowTiles, kWaves, kSteps, false>(p, g, bx, lds);
}

// ---- launch ---------------------------------------------------------------

// Token columns per pass: enough 16-wide tiles for the expected rows of a
// work item (the rows of the forward spread over max_work items, at most
// DMOE_WORK_ROWS), at most 4.
// rows per item of the launch: the routed rows spread over max_work items, or
// (max_work == 0, the shared expert alone) its pieces of up to DMOE_WORK_ROWS.
long rows_per_item(int T, int k, int max_work) {
  if (max_work == 0) return std::min<long>(DMOE_WORK_ROWS, T);
  return std::min<long>(DMOE_WORK_ROWS, (static_cast<long>(T) * k + max_work - 1) / max_work);
}

int pick_ntiles(int T, int k, int max_work) {
  const long rows = rows_per_item(T, k, max_work);
  return rows <= 16 ? 1 : (rows <= 32 ? 2 : 4);
}

// Launch shapes per token-tile count NT: weight burst KMAX steps, token
// chunks of BC steps, occupancy floor MINW (waves per SIMD), weight tiles
// per wave (kGuRows / kDnRows: each token fragment feeds that many matrix
// instructions), and the order of the grid rows (kSharedFirst, see the top
// of the file).  The one-tile variants serve token-level schedules, items of
// a few rows over many experts: two weight tiles per wave in both kernels
// halve the token-fragment reads from L2 per weight byte (measured 12 %
// faster at 512 tokens over 256 experts, equal at 32 tokens).  The two-tile
// variants serve block-routed decode steps, whose launches are small enough
// that a higher floor keeps every workgroup resident at once; their down
// kernel applies each h fragment to two weight tiles (half the h reads from
// L2; measured 0.4 us faster per step than one tile, while two gate/up tiles
// per wave measured 1.2 us slower).
// Burst lengths set the registers and so the resident workgroups, which set
// how much is in flight for workgroups of tens of KB: the one-tile down
// kernel at bursts of four K-steps (intermediate 512 in one) holds five per
// CU where eight-step bursts held three (32 tokens of the decode layer, token
// routing 186 -> 179 us per layer, Top-P 106 -> 102; forced to six per CU
// 201).  Slices of five to eight steps keep the eight-step burst: only a
// one-burst slice stays in registers across the 16-row passes of an item,
// and an expert with many rows would read it once per pass (token routing of
// 192 tokens over 128 Zipf-biased experts of intermediate 1024: 204 us per
// layer, in two bursts of four 256; 64 tokens 126 against 140, intermediate
// 768 107 against 117; without the bias equal to 3 %).  The two-tile
// gate/up kernel at eight steps holds four (five blocks of 24 tokens over 48
// experts 47.2 -> 45.1, two blocks of 32 of the decode layer 56.5 -> 55.5).
// Other gate/up bursts at one token tile measured within 1.5 % (four and
// eight steps, one weight tile).
template <int NT>
struct Shape;
template <>
struct Shape<1> {
  static constexpr int kGuMax = 16, kGuChunk = 4, kGuWaves = 2, kDnMax = 4, kDnChunk = 4, kDnWaves = 4;
  static constexpr int kDnLong = 8, kDnLongWaves = 3;  // down slices longer than kDnMax
  static constexpr int kGuRows = 2, kDnRows = 2;
  static constexpr bool kSharedFirst = true;
};
template <>
struct Shape<2> {
  static constexpr int kGuMax = 8, kGuChunk = 4, kGuWaves = 4, kDnMax = 4, kDnChunk = 4, kDnWaves = 3;
  static constexpr int kGuLong = 16, kGuLongWaves = 3;  // a slice held across passes, or of one pass
  static constexpr int kGuRows = 1, kDnRows = 2;
  static constexpr bool kSharedFirst = false;
};
template <>
struct Shape<4> {
  static constexpr int kGuMax = 8, kGuChunk = 4, kGuWaves = 1, kDnMax = 8, kDnChunk = 4, kDnWaves = 1;
  static constexpr int kGuRows = 1, kDnRows = 1;
  static constexpr bool kSharedFirst = false;
};

// kSplit: a pass per workgroup.
template <int NT, bool kSplit, int kGuMax = Shape<NT>::kGuMax, int kGuWaves = Shape<NT>::kGuWaves,
          int kDnMax = Shape<NT>::kDnMax, int kDnWaves = Shape<NT>::kDnWaves>
hipError_t launch_decode(const FfnParams& p, int ldh, int groups, int passes, hipStream_t s) {
  using S = Shape<NT>;
  // tiles: a multiple of 8 (see the kernels), the down projection's rounded up
  const int gx_gu = ldh / (8 * S::kGuRows), gx_dn = (p.H / (16 * S::kDnRows) + 7) / 8 * 8;
  const int gy = p.adjacent ? passes : groups, gz = p.adjacent ? groups : passes;
  ffn_gateup_bf16_kernel<NT, kGuMax, S::kGuChunk, kGuWaves, S::kSharedFirst, S::kGuRows, kSplit>
      <<<dim3(gx_gu, gy, gz), kThreads, 0, s>>>(p);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  ffn_down_bf16_kernel<NT, kDnMax, S::kDnChunk, kDnWaves, S::kSharedFirst, S::kDnRows, kSplit>
      <<<dim3(gx_dn, gy, gz), kThreads, 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_one_tile(const FfnParams& p, int ldh, int items, hipStream_t s) {
  using S = Shape<1>;
  if (ldh / 128 > S::kDnMax)
    return launch_decode<1, false, S::kGuMax, S::kGuWaves, S::kDnLong, S::kDnLongWaves>(p, ldh, items, 1, s);
  return launch_decode<1, false>(p, ldh, items, 1, s);
}

// Two token tiles.  How the passes of an item run, us per layer, one
// workgroup for all / a grid layer per pass / adjacent:
//  * Adjacent where the weights stream long enough (hidden 1024 and up: slices
//    of a whole burst and more) for the later passes to miss the caches, and
//    some item is sure to have several (the shared expert) or the launch is
//    large: nine blocks of 32 under Top-P, hidden 3840, intermediate 1408, 521 /
//    540 / 462; six of 24 with a shared expert, hidden 4096, intermediate 1536,
//    432 / 383 / 346, hidden 1024, intermediate 1024, Zipf-biased, 91 / 80 / 72;
//    three of 32, hidden 2048, intermediate 512, Zipf-biased, 58.5 / 57.0 / 55.0.
//    Not with few tiles: dispatch is round-robin over the CUs, and the passes
//    without rows, a few workgroups each between those that have some, leave
//    CUs without work (intermediate 384, 48 tiles, 36 blocks of 16 tokens over
//    148 experts 367 / 354 / 377; intermediate 256, two of 32 52.0 / 51.8 / 57.2;
//    intermediate 128, ten of 10 43.2 / 43.3 / 47.7).
//  * One workgroup for all in launches of many items, most of whose passes
//    would have no rows, where holding the weights saves reads: slices that are
//    one burst at its length but two at the others' (hidden 1280, intermediate
//    384, 14 blocks of 40 under Top-P, 162 items 135 / 149 / 137; hidden 1536, 19
//    of 32, 194 items 112 / 122 / 124), and in large launches those of more than
//    half a short burst (hidden 1024, intermediate 384, 12 of 61, token routing,
//    308 items 133 / 144 / 149; hidden 768, 11 of 64 under Top-P, 267 items 156 /
//    160 / 165; at hidden 384, 34 of 32, 271 items, 374 / 353 / 366).
//  * A grid layer per pass otherwise (five blocks of 24 over 48, hidden 768,
//    intermediate 384: 45.5 / 38.8 / 39.1).
constexpr int kAdjacentHidden = 1024, kAdjacentTiles = 64;
constexpr long kLargeLaunch = 8192;  // gate/up workgroups of one pass
constexpr int kManyItems = 128;

hipError_t launch_two_tiles(FfnParams p, int ldh, int items, hipStream_t s) {
  using S = Shape<2>;
  const int passes = (std::min(p.T, DMOE_WORK_ROWS) + 31) / 32;
  const int gx = ldh / 8, steps = p.H / 128;
  // One pass over slices longer than the burst (one block of 32 tokens, hidden
  // 2048): the whole slice in one burst, issued before the row list, 20.3
  // against 20.7 us for the FFN (two such blocks, two passes: 56.5 against
  // 55.5 per layer).
  if (passes == 1 && steps > S::kGuMax)
    return launch_decode<2, true, S::kGuLong, S::kGuLongWaves>(p, ldh, items, 1, s);
  const bool large = static_cast<long>(gx) * items >= kLargeLaunch;
  p.adjacent = p.H >= kAdjacentHidden && gx >= kAdjacentTiles && (large || p.shared_items > 0);
  const bool hold = steps > S::kGuMax ? steps <= S::kGuLong : large && steps > S::kGuMax / 2;
  if (passes > 1 && !p.adjacent && items >= kManyItems && hold)
    return launch_decode<2, false, S::kGuLong, S::kGuLongWaves>(p, ldh, items, 1, s);
  return launch_decode<2, true>(p, ldh, items, passes, s);
}

hipError_t launch_four_tiles(const FfnParams& p, int ldh, int items, hipStream_t s) {
  return launch_decode<4, true>(p, ldh, items, (std::min(p.T, DMOE_WORK_ROWS) + 63) / 64, s);
}

// Tile kernels, one item per workgroup.  Two weight tiles per wave halve the
// LDS reads per weight byte; one tile per wave doubles the workgroups.  A
// gate/up grid of fewer than two rounds of the chip (three resident
// workgroups on each of 256 CUs) ends in a long partial round, which the
// finer split shortens.  The down projection always takes two tiles per wave:
// its reduction (I) is short, and at one tile per wave a workgroup reads
// twice as many token bytes as weight bytes.
//
// Wide workgroups (eight waves, 256 weight rows, one K-step per stage so that
// two of them fit a CU) read a quarter fewer bytes per flop than the four-wave
// ones, but leave fewer, longer workgroups to balance.  Whole layer, us,
// four waves -> wide, on layers of the decode shape (hidden 2048, 256 experts
// of intermediate 512, top-8): gate/up wide at 64 x 64 tokens 441 -> 431,
// 32 x 64 319 -> 302, 64 x 32 360 -> 345 (wide grids of 1088 workgroups and
// up, 43 rows per item and up); the Zipf-biased hidden-4096 layer of 8 x 32
// tokens 173 -> 196 (792 workgroups, 32 rows), 512 tokens under Top-P
// 298 -> 304 (15 rows).  Down wide as well: 64 x 64 431 -> 428 (4352
// workgroups), 32 x 64 302 -> 312 (2176), 64 x 32 345 -> 352 (3200).
constexpr long kTileRound = 3L * 256;
constexpr int kWideMinRows = 32;                             // rows per item
constexpr long kWideMinGateUp = 1024, kWideMinDown = 4096;  // workgroups of the wide grid

template <bool kGateUp>
hipError_t launch_tile_bf16(const FfnParams& p, int ldh, int items, long rows, hipStream_t s) {
  const int tiles = kGateUp ? ldh / 8 : p.H / 16;  // packed 16-row tiles
  const int items8 = (items + 7) / 8 * 8;
  if constexpr (kGateUp) {
    if (static_cast<long>(ldh / 64) * items < 2 * kTileRound) {
      ffn_tile_bf16_kernel<true, 1, 4, 2, 2><<<dim3(tiles / 4 * items8), 4 * kWave, 0, s>>>(p, tiles / 4);
      return hipGetLastError();
    }
  }
  const int wide = (tiles + 15) / 16;
  if (rows >= kWideMinRows && static_cast<long>(wide) * items >= (kGateUp ? kWideMinGateUp : kWideMinDown))
    ffn_tile_bf16_kernel<kGateUp, 2, 8, 1, 4><<<dim3(wide * items8), 8 * kWave, 0, s>>>(p, wide);
  else
    ffn_tile_bf16_kernel<kGateUp, 2, 4, 2, 2><<<dim3(tiles / 8 * items8), 4 * kWave, 0, s>>>(p, tiles / 8);
  return hipGetLastError();
}

hipError_t launch_tiles(const FfnParams& p, int ldh, int items, long rows, hipStream_t s) {
  const hipError_t err = launch_tile_bf16<true>(p, ldh, items, rows, s);
  if (err != hipSuccess) return err;
  return launch_tile_bf16<false>(p, ldh, items, rows, s);
}

constexpr int kPassRows = 16;    // token rows of one decode-kernel pass

bool use_tile_kernels(int T, int k, int max_work, int items, int ldh) {
  return rows_per_item(T, k, max_work) >= 32 && static_cast<long>(ldh / 32) * items >= 512;
}

}  // namespace

size_t ffn_workspace_bytes(int T, int I, int I_s, int k, dmoe_dtype dt) {
  const size_t rows = static_cast<size_t>(T) * k + (I_s > 0 ? T : 0);
  const size_t ldh = static_cast<size_t>(std::max(I, I_s));
  return rows * ldh * (dt == DMOE_F32 ? 4 : 2);
}

hipError_t launch_ffn(const FfnArgs& a, dmoe_dtype dt, hipStream_t s) {
  const int Tk = a.T * a.k;
  const int R = Tk + (a.I_s > 0 ? a.T : 0);
  const int ldh = std::max(a.I, a.I_s);
  const int shared_items = a.I_s > 0 ? (a.T + DMOE_WORK_ROWS - 1) / DMOE_WORK_ROWS : 0;
  const int items = a.max_work + shared_items;
  if (dt == DMOE_BF16) {
    FfnParams p{static_cast<const bf16_t*>(a.x), static_cast<const bf16_t*>(a.xr),
                static_cast<const bf16_t*>(a.w13), static_cast<const bf16_t*>(a.w2),
                static_cast<const bf16_t*>(a.ws13),
                static_cast<const bf16_t*>(a.ws2), a.sched.n_work, a.sched.work, a.sched.row_token,
                a.sched.row_slot, a.T, a.H, a.E, a.I, a.I_s, a.k, Tk, R, a.max_work, shared_items,
                static_cast<bf16_t*>(a.workspace), a.slot_out, a.shared_out,
                a.slot_fmt == DMOE_SLOT_F16S ? 1 : 0, 0};
    if (use_tile_kernels(a.T, a.k, a.max_work, items, ldh)) {
      return launch_tiles(p, ldh, items, rows_per_item(a.T, a.k, a.max_work), s);
    }
    switch (pick_ntiles(a.T, a.k, a.max_work)) {
      case 1: {
        // Items of a one-tile schedule average few rows, but an expert can
        // still collect many (a popular expert, a small Top-P coreset, the
        // shared expert over more than 16 tokens).  The decode kernels keep a
        // wave's weight slice in registers across 16-row passes when it is
        // one burst; long slices they would stream once per pass, so such
        // layers run every item on the tile kernels (measured
        // faster than leaving the items of one pass to the decode kernels,
        // whose grids, sized for the worst case, cost ~17 us each when few
        // items are that small).  So do schedules of at least one pass per
        // expert on average (T*k >= 16 E), where the tile kernels measured
        // faster too (512 tokens over 256 experts at hidden 2048: token
        // routing 321 -> 283 us, Top-P 317 -> 306; 256 tokens and fewer
        // favour the decode kernels).
        const bool multi_burst = a.H / 128 > Shape<1>::kGuMax || ldh / 128 > Shape<1>::kDnLong;
        const bool pass_per_expert = static_cast<long>(a.T) * a.k >= static_cast<long>(kPassRows) * a.E;
        if (a.T > kPassRows && (multi_burst || pass_per_expert)) {
          return launch_tiles(p, ldh, items, rows_per_item(a.T, a.k, a.max_work), s);
        }
        return launch_one_tile(p, ldh, items, s);
      }
      case 2: return launch_two_tiles(p, ldh, items, s);
      default: return launch_four_tiles(p, ldh, items, s);
    }
  }
  return launch_ffn_f32(a, ldh, items, s);
}

}  // namespace dmoe
