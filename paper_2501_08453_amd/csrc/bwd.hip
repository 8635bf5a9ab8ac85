// Backward joint text-video attention for gfx950.
//
// Prepare: per query row, -D_i = -<dO_i, O_i> and -LSE_i / c in fp32, padded
//   to whole tiles of 64 rows (padding rows get -inf for the latter so that their
//   probabilities vanish, and D = 0). So dP - D is what the dP accumulator holds
//   when it starts from -D, and S - LSE / c (P = exp2 of it times c log2(e)) what
//   the score accumulator holds when it starts from -LSE / c. (For scales so small that
//   LSE / c could overflow, a power of two is moved from K to c there.)
// dK/dV (key-stationary): one workgroup of eight waves owns 256 keys of one
//   (sample, head), each wave 32, with K and V of its keys in registers and
//   dK^T, dV^T accumulated in registers. It walks over all query tiles of 32,
//   whose row-major Q and dO rows are copied asynchronously global -> LDS into a
//   two-stage ring one tile ahead; one barrier per tile. Per tile it recomputes
//   S = Q K^T and P = exp2((S - LSE / c) c log2(e)), forms dP - D = -D + dO V^T
//   and dS = P o (dP - D) with the matrix cores, and accumulates dV^T += dO^T P and
//   dK^T += Q^T dS straight from the accumulator layout (lane column = key). The
//   transposed operands Q^T, dO^T come from the row-major rows through transposing
//   LDS reads. What bounds it: each wave's in-order stream of matrix-core ops, LDS
//   reads and vector arithmetic, at the power-limited matrix rate; so the reads are
//   placed ahead of their products and the arithmetic between them by hand, and the
//   copies cost scalar arithmetic only. 24 heads x 57,856 tokens, D = 128, no dQ:
//   68.4 -> 62 ms; with dQ of 65% of the keys 97.2 -> 90 ms (one box).
// dQ, fused (the default for joint attention at head_dim 128): in the workgroups
//   of the first key blocks (a fraction set by the host), after the dK/dV products
//   of a tile, the waves exchange dS^T through LDS and, one tile later, D/32 of
//   them (in turns) each compute one 32x32 block of the tile's dQ / scale = dS K
//   over the workgroup's 256 keys, with K^T held in LDS for the workgroup's
//   lifetime, and add it to an fp32 accumulator with atomics; the
//   workgroups of each XCD start their walk at a different query tile so that
//   concurrent atomics spread over the accumulator. For those keys S and dP are
//   computed once per (query, key) pair; the atomic traffic (fp32 dQ rows per key
//   block, performed at the memory side) is what limits the fraction: the dQ pass
//   below then covers only the other key blocks' tiles and adds the accumulator.
//   The order of the atomic additions, and so the rounding of dQ, varies from run
//   to run.
// dQ, separate (deterministic): one workgroup of eight waves owns 256 queries,
//   each wave 32, with Q^T and dO^T of its queries in registers and the lane's
//   LSE and -D as scalars. It walks over the key tiles like the forward,
//   computing S^T = K Q^T and dP^T = V dO^T, dS^T, and dQ^T += K^T dS^T with
//   dS^T taken straight from the accumulator layout (lane column = query) and K^T
//   from K's own rows by transposing LDS reads; reads, arithmetic and copies are
//   placed as in the dK/dV walk.
//   (Over 35% of the keys of 24 heads x 57,856 tokens: 19.4 -> 17.6 ms, and no
//   token-major copy of K, 128 us.)
//   This recomputes S and dP once more instead of scattering dQ partial sums
//   with atomics; the result is bitwise reproducible.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace vcja {
namespace {

constexpr int kDkdvWaves = 8;
constexpr int kBKV = 32 * kDkdvWaves;  // keys per dK/dV workgroup
static_assert(kBKV == kDkdvKeys, "dK/dV key block");
constexpr int kBQ = 32;                // queries per dK/dV tile
constexpr int kDqWaves = 8;
constexpr int kDqBM = 32 * kDqWaves;  // queries per dQ workgroup
constexpr int kBN = kTileTok;         // keys per dQ tile

template <int D>
__global__ __launch_bounds__(256) void bwd_prepare_kernel(const __bf16* __restrict__ o,
                                                          const float* __restrict__ lse,
                                                          const __bf16* __restrict__ dout,
                                                          float* __restrict__ dd, float* __restrict__ nls, int B,
                                                          int H, int N, int Npad, float inv_scale,
                                                          float* __restrict__ zero_acc) {
  constexpr int CPR = D / 8;  // 16-byte chunks per (token, head) row
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t rows = (size_t)B * N * H;
  const size_t row = gid / CPR;
  const int chunk = (int)(gid % CPR);
  float sum = 0.0f;
  if (row < rows) {
    const bf16x8 x = *(const bf16x8*)(o + row * D + chunk * 8);
    const bf16x8 y = *(const bf16x8*)(dout + row * D + chunk * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) sum = fmaf((float)x[e], (float)y[e], sum);
    if (zero_acc) {  // the dQ accumulator of a fused pass, cleared on the way
      *(f32x4*)(zero_acc + row * D + chunk * 8) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      *(f32x4*)(zero_acc + row * D + chunk * 8 + 4) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
  }
#pragma unroll
  for (int off = 1; off < CPR; off <<= 1) sum += __shfl_xor(sum, off, 64);
  if (row < rows && chunk == 0) {
    const int h = (int)(row % H);
    const size_t bn = row / H;
    const int n = (int)(bn % N);
    const int b = (int)(bn / N);
    const size_t bh = (size_t)b * H + h;
    const float x = lse[bh * N + n];
    dd[bh * Npad + n] = -sum;
    nls[bh * Npad + n] = (x == -INFINITY) ? -INFINITY : -x * inv_scale;
  }
  // Padding rows [N, Npad) of every (sample, head).
  const size_t pads = (size_t)B * H * (Npad - N);
  if (gid < pads) {
    const size_t bh = gid / (Npad - N);
    const int n = N + (int)(gid % (Npad - N));
    dd[bh * Npad + n] = 0.0f;
    nls[bh * Npad + n] = -INFINITY;
  }
}

// LDS layout of the dK/dV kernel. A stage holds one tile of 32 queries: their Q rows, their
// dO rows (swizzled rows in perm_row order); two stages. Two buffers of -LSE/c[256] |
// -D[256] follow, for 8 tiles each (copied once per 8 tiles: a 32-query copy per tile, by
// two of the waves, held up every tile's barrier). With dQ fused, K^T of the workgroup's keys ([D][256 + 8] bf16) and two buffers of a tile's dS^T
// ([256 keys][32] bf16) follow, read by the dQ products.
// dS^T rows are 72 bytes (32 queries + 4 pad), and key 32u + 4j + e sits in row
// 32u + 8e + j: the writes (32 consecutive keys, one per lane) hit 64 distinct banks, the
// transposing reads (4 consecutive keys x 32 queries per half-wave) too, as the 4 keys'
// rows lie 8 apart; every address is a per-lane base plus an immediate offset.
template <int D, bool FUSED>
struct DkdvLds {
  using Rows = SwzRows<D>;
  static constexpr int RT = Rows::bytes(kBQ);        // Q or dO rows of a tile
  static constexpr int COPIES = kBQ / Rows::RPC;     // wave copies of each
  static constexpr int STAGE = 2 * RT;
  static constexpr int SQ = 256;                     // queries per copy of row statistics
  static constexpr int SB = 2 * SQ * 4;              // -LSE/c[SQ] | -D[SQ]
  static constexpr int ST_OFF = 2 * STAGE;           // row statistics, two buffers
  static constexpr int KTS = (kBKV + 8) * 2;         // K^T row stride (bytes)
  static constexpr int DSS = (kBQ + 4) * 2;          // dS^T row stride (bytes)
  static constexpr int DSB = kBKV * DSS;             // dS^T of one tile
  static constexpr int KT_OFF = ST_OFF + 2 * SB;
  static constexpr int DS_OFF = KT_OFF + D * KTS;
  static constexpr int BYTES = FUSED ? DS_OFF + 2 * DSB : KT_OFF;
  // Byte offset of the 8-byte unit u (queries 4u .. 4u+3) of dS^T row j; row of key k.
  static __device__ __forceinline__ int ds_at(int j, int u) { return j * DSS + 8 * u; }
  static __device__ __forceinline__ int ds_row(int k) { return (k & ~31) | ((k & 3) << 3) | ((k >> 2) & 7); }
};

template <int D, bool SPATIAL, bool FUSED>
__global__ __launch_bounds__(64 * kDkdvWaves, 1) void bwd_dkdv_kernel(DkdvArgs a) {
  using Lds = DkdvLds<D, FUSED>;
  using Rows = SwzRows<D>;
  constexpr int RT = Lds::RT;
  constexpr int STAGE = Lds::STAGE;
  __shared__ __attribute__((aligned(1024))) char smem[Lds::BYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index (uniform)
  const int l32 = lane & 31;
  const int hi = lane >> 5;
  // Spatial branch: 3-D grid (key block slot, head, sample), renumbered by XCD. Joint: 1-D
  // grid of items with the split tail dispatched last.
  int gx, h, b;
  TailItem ti{0, 0, 0, -1, 0};
  if (SPATIAL) {
    const int3 gp = xcd_grid_pos(true);
    gx = gp.x;
    h = gp.y;
    b = gp.z;
  } else {
    ti = tail_item(blockIdx.x, (a.N + kBKV - 1) / kBKV, a.H, a.B, a.tail_blocks);
    gx = ti.blk;
    h = ti.h;
    b = ti.b;
  }
  const bool tail = !SPATIAL && ti.chunk >= 0;
  const int N = a.N;
  const int ntq = (N + kBQ - 1) / kBQ;  // query tiles
  const size_t tok = (size_t)a.H * D;
  const size_t base = (size_t)b * N * tok + (size_t)h * D;
  const size_t bh = (size_t)b * a.H + h;
  const int npad = a.ntile * kTileTok;
  // Spatial branch with split text blocks: workgroups [0, text_blocks*text_chunks) of a head
  // take (text block, chunk of its query tiles) and come first in dispatch order, the rest
  // the other key blocks in order.
  int kb = gx, chunk = 0;
  bool split = false;
  if (SPATIAL && a.text_chunks > 1) {
    const int nsplit = a.text_blocks * a.text_chunks;
    split = gx < nsplit;
    kb = split ? gx % a.text_blocks : gx - nsplit + a.text_blocks;
    chunk = split ? gx / a.text_blocks : 0;
  }
  // This workgroup's keys (spatial branch: text keys, or keys of one frame).
  const RowBlock rb = row_block(kb, N, a.T, SPATIAL ? a.frame_len : 0, kBKV, true);
  const bool do_dq = FUSED && kb < a.dq_blocks;  // this key block carries its share of dQ
  // This lane's key (accumulator column), formed where it is used from a lane index that the
  // compiler must treat as new, so that no register holds it across the walk (registers are
  // the limit there); so are the per-lane addresses of the walk's steps.
  auto fresh_lane = [&]() {
    int x = lane;
    asm volatile("" : "+v"(x));
    return x;
  };
  auto lane_key = [&]() { return rb.r0 + w * 32 + (fresh_lane() & 31); };
  // Partial dK of this lane's key in its chunk (dV partials follow all dK partials); formed
  // only where it is written, so that no register holds it across the main loop.
  const size_t part_stride = (size_t)a.text_chunks * a.B * a.H * a.text_blocks * kBKV * D;
  auto part_k = [&](int key) {
    return a.text_part + ((((size_t)chunk * a.B + b) * a.H + h) * a.text_blocks * kBKV + key) * D;
  };
  // Joint tail: partial dK of this lane's key (dV partials follow all dK partials).
  const size_t tail_stride = (size_t)a.tail_blocks * a.tail_chunks * kBKV * D;
  auto tail_k = [&](int key) {
    return a.tail_part + (((size_t)ti.slot * a.tail_chunks + ti.chunk) * kBKV + (key - rb.r0)) * D;
  };

  AttendRule rule;
  rule.N = N;
  rule.T = a.T;
  rule.tl = a.text_len ? min(max(a.text_len[b], 0), a.T) : a.T;
  rule.L = SPATIAL ? a.frame_len : 0;
  rule.km = a.key_mask ? a.key_mask + (size_t)b * N : nullptr;
  const bool valid = lane_key() < rb.r1 && rule.key_valid(lane_key());

  if (!__syncthreads_or(valid)) {
    // No valid key in this workgroup: its dK, dV (or partials) are zero.
    const int key = lane_key();
    if (tail || split) {
      const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
      float* pk = tail ? tail_k(key) : part_k(key);
      for (int c = 0; c < D / 4; ++c) {
        *(f32x4*)(pk + 4 * c) = z;
        *(f32x4*)(pk + (tail ? tail_stride : part_stride) + 4 * c) = z;
      }
    } else if (key < rb.r1) {
      const bf16x8 z = zero_bf16x8();
      for (int c = 0; c < D / 8; ++c) {
        *(bf16x8*)(a.dk + base + (size_t)key * tok + 8 * c) = z;
        *(bf16x8*)(a.dv + base + (size_t)key * tok + 8 * c) = z;
      }
    }
    return;
  }

  // This wave's copies of query tile qt into stage st: j = 0 Q rows, j = 1 dO rows (at
  // head_dim 64 each wave has one of the two). Rows past N repeat row N-1; the padded -LSE
  // (-inf) makes their probabilities zero. The lane index is made opaque, so that the lane's
  // part of the addresses is formed once per tile instead of being held across the walk.
  static_assert(Lds::COPIES == (D == 128 ? kDkdvWaves : kDkdvWaves / 2), "copies of a tile over the waves");
  struct TileCopy {
    int first;
    unsigned off;
  };
  auto tile_copy = [&](int qt) {
    unsigned cl = lane;
    asm volatile("" : "+v"(cl));
    const int first = swz_copy_row<D, true>(qt * kBQ, N, w % Lds::COPIES);
    return TileCopy{first, swz_copy_off<D, true>(first, (unsigned)tok, N, cl)};
  };
  auto issue_j = [&](int j, const TileCopy& tc, int st) {
    if (D == 64 && j == 1) return;
    const bool is_q = D == 128 ? j == 0 : w < Lds::COPIES;
    copy16_to_lds_opaque((is_q ? a.q : a.dout) + base + (size_t)tc.first * tok, tc.off,
                         (VC_LDS char*)smem + st * STAGE + (is_q ? 0 : RT) + (w % Lds::COPIES) * Rows::GS);
  };
  // The dO rows past N - 1 that this wave copied into stage st: zero, as the probability 0 of such
  // a row times an infinite dO of row N - 1, which it repeats, would be a NaN in dV. (Not where dQ
  // is fused in, whose instances have no register left for it: 4 to 8 would spill.)
  auto zero_do_padding = [&](int row0, int st) {
    if (D == 64 && w < Lds::COPIES) return;
    const int cl = fresh_lane(), idx = w % Lds::COPIES;
    f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    asm volatile("" : "+v"(z));  // formed here: no registers hold it across the walk
    if (row0 + perm_row(Rows::RPC * idx + cl / Rows::CPR) >= N)
      *(VC_LDS f32x4*)((VC_LDS char*)smem + st * STAGE + RT + idx * Rows::GS + 16 * cl) = z;
  };
  // Query tiles this workgroup visits (the same sequence for every wave): all of them in
  // joint attention; in the spatial branch the video tiles its keys are attended from. The
  // host's spans count tiles of kTileTok queries.
  constexpr int TPS = kTileTok / kBQ;
  TileRuns runs = rule.query_tiles(rb.r0, rb.r1, ntq, kBQ);
  if (split) {  // this chunk's part of the video query tiles
    const int c0 = (a.T / kTileTok + chunk * a.text_span) * TPS;
    runs.b0 = max(runs.b0, c0);
    runs.b1 = min(runs.b1, c0 + a.text_span * TPS);
    if (runs.b0 >= runs.b1) runs.b1 = 0;
  }
  if (tail) {  // this chunk's run of query tiles
    runs.b0 = ti.chunk * a.tail_span * TPS;
    runs.b1 = min(ntq, runs.b0 + a.tail_span * TPS);
    if (runs.b0 >= runs.b1) runs.b1 = 0;
  }
  auto next_q = [&](int qt) { return (SPATIAL || tail) ? runs.next(qt) : qt; };
  // Spatial branch: the queries attending to this workgroup's keys, [kx, ky) (its keys are all
  // text, attended from every video row, or all of one frame); a tile needs the per-query
  // test unless it lies inside.
  const bool text_keys = SPATIAL && rb.r0 < a.T;
  const int kx = SPATIAL ? (text_keys ? a.T : rule.frame_start(rb.r0)) : 0;
  const int ky = text_keys ? N : kx + rule.L;

  // dQ: the workgroups of each XCD (dispatch is round-robin over the XCDs) start
  // their walk over the query tiles at a different eighth of them, so that the atomics
  // of concurrent workgroups land on different rows of the accumulator. Walk position u
  // visits tile phys(u).
  const int xs = (FUSED && !SPATIAL && !tail) ? (int)((blockIdx.x % kXcds) * ((ntq + kXcds - 1) / kXcds)) % ntq : 0;
  auto phys = [&](int u) { return u + xs >= ntq ? u + xs - ntq : u + xs; };
  // The statistics of the SQ / kBQ walk positions around u (the aligned run holding it) into
  // their buffer, by the last two waves (past the padded length: its last four repeated).
  constexpr int SPT = Lds::SQ / kBQ;
  auto issue_stats = [&](int u) {
    if (w < kDkdvWaves - 2) return;
    int cl = lane;
    asm volatile("" : "+v"(cl));
    const bool is_l = w == kDkdvWaves - 2;
    int q = ((u & -SPT) + xs) * kBQ + 4 * cl;
    q = q >= ntq * kBQ ? q - ntq * kBQ : q;  // the walk wraps past the last tile
    copy16_to_lds_opaque((is_l ? a.nls : a.dd) + bh * npad, 4u * (unsigned)min(q, npad - 4),
                         (VC_LDS char*)smem + Lds::ST_OFF + (u / SPT % 2) * Lds::SB + (is_l ? 0 : Lds::SQ * 4));
  };
  // The first tile's copies, in flight with the loads of K and V.
  const int qt0 = next_q(0);
  if (qt0 < ntq) {
    const TileCopy tc = tile_copy(phys(qt0));
    issue_stats(qt0);
    issue_j(0, tc, 0);
    issue_j(1, tc, 0);
  }
  // K, V of this lane's key as B operands (dims 16*ks + 8*hi .. +7).
  bf16x8 kf[D / 16], vf[D / 16];
  {
    const size_t kr = base + (size_t)min(lane_key(), rb.r1 - 1) * tok + 8 * hi;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      kf[ks] = *(const bf16x8*)(a.k + kr + 16 * ks);
      vf[ks] = *(const bf16x8*)(a.v + kr + 16 * ks);
    }
    wait_all_memory();  // and the first tile's copies: no later wait stands among copies
  }

  // dQ: K^T of the workgroup's keys (row d holds K[key][d] of its 256 keys).
  if (FUSED && do_dq) {
    VC_LDS __bf16* ktl = (VC_LDS __bf16*)(smem + Lds::KT_OFF);
    const int kl = w * 32 + l32;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
      for (int t = 0; t < 8; ++t) ktl[(16 * ks + 8 * hi + t) * (Lds::KTS / 2) + kl] = kf[ks][t];
  }
  if (a.score_down != 1.0f) scale_operand(kf, a.score_down);  // the scores' copy of K

  f32x16 dk_acc[D / 32], dv_acc[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; ++i) {
    dk_acc[i] = zero_f32x16();
    dv_acc[i] = zero_f32x16();
  }

  // A tile's dQ has D/32 blocks of 32 queries x 32 dims. The waves form them in turns, D/32
  // waves per tile (of different SIMDs: wave w shares its SIMD with wave w + 4): group
  // w / (D/32) takes every DQ_TURNS-th tile, wave w of it the dims 32*(w % (D/32)). While one
  // of a SIMD's two waves forms its dQ block of the previous tile, the other is already in
  // this tile's products, so the two run out of step and one's vector arithmetic overlaps
  // the other's matrix-core work; with every wave taking a block of every tile they ran in
  // step from barrier to barrier.
  constexpr int NB = D / 32;
  constexpr int DQ_STEPS = kBKV / 16;
  constexpr int DQ_TURNS = kDkdvWaves / NB;
  const int dq_turn = w / NB, dq_db = w % NB;
  // Bases of the operand reads: plain (the lane's query row) and transposing.
  using Reads = SwzReads<D>;
  const int row_base = Reads::row_base(perm_row(l32), hi);
  const int tr_base = Reads::tr_base(lane);

  // dQ block of the tile starting at query row0, whose dS^T is in buffer `buf`: A = dS
  // (queries x keys) by transposing reads of dS^T, B = K from K^T. Lane l of 16-lane group G
  // supplies key 16*st + 8*hi + (l%16)/4 (+4), i.e. row 32*(st/2) + 4*(st%2) + 8*((l%16)/4) +
  // 2*hi (+1), and unit 4*(G%2) + l%4 of that row. The block is added to the accumulator with
  // a uniform 64-bit base plus a 32-bit per-lane offset (4 rows at most); rows past N are
  // padding.
  auto dq_step = [&](int row0, int buf) {
    const int ln = fresh_lane();
    const VC_LDS char* ds_src = (const VC_LDS char*)smem + Lds::DS_OFF + buf * Lds::DSB;
    const int arow = 8 * ((ln & 15) >> 2) + 2 * (ln >> 5), aunit = 4 * ((ln >> 4) & 1) + (ln & 3);
    const VC_LDS char* b_base =
        (const VC_LDS char*)smem + Lds::KT_OFF + (dq_db * 32 + (ln & 31)) * Lds::KTS + 8 * (ln >> 5) * 2;
    f32x16 blk = zero_f32x16();
    constexpr int PF = 4;  // operands read this many ops ahead
    bf16x8 da[DQ_STEPS], kb8[DQ_STEPS];
    auto rd = [&](int st) {
      const int j = arow + 32 * (st >> 1) + 4 * (st & 1);
      da[st] = cat4(lds_read_tr(ds_src + Lds::ds_at(j, aunit)), lds_read_tr(ds_src + Lds::ds_at(j + 1, aunit)));
      kb8[st] = *(const VC_LDS bf16x8*)(b_base + st * 32);
    };
#pragma unroll
    for (int st = 0; st < PF; ++st) rd(st);
#pragma unroll
    for (int st = 0; st < DQ_STEPS; ++st) {
      sched_fence();
      if (st + PF < DQ_STEPS) rd(st + PF);
      blk = mfma32(da[st], kb8[st], blk);
    }
    sched_fence();
    // Register r of lane (col, half): query row0 + 8*(r/4) + r%4 + 4*half, dim dq_db*32 + col.
    float* const dst = a.dq_acc + (size_t)b * N * tok + (size_t)h * D + dq_db * 32 + (size_t)row0 * tok;
    const int ln2 = fresh_lane();
    const int half = ln2 >> 5;
    const unsigned loff = (unsigned)(4 * half) * (unsigned)tok + (unsigned)(ln2 & 31);
    if (row0 + kBQ <= N) {
#pragma unroll
      for (int r = 0; r < 16; ++r) atomicAdd(dst + (size_t)(8 * (r >> 2) + (r & 3)) * tok + loff, blk[r]);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (row0 + acc_row(r, half) < N) atomicAdd(dst + (size_t)(8 * (r >> 2) + (r & 3)) * tok + loff, blk[r]);
    }
  };

  // The walk over the query tiles; DQ: this workgroup also adds its dQ share (a separate
  // instance of the loop, so that neither carries the other's registers). One barrier per
  // tile: past it, stage st holds the tile, dS^T of the previous tile is complete, and no
  // wave reads the other stage or the other dS^T buffer.
  auto walk = [&](auto dq_tag) {
    constexpr bool DQ = decltype(dq_tag)::value;
    int qt = qt0;
    int prev0 = -1;  // first query row of the previous tile, -1: none
    int turn = 0;    // whose turn the previous tile's dQ is
    for (int st = 0; qt < ntq; st ^= 1) {  // stage st holds tile qt, stage st ^ 1 takes the next
      const int qn = next_q(qt + 1);
      wait_all_memory();
      if (!FUSED && __builtin_expect(qt * kBQ + kBQ > N, 0)) zero_do_padding(qt * kBQ, st);
      __syncthreads();
      if constexpr (DQ) {
        if (prev0 >= 0) {
          if (turn == dq_turn) dq_step(prev0, st ^ 1);
          turn = (turn + 1) % DQ_TURNS;
        }
        sched_fence();
      }
      const int q0 = phys(qt) * kBQ;
      const TileCopy tc = tile_copy(phys(qn < ntq ? qn : qt));  // past the last tile: any tile, never read
      if (qn % SPT == 0 && qn < ntq) issue_stats(qn);
      const bool pair_mask = SPATIAL && !(q0 >= kx && q0 + kBQ <= ky);
      const VC_LDS char* q_lds = (const VC_LDS char*)smem + st * STAGE;
      const VC_LDS float* nls_lds =
          (const VC_LDS float*)((const VC_LDS char*)smem + Lds::ST_OFF + (qt / SPT % 2) * Lds::SB) + qt % SPT * kBQ + 4 * (fresh_lane() >> 5);
      const VC_LDS float* dd_lds = nls_lds + Lds::SQ;

      // The tile's products in one stretch of 4 * KSN matrix-core ops, every LDS operand read
      // PF ops ahead of its use, each phase's vector arithmetic placed between the ops of the
      // next one (which do not depend on it): S = Q K^T; dP = -D + dO V^T while P is formed;
      // dV^T += dO^T P while dS is formed; dK^T += Q^T dS. Left to the compiler, the reads
      // came two ops ahead at most and the arithmetic stood between the products.
      constexpr int KSN = D / 16;
      constexpr int PF = 2;
      constexpr int EP = 16 / KSN;       // elements of P per dP op
      constexpr int ED = 16 / (2 * NB);  // elements of dS per dV op
      f32x16 s, dp;
      bf16x8 f[2 * KSN];
      auto rd = [&](int i) {
        f[i] = *(const VC_LDS bf16x8*)(Reads::row_at(q_lds + row_base, i % KSN) + (i < KSN ? 0 : RT));
      };
      // Operand element t of k-step st2 is query 16*st2 + 8*(t/4) + 4*hi + t%4, read from the
      // row-major tiles by two transposing reads (queries +0..3 and +8..11). Operand i: dO^T,
      // then Q^T, k-step st2 = (i / NB) % 2 major, dim block i % NB minor.
      bf16x8 g[4 * NB];
      auto rdt = [&](int i) {
        g[i] = Reads::tr_operand(q_lds + (i < 2 * NB ? RT : 0) + tr_base, i / NB % 2, i % NB);
      };
      // Register r holds query row 8*(r/4) + 4*hi + r%4 of the tile: four runs of 4 rows.
      auto form_p = [&](int r) {
        s[r] = fast_exp2(s[r] * a.scale_log2);
      };
      auto operand = [&](const f32x16& x, int half) {
        bf16x8 y;
#pragma unroll
        for (int t = 0; t < 8; ++t) y[t] = (__bf16)x[8 * half + t];
        return y;
      };
      auto form_ds = [&](int r) { dp[r] = s[r] * dp[r]; };
      // dS as operand `half`. An invalid key needs no test for dK, dV: its probabilities
      // reach only its own lane's dK, dV, which are written as zero at the end.
      // Its dS also reaches dQ, so with dQ formed here it is zeroed (its P may even be inf).
      auto ds_operand = [&](int half) {
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        u32x4 y = __builtin_bit_cast(u32x4, operand(dp, half));
        if (DQ) {
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = valid ? y[e] : 0u;
        }
        return __builtin_bit_cast(bf16x8, y);
      };
#pragma unroll
      for (int i = 0; i < PF; ++i) rd(i);
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // S accumulates on top of -LSE/c, dP on top of -D of its query rows
        const f32x4 nl = *(const VC_LDS f32x4*)(nls_lds + 8 * j), nd = *(const VC_LDS f32x4*)(dd_lds + 8 * j);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[4 * j + i] = nl[i];
          dp[4 * j + i] = nd[i];
        }
      }
#pragma unroll
      for (int i = 0; i < KSN; ++i) {
        sched_fence();
        rd(i + PF);
        s = mfma32(f[i], kf[i], s);
        // The next tile's copies, one at a time: issued together at the top of the step, eight
        // waves' copies would hold up the start of every wave's products.
        if (i == 0 || i == 2) issue_j(i / 2, tc, st ^ 1);
      }
      if (SPATIAL && pair_mask) {  // queries outside [kx, ky) get probability zero
        sched_fence();
        const int half = fresh_lane() >> 5;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int qrow = q0 + acc_row(r, half);
          s[r] = (qrow >= kx) & (qrow < ky) ? s[r] : -INFINITY;
        }
      }
#pragma unroll
      for (int i = 0; i < KSN; ++i) {
        sched_fence();
        if (i + PF < KSN)
          rd(KSN + i + PF);
        else
          rdt(i + PF - KSN);
        dp = mfma32(f[KSN + i], vf[i], dp);
        if (i > 0) {
#pragma unroll
          for (int e = 0; e < EP; ++e) form_p((i - 1) * EP + e);
        }
      }
      bf16x8 pb[2], sb[2];
      sched_fence();
      pb[0] = operand(s, 0);
#pragma unroll
      for (int i = 0; i < 2 * NB; ++i) {
        sched_fence();
        rdt(i + PF);
        dv_acc[i % NB] = mfma32(g[i], pb[i / NB], dv_acc[i % NB]);
        if (i == 0) {
#pragma unroll
          for (int e = 0; e < EP; ++e) form_p((KSN - 1) * EP + e);
          pb[1] = operand(s, 1);
        } else {
#pragma unroll
          for (int e = 0; e < ED; ++e) form_ds((i - 1) * ED + e);
        }
      }
      sched_fence();
      sb[0] = ds_operand(0);
#pragma unroll
      for (int i = 0; i < 2 * NB; ++i) {
        sched_fence();
        if (2 * NB + i + PF < 4 * NB) rdt(2 * NB + i + PF);
        dk_acc[i % NB] = mfma32(g[2 * NB + i], sb[i / NB], dk_acc[i % NB]);
        if (i == 0) {
#pragma unroll
          for (int e = 0; e < ED; ++e) form_ds((2 * NB - 1) * ED + e);
          sb[1] = ds_operand(1);
        }
        if (i == 1) {
          if constexpr (DQ) {
            // dS^T: element t of operand st2 is query 16*st2 + 8*(t/4) + 4*hi + t%4, i.e. units
            // 4*st2 + hi and 4*st2 + 2 + hi.
            const int ln = fresh_lane();
            VC_LDS char* ds_dst = (VC_LDS char*)smem + Lds::DS_OFF + st * Lds::DSB;
            const int kl = Lds::ds_row(w * 32 + (ln & 31)), hl = ln >> 5;  // dS^T row, lane half
#pragma unroll
            for (int st2 = 0; st2 < 2; ++st2) {
              const bf16x8 x = sb[st2];
              *(VC_LDS bf16x4*)(ds_dst + Lds::ds_at(kl, 4 * st2 + hl)) = bf16x4{x[0], x[1], x[2], x[3]};
              *(VC_LDS bf16x4*)(ds_dst + Lds::ds_at(kl, 4 * st2 + 2 + hl)) = bf16x4{x[4], x[5], x[6], x[7]};
            }
          }
        }
      }
      sched_fence();
      if constexpr (DQ) prev0 = q0;
      qt = qn;
      if constexpr (DQ) {
        if (qn >= ntq) {  // the last tile's dQ
          __syncthreads();
          if (turn == dq_turn) dq_step(prev0, st);
        }
      }
    }
  };
  if constexpr (FUSED) {
    if (do_dq)
      walk(std::true_type{});
    else
      walk(std::false_type{});
  } else {
    walk(std::false_type{});
  }

  wait_all_memory();  // no copy outlives the workgroup
  const int key = lane_key();

  if (tail || split) {
    // fp32 partials; an invalid key's are zero (its accumulators may hold anything).
    float* pk = tail ? tail_k(key) : part_k(key);
    float* pv = pk + (tail ? tail_stride : part_stride);
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        f32x4 tk, tv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          tk[e] = valid ? dk_acc[db][4 * j + e] * a.scale : 0.0f;
          tv[e] = valid ? dv_acc[db][4 * j + e] : 0.0f;
        }
        *(f32x4*)(pk + db * 32 + 8 * j + 4 * hi) = tk;
        *(f32x4*)(pv + db * 32 + 8 * j + 4 * hi) = tv;
      }
  } else if (key < rb.r1) {
    __bf16* dkp = a.dk + base + (size_t)key * tok;
    __bf16* dvp = a.dv + base + (size_t)key * tok;
    // An invalid key gets exactly zero (its accumulators may hold anything, even inf).
    auto kv = [&](float x) { return (__bf16)(valid ? x * a.scale : 0.0f); };
    auto vv = [&](float x) { return (__bf16)(valid ? x : 0.0f); };
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x4 tk = {kv(dk_acc[db][4 * j + 0]), kv(dk_acc[db][4 * j + 1]), kv(dk_acc[db][4 * j + 2]),
                     kv(dk_acc[db][4 * j + 3])};
        bf16x4 tv = {vv(dv_acc[db][4 * j + 0]), vv(dv_acc[db][4 * j + 1]), vv(dv_acc[db][4 * j + 2]),
                     vv(dv_acc[db][4 * j + 3])};
        *(bf16x4*)(dkp + db * 32 + 8 * j + 4 * hi) = tk;
        *(bf16x4*)(dvp + db * 32 + 8 * j + 4 * hi) = tv;
      }
  }
}

// Spatial branch: dK, dV of the text rows [0, nrow) as the sum of the chunks' fp32
// partials (rows = text_blocks * 256 per partial). One thread per 4 dims of one row.
template <int D>
__global__ void text_reduce_kernel(const float* part, __bf16* dk, __bf16* dv, int B, int H, int N, int rows,
                                   int nrow, int chunks) {
  const size_t total = (size_t)B * H * nrow * (D / 4);
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int d = (int)(i % (D / 4)) * 4;
  size_t t = i / (D / 4);
  const int row = (int)(t % nrow);
  t /= nrow;
  const int h = (int)(t % H);
  const int b = (int)(t / H);
  const size_t stride = (size_t)B * H * rows * D;  // one chunk
  const size_t off = (((size_t)b * H + h) * rows + row) * D + d;
  f32x4 sk = {0.0f, 0.0f, 0.0f, 0.0f}, sv = sk;
  for (int c = 0; c < chunks; ++c) {
    sk += *(const f32x4*)(part + c * stride + off);
    sv += *(const f32x4*)(part + (size_t)chunks * stride + c * stride + off);
  }
  const size_t o = (((size_t)b * N + row) * H + h) * D + d;
  *(bf16x4*)(dk + o) = bf16x4{(__bf16)sk[0], (__bf16)sk[1], (__bf16)sk[2], (__bf16)sk[3]};
  *(bf16x4*)(dv + o) = bf16x4{(__bf16)sv[0], (__bf16)sv[1], (__bf16)sv[2], (__bf16)sv[3]};
}

// Joint tail of the dK/dV kernel: dK, dV of the split items as the sum of their chunks'
// fp32 partials. One thread per 4 dims of one key row.
template <int D>
__global__ void tail_reduce_kernel(const float* part, __bf16* dk, __bf16* dv, int B, int H, int N, int items,
                                   int chunks) {
  const int nblk = (N + kBKV - 1) / kBKV;
  const size_t total = (size_t)items * kBKV * (D / 4);
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int d = (int)(i % (D / 4)) * 4;
  const int k = (int)((i / (D / 4)) % kBKV);
  const int slot = (int)(i / ((size_t)(D / 4) * kBKV));
  const int item = nblk * H * B - items + slot;
  const int row = (item % nblk) * kBKV + k;
  if (row >= N) return;
  const int h = (item / nblk) % H, b = item / (nblk * H);
  const size_t stride = (size_t)items * chunks * kBKV * D;  // dK partials, then dV
  f32x4 sk = {0.0f, 0.0f, 0.0f, 0.0f}, sv = sk;
#pragma unroll 4
  for (int c = 0; c < chunks; ++c) {
    const size_t off = (((size_t)slot * chunks + c) * kBKV + k) * D + d;
    sk += *(const f32x4*)(part + off);
    sv += *(const f32x4*)(part + stride + off);
  }
  const size_t o = (((size_t)b * N + row) * H + h) * D + d;
  *(bf16x4*)(dk + o) = bf16x4{(__bf16)sk[0], (__bf16)sk[1], (__bf16)sk[2], (__bf16)sk[3]};
  *(bf16x4*)(dv + o) = bf16x4{(__bf16)sv[0], (__bf16)sv[1], (__bf16)sv[2], (__bf16)sv[3]};
}

// KM: a key mask is given (a separate instance, so that the unmasked one carries none of
// its per-tile work).
template <int D, bool KM>
__global__ __launch_bounds__(64 * kDqWaves, 1) void bwd_dq_kernel(DqArgs a) {
  using Rows = SwzRows<D>;
  using Reads = SwzReads<D>;
  constexpr int RT = Rows::bytes(kBN);  // K or V rows of a tile
  constexpr int STAGE = 2 * RT;         // K | V
  constexpr int COPIES = kBN / Rows::RPC;
  constexpr int CPW = COPIES / kDqWaves;  // copies of each per wave and tile
  static_assert(CPW * kDqWaves == COPIES, "copies of a tile over the waves");
  __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index (uniform)
  const int l32 = lane & 31;
  const int hi = lane >> 5;
  // Spatial branch: 3-D grid renumbered by XCD. Joint: 1-D grid of items, split tail last.
  int gx, h, b;
  TailItem ti{0, 0, 0, -1, 0};
  if (a.frame_len) {
    const int3 gp = xcd_grid_pos(true);
    gx = gp.x;
    h = gp.y;
    b = gp.z;
  } else {
    ti = tail_item(blockIdx.x, (a.N + kDqBM - 1) / kDqBM, a.H, a.B, a.tail_blocks);
    gx = ti.blk;
    h = ti.h;
    b = ti.b;
  }
  if (a.frame_len)  // text rows are not queries of the spatial branch
    write_text_rows<D>(TextRows{a.dq, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr}, a.B, a.H, a.N, a.T, tid,
                       blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), gridDim.x * gridDim.y * gridDim.z);
  const bool tail = ti.chunk >= 0;
  const int N = a.N;
  const size_t tok = (size_t)a.H * D;
  const size_t base = (size_t)b * N * tok + (size_t)h * D;
  const size_t bh = (size_t)b * a.H + h;
  // This workgroup's queries (spatial branch: inside one frame).
  const RowBlock rb = row_block(gx, N, a.T, a.frame_len, kDqBM, false);
  const int qi = rb.r0 + w * 32 + l32;  // this lane's query (accumulator column)
  const int qr = min(qi, rb.r1 - 1);

  // Q^T and dO^T as B operands (dims 16*ks + 8*hi .. +7), -LSE/c and -D as scalars.
  bf16x8 qf[D / 16], dof[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    qf[ks] = *(const bf16x8*)(a.q + base + (size_t)qr * tok + 16 * ks + 8 * hi);
    dof[ks] = *(const bf16x8*)(a.dout + base + (size_t)qr * tok + 16 * ks + 8 * hi);
  }
  const float nls = a.nls[bh * (size_t)a.ntile * kBN + qr];
  const float dd = a.dd[bh * (size_t)a.ntile * kBN + qr];

  f32x16 dq_acc[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; ++i) dq_acc[i] = zero_f32x16();

  AttendRule rule;
  rule.N = N;
  rule.T = a.T;
  rule.tl = a.text_len ? min(max(a.text_len[b], 0), a.T) : a.T;
  rule.L = a.frame_len;
  rule.km = a.key_mask ? a.key_mask + (size_t)b * N : nullptr;  // non-null exactly when KM
  // This wave's queries (past the end of a short block: its last row).
  const int qw0 = min(rb.r0 + w * 32, rb.r1 - 1), qw1 = min(rb.r0 + w * 32 + 31, rb.r1 - 1);
  const bool wave_all_video = qw0 >= a.T && qw1 < N;
  const int wqs = a.frame_len ? rule.frame_start(qw0) : 0;
  const bool wave_one_frame = wave_all_video && a.frame_len && rule.frame_start(qw1) == wqs;
  const QueryRange qrange = query_range(rule, qi);
  // Key tiles this workgroup visits (the same sequence for every wave).
  TileRuns runs = rule.key_tiles(rb.r0, rb.r1, a.ntile);
  // Completing a fused backward: keys >= kt_min only; joint tail: this chunk's key tiles of them.
  const int kt0 = a.kt_min + (tail ? ti.chunk * a.tail_span : 0);
  if (tail) {
    runs = runs.clipped(kt0 + a.tail_span);
  }
  auto next_tile = [&](int kt) { return runs.next(kt); };
  // This wave's j-th copies of tile kt's K and V rows into stage st (rows past N repeat row
  // N-1; such keys are masked). K rows, and V rows alike, in perm_row order: K^T comes from
  // them by transposing reads.
  const unsigned tok32 = (unsigned)tok;
  const SwzCopy<D, true> cp(tok32, lane);
  auto issue_j = [&](int j, bool is_k, int kt, int st) {
    const int idx = w + j * kDqWaves, first = swz_copy_row<D, true>(kt * kBN, N, idx);
    copy16_to_lds_opaque((is_k ? a.k : a.v) + base + (size_t)first * tok, cp.offset(first, N, tok32),
                         (VC_LDS char*)smem + st * STAGE + (is_k ? 0 : RT) + idx * Rows::GS);
  };
  const int row_base = Reads::row_base(perm_row(l32), hi), tr_base = Reads::tr_base(lane);

  int kt = next_tile(kt0);
  if (kt < a.ntile) {
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
      issue_j(j, true, kt, 0);
      issue_j(j, false, kt, 0);
    }
  }
  wait_all_memory();  // the loads above and the first copies: no later wait stands among copies
  const float nlse2 = nls * a.nls_log2;
  // Key-mask bytes of each tile loaded a step ahead (waited for at the barrier with the
  // tile's copies), turned into the tile's bits there.
  int kmb = KM && kt < a.ntile ? rule.key_mask_byte(kt, lane) : 1;
  int st = 0;
  while (kt < a.ntile) {
    const int kn = next_tile(kt + 1);
    wait_all_memory();
    __syncthreads();
    const unsigned long long kbits = KM ? key_mask_bits(kmb) : ~0ull;
    if (KM && kn < a.ntile) kmb = rule.key_mask_byte(kn, lane);
    // a joint tile whose keys are all real (no padding, no text cut): masked by its bits only
    const bool plain_tile = KM && rule.L == 0 && kt * kBN + kBN <= N && (kt * kBN >= a.T || kt * kBN + kBN <= rule.tl);
    const int k0 = kt * kBN;
    bool need_mask;
    if (rule.km || k0 + kBN > N)
      need_mask = true;
    else if (rule.L == 0)
      need_mask = rule.tl < a.T && k0 < a.T && k0 + kBN > rule.tl;
    else if (k0 + kBN <= rule.tl)
      need_mask = !wave_all_video;
    else
      need_mask = !(wave_one_frame && k0 >= wqs && k0 + kBN <= wqs + rule.L);

    // The two key blocks' products in one stretch of matrix-core ops, every LDS operand read
    // PF ops ahead, the vector arithmetic of a phase placed between the ops of the next ones:
    // S0 | dP0, P0 | S1, dS0 | dP1, P1 | dQ += K0^T dS0, dS1 | dQ += K1^T dS1.
    constexpr int KSN = D / 16;
    constexpr int NB = D / 32;
    constexpr int PF = 3;
    constexpr int EP = 16 / KSN;       // elements per op of a score phase
    const VC_LDS char* tile = (const VC_LDS char*)smem + st * STAGE;
    const int kc = kn < a.ntile ? kn : kt;  // next tile's copies (past the last: any tile, never read)
    bf16x8 f[4 * KSN], g[4 * NB];
    auto rd = [&](int i) {  // S0, dP0, S1, dP1, then the dQ operands
      if (i < 4 * KSN) {
        const int kb = i / (2 * KSN), v = i / KSN % 2;
        f[i] = *(const VC_LDS bf16x8*)(Reads::row_at(tile + row_base, i % KSN) + v * RT + kb * Rows::bytes(32));
      } else if (i - 4 * KSN < 4 * NB) {
        g[i - 4 * KSN] = Reads::tr_operand(tile + tr_base, (i - 4 * KSN) / NB, (i - 4 * KSN) % NB);
      }
    };
    f32x16 s[2], dp[2];
    bf16x8 sb[4];
    auto form_p = [&](int kb, int r) { s[kb][r] = fast_exp2(fmaf(s[kb][r], a.scale_log2, nlse2)); };
    auto form_ds = [&](int kb, int r) { dp[kb][r] *= s[kb][r]; };
    auto operand = [&](const f32x16& x, int half) {
      bf16x8 y;
#pragma unroll
      for (int t = 0; t < 8; ++t) y[t] = (__bf16)x[8 * half + t];
      return y;
    };
#pragma unroll
    for (int i = 0; i < PF; ++i) rd(i);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      s[kb] = zero_f32x16();
#pragma unroll
      for (int i = 0; i < KSN; ++i) {
        sched_fence();
        rd(2 * KSN * kb + i + PF);
        s[kb] = mfma32(f[2 * KSN * kb + i], qf[i], s[kb]);
        if (kb == 0 && i % 2 == 0 && i / 2 < 2 * CPW) issue_j(i / 4, i / 2 % 2 == 0, kc, st ^ 1);
        if (kb == 1 && i == 0)
#pragma unroll
          for (int e = 0; e < EP; ++e) form_p(0, (KSN - 1) * EP + e);
        if (kb == 1 && i > 0)
#pragma unroll
          for (int e = 0; e < EP; ++e) form_ds(0, (i - 1) * EP + e);
      }
      if (kb == 1) {
#pragma unroll
        for (int e = 0; e < EP; ++e) form_ds(0, (KSN - 1) * EP + e);
        sb[0] = operand(dp[0], 0);
        sb[1] = operand(dp[0], 1);
      }
      // Register r holds key k0 + kb*32 + 8*(r/4) + 4*hi + r%4 of this lane's query.
      if (need_mask) {
        sched_fence();
        if (plain_tile) {  // joint tile of real keys: the key mask's bits alone
          const unsigned bits = (unsigned)(kbits >> (32 * kb)) >> (4 * hi);
#pragma unroll
          for (int r = 0; r < 16; ++r) s[kb][r] = ((bits >> (8 * (r >> 2) + (r & 3))) & 1u) ? s[kb][r] : -INFINITY;
        } else {  // branch-free per element; the key mask from the tile's bits
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = k0 + kb * 32 + acc_row(r, hi);
            bool ok = rule.key_valid_bits(key, k0, kbits);  // all bits set without a mask
            if (rule.L) ok = ok & qrange.ok(key, a.T);
            s[kb][r] = ok ? s[kb][r] : -INFINITY;
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) dp[kb][r] = dd;  // dP - D
#pragma unroll
      for (int i = 0; i < KSN; ++i) {
        sched_fence();
        rd(2 * KSN * kb + KSN + i + PF);
        dp[kb] = mfma32(f[2 * KSN * kb + KSN + i], dof[i], dp[kb]);
        if (i > 0)
#pragma unroll
          for (int e = 0; e < EP; ++e) form_p(kb, (i - 1) * EP + e);
      }
    }
    constexpr int ED = 16 / (2 * NB);  // elements per op of a dQ phase
#pragma unroll
    for (int i = 0; i < 4 * NB; ++i) {
      sched_fence();
      rd(4 * KSN + i + PF);
      dq_acc[i % NB] = mfma32(g[i], sb[i / NB], dq_acc[i % NB]);
      if (i == 0)
#pragma unroll
        for (int e = 0; e < EP; ++e) form_p(1, (KSN - 1) * EP + e);
      else if (i < 2 * NB)
#pragma unroll
        for (int e = 0; e < ED; ++e) form_ds(1, (i - 1) * ED + e);
      if (i == 2 * NB - 1) {
#pragma unroll
        for (int e = 0; e < ED; ++e) form_ds(1, (2 * NB - 1) * ED + e);
        sb[2] = operand(dp[1], 0);
        sb[3] = operand(dp[1], 1);
      }
    }
    sched_fence();
    st ^= 1;
    kt = kn;
  }

  wait_all_memory();  // no copy outlives the workgroup

  if (tail) {  // partial dQ of this lane's query row
    float* pq = a.tail_part + (((size_t)ti.slot * a.tail_chunks + ti.chunk) * kDqBM + (qi - rb.r0)) * D;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 t = {dq_acc[db][4 * j + 0] * a.scale, dq_acc[db][4 * j + 1] * a.scale,
                         dq_acc[db][4 * j + 2] * a.scale, dq_acc[db][4 * j + 3] * a.scale};
        *(f32x4*)(pq + db * 32 + 8 * j + 4 * hi) = t;
      }
  } else if (qi < rb.r1) {
    __bf16* qp = a.dq + base + (size_t)qi * tok;
    const float* fp = a.dq_acc ? a.dq_acc + base + (size_t)qi * tok : nullptr;  // the fused keys' share
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        f32x4 x = {dq_acc[db][4 * j + 0], dq_acc[db][4 * j + 1], dq_acc[db][4 * j + 2], dq_acc[db][4 * j + 3]};
        if (fp) x += *(const f32x4*)(fp + db * 32 + 8 * j + 4 * hi);
        bf16x4 t = {(__bf16)(x[0] * a.scale), (__bf16)(x[1] * a.scale), (__bf16)(x[2] * a.scale),
                    (__bf16)(x[3] * a.scale)};
        *(bf16x4*)(qp + db * 32 + 8 * j + 4 * hi) = t;
      }
  }
}

// Joint tail of the dQ kernel: dQ of the split items as the sum of their chunks' partials.
template <int D>
__global__ void tail_reduce_dq_kernel(const float* part, __bf16* dq, int B, int H, int N, int items, int chunks,
                                      const float* dq_acc, float scale) {
  const int nblk = (N + kDqBM - 1) / kDqBM;
  const size_t total = (size_t)items * kDqBM * (D / 4);
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int d = (int)(i % (D / 4)) * 4;
  const int k = (int)((i / (D / 4)) % kDqBM);
  const int slot = (int)(i / ((size_t)(D / 4) * kDqBM));
  const int item = nblk * H * B - items + slot;
  const int row = (item % nblk) * kDqBM + k;
  if (row >= N) return;
  const int h = (item / nblk) % H, b = item / (nblk * H);
  f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int c = 0; c < chunks; ++c) s += *(const f32x4*)(part + (((size_t)slot * chunks + c) * kDqBM + k) * D + d);
  const size_t off = (((size_t)b * N + row) * H + h) * D + d;
  if (dq_acc) s += scale * *(const f32x4*)(dq_acc + off);  // the fused keys' share (unscaled)
  *(bf16x4*)(dq + off) = bf16x4{(__bf16)s[0], (__bf16)s[1], (__bf16)s[2], (__bf16)s[3]};
}

}  // namespace

hipError_t launch_bwd_prepare(const __bf16* o, const float* lse, const __bf16* dout, float* dd, float* nls, int B,
                              int H, int N, int Npad, int head_dim, float scale, float* zero_acc, hipStream_t s) {
  const size_t threads = std::max((size_t)B * N * H * (head_dim / 8), (size_t)B * H * (Npad - N));
  dim3 grid((unsigned)((threads + 255) / 256));
  if (head_dim == 128)
    hipLaunchKernelGGL(bwd_prepare_kernel<128>, grid, dim3(256), 0, s, o, lse, dout, dd, nls, B, H, N, Npad, 1.0f / scale,
                       zero_acc);
  else
    hipLaunchKernelGGL(bwd_prepare_kernel<64>, grid, dim3(256), 0, s, o, lse, dout, dd, nls, B, H, N, Npad, 1.0f / scale,
                       zero_acc);
  return hipGetLastError();
}

hipError_t launch_bwd_dkdv(const DkdvArgs& a, int head_dim, hipStream_t s) {
  const bool spatial = a.frame_len > 0;
  const bool split = spatial && a.text_chunks > 1;
  const int nblk = row_blocks(a.N, a.T, spatial ? a.frame_len : 0, kBKV, true);
  // Spatial: 3-D grid renumbered by XCD. Joint: 1-D grid of items, the split tail last.
  dim3 grid = spatial ? dim3(nblk + (split ? (a.text_chunks - 1) * a.text_blocks : 0), a.H, a.B)
                      : dim3(nblk * a.H * a.B + a.tail_blocks * (a.tail_chunks - 1));
  const bool fused = a.dq_acc != nullptr;
  if (fused && a.zero_acc) {
    const hipError_t e = launch_zero_f32(a.dq_acc, (size_t)a.B * a.N * a.H * head_dim, s);
    if (e != hipSuccess) return e;
  }
  if (head_dim == 128 && spatial && fused)
    hipLaunchKernelGGL((bwd_dkdv_kernel<128, true, true>), grid, dim3(64 * kDkdvWaves), 0, s, a);
  else if (head_dim == 128 && spatial)
    hipLaunchKernelGGL((bwd_dkdv_kernel<128, true, false>), grid, dim3(64 * kDkdvWaves), 0, s, a);
  else if (head_dim == 128 && fused)
    hipLaunchKernelGGL((bwd_dkdv_kernel<128, false, true>), grid, dim3(64 * kDkdvWaves), 0, s, a);
  else if (head_dim == 128)
    hipLaunchKernelGGL((bwd_dkdv_kernel<128, false, false>), grid, dim3(64 * kDkdvWaves), 0, s, a);
  else if (spatial && fused)
    hipLaunchKernelGGL((bwd_dkdv_kernel<64, true, true>), grid, dim3(64 * kDkdvWaves), 0, s, a);
  else if (spatial)
    hipLaunchKernelGGL((bwd_dkdv_kernel<64, true, false>), grid, dim3(64 * kDkdvWaves), 0, s, a);
  else if (fused)
    hipLaunchKernelGGL((bwd_dkdv_kernel<64, false, true>), grid, dim3(64 * kDkdvWaves), 0, s, a);
  else
    hipLaunchKernelGGL((bwd_dkdv_kernel<64, false, false>), grid, dim3(64 * kDkdvWaves), 0, s, a);
  if (!spatial && a.tail_blocks > 0) {
    const size_t threads = (size_t)a.tail_blocks * kBKV * (head_dim / 4);
    dim3 rgrid((unsigned)((threads + 255) / 256));
    if (head_dim == 128)
      hipLaunchKernelGGL(tail_reduce_kernel<128>, rgrid, dim3(256), 0, s, a.tail_part, a.dk, a.dv, a.B, a.H, a.N,
                         a.tail_blocks, a.tail_chunks);
    else
      hipLaunchKernelGGL(tail_reduce_kernel<64>, rgrid, dim3(256), 0, s, a.tail_part, a.dk, a.dv, a.B, a.H, a.N,
                         a.tail_blocks, a.tail_chunks);
  }
  if (split) {
    const int rows = a.text_blocks * kBKV;
    const int nrow = std::min(a.T, a.N);  // the text keys
    const size_t threads = (size_t)a.B * a.H * nrow * (head_dim / 4);
    dim3 rgrid((unsigned)((threads + 255) / 256));
    if (head_dim == 128)
      hipLaunchKernelGGL(text_reduce_kernel<128>, rgrid, dim3(256), 0, s, a.text_part, a.dk, a.dv, a.B, a.H, a.N,
                         rows, nrow, a.text_chunks);
    else
      hipLaunchKernelGGL(text_reduce_kernel<64>, rgrid, dim3(256), 0, s, a.text_part, a.dk, a.dv, a.B, a.H, a.N,
                         rows, nrow, a.text_chunks);
  }
  return hipGetLastError();
}

hipError_t launch_bwd_dq(const DqArgs& args, int head_dim, hipStream_t s) {
  DqArgs a = args;
  const int nblk = row_blocks(a.N, a.T, a.frame_len, kDqBM, false);
  int text_rows = a.T;  // of them in the spatial kernel's grid
  if (a.frame_len) {
    const hipError_t e = place_text_rows(TextRows{a.dq, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr}, a.B, a.H, a.N, a.T,
                                         head_dim, (size_t)nblk * a.H * a.B * 64 * kDqWaves, s, &text_rows);
    if (e != hipSuccess) return e;
  }
  // Spatial: 3-D grid renumbered by XCD. Joint: 1-D grid of items, the split tail last.
  dim3 grid = a.frame_len ? dim3(nblk, a.H, a.B) : dim3(nblk * a.H * a.B + a.tail_blocks * (a.tail_chunks - 1));
  if (a.frame_len && !text_rows) a.B = 0;
  const bool km = a.key_mask != nullptr;
  if (head_dim == 128 && km)
    hipLaunchKernelGGL((bwd_dq_kernel<128, true>), grid, dim3(64 * kDqWaves), 0, s, a);
  else if (head_dim == 128)
    hipLaunchKernelGGL((bwd_dq_kernel<128, false>), grid, dim3(64 * kDqWaves), 0, s, a);
  else if (km)
    hipLaunchKernelGGL((bwd_dq_kernel<64, true>), grid, dim3(64 * kDqWaves), 0, s, a);
  else
    hipLaunchKernelGGL((bwd_dq_kernel<64, false>), grid, dim3(64 * kDqWaves), 0, s, a);
  if (!a.frame_len && a.tail_blocks > 0) {
    const size_t threads = (size_t)a.tail_blocks * kDqBM * (head_dim / 4);
    dim3 rgrid((unsigned)((threads + 255) / 256));
    if (head_dim == 128)
      hipLaunchKernelGGL(tail_reduce_dq_kernel<128>, rgrid, dim3(256), 0, s, a.tail_part, a.dq, a.B, a.H, a.N,
                         a.tail_blocks, a.tail_chunks, a.dq_acc, a.scale);
    else
      hipLaunchKernelGGL(tail_reduce_dq_kernel<64>, rgrid, dim3(256), 0, s, a.tail_part, a.dq, a.B, a.H, a.N,
                         a.tail_blocks, a.tail_chunks, a.dq_acc, a.scale);
  }
  return hipGetLastError();
}

}  // namespace vcja
