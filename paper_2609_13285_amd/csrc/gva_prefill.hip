// libgva.so -- causal prefill of GVA (Algorithm 1 for every prompt position at
// once): prefill_lds_kernel (key tiles shared through LDS, the absorption
// fused), prefill_bf16_kernel (the waves of a workgroup split its key tiles,
// for launches of few workgroups), gva_prefill, gva_prefill_attention and the
// matched-GQA baseline gva_gqa_prefill_attention.

#include <cfloat>
#include <type_traits>

#include "gva_common.h"

namespace {

// =============================================================== prefill
// Causal attention for the last N cached rows of every sequence (a prompt,
// after any cached prefix): query i of sequence b sits at position
// p = L_b - N + i and sees rows 0..p (Algorithm 1's loop for every prompt
// position at once; Section 3.3's absorbed scores).  Unlike a decode step
// this is a dense contraction: a workgroup takes C (position, head)
// columns of one group -- C / (H/G) consecutive positions times the H/G
// heads that share the group's value rows; C = 64, or 32 at d_v = 128 to
// stay within 256 registers -- and its four waves split the key tiles up to
// the block's last position.  Per 32-row key tile a wave forms the scores
// of all C columns on the matrix cores (keys = [V | k_r] rows as stored),
// masks rows past each column's position, updates the online softmax and
// accumulates P.V (V transposed once per tile with the identity MFMA,
// shared by the column blocks).
// Precision.  The absorbed and rotated queries enter the score product as
// bf16 high + low pairs (x = hi + lo to ~2^-16 of x, as in the decode
// kernel): a single bf16 query moves every logit by up to 2^-9 of its size,
// an error that grows with the sharpness of the scores.  The high parts
// stay in registers; the low parts, the same for every tile and every wave
// of the workgroup, are read from LDS each tile (registers are the limit).
// A positional slice of at most 16 entries fills half of its 32-wide
// K-chunk, so its low part rides in the other half of the same product.
// P.V runs in fp16: the transposed rows come out of the identity product in
// fp32 and every bf16 value of magnitude 2^-14 .. 65504 is exact in fp16,
// while the weights in [0, 1] keep 3 more bits than bf16.
// The waves merge through LDS.
// Query blocks are dealt longest first, so the triangle's tail is short.
// GQA = true is the matched grouped-query prefill the paper compares
// against: scores read an explicit key stream, no positional term; its
// queries take the same high + low pairs.
// (position, head) columns per workgroup: 64, fewer where a wider value
// row (or the baseline's separate key tile) needs the registers
__host__ __device__ constexpr int prefill_cols(int dv, bool gqa) { return dv >= 128 ? (gqa ? 16 : 32) : 64; }

struct PrefillParams {
  const float* q_abs;     // [B][N][H][d_v]: absorbed queries (GQA: the raw query)
  const float* q_rot;     // [B][N][H][d_r]: rotated positional queries
  const void* v;          // tiled caches, the prompt's rows already appended
  const void* kr;
  const void* k_gqa;      // matched-GQA baseline: explicit key stream (tiled like v)
  const int32_t* lens;
  float* o;               // [B][N][H][d_v]
  float* lse;             // [B][N][H]
  int32_t B, H, G, N, d_r, t_max, n_qblocks;
  float scale_log2;
  const void* q;          // fused absorption: the raw query [B][N][H][d_c + d_r] and the
  const void* m;          // maps [H][d_v][d_c] (q_abs and q_rot NULL)
  int32_t d_c;
  double inv_freq[kMaxPairs];
};

constexpr float kLazyMax = 8.f;

// Two workgroups per CU where the registers allow it without spilling.
constexpr int prefill_min_blocks(int nrc) { return nrc >= 2 ? 1 : 2; }

// KPACK: the positional slice has at most 16 entries (one K-chunk, half
// used), so its low part shares that chunk.
template <int HPG, int DV, int NRC, bool GQA, bool KPACK>
__global__ void __launch_bounds__(kThreads, prefill_min_blocks(NRC)) prefill_bf16_kernel(PrefillParams p) {
  static_assert(!KPACK || NRC == 1, "a packed positional chunk is a single chunk");
  constexpr int COLS = prefill_cols(DV, GQA), NC = DV / 32, NB = DV / 16, CB = COLS / 16;
  constexpr int QB = COLS / HPG;               // positions per workgroup
  constexpr int DEPTH = 2;
  constexpr int RS = DV + 2;                   // per-(wave, column) record: [m, l, o[DV]]
  constexpr int NLO = NC + (KPACK ? 0 : NRC);  // low-part K-chunks read from LDS per column block
  constexpr int RED_FLOATS = kWaves * COLS * RS;
  constexpr int LO_FLOATS = CB * NLO * 64 * 4; // bf16x8 per lane, [cb][chunk][lane]
  // the low parts are read during the key loop, the records only after it
  __shared__ __attribute__((aligned(16))) float lds[RED_FLOATS > LO_FLOATS ? RED_FLOATS : LO_FLOATS];
  float* red = lds;
  bf16x8* lo_lds = reinterpret_cast<bf16x8*>(lds);

  const int nbg = p.B * p.G;
  const int x = blockIdx.x;
  const int qb = p.n_qblocks - 1 - x / nbg;    // longest query blocks first
  const int b = (x % nbg) / p.G, g = (x % nbg) % p.G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, qd = lane >> 4;
  const int h0 = g * HPG;
  const bf16x8 zero8 = as_bf16x8(u32x4{0u, 0u, 0u, 0u});

  const int L = clamp_len(p.lens, b, p.t_max);
  const int i_end = min(p.N, (qb + 1) * QB);
  const int kend = L - p.N + i_end;            // rows the block's last position sees
  // column 16 cb + n of this lane: position i = qb QB + col / HPG, head
  // h0 + col % HPG; pos[cb] = its position, or -1 if it has none
  int pos[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int col = 16 * cb + n;
    const int i = qb * QB + col / HPG;
    const int ps = L - p.N + i;
    pos[cb] = (i < p.N && ps >= 0) ? ps : -1;
  }
  const int p_first = L - p.N + qb * QB;       // the block's first position

  // ---- key tiles: rows [0, kend), read through descriptors that end at
  // the last layout tile (reads past it return zeros)
  const int kend16 = kend > 0 ? ((kend + kLayoutRows - 1) / kLayoutRows) * kLayoutRows : 0;
  const uint16_t* vbase = static_cast<const uint16_t*>(p.v) + ((int64_t)b * p.G + g) * p.t_max * DV;
  const uint16_t* kbase = static_cast<const uint16_t*>(p.kr) + (int64_t)b * p.t_max * p.d_r;
  const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(vbase), (short)0, kend16 * DV * 2, kBufferWord3);
  const __amdgpu_buffer_rsrc_t kres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(kbase), (short)0, NRC > 0 ? kend16 * p.d_r * 2 : 0, kBufferWord3);
  const __amdgpu_buffer_rsrc_t kcres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(GQA ? static_cast<const void*>(static_cast<const uint16_t*>(p.k_gqa) +
                                                       ((int64_t)b * p.G + g) * p.t_max * DV)
                            : static_cast<const void*>(vbase)),
      (short)0, kend16 * DV * 2, kBufferWord3);
  const int kpieces = p.d_r / 8;
  const int v_lane = qd * 256 + n * 16;
  // positional K-slots: piece qd of the row (lanes past d_r re-read a valid
  // piece against a zero query); packed, slots kpieces .. 2 kpieces - 1
  // repeat the row's pieces for the query's low part
  int k_lane[NRC > 0 ? NRC : 1];
#pragma unroll
  for (int rc = 0; rc < NRC; ++rc) {
    const int piece = KPACK ? (qd < 2 * kpieces ? qd % kpieces : 0) : min(4 * rc + qd, kpieces - 1);
    k_lane[rc] = piece * 256 + n * 16;
  }
  const int v_tile_bytes = 16 * DV * 2, k_tile_bytes = 16 * p.d_r * 2;
  const int ntiles = kend > 0 ? (kend + kTileRows - 1) / kTileRows : 0;
  const int my_tiles = ntiles > w ? (ntiles - w + kWaves - 1) / kWaves : 0;
  auto tile_row = [&](int j) { return (w + kWaves * j) * kTileRows; };
  using TileT = Tile<DV, NRC, GQA>;
  auto load_tile = [&](TileT& t, int row0) {
    const int lt = row0 / kLayoutRows;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const int vsoff = (lt + hf) * v_tile_bytes;
      if constexpr (GQA) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
          t.kc[hf][c] = as_bf16x8(__builtin_amdgcn_raw_buffer_load_b128(kcres, v_lane + 1024 * c, vsoff, 0));
      }
#pragma unroll
      for (int c = 0; c < NC; ++c)
        t.v[hf][c] = as_bf16x8(__builtin_amdgcn_raw_buffer_load_b128(vres, v_lane + 1024 * c, vsoff, 0));
#pragma unroll
      for (int rc = 0; rc < NRC; ++rc)
        t.k[hf][rc] = as_bf16x8(__builtin_amdgcn_raw_buffer_load_b128(kres, k_lane[rc], (lt + hf) * k_tile_bytes, 0));
    }
  };
  TileT buf[DEPTH];
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d) {
    load_tile(buf[d], tile_row(d));
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- the queries as bf16 high + low B operands (zero for columns with
  // no position).  Every wave forms the high parts of all the workgroup's
  // columns; the low parts go to LDS, each chunk written by one wave.
  bf16x8 bq[CB][NC];
  bf16x8 bk[CB][NRC > 0 ? NRC : 1];
  auto put_lo = [&](int cb, int c, const float* xv, bool live) {
    if ((cb * NLO + c) % kWaves == w) lo_lds[(cb * NLO + c) * 64 + lane] = live ? split_hi_lo(xv, true) : zero8;
  };
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int col = 16 * cb + n;
    const int i = min(qb * QB + col / HPG, p.N - 1);
    const int64_t qrow = ((int64_t)b * p.N + i) * p.H + h0 + col % HPG;
    const float* qa = p.q_abs + qrow * DV + 8 * qd;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const f32x4 u0 = *reinterpret_cast<const f32x4*>(qa + 32 * c);
      const f32x4 u1 = *reinterpret_cast<const f32x4*>(qa + 32 * c + 4);
      float xv[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        xv[j] = u0[j] * p.scale_log2;
        xv[4 + j] = u1[j] * p.scale_log2;
      }
      bq[cb][c] = pos[cb] >= 0 ? split_hi_lo(xv, false) : zero8;
      put_lo(cb, c, xv, pos[cb] >= 0);
    }
#pragma unroll
    for (int rc = 0; rc < NRC; ++rc) {
      // the positional piece this lane's K-slot carries: high part of piece
      // 4 rc + qd, or (packed) the low part of piece qd - kpieces
      const bool hi_slot = KPACK ? qd < kpieces : 32 * rc + 8 * qd < p.d_r;
      const bool lo_slot = KPACK && qd >= kpieces && qd < 2 * kpieces;
      const int j0 = KPACK ? 8 * (lo_slot ? qd - kpieces : qd) : 32 * rc + 8 * qd;
      float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (hi_slot || lo_slot) {
        const float* qr = p.q_rot + qrow * p.d_r + j0;
        const f32x4 u0 = *reinterpret_cast<const f32x4*>(qr);
        const f32x4 u1 = *reinterpret_cast<const f32x4*>(qr + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          xv[j] = u0[j] * p.scale_log2;
          xv[4 + j] = u1[j] * p.scale_log2;
        }
      }
      bk[cb][rc] = (pos[cb] >= 0 && (hi_slot || lo_slot)) ? split_hi_lo(xv, lo_slot) : zero8;
      if constexpr (!KPACK) put_lo(cb, NC + rc, xv, pos[cb] >= 0 && hi_slot);
    }
  }
  __syncthreads();                             // the low parts are in LDS

  bf16x8 esel[2];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    u32x4 u = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (8 * qd + j == n + 16 * half) u[j >> 1] |= 0x3F80u << (16 * (j & 1));
    esel[half] = as_bf16x8(u);
  }

  float m_run[CB], l_run[CB];
  f32x4 acc[CB][NB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    m_run[cb] = -INFINITY;
    l_run[cb] = 0.f;
#pragma unroll
    for (int ib = 0; ib < NB; ++ib) acc[cb][ib] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  auto compute_tile = [&](TileT& t, int row0) {
    if (row0 + kTileRows > kend) {             // rows past the block's keys: zero
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const bool dead = row0 + 16 * hf + n >= kend;
#pragma unroll
        for (int c = 0; c < NC; ++c) t.v[hf][c] = dead ? zero8 : t.v[hf][c];
        if constexpr (GQA) {
#pragma unroll
          for (int c = 0; c < NC; ++c) t.kc[hf][c] = dead ? zero8 : t.kc[hf][c];
        }
#pragma unroll
        for (int rc = 0; rc < NRC; ++rc) t.k[hf][rc] = dead ? zero8 : t.k[hf][rc];
      }
    }
    const bool masked = row0 + kTileRows - 1 > p_first;   // some column may not see every row
    // the LDS offset is opaque to the compiler, so the low parts are read
    // here, tile by tile, instead of being hoisted into registers
    int lo_off = lane;
    asm volatile("" : "+v"(lo_off));
    // scores of one column block: the high and the low query parts
    // accumulate into one sum per 16-row half
    auto scores = [&](int cb, f32x4 (&sc)[2]) {
      bf16x8 lo[NLO];
#pragma unroll
      for (int c = 0; c < NLO; ++c) lo[c] = lo_lds[(cb * NLO + c) * 64 + lo_off];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        sc[hf] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          sc[hf] = mfma16(GQA ? t.kc[hf][c] : t.v[hf][c], bq[cb][c], sc[hf]);
          sc[hf] = mfma16(GQA ? t.kc[hf][c] : t.v[hf][c], lo[c], sc[hf]);
        }
#pragma unroll
        for (int rc = 0; rc < NRC; ++rc) {
          sc[hf] = mfma16(t.k[hf][rc], bk[cb][rc], sc[hf]);
          if constexpr (!KPACK) sc[hf] = mfma16(t.k[hf][rc], lo[NC + rc], sc[hf]);
        }
      }
    };
    // the online softmax of one column block, its weights as fp16
    auto softmax = [&](int cb, const f32x4 (&sc)[2]) {
      float xv[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) xv[k] = sc[k >> 2][k & 3];
      if (masked) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (row0 + 16 * (k >> 2) + 4 * qd + (k & 3) > pos[cb]) xv[k] = -INFINITY;
      }
      float mt = xv[0];
#pragma unroll
      for (int k = 1; k < 8; ++k) mt = fmaxf(mt, xv[k]);
      mt = max_over_rows(mt);
      const float m_new = fmaxf(m_run[cb], mt);
      // The running maximum moves only once some column's tile maximum
      // exceeds it by more than kLazyMax (log2 units): the weights then stay
      // below 2^kLazyMax (fp16 holds them; the sums are fp32), and the
      // accumulators are rescaled on few tiles.
      if (__ballot(mt > m_run[cb] + kLazyMax) != 0) {
        // columns whose rows so far are all masked keep m = -inf: scale 1
        const float alpha = m_new > m_run[cb] ? __builtin_amdgcn_exp2f(m_run[cb] - m_new) : 1.f;
        l_run[cb] *= alpha;
#pragma unroll
        for (int ib = 0; ib < NB; ++ib) acc[cb][ib] *= alpha;
        m_run[cb] = m_new;
      }
      const float m_use = m_run[cb] == -INFINITY ? 0.f : m_run[cb];   // all masked so far
      float pr[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        pr[k] = __builtin_amdgcn_exp2f(xv[k] - m_use);
        l_run[cb] += pr[k];
      }
      return to_f16x8(pr);
    };
    // The next column block's score products are issued before this
    // block's softmax, so the matrix cores run them while the vector units
    // work (the order is pinned by scheduling barriers).
    f16x8 bp[CB];
    f32x4 sc[2][2];
    scores(0, sc[0]);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      if (cb + 1 < CB) scores(cb + 1, sc[(cb + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      bp[cb] = softmax(cb, sc[cb & 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // P.V over the 2 NC 16-wide output blocks; the identity products that
    // transpose block k + 1 of V are issued before block k's conversion to
    // fp16 and its products
    auto transpose = [&](int k, f32x4 (&tq)[2]) {
      const int c = k >> 1, half = k & 1;
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      tq[0] = mfma16(t.v[0][c], esel[half], z);
      tq[1] = mfma16(t.v[1][c], esel[half], z);
    };
    f32x4 tq[2][2];
    transpose(0, tq[0]);
#pragma unroll
    for (int k = 0; k < 2 * NC; ++k) {
      if (k + 1 < 2 * NC) transpose(k + 1, tq[(k + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      const f32x4* tk = tq[k & 1];
      const float tv[8] = {tk[0][0], tk[0][1], tk[0][2], tk[0][3], tk[1][0], tk[1][1], tk[1][2], tk[1][3]};
      const f16x8 av = to_f16x8(tv);           // bf16 values: exact in fp16 at these magnitudes
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[cb][k] = mfma16(av, bp[cb], acc[cb][k]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  for (int jt = 0; jt < my_tiles; jt += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const int j = jt + d;
      if (j >= my_tiles) break;
      load_tile(buf[(d + DEPTH - 1) % DEPTH], tile_row(j + DEPTH - 1));
      __builtin_amdgcn_sched_barrier(0);
      compute_tile(buf[d], tile_row(j));
    }
  }

  // ---- merge the waves: per column the records (m, l, o) of the 4 waves
  __syncthreads();                             // every wave is done with the low parts
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const float l = sum_over_rows(l_run[cb]);
    float* rec = red + (w * COLS + 16 * cb + n) * RS;
    if (qd == 0) {
      rec[0] = m_run[cb];
      rec[1] = l;
    }
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) rec[2 + 16 * ib + 4 * qd + jj] = acc[cb][ib][jj];
  }
  __syncthreads();
  for (int idx = tid; idx < COLS * DV; idx += kThreads) {
    const int col = idx / DV, i = idx % DV;
    const int qi = qb * QB + col / HPG;
    if (qi >= p.N) continue;
    float mx = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) mx = fmaxf(mx, red[(ww * COLS + col) * RS]);
    float o = 0.f, lsum = 0.f;
    if (mx != -INFINITY && L - p.N + qi >= 0) {
#pragma unroll
      for (int ww = 0; ww < kWaves; ++ww) {
        const float* rec = red + (ww * COLS + col) * RS;
        if (rec[0] == -INFINITY) continue;       // this wave saw no row of the column
        const float sc = __builtin_amdgcn_exp2f(rec[0] - mx);
        lsum += rec[1] * sc;
        o += rec[2 + i] * sc;
      }
      o /= lsum;
    } else {
      mx = -INFINITY;
    }
    const int64_t orow = ((int64_t)b * p.N + qi) * p.H + h0 + col % HPG;
    __builtin_nontemporal_store(o, p.o + orow * DV + i);   // written once: kept out of the L2
    if (i == 0) p.lse[orow] = mx == -INFINITY ? -INFINITY : (mx + log2f(lsum)) * kLn2;
  }
}

using PrefillFn = void (*)(PrefillParams);

constexpr int kPrefillCols = 128;             // (position, head) columns per workgroup of prefill_lds_kernel

// ------------------------------------------ prefill, key tiles shared in LDS
// The prompt kernel.  A workgroup takes 128 (position, head) columns of one
// group, 32 per wave (a wave's columns: 32 positions of one head, or 16 of
// each of two at H/G = 8), and its four waves walk the key tiles together;
// with KS = 2 a second set of four waves takes every other tile of the same
// columns and the two are merged at the end.
//
// Per 32-row tile, on 32x32x16 products (lane = column, registers = rows):
//  - the tile's value and positional-key rows are copied into LDS by the
//    waves, a quarter each, two tiles ahead (buffer loads straight to LDS,
//    three buffers), so no wave holds a tile in registers and each row is
//    requested once per workgroup;
//  - every wave reads them as A operands for its scores S^T = [V | kr] q^T,
//    the query's bf16 high and low parts both in registers as B operands;
//  - wave w turns value block w (at d_v = 64, waves 0 and 1) into V^T in fp16
//    with identity products and puts it in LDS for all four (two buffers), in
//    the row order in which the score registers lie, so a wave's softmax
//    weights are the B operand of its P.V as they are;
//  - the softmax and P.V run one tile behind the scores: the previous tile's
//    exponentials stand between this tile's score products, this tile's maxima
//    between the previous tile's P.V.  (Two or three vector instructions
//    beside a 32x32x16 product are nearly free, a run of them between products
//    costs its full time: softmax and P.V of one tile together, after its
//    scores, took 80.9 us where this takes 76.5, four 2048-token prompts at
//    H16 G4 d 64/16 with their append, and 200.6 against 196.7 for the
//    baseline below.)
// One barrier per tile.
//
// What bounds it: at d_v = 128 the matrix cores' power.  They are busy 70% of
// the cycles, at which the clock settles at 1.7 GHz (a large bf16 library
// product: 69% at 1.9 GHz).  At d_v = 64, busy 44% at 2.0 GHz, the softmax,
// twice as much per product, and each workgroup's start.  Measured, append and
// prompt from the raw queries against the separate absorption and the kernels
// before: H32 G8 d 128/16, 8192 tokens 900 -> 778 us; H16 G4 d 64/16, four
// 2048-token prompts 141 -> 76.7 us; the matched-GQA baseline at H32 G8 d 128,
// 4096 tokens 311 -> 193 us.  Registers: d_v = 128 takes all of two waves per
// SIMD, and its instances of two and four positional chunks keep 8 or 9 and 26
// to 28 of them in scratch around the key loop (none inside it); d_v = 64 with
// d_r <= 16 takes 161 to 163, so three workgroups of one set fit a CU.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma32(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ i32x4 buffer_desc(const void* p, int bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)p;
  return i32x4{(int)(uint32_t)a, (int)((a >> 32) & 0xFFFFu), bytes, kBufferWord3};
}

// One wave copies 1 KB into LDS, 16 bytes per lane in lane order: bytes
// [soff, soff + 1024) behind the descriptor (zeros past its end) to LDS
// address dst.  In asm because the compiler, which cannot tell the tile
// buffers apart, would otherwise drain every copy in flight before each LDS
// read; the kernel waits for its own copies (wait_copies) before the barrier
// that hands a tile over.  The copy writes no register but m0.
__device__ __forceinline__ void copy_kb(i32x4 desc, uint32_t dst, int voff, int soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               ::"s"(dst), "v"(voff), "s"(desc), "s"(soff)
               : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_copies() {   // until at most N of this wave's copies are in flight
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The weights of the first kLowRows rows take a second, low part through P.V.
// A short row of outputs is a sum of few weights, whose roundings to fp16 then
// do not average out: with one running maximum per column (the tile-split
// kernel has four, one per wave, and each makes one weight exact) the error of
// short prompts was 5 to 16% above the tile-split kernel's.  With it the
// rounding of the first 128 rows, where those four lie, is gone (off a 64-bit
// evaluation, tile-split, without and with it: four 2048-token prompts at H16
// G4 d 64/16 1.01e-4, 1.10e-4, 7.3e-5; 512 tokens 1.17e-4, 1.32e-4, 6.2e-5).
// It costs the 350M prompts 77.2 -> 80.9 us, 8192 tokens 752 -> 766.
constexpr int kLowRows = 128;
// The maximum's own weight is exact, so with sharp scores, whose outputs hang
// on few weights, it moves sooner than the tile-split kernel's four do: at 8,
// queries of 6 times the usual size came out up to 1.48 times as far off as
// there, at 4 nowhere further (70 shapes at 1, 2.5 and 6 times; 0.50, 0.57 and
// 0.62 of its error on average; at 10 times 7 of 70, up to 1.13).  8192 tokens 812 and 819 us, four 350M prompts
// 77.4 and 78.1; at 2, 836 and 79.5.
constexpr float kLdsLazyMax = 4.f;

// The workgroup's barrier, which alone orders no memory access for the
// compiler: accesses stay on their side of it.
__device__ __forceinline__ void tile_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// LDS written by this wave's lanes is readable by its others from here on,
// and what they have read may be written again.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// row of a 32-row tile in score register r of a lane in half h
__device__ __forceinline__ constexpr int score_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

template <int DV, int NRC, bool GQA, int KS>
struct PrefillCfg {
  static constexpr int NCH = DV / 16;                      // 16-wide K-chunks of a value row
  static constexpr int NIB = DV / 32;                      // 32-wide output blocks
  static constexpr int V_BYTES = kTileRows * DV * 2;
  static constexpr int KB = V_BYTES / 1024;                // KB per value tile
  static constexpr int TILE_BYTES = V_BYTES * (GQA ? 2 : 1) + NRC * 1024;
  static constexpr int VT_BYTES = V_BYTES;
  static constexpr int GROUP_BYTES = 3 * TILE_BYTES + 2 * VT_BYTES;   // one set of four waves
  // operands read from LDS ahead of their products: of the scores, and of the
  // P.V's V^T before it begins (fewer where the positional chunks hold the registers)
  static constexpr int READ_AHEAD = DV >= 128 && NRC > 1 ? 3 : 4;
  static constexpr int VT_AHEAD = DV >= 128 && NRC > 1 ? 2 : 4;
  static constexpr int COPIES = KB / 4 * (GQA ? 2 : 1) + (NRC > 0 ? 1 : 0);   // per wave and tile
  static constexpr int MERGE_BYTES = KS > 1 ? kWaves * 64 * (NIB * 16 + 2) * 4 : 0;
  static constexpr int LDS = KS * GROUP_BYTES > MERGE_BYTES ? KS * GROUP_BYTES : MERGE_BYTES;
  static_assert(GROUP_BYTES >= kWaves * 32 * 36 * 4, "the outputs pass through the tiles' LDS");
};

template <int DV, int NRC, bool GQA, int KS>
__global__ void __launch_bounds__(256 * KS, 2) prefill_lds_kernel(PrefillParams p) {
  using Cfg = PrefillCfg<DV, NRC, GQA, KS>;
  static_assert(!GQA || NRC == 0, "the GQA baseline has no positional term");
  constexpr int NCH = Cfg::NCH, NIB = Cfg::NIB, RA = Cfg::READ_AHEAD, VA = Cfg::VT_AHEAD;
  __shared__ __attribute__((aligned(1024))) char lds[Cfg::LDS];

  const int hpg = p.H / p.G;
  const int nbg = p.B * p.G;
  const int x = blockIdx.x;
  const int qb = p.n_qblocks - 1 - x / nbg;    // longest query blocks first
  const int b = (x % nbg) / p.G, g = (x % nbg) % p.G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = KS > 1 ? wave >> 2 : 0, w = wave & 3;
  const int n = lane & 31, h = lane >> 5;      // column, and half of the rows / K-chunk
  const bf16x8 zero8 = as_bf16x8(u32x4{0u, 0u, 0u, 0u});

  // ---- this wave's columns: position i (of the prompt), head
  const int ppb = kPrefillCols / hpg;          // positions per workgroup
  const int wpos = qb * ppb + (hpg < 4 ? (w / hpg) * 32 : 0);   // the wave's first position
  const int head = g * hpg + (hpg < 4 ? w % hpg : (hpg == 4 ? w : 2 * w + (n >> 4)));
  const int i_col = wpos + (hpg == 8 ? n & 15 : n);
  const int L = clamp_len(p.lens, b, p.t_max);
  const int kend = L - p.N + min(p.N, (qb + 1) * ppb);          // rows the block's last position sees
  const int p_first = L - p.N + wpos;
  const int pos = (i_col < p.N && L - p.N + i_col >= 0) ? L - p.N + i_col : -1;
  const int64_t qrow = ((int64_t)b * p.N + min(i_col, p.N - 1)) * p.H + head;

  // ---- tile copies.  The descriptors end at the last layout tile.
  const int kend16 = kend > 0 ? (kend + kLayoutRows - 1) / kLayoutRows * kLayoutRows : 0;
  const int64_t vstream = ((int64_t)b * p.G + g) * p.t_max * DV;
  const i32x4 vdesc = buffer_desc(static_cast<const uint16_t*>(p.v) + vstream, kend16 * DV * 2);
  const i32x4 kcdesc = buffer_desc(GQA ? static_cast<const uint16_t*>(p.k_gqa) + vstream : nullptr, kend16 * DV * 2);
  const i32x4 kdesc = buffer_desc(static_cast<const uint16_t*>(p.kr) + (int64_t)b * p.t_max * p.d_r,
                                  NRC > 0 ? kend16 * p.d_r * 2 : 0);
  char* const grp_lds = lds + grp * Cfg::GROUP_BYTES;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)grp_lds;
  const int ntiles = kend > 0 ? (kend + kTileRows - 1) / kTileRows : 0;
  const int nit = (ntiles + KS - 1) / KS;      // the same for both sets of waves (they share the barriers)
  auto tile_row = [&](int j) { return (KS * j + grp) * kTileRows; };
  auto copy_tile = [&](int row0, int buf) {
    const uint32_t dst = lds0 + buf * Cfg::TILE_BYTES;
#pragma unroll
    for (int k = 0; k < Cfg::KB / 4; ++k) {
      const int kb = w * (Cfg::KB / 4) + k;
      copy_kb(vdesc, dst + kb * 1024, lane * 16, row0 * DV * 2 + kb * 1024);
      if constexpr (GQA) copy_kb(kcdesc, dst + Cfg::V_BYTES + kb * 1024, lane * 16, row0 * DV * 2 + kb * 1024);
    }
    // the positional tile is 32 d_r 2 bytes <= NRC KB: copied in whole KBs
    // (what follows it lands in padding), by as many waves as it takes, the
    // others repeating one of them so that every wave makes as many copies
    if constexpr (NRC > 0) {
      const int kb = w % NRC;
      copy_kb(kdesc, dst + Cfg::V_BYTES + kb * 1024, lane * 16, row0 * p.d_r * 2 + kb * 1024);
    }
  };
  copy_tile(tile_row(0), 0);
  copy_tile(tile_row(1), 1);

  // ---- the queries as bf16 high and low B operands: lane (n, h) holds
  // entries 16 c + 8 h .. + 7 of its column's query
  bf16x8 qh[NCH], ql[NCH], rh[NRC > 0 ? NRC : 1], rl[NRC > 0 ? NRC : 1];
  auto put_query = [&](bf16x8& hi, bf16x8& lo, float* xv) {
#pragma unroll
    for (int j = 0; j < 8; ++j) xv[j] *= p.scale_log2;
    hi = pos >= 0 ? split_hi_lo(xv, false) : zero8;
    lo = pos >= 0 ? split_hi_lo(xv, true) : zero8;
  };
  if (!GQA && p.q != nullptr) {
    // Fused absorption: q~^T[i][col] = sum_k M_h[i][k] q[col][k] on the same
    // products.  Row m of an A operand is row i(m) of M_h, bits 2 and 3 of m
    // swapped, so that a lane's 16 results of a block are two B operands of
    // the score product as they lie.  At H/G = 8 a wave holds two heads, each
    // with half of the columns: one pass per head, each keeping its own columns.
    const int W = p.d_c + p.d_r;
    const uint16_t* qraw = static_cast<const uint16_t*>(p.q) + qrow * W;
    f32x16 d[NIB];
    const int mrow = (n & 19) | ((n & 4) << 1) | ((n & 8) >> 1);
    const int npass = hpg == 8 ? 2 : 1;
    constexpr int CS = 4;                      // 16-column chunks per load round
    const int nround = (p.d_c + 16 * CS - 1) / (16 * CS);
    for (int ps = 0; ps < npass; ++ps) {
      const bool mine = npass == 1 || (n >> 4) == ps;
      const int hd = npass == 1 ? g * hpg + (hpg < 4 ? w % hpg : w) : g * hpg + 2 * w + ps;
      const uint16_t* mh = static_cast<const uint16_t*>(p.m) + ((int64_t)hd * DV + mrow) * p.d_c;
      f32x16 e[NIB];
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
        for (int r = 0; r < 16; ++r) e[ib][r] = 0.f;
      for (int ro = 0; ro < nround; ++ro) {
        u32x4 xq[CS], xm[CS][NIB];
#pragma unroll
        for (int c = 0; c < CS; ++c) {         // columns past d_c: any valid ones against zeros
          const int col = min(16 * (CS * ro + c) + 8 * h, p.d_c - 8);
          xq[c] = *reinterpret_cast<const u32x4*>(qraw + col);
#pragma unroll
          for (int ib = 0; ib < NIB; ++ib)
            xm[c][ib] = *reinterpret_cast<const u32x4*>(mh + (int64_t)(32 * ib) * p.d_c + col);
        }
#pragma unroll
        for (int c = 0; c < CS; ++c) {
          const bf16x8 bq = 16 * (CS * ro + c) < p.d_c ? as_bf16x8(xq[c]) : zero8;
#pragma unroll
          for (int ib = 0; ib < NIB; ++ib) e[ib] = mfma32(as_bf16x8(xm[c][ib]), bq, e[ib]);
        }
      }
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
        for (int r = 0; r < 16; ++r) d[ib][r] = ps == 0 || mine ? e[ib][r] : d[ib][r];
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      float xv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) xv[j] = d[c >> 1][8 * (c & 1) + j];
      put_query(qh[c], ql[c], xv);
    }
#pragma unroll
    for (int rc = 0; rc < NRC; ++rc) {
      const int piece = 2 * rc + h;
      float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (8 * piece < p.d_r) {
        const u32x4 raw = *reinterpret_cast<const u32x4*>(qraw + p.d_c + 8 * piece);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          rotate_query_pair(bf16_bits_to_f32(raw[k] & 0xFFFFu), bf16_bits_to_f32(raw[k] >> 16),
                            (double)(pos > 0 ? pos : 0) * p.inv_freq[4 * piece + k], 1.f, xv[2 * k], xv[2 * k + 1]);
      }
      put_query(rh[rc], rl[rc], xv);
    }
  } else {
    const float* qa = p.q_abs + qrow * DV + 8 * h;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const f32x4 u0 = *reinterpret_cast<const f32x4*>(qa + 16 * c);
      const f32x4 u1 = *reinterpret_cast<const f32x4*>(qa + 16 * c + 4);
      float xv[8] = {u0[0], u0[1], u0[2], u0[3], u1[0], u1[1], u1[2], u1[3]};
      put_query(qh[c], ql[c], xv);
    }
#pragma unroll
    for (int rc = 0; rc < NRC; ++rc) {
      const int piece = 2 * rc + h;
      float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (8 * piece < p.d_r) {
        const float* qr = p.q_rot + qrow * p.d_r + 8 * piece;
        const f32x4 u0 = *reinterpret_cast<const f32x4*>(qr);
        const f32x4 u1 = *reinterpret_cast<const f32x4*>(qr + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          xv[j] = u0[j];
          xv[4 + j] = u1[j];
        }
      }
      put_query(rh[rc], rl[rc], xv);
    }
  }
  int k_off[NRC > 0 ? NRC : 1];                // LDS offset of this lane's positional piece
#pragma unroll
  for (int rc = 0; rc < NRC; ++rc) {           // pieces past d_r: any valid one against a zero query
    const int piece = 8 * (2 * rc + h) < p.d_r ? 2 * rc + h : 0;
    k_off[rc] = (n >> 4) * 32 * p.d_r + piece * 256 + (n & 15) * 16;
  }
  // identity selectors: E_c[k][n] = (n == k + 16 c)
  bf16x8 esel[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    u32x4 u = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (8 * h + j + 16 * c == n) u[j >> 1] |= 0x3F80u << (16 * (j & 1));
    esel[c] = as_bf16x8(u);
  }

  f32x16 acc[NIB];
  // the running maximum starts below every score but -inf (a row hidden from
  // the column): an exponential against it is 0, and the first score that
  // counts replaces it
  float m_run = -FLT_MAX, l_run = 0.f;
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[ib][r] = 0.f;

  const int v_off = (n >> 4) * (DV * 32) + h * 256 + (n & 15) * 16;   // this lane's piece of chunk 0
  const char* const vt_lane = grp_lds + 3 * Cfg::TILE_BYTES + lane * 16;
  auto vt_piece = [&](int vbuf, int k) {       // A operand k = 2 ib + c of a tile's V^T
    return *reinterpret_cast<const f16x8*>(vt_lane + vbuf * Cfg::VT_BYTES + k * 1024);
  };

  // element r of the softmax weights of scores sc; the tile's sum joins the
  // running one when it is whole (a running sum over single weights has
  // sixteen times the roundings)
  float tile_sum = 0.f;
  auto exps = [&](const f32x16& sc, float (&pr)[16], int r) {
    pr[r] = __builtin_amdgcn_exp2f(sc[r] - m_run);
    tile_sum = r == 0 ? pr[r] : tile_sum + pr[r];
    if (r == 15) l_run += tile_sum;
  };
  // What a tile's fp16 weights leave over, through the same V^T: run for the
  // tiles below kLowRows, ahead of the tile's P.V.
  auto add_low = [&](const f32x16& sc, int vbuf) __attribute__((always_inline)) {
    float m = m_run;                           // opaque: formed again here, not kept for the tile's own P.V
    asm volatile("" : "+v"(m));
#pragma unroll
    for (int c = 0; c < 2; ++c) {              // a half at a time: few registers beside the loop's
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = __builtin_amdgcn_exp2f(sc[8 * c + e] - m);
      const f16x8 hi = to_f16x8(x);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] -= (float)hi[e];
      const f16x8 lo = to_f16x8(x);
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib) {
        acc[ib] = mfma32(vt_piece(vbuf, 2 * ib + c), lo, acc[ib]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // One tile: scores sn of tile j, beside them the softmax weights of the
  // tile before (scores sp), then that tile's P.V, beside it tile j's maxima.
  // The orders are pinned (scheduling barriers): on these matrix cores a few
  // vector instructions between two products are nearly free, a run of them
  // is not.  FIRST: the workgroup's first tile, with none before it.
  auto step = [&](auto first_tag, int j, int buf, const f32x16& sp, f32x16& sn) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(first_tag)::value;
    const int row0 = tile_row(j);
    if constexpr (!FIRST) {
      if (tile_row(j - 1) < kLowRows) add_low(sp, (j & 1) ^ 1);
    }
    copy_tile(tile_row(j + 2), buf == 0 ? 2 : buf - 1);
    const char* vtile = grp_lds + buf * Cfg::TILE_BYTES;
    const char* ktile = vtile + Cfg::V_BYTES;
    const int tw = w < NIB ? w : 0;            // this wave's block of V^T (waves past it repeat block 0 and drop it)
    // operand k of the tile: the score chunks, the positional ones, the V^T block's
    constexpr int NA = NCH + NRC, NOP = NA + 2;
    auto operand = [&](int k) {
      if (k < NCH) return *reinterpret_cast<const bf16x8*>((GQA ? ktile : vtile) + v_off + k * 512);
      if (k < NA) return *reinterpret_cast<const bf16x8*>(ktile + k_off[k < NA && k >= NCH ? k - NCH : 0]);
      return *reinterpret_cast<const bf16x8*>(vtile + v_off + (2 * tw + k - NA) * 512);
    };
    bf16x8 a[NOP];
    f16x8 av[2 * NIB];
    float pr[16];
    f16x8 bn[2];
    f32x16 t;
#pragma unroll
    for (int k = 0; k < RA; ++k) a[k] = operand(k);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 16; ++r) sn[r] = t[r] = 0.f;
    constexpr int NM = 2 * NA + 2;             // products of this phase
    __builtin_amdgcn_s_setprio(1);             // ahead of the other wave's P.V, which has less to interleave
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      const int k = i < 2 * NA ? i / 2 : i - NA;
      if (k < NCH) sn = mfma32(a[k], (i & 1) ? ql[k < NCH ? k : 0] : qh[k < NCH ? k : 0], sn);
      else if (k < NA) sn = mfma32(a[k], (i & 1) ? rl[k < NA && k >= NCH ? k - NCH : 0] : rh[k < NA && k >= NCH ? k - NCH : 0], sn);
      else t = mfma32(a[k], esel[k - NA], t);
      if ((i & 1) == 1 || i >= 2 * NA) {
        if (k + RA < NOP) a[k + RA] = operand(k + RA);
        else if (!FIRST && k + RA - NOP < VA) av[k + RA - NOP] = vt_piece((j & 1) ^ 1, k + RA - NOP);
      }
      if constexpr (!FIRST) {
        // sixteen exponentials over the phase's products
#pragma unroll
        for (int r = i * 16 / NM; r < (i + 1) * 16 / NM; ++r) {
          exps(sp, pr, r);
          if (r == 7) bn[0] = to_f16x8(pr);
          if (r == 15) bn[1] = to_f16x8(pr + 8);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!FIRST) asm volatile("" ::"v"(bn[0]), "v"(bn[1]), "v"(l_run));   // formed here, beside the products
    __builtin_amdgcn_sched_barrier(0);
    if (row0 + kTileRows - 1 > p_first) {      // some column may not see every row
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (row0 + score_row(r, h) > pos) sn[r] = -INFINITY;
    }
    // rows past the block's keys may hold anything (a wave whose columns all
    // lie past the prompt's last row masks nothing, but its V^T block counts)
    if (row0 + kTileRows > kend) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (row0 + score_row(r, h) >= kend) t[r] = 0.f;
    }
    __builtin_amdgcn_s_setprio(0);
    float mt = -INFINITY;
    char* vt = grp_lds + 3 * Cfg::TILE_BYTES + (j & 1) * Cfg::VT_BYTES + lane * 16;
#pragma unroll
    for (int k = 0; k < 2 * NIB; ++k) {
      if constexpr (!FIRST) {
        acc[k >> 1] = mfma32(av[k], bn[k & 1], acc[k >> 1]);
        if (k + VA < 2 * NIB) av[k + VA] = vt_piece((j & 1) ^ 1, k + VA);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int r = k * (8 / NIB); r < (k + 1) * (8 / NIB); ++r) mt = fmaxf(mt, sn[r]);
      if (k == 0 || k == NIB) {
        float x8[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x8[e] = t[8 * (k / NIB) + e];
        const f16x8 tv = to_f16x8(x8);         // bf16 values: exact in fp16 at these magnitudes
        if (w < NIB) *reinterpret_cast<f16x8*>(vt + (2 * w + k / NIB) * 1024) = tv;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mt), __float_as_uint(mt), false, false);
      mt = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    // The maximum is the first tile's with a row that counts, and moves when
    // a column's tile maximum exceeds it by more than kLdsLazyMax (log2 units).
    if (FIRST || __ballot(mt > m_run + kLdsLazyMax) != 0) {
      const float m_new = fmaxf(mt, m_run);
      if constexpr (!FIRST) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int ib = 0; ib < NIB; ++ib) acc[ib] *= alpha;
      }
      m_run = m_new;
    }
    wait_copies<Cfg::COPIES>();                // the next tile has landed (the one after it may be in flight)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's V^T block is in LDS
    tile_barrier();
  };
  auto last = [&](const f32x16& sp) {          // the last tile's weights and P.V
    if (tile_row(nit - 1) < kLowRows) add_low(sp, (nit - 1) & 1);
    float pr[16];
    f16x8 bn[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) exps(sp, pr, r);
    bn[0] = to_f16x8(pr);
    bn[1] = to_f16x8(pr + 8);
#pragma unroll
    for (int k = 0; k < 2 * NIB; ++k) acc[k >> 1] = mfma32(vt_piece((nit - 1) & 1, k), bn[k & 1], acc[k >> 1]);
  };

  wait_copies<Cfg::COPIES>();
  tile_barrier();
  if (nit > 0) {
    f32x16 s0, s1;                             // the scores of even and odd tiles
    step(std::true_type{}, 0, 0, s0, s0);
    int buf = 1, j = 1;
    for (; j + 1 < nit; j += 2) {
      step(std::false_type{}, j, buf, s0, s1);
      buf = buf == 2 ? 0 : buf + 1;
      step(std::false_type{}, j + 1, buf, s1, s0);
      buf = buf == 2 ? 0 : buf + 1;
    }
    if (j < nit) {
      step(std::false_type{}, j, buf, s0, s1);
      last(s1);
    } else {
      last(s0);
    }
  }

  // ---- merge the two sets of waves, normalise, write
  {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
    l_run = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  if constexpr (KS > 1) {
    float* rec = reinterpret_cast<float*>(lds) + w * 64 * (NIB * 16 + 2) + lane;
    wait_copies<0>();                          // copies past the end still write LDS
    __syncthreads();
    if (grp == 1) {
      rec[0] = m_run;
      rec[64] = l_run;
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
        for (int r = 0; r < 16; ++r) rec[64 * (2 + 16 * ib + r)] = acc[ib][r];
    }
    __syncthreads();
    if (grp == 1) return;
    const float m1 = rec[0], l1 = rec[64];
    const bool has0 = !(l_run == 0.f), has1 = !(l1 == 0.f);
    const float mx = has0 && has1 ? fmaxf(m_run, m1) : (has0 ? m_run : m1);
    const float a0 = has0 ? __builtin_amdgcn_exp2f(m_run - mx) : 0.f;
    const float a1 = has1 ? __builtin_amdgcn_exp2f(m1 - mx) : 0.f;
    l_run = l_run * a0 + l1 * a1;
    m_run = mx;
#pragma unroll
    for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ib][r] = acc[ib][r] * a0 + rec[64 * (2 + 16 * ib + r)] * a1;
  } else {
    wait_copies<0>();
    __syncthreads();                           // every wave is done with the tiles
  }
  // A lane holds 16 bytes of its column at a time, two lanes of a column 32:
  // as they lie, streaming stores of parts of a line, which the memory has to
  // merge.  They go through the wave's own LDS a 32-wide block at a time and
  // leave as whole 128-byte lines.
  const bool seen = pos >= 0 && !(l_run == 0.f);
  const float inv = seen ? 1.f / l_run : 0.f;
  constexpr int OP = 36;                       // floats per padded LDS row
  float* const ob = reinterpret_cast<float*>(lds + w * (KS > 1 ? Cfg::MERGE_BYTES / kWaves : 32 * OP * 4));
#pragma unroll
  for (int ib = 0; ib < NIB; ++ib) {
    wave_fence();                              // the block before has been read
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      f32x4 o;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) o[jj] = acc[ib][4 * r4 + jj] * inv;
      if (!seen) o = f32x4{0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f32x4*>(ob + n * OP + 8 * r4 + 4 * h) = o;
    }
    wave_fence();
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int col = 8 * it + (lane >> 3);
      const f32x4 o = *reinterpret_cast<const f32x4*>(ob + col * OP + 4 * (lane & 7));
      const int i = wpos + (hpg == 8 ? col & 15 : col);
      const int hd = hpg == 8 ? g * hpg + 2 * w + (col >> 4) : head;
      // written once and not read again here: kept out of the L2, which holds
      // the group's key and value rows
      if (i < p.N)
        __builtin_nontemporal_store(
            o, reinterpret_cast<f32x4*>(p.o + (((int64_t)b * p.N + i) * p.H + hd) * DV + 32 * ib + 4 * (lane & 7)));
    }
  }
  if (h == 0 && i_col < p.N) p.lse[qrow] = seen ? (m_run + log2f(l_run)) * kLn2 : -INFINITY;
}

template <int DV, int KS>
PrefillFn pick_prefill_lds_nrc(int d_r, bool gqa) {
  if (gqa) return prefill_lds_kernel<DV, 0, true, KS>;
  if (d_r == 0) return prefill_lds_kernel<DV, 0, false, KS>;
  if (d_r <= 16) return prefill_lds_kernel<DV, 1, false, KS>;
  if (d_r <= 32) return prefill_lds_kernel<DV, 2, false, KS>;
  return prefill_lds_kernel<DV, 4, false, KS>;
}

PrefillFn pick_prefill_lds(int dv, int d_r, bool gqa, int ks) {
  if (dv == 128) return ks == 2 ? pick_prefill_lds_nrc<128, 2>(d_r, gqa) : pick_prefill_lds_nrc<128, 1>(d_r, gqa);
  return ks == 2 ? pick_prefill_lds_nrc<64, 2>(d_r, gqa) : pick_prefill_lds_nrc<64, 1>(d_r, gqa);
}


template <int HPG, int DV>
PrefillFn pick_prefill_nrc(int d_r, bool gqa) {
  if (gqa) return prefill_bf16_kernel<HPG, DV, 0, true, false>;
  if (d_r == 0) return prefill_bf16_kernel<HPG, DV, 0, false, false>;
  if (d_r <= 16) return prefill_bf16_kernel<HPG, DV, 1, false, true>;
  if (d_r <= 32) return prefill_bf16_kernel<HPG, DV, 1, false, false>;
  if (d_r <= 64) return prefill_bf16_kernel<HPG, DV, 2, false, false>;
  return nullptr;
}

template <int HPG>
PrefillFn pick_prefill_dv(int dv, int d_r, bool gqa) {
  switch (dv) {
    case 64: return pick_prefill_nrc<HPG, 64>(d_r, gqa);
    case 128: return pick_prefill_nrc<HPG, 128>(d_r, gqa);
  }
  return nullptr;
}

PrefillFn pick_prefill(int hpg, int dv, int d_r, bool gqa) {
  switch (hpg) {
    case 1: return pick_prefill_dv<1>(dv, d_r, gqa);
    case 2: return pick_prefill_dv<2>(dv, d_r, gqa);
    case 4: return pick_prefill_dv<4>(dv, d_r, gqa);
    case 8: return pick_prefill_dv<8>(dv, d_r, gqa);
  }
  return nullptr;
}

// Which kernel a prompt takes: the sets of four waves per workgroup of
// prefill_lds_kernel, or 0 for the tile-split kernel, whose workgroups are a
// half to an eighth the size and split the keys over the four waves.  By its
// workgroups of 128 columns against the CUs (us below are single calls):
//  - two per CU and more: one set, two workgroups per CU (2048 tokens at H32
//    G8 d 128, 512 workgroups: 77 us, 88 with two sets, 123 tile-split);
//  - from 3/4 per CU (the baseline at d_v = 128, whose tile-split workgroups
//    hold only 16 columns but whose chains are half as long: 1/2): two sets,
//    so that each SIMD has two waves (H16 G4 d 128, 2048 tokens, 256
//    workgroups: 54, 58 and 70; H32 G8, 768 rows after 3328, 192 workgroups:
//    90, 102 and 108).  But the launch then takes as long as the longest
//    block's keys, the tile-split one as long as all of them together, and the
//    blocks of a prompt without a prefix average half the longest: counted in
//    blocks of that average, long caches need more than 1/2 per CU (H3 G3 d
//    128, 8192 tokens, 192 workgroups: 154 us, 127 tile-split; at 256, H4 G1,
//    158 and 155; d_v = 64 from 8192 rows only, 4096 tokens with 192
//    workgroups 59 and 66), the baseline 3/8, from 1024 rows on 7/16 (H8 G8
//    d 128, 2048 tokens, 128 workgroups: 42 and 36; 512 after 1536: 42 and 46);
//  - fewer: the tile-split kernel (H32 G8 d 128, 512 rows after 7680, 128
//    workgroups: 128 us, 153 with two sets; baseline, 64 rows after 960: 12
//    and 27), except where the cache is short, so that a workgroup's chain of
//    tiles is, and at least 32 columns of a group have a query (a single row
//    of 8 x 1 heads after 1023: 18 us tile-split, 29 with two sets).  At
//    d_v = 64, whose tile-split workgroup starts slowly, up to 1024 rows, one
//    set to 128 rows, or 256 with the absorption inside, and two sets past
//    that (H32 G8, 512 tokens: 17 us, 30 tile-split; 64 rows after 960: 22
//    and 28).  At d_v = 128 up to 128 rows, or 256 with the absorption's
//    launch to save (H32 G8, 256 tokens: 19 and 24), to 512 the larger the
//    prompt (512 tokens, 128 workgroups: 25 and 33; H4 G2, 16 workgroups: 24
//    and 22; H24 G6, 720 tokens, 138 workgroups, which are two rounds of
//    tile-split ones: 29 and 44), to 1024 at 128 workgroups if its blocks are
//    long on average too (512 after 512: 38 and 40; H16 G16, 1024 tokens: 36
//    and 31), and never for the baseline (128 tokens: 11 us, 9 tile-split).
enum class Prompt { kAttention, kWhole, kGqa };   // absorbed queries, raw ones (gva_prefill), the baseline

struct PrefillPlan {
  int sets;
  bool inside;                                 // kWhole: the absorption inside the attention launch
};

// Whether gva_prefill absorbs inside the attention launch.  Each workgroup
// then reads its heads' maps, each set of waves for itself and at H/G = 8 in
// two passes: a launch of one workgroup or more per CU bears more of it
// (`full`) than a small one, whose absorption's own launch is short (us,
// inside and apart: H16 G2 d 128/512, 4 x 1024 tokens, one set 110 and 89,
// 256 columns 73 and 72; H4 G4 d 64/1024 the same tokens 74 and 101; H32 G8
// d 128/512, 512 tokens after 7680, two sets 222 and 211, 256 columns 203 and
// 203; few workgroups: H16 G2 d 128/512, 256 tokens 49 and 24, d 128/128 23
// and 20; H16 G4 d 64/512 22 and 19, d 64/256 16 and 17).
bool absorb_inside(const gva_dims* d, int sets, bool full) {
  const long long maps = (long long)(d->n_heads / d->n_groups == 8 ? 2 : 1) * sets;   // read per workgroup
  if (full) return maps * d->d_c <= (maps == 1 ? 1024 : 640);
  return maps * d->d_c * d->d_v <= 16384;
}

PrefillPlan prefill_plan(const gva_dims* d, int n_new, Prompt kind) {
  const int hpg = d->n_heads / d->n_groups;
  if (hpg > 8) return {0, false};              // no kernel takes it
  const bool whole = kind == Prompt::kWhole;
  const int rows = kPrefillCols / hpg;         // positions per workgroup
  const long long items = (long long)d->batch * d->n_groups * (((long long)n_new + rows - 1) / rows);
  const long long n_cu = device_cu_count(), T = d->t_max;
  if (items >= 2 * n_cu) return {1, whole && absorb_inside(d, 1, true)};
  // twice the blocks of average length: all rows' keys over those of the longest
  const double mean2 = (double)items * (double)(2 * T - n_new) / (double)T;
  bool two_sets;
  if (kind == Prompt::kGqa && d->d_v >= 128)
    two_sets = 4 * items >= 3 * n_cu ||
               (2 * items >= n_cu && (T <= 512 || 8 * mean2 >= (T > 1024 ? 7 : 6) * (double)n_cu));
  else
    two_sets = 4 * items >= 3 * n_cu && (T < (d->d_v >= 128 || !whole ? 4096 : 8192) || mean2 > (double)n_cu);
  if (two_sets) return {2, whole && absorb_inside(d, 2, true)};
  const bool cols32 = (long long)n_new * hpg >= 32;
  if (d->d_v < 128) {
    if (T <= (whole ? 256 : 128)) return {1, whole && absorb_inside(d, 1, false)};
    if (cols32 && T <= 1024) return {2, whole && absorb_inside(d, 2, false)};
    return {0, false};
  }
  if (!cols32 || kind == Prompt::kGqa) return {0, false};
  const int passes = hpg == 8 ? 2 : 1;         // of a wave's absorption
  const bool larger = T <= 512 || 2 * items > n_cu || 4 * mean2 >= 3 * (double)n_cu;
  if (whole && T <= 1024 && passes * T * n_cu <= (larger ? 2048 : 1664) * items && passes * d->d_c <= 256)
    return {1, true};
  if (T <= (whole ? 256 : 128)) return {1, whole && absorb_inside(d, 1, false)};
  return {0, false};
}

// The launch behind gva_prefill_attention, gva_prefill (raw query q and maps
// m in place of q_abs and q_rot) and, with k_gqa given,
// gva_gqa_prefill_attention, with the sets of its plan.
int prefill_impl(int sets, const gva_dims* dims, int32_t n_new, const float* q_abs, const float* q_rot, const void* q,
                 const void* m, const void* v_cache, const void* kr_cache, const void* k_gqa, const int32_t* lens,
                 float* o, float* lse, void* stream, bool launch = true) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  const bool gqa = k_gqa != nullptr, fused = q != nullptr;
  const int d_r = gqa ? 0 : dims->d_r;
  if (n_new < 1 || n_new > dims->t_max) return GVA_ERR_INVALID_ARG;
  if (!v_cache || !lens || !o || !lse) return GVA_ERR_INVALID_ARG;
  if (fused ? !m : (!q_abs || (d_r > 0 && !q_rot))) return GVA_ERR_INVALID_ARG;
  if (d_r > 0 && !kr_cache) return GVA_ERR_INVALID_ARG;
  if (!aligned(q_abs, 16) || !aligned(q, 16) || !aligned(m, 16) || !aligned(v_cache, 16) || !aligned(lens, 4) ||
      !aligned(o, 16) || !aligned(lse, 4) || (d_r > 0 && (!aligned(q_rot, 16) || !aligned(kr_cache, 16))) ||
      (gqa && !aligned(k_gqa, 16)))
    return GVA_ERR_INVALID_ARG;
  if (dims->dtype != GVA_DTYPE_BF16) return GVA_ERR_UNSUPPORTED;
  st = check_cache_layout(dims);
  if (st != GVA_OK) return st;
  if (d_r % 8 != 0 || d_r > 64) return GVA_ERR_UNSUPPORTED;
  const int hpg = dims->n_heads / dims->n_groups;
  if (hpg != 1 && hpg != 2 && hpg != 4 && hpg != 8) return GVA_ERR_UNSUPPORTED;
  if (dims->d_v != 64 && dims->d_v != 128) return GVA_ERR_UNSUPPORTED;
  if (fused && sets == 0) return GVA_ERR_UNSUPPORTED;
  const PrefillFn fn = sets > 0 ? pick_prefill_lds(dims->d_v, d_r, gqa, sets) : pick_prefill(hpg, dims->d_v, d_r, gqa);
  if (fn == nullptr) return GVA_ERR_UNSUPPORTED;
  const int qb_rows = (sets > 0 ? kPrefillCols : prefill_cols(dims->d_v, gqa)) / hpg;
  const long long n_qblocks = (n_new + qb_rows - 1) / qb_rows;
  const long long n_items = (long long)dims->batch * dims->n_groups * n_qblocks;
  if (n_items > 0x7FFFFFFFLL) return GVA_ERR_UNSUPPORTED;

  if (!launch) return GVA_OK;

  PrefillParams p{};
  memset(&p, 0, sizeof(p));
  p.q_abs = q_abs;
  p.q_rot = q_rot;
  p.v = v_cache;
  p.kr = kr_cache;
  p.k_gqa = k_gqa;
  p.q = q;
  p.m = m;
  p.d_c = dims->d_c;
  fill_inv_freq(dims, p.inv_freq);
  p.lens = lens;
  p.o = o;
  p.lse = lse;
  p.B = dims->batch;
  p.H = dims->n_heads;
  p.G = dims->n_groups;
  p.N = n_new;
  p.d_r = d_r;
  p.t_max = dims->t_max;
  p.n_qblocks = (int32_t)n_qblocks;
  if (gqa) {
    const double sc = dims->scale > 0.0 ? dims->scale : 1.0 / sqrt((double)dims->d_v);
    p.scale_log2 = (float)(sc * kLog2e);
  } else {
    p.scale_log2 = scale_log2(dims);
  }
  hipLaunchKernelGGL(fn, dim3((unsigned)n_items), dim3(sets == 2 ? 2 * kThreads : kThreads), 0, static_cast<hipStream_t>(stream), p);
  return launch_status();
}

// gva_prefill's plan, and where its two launches keep the absorbed queries
// (bytes = 0 with the absorption inside).
struct PrefillLayout {
  PrefillPlan plan;
  size_t q_rot, bytes;
};

void prefill_layout(const gva_dims* d, int n_new, PrefillLayout& L) {
  L = PrefillLayout{prefill_plan(d, n_new, Prompt::kWhole), 0, 0};
  if (L.plan.inside) return;
  const size_t rows = (size_t)d->batch * n_new * d->n_heads;
  L.q_rot = (rows * d->d_v * 4 + 255) / 256 * 256;
  L.bytes = L.q_rot + (rows * d->d_r * 4 + 255) / 256 * 256;
}

}  // namespace

extern "C" {

int gva_prefill_attention(const gva_dims* dims, int32_t n_new, const float* q_abs, const float* q_rot,
                          const void* v_cache, const void* kr_cache, const int32_t* lens, float* o,
                          float* lse, void* stream) {
  const int st = check_dims(dims);
  if (st != GVA_OK) return st;
  return prefill_impl(prefill_plan(dims, n_new, Prompt::kAttention).sets, dims, n_new, q_abs, q_rot, nullptr, nullptr,
                      v_cache, kr_cache, nullptr, lens, o, lse, stream);
}

int gva_prefill_workspace_size(const gva_dims* dims, int32_t n_new, size_t* bytes) {
  if (bytes == nullptr) return GVA_ERR_INVALID_ARG;
  const int st = check_dims(dims);
  if (st != GVA_OK) return st;
  if (n_new < 1 || n_new > dims->t_max) return GVA_ERR_INVALID_ARG;
  PrefillLayout L;
  prefill_layout(dims, n_new, L);
  *bytes = L.bytes;
  return GVA_OK;
}

int gva_prefill(const gva_dims* dims, int32_t n_new, const void* q, const void* m, const void* v_cache,
                const void* kr_cache, const int32_t* lens, void* workspace, size_t workspace_bytes, float* o,
                float* lse, void* stream) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  if (n_new < 1 || n_new > dims->t_max) return GVA_ERR_INVALID_ARG;
  if (!q || !m || !v_cache || !lens || !o || !lse) return GVA_ERR_INVALID_ARG;
  // the absorption's bounds hold for both forms
  const long long rows = (long long)dims->batch * n_new;
  if (rows > (1LL << 20) || rows * dims->n_heads > 0x7FFFFFFFLL || dims->d_c % 32 != 0) return GVA_ERR_UNSUPPORTED;
  PrefillLayout L;
  prefill_layout(dims, n_new, L);
  if (L.bytes == 0)
    return prefill_impl(L.plan.sets, dims, n_new, nullptr, nullptr, q, m, v_cache, kr_cache, nullptr, lens, o, lse,
                        stream);
  if (workspace == nullptr || workspace_bytes < L.bytes || !aligned(workspace, 256)) return GVA_ERR_INVALID_ARG;
  float* q_abs = static_cast<float*>(workspace);
  float* q_rot = dims->d_r > 0 ? reinterpret_cast<float*>(static_cast<char*>(workspace) + L.q_rot) : nullptr;
  // every check of the second launch before the first is enqueued
  st = prefill_impl(L.plan.sets, dims, n_new, q_abs, q_rot, nullptr, nullptr, v_cache, kr_cache, nullptr, lens, o, lse,
                    stream, false);
  if (st != GVA_OK) return st;
  st = gva_prefill_absorb(dims, n_new, q, m, lens, q_abs, q_rot, stream);
  if (st != GVA_OK) return st;
  return prefill_impl(L.plan.sets, dims, n_new, q_abs, q_rot, nullptr, nullptr, v_cache, kr_cache, nullptr, lens, o, lse,
                      stream);
}

int gva_gqa_prefill_attention(const gva_dims* dims, int32_t n_new, const float* q, const void* k_cache,
                              const void* v_cache, const int32_t* lens, float* o, float* lse,
                              void* stream) {
  if (k_cache == nullptr) return GVA_ERR_INVALID_ARG;
  const int st = check_dims(dims);
  if (st != GVA_OK) return st;
  return prefill_impl(prefill_plan(dims, n_new, Prompt::kGqa).sets, dims, n_new, q, nullptr, nullptr, nullptr, v_cache,
                      nullptr, k_cache, lens, o, lse, stream);
}

}  // extern "C"
