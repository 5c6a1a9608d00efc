// libgva.so -- GVA decode-step attention for MI355X (gfx950, CDNA4).
//
// The method is Grouped Value Attention with decoupled RoPE: the cache keeps
// G value streams plus one shared, already-rotated positional key; the
// per-head key map M_h is absorbed into the query (eq. absorb, Section 3.2),
// so the content score against cached position t is q~_h . v_t and no
// content key is ever formed (Section 3.3, Algorithm 1).
//
// Kernels
//   append_kernel        Algorithm 1 append steps + eq. krope (fp64 rotation)
//   absorb_bf16_kernel   eq. absorb + query rotation on the matrix cores
//   absorb_f32_kernel    the same on the vector ALUs, fp32 storage
//   decode_bf16_kernel   the hot path: split-KV streaming over the value and
//                        positional-key rows of one (sequence, group, split)
//                        on the matrix cores, online softmax, optional fused
//                        absorption prologue
//   decode_f32_kernel    fp32-storage variant on the fp32 matrix products
//   combine_kernel       log-sum-exp merge of the split partials
//
// Cache layout (MFMA-native).  Each (sequence, group) value stream and each
// sequence's positional-key stream is stored in tiles of 16 rows; inside a
// tile the row pieces of 16 bytes are ordered piece-major:
//   element (t, i) of a stream with D columns of E bytes, P = 16/E:
//     (t/16)*16*D + ((i/P)*16 + t%16)*P + i%P
// A wave's 16-byte-per-lane load of 64 consecutive pieces then covers 1 KB
// of contiguous memory while every lane receives exactly the 8 bf16 of one
// row that its matrix-core operand slot needs (row = lane%16, columns
// 8*(lane/16) .. +7 of a 32-column chunk).
//
// Hot-loop design (bf16).  A workgroup owns one (b, g, split); its 4 waves
// take interleaved 32-row tiles and keep DEPTH tiles in registers.  Every V
// tile serves all H/G heads of the group:
//   scores  S^T[t][n] = V[t][:] . Bq[:][n]           (v_mfma 16x16x32 bf16)
//           column n holds one head's absorbed query as a bf16 high part or
//           low part (q~ = hi + lo to ~2^-16); the columns are mirrored so a
//           DPP mirror adds the pair; the positional key rides as one more
//           K-chunk of the same product
//   P.V     O^T[i][n] += V^T[i][t] P[t][n]            (v_mfma 16x16x32 bf16)
//           V^T comes from an identity-selector MFMA on the same registers;
//           P is split hi + lo again, so both products keep ~fp32 accuracy
// The score layout the MFMA returns (lane = column, registers = 4 rows) is
// exactly the B-operand layout of the P.V product, so the softmax needs no
// cross-lane traffic except the max over the four 16-lane rows.

#include <cfloat>
#include <mutex>
#include <type_traits>

#include "gva_common.h"

namespace {

// ================================================================ append
// Sixteen new rows per workgroup row; a wave moves 4 KP pieces of each for one
// group: lane (n, qd) moves pieces 4 k + qd of row n, so for rows at
// consecutive positions of one layout tile (a prompt) a store covers 1 KB of
// contiguous memory and a row's reads share cache lines; rows of different
// sequences (a decode batch) scatter as they must.  The pieces are requested
// before seq/pos are known (they are indexed by the row alone): a single
// dependent round trip.  The positional pairs, an fp64 rotation each, have
// workgroups of their own (the last of gridDim.y), one pair per thread.
// Bound by HBM for a prompt (8192 rows of 8 x 128 + 16 bf16 are read and
// written, 34 MB), by latency for a batch.  KP = 4 for a prompt (one workgroup
// per row, half of its threads idle, took 20.3 us for those 8192 rows; now 7
// us), 1 below 3/8 of such a workgroup per CU, so that a wide row is spread
// over waves and nothing follows the first request (64 rows of G2 d 256 fp32
// 2.8 us, 5.1 with the pieces past the first four of a lane in a loop and two
// pairs per thread at d_r = 64).  At the line, KP = 4 and 1: 700 prompt rows of
// G8 d 128, 88 workgroups, 3.3 and 3.3 us; 1000, 126, 3.4 and 3.6; 512 scattered
// ones, 64, 4.0 and 3.6.
constexpr int kAppendRows = 16;

// waves over a row block's values: one per group and 4 KP pieces of its rows
__host__ __device__ __forceinline__ int append_segs(int npc, int kp) { return (npc + 4 * kp - 1) / (4 * kp); }
// workgroups over them (gridDim.y but for the positional keys')
__host__ __device__ __forceinline__ int append_value_blocks(int G, int npc, int kp) {
  const long long n = ((long long)G * append_segs(npc, kp) + kWaves - 1) / kWaves;
  return (int)(n < 4096 ? n : 4096);
}
// and those over its positional pairs
__host__ __device__ __forceinline__ int append_pair_blocks(int d_r) {
  return (kAppendRows * (d_r / 2) + kThreads - 1) / kThreads;
}

// The streams holding row ps of sequence b: contiguous (b, g) streams, or,
// paged, page block_table[b][ps / page_rows].  False: out of range, skipped.
struct AppendPlace {
  int64_t vstream0, vstride, kstream0;
  int row;
};

__device__ __forceinline__ bool append_place(const AppendParams& p, int b, int ps, AppendPlace& at) {
  if (b < 0 || b >= p.B || ps < 0 || ps >= p.t_max) return false;
  at.row = ps;
  if (p.block_table != nullptr) {
    const int page = p.block_table[(int64_t)b * p.max_pages + ps / p.page_rows];
    if (page < 0 || page >= p.n_pages) return false;
    at.row = ps % p.page_rows;
    at.vstride = (int64_t)p.page_rows * p.d_v;
    at.vstream0 = (int64_t)page * p.G * at.vstride;
    at.kstream0 = (int64_t)page * p.page_rows * p.d_r;
  } else {
    at.vstride = (int64_t)p.t_max * p.d_v;
    at.vstream0 = (int64_t)b * p.G * at.vstride;
    at.kstream0 = (int64_t)b * p.t_max * p.d_r;
  }
  return true;
}

template <typename T, int KP>
__global__ void __launch_bounds__(kThreads) append_kernel(AppendParams p) {
  constexpr int P = 16 / sizeof(T);
  const int r0 = blockIdx.x * kAppendRows;
  const int tid = threadIdx.x;
  const int npc = p.d_v / P;
  const int nvb = append_value_blocks(p.G, npc, KP);
  AppendPlace at;
  if ((int)blockIdx.y < nvb) {
    const int lane = tid & 63, n = lane & 15, qd = lane >> 4;
    const int r = r0 + n;
    if (r >= p.n_rows) return;
    const int nseg = append_segs(npc, KP);
    for (int64_t t = blockIdx.y * kWaves + (tid >> 6); t < (int64_t)p.G * nseg; t += nvb * kWaves) {
      const int g = (int)(t / nseg), c0 = (int)(t % nseg) * 4 * KP + qd;
      const u32x4* src =
          reinterpret_cast<const u32x4*>(static_cast<const T*>(p.v_new) + ((int64_t)r * p.G + g) * p.d_v);
      u32x4 piece[KP];
#pragma unroll
      for (int k = 0; k < KP; ++k)
        if (c0 + 4 * k < npc) piece[k] = src[c0 + 4 * k];
      if (!append_place(p, p.seq[r], p.pos[r], at)) return;
      T* stream = static_cast<T*>(p.v_cache) + at.vstream0 + g * at.vstride + tiled_off<T>(at.row, c0 * P, p.d_v);
      constexpr int kStep = 4 * kLayoutRows * P; // elements between pieces c and c + 4 of a row
#pragma unroll
      for (int k = 0; k < KP; ++k)
        if (c0 + 4 * k < npc) *reinterpret_cast<u32x4*>(stream + k * kStep) = piece[k];
    }
    return;
  }
  // positional keys: rotate pair i of row r at its position in fp64 (eq. krope)
  const int npair = p.d_r / 2;
  const int task = ((int)blockIdx.y - nvb) * kThreads + tid;
  if (task >= kAppendRows * npair) return;
  const int r = r0 + task / npair, i = task % npair;
  if (r >= p.n_rows) return;
  const T* kin = static_cast<const T*>(p.kr_new) + (int64_t)r * p.d_r + 2 * i;
  const double k0 = load_elem<T>(kin, 0), k1 = load_elem<T>(kin, 1);
  const int ps = p.pos[r];
  if (!append_place(p, p.seq[r], ps, at)) return;
  double y0, y1;
  rotate_pair(k0, k1, (double)ps * p.inv_freq[i], y0, y1);
  T* kstream = static_cast<T*>(p.kr_cache) + at.kstream0;
  const int64_t o = tiled_off<T>(at.row, 2 * i, p.d_r);  // the pair shares a piece
  store_from_f64<T>(kstream, o, y0);
  store_from_f64<T>(kstream, o + 1, y1);
}

// ================================================================ absorb
// Position of query row r: a sequence's n_per_seq query rows are its last
// n_per_seq cached rows (one row, at L-1, for a decode step).
__device__ __forceinline__ int query_pos(const AbsorbParams& p, int r) {
  const int seq = r / p.n_per_seq, i = r % p.n_per_seq;
  const int pos = clamp_len(p.lens, seq, p.t_max) - p.n_per_seq + i;
  return pos > 0 ? pos : 0;
}

// bf16, matrix cores.  Workgroup = (head h, 16 RB query rows); wave w
// computes the output blocks ib = w, w+4, ... of
// q~^T[i][r] = sum_k M_h[i][k] q[r][h][k] (A = rows of M_h, B = the query
// rows, K = d_c).  M_h is staged through LDS in passes of 128 rows x 128
// columns: the workgroup reads each pass as whole rows (16 threads x 16 B
// per row, so every load covers whole cache lines; the MFMA operand order,
// 64 bytes of 16 rows per load, took four times as long to arrive), and the
// waves take their A operands from LDS (rows padded by 16 bytes: the 16
// rows of an operand fall in distinct banks).
constexpr int kAbsorbRows = 128, kAbsorbCols = 128, kAbsorbStride = kAbsorbCols + 8;
constexpr int kAbsorbMaxRB = 4;

__global__ void __launch_bounds__(kThreads) absorb_bf16_kernel(AbsorbParams p) {
  __shared__ __attribute__((aligned(16))) uint16_t ms[kAbsorbRows * kAbsorbStride];
  const int h = blockIdx.x;
  const int RB = p.row_blocks;                            // M_h rows reused for RB row blocks
  const int b0 = blockIdx.y * 16 * RB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, qd = lane >> 4;
  const int W = p.d_c + p.d_r;
  const int nck = p.d_c / 32;
  const uint16_t* qg = static_cast<const uint16_t*>(p.q);
  const uint16_t* mh = static_cast<const uint16_t*>(p.m) + (int64_t)h * p.d_v * p.d_c;
  const int nseg = (p.d_c + kAbsorbCols - 1) / kAbsorbCols;
  constexpr int kFill = kAbsorbRows * kAbsorbCols / 8 / kThreads;   // 16-byte pieces per thread and pass
  for (int rbase = 0; rbase < p.d_v; rbase += kAbsorbRows) {
    f32x4 acc[2][kAbsorbMaxRB];
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
      for (int rb = 0; rb < kAbsorbMaxRB; ++rb) acc[k2][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int seg = 0; seg < nseg; ++seg) {
      u32x4 piece[kFill];
#pragma unroll
      for (int k = 0; k < kFill; ++k) {
        const int pc = tid + kThreads * k, row = pc >> 4, col = seg * kAbsorbCols + 8 * (pc & 15);
        piece[k] = (rbase + row < p.d_v && col < p.d_c)
                       ? *reinterpret_cast<const u32x4*>(mh + (int64_t)(rbase + row) * p.d_c + col)
                       : u32x4{0u, 0u, 0u, 0u};
      }
      // the query rows' chunks of this segment, requested with the pass (one
      // memory round trip for both)
      u32x4 xq[kAbsorbMaxRB][4];
#pragma unroll
      for (int rb = 0; rb < kAbsorbMaxRB; ++rb) {
        const int bq = min(b0 + 16 * rb + n, p.B - 1);    // rows past B compute a duplicate
        const uint16_t* qrow = qg + ((int64_t)bq * p.H + h) * W + seg * kAbsorbCols + 8 * qd;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          xq[rb][c] = (rb < RB && seg * 4 + c < nck) ? *reinterpret_cast<const u32x4*>(qrow + 32 * c)
                                                      : u32x4{0u, 0u, 0u, 0u};
      }
      if (rbase > 0 || seg > 0) __syncthreads();         // the previous pass has been read
#pragma unroll
      for (int k = 0; k < kFill; ++k) {
        const int pc = tid + kThreads * k;
        *reinterpret_cast<u32x4*>(ms + (pc >> 4) * kAbsorbStride + 8 * (pc & 15)) = piece[k];
      }
      __syncthreads();
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        const int ibl = w + kWaves * k2;                  // 16-row block of the pass
        if (rbase + 16 * ibl >= p.d_v) break;
        bf16x8 a[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
          a[c] = *reinterpret_cast<const bf16x8*>(ms + (16 * ibl + n) * kAbsorbStride + 32 * c + 8 * qd);
#pragma unroll
        for (int rb = 0; rb < kAbsorbMaxRB; ++rb) {
          if (rb >= RB || b0 + 16 * rb >= p.B) break;
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (seg * 4 + c < nck) acc[k2][rb] = mfma16(a[c], as_bf16x8(xq[rb][c]), acc[k2][rb]);
        }
      }
    }
    // lane (n, qd) holds q~[r0 + n][rbase + 16 ibl + 4 qd + jj]
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      const int i0 = rbase + 16 * (w + kWaves * k2);
      if (i0 >= p.d_v) break;
#pragma unroll
      for (int rb = 0; rb < kAbsorbMaxRB; ++rb) {
        const int r0 = b0 + 16 * rb;
        if (rb >= RB || r0 >= p.B) break;
        if (r0 + n < p.B)
          *reinterpret_cast<f32x4*>(p.q_abs + ((int64_t)(r0 + n) * p.H + h) * p.d_v + i0 + 4 * qd) = acc[k2][rb];
      }
    }
  }
  // the positional pairs of the workgroup's rows: 16 RB d_r / 2 tasks
  const int npair = p.d_r / 2;
  for (int task = tid; task < 16 * RB * npair; task += kThreads) {
    const int pb = b0 + task / npair, pi = task % npair;
    if (pb >= p.B) break;
    const uint32_t two = *reinterpret_cast<const uint32_t*>(qg + ((int64_t)pb * p.H + h) * W + p.d_c + 2 * pi);
    float y0, y1;
    rotate_query_pair(bf16_bits_to_f32(two & 0xFFFFu), bf16_bits_to_f32(two >> 16),
                      (double)query_pos(p, pb) * p.inv_freq[pi], 1.f, y0, y1);
    float* out = p.q_rot + ((int64_t)pb * p.H + h) * p.d_r + 2 * pi;
    out[0] = y0;
    out[1] = y1;
  }
}

// fp32 storage, vector ALUs: one workgroup per (b, h).
// sum_k x[k] y[k] over fp32 rows of n.  Rows that are 16-byte aligned with
// n a multiple of 4 are read as 16-byte pieces, eight of each row requested
// per step (32 terms per memory round trip); any others element by element,
// eight per step.
__device__ __forceinline__ float dot_f32(const float* x, const float* y, int n) {
  if ((((uintptr_t)x | (uintptr_t)y) & 15) == 0 && (n & 3) == 0) {
    const f32x4* x4 = reinterpret_cast<const f32x4*>(x);
    const f32x4* y4 = reinterpret_cast<const f32x4*>(y);
    const int n4 = n >> 2;
    f32x4 a4 = {0.f, 0.f, 0.f, 0.f};
    int k = 0;
    for (; k + 8 <= n4; k += 8) {
      f32x4 xv[8], yv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        xv[j] = x4[k + j];
        yv[j] = y4[k + j];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) a4[e] = fmaf(xv[j][e], yv[j][e], a4[e]);
    }
    for (; k < n4; ++k) {
      const f32x4 xv = x4[k], yv = y4[k];
#pragma unroll
      for (int e = 0; e < 4; ++e) a4[e] = fmaf(xv[e], yv[e], a4[e]);
    }
    return (a4[0] + a4[1]) + (a4[2] + a4[3]);
  }
  float acc8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int k = 0;
  for (; k + 8 <= n; k += 8) {
    float xv[8], yv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      xv[j] = x[k + j];
      yv[j] = y[k + j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) acc8[j] = fmaf(xv[j], yv[j], acc8[j]);
  }
  for (; k < n; ++k) acc8[0] = fmaf(x[k], y[k], acc8[0]);
  return ((acc8[0] + acc8[1]) + (acc8[2] + acc8[3])) + ((acc8[4] + acc8[5]) + (acc8[6] + acc8[7]));
}

__global__ void __launch_bounds__(128) absorb_f32_kernel(AbsorbParams p) {
  const int bh = blockIdx.x;
  const int b = bh / p.H, h = bh % p.H;
  const int W = p.d_c + p.d_r;
  const float* q = static_cast<const float*>(p.q) + (int64_t)bh * W;
  const float* m = static_cast<const float*>(p.m) + (int64_t)h * p.d_v * p.d_c;
  for (int i = threadIdx.x; i < p.d_v; i += blockDim.x) {
    p.q_abs[(int64_t)bh * p.d_v + i] = dot_f32(q, m + (int64_t)i * p.d_c, p.d_c);
  }
  const int pos = query_pos(p, b);
  for (int i = threadIdx.x; i < p.d_r / 2; i += blockDim.x) {
    double y0, y1;
    rotate_pair(q[p.d_c + 2 * i], q[p.d_c + 2 * i + 1], (double)pos * p.inv_freq[i], y0, y1);
    p.q_rot[(int64_t)bh * p.d_r + 2 * i] = (float)y0;
    p.q_rot[(int64_t)bh * p.d_r + 2 * i + 1] = (float)y1;
  }
}

// ========================================================= decode (bf16)
// HPG heads per group, DV value width, NRC = ceil(d_r / 32) positional
// K-chunks, DEPTH tiles of V held in registers (DEPTH-1 loads in flight).
template <int HPG, int DV, int NRC, int NW, bool GQA>
struct DecodeCfg {
  static constexpr int NC = DV / 32;                         // K-chunks per V row
  static constexpr int NB = DV / 16;                         // 16-wide i-blocks of the output
  // (eight-wave workgroups keep three tiles in flight at d_v = 64: five
  // measured 1 us slower on the 350M shape)
  static constexpr int DEPTH = DV >= 128 ? 2 : (NW > kWaves ? 4 : 3);
  // fused absorption: 16-byte pieces of M_h per lane and load round, one
  // round of 32 where the registers allow it (no spills), else rounds of 16
  static constexpr int AR = (DV >= 128 && NRC < 2 && NW <= 8) ? 32 : 16;
  static constexpr int QS_STRIDE = DV + 4;                   // padded LDS rows (floats)
  static constexpr int QR_STRIDE = 32 * NRC + 4;
  static constexpr int LDS_PRO = HPG * (QS_STRIDE + QR_STRIDE);
  static constexpr int LDS_RED = NW * HPG * (DV + 2);
  static constexpr int LDS_FLOATS = LDS_PRO > LDS_RED ? LDS_PRO : LDS_RED;
};

// GQA = true builds the matched grouped-query baseline the paper compares
// against (Section 2): the scores read an explicit, already-rotated key
// stream per group instead of the value rows, with no positional term and
// the raw query; P.V, the softmax, the splits and the layout are shared, so
// the two kernels differ only in the bytes they must stream.
// PAGED reads the caches from page pools through a block table: only the
// addressing of a tile (and of the current row) changes.
// KR_STREAM loads the positional-key tiles with the non-temporal policy too
// (decode_kr_stream decides).
template <int HPG, int DV, int NRC, bool GQA, bool FUSED, bool PAGED, bool KR_STREAM = false, int NW = kWaves>
__global__ void __launch_bounds__(64 * NW, NW == kWaves ? 2 : 1)
    decode_bf16_kernel(GVA_DECODE_HEAD_ARGS, DecodeParams p) {
  static_assert(!(GQA && FUSED), "the GQA baseline takes the raw query");
  static_assert(!(GQA && PAGED), "the GQA baseline reads contiguous caches");
  const DecodeArgs a = decode_args<FUSED || GQA>(GVA_DECODE_HEAD_NAMES, p);
  using Cfg = DecodeCfg<HPG, DV, NRC, NW, GQA>;
  constexpr int NT = 64 * NW;                  // threads per workgroup
  using TileT = Tile<DV, NRC, GQA>;
  constexpr int NC = Cfg::NC, NB = Cfg::NB, DEPTH = Cfg::DEPTH, AR = Cfg::AR;
  __shared__ __attribute__((aligned(16))) float lds[Cfg::LDS_FLOATS];

  int b, s, g;
  bool empty_slot;
  if (!work_item(a, b, s, g, empty_slot)) return;   // grid padding
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index, uniform (SGPR)
  const int n = lane & 15, qd = lane >> 4;     // MFMA column / row slot and 16-lane row
  const int h0 = g * HPG;
  // Column roles: [hi_0 .. hi_{HPG-1}, lo_{HPG-1} .. lo_0, zero padding].
  const bool active = n < 2 * HPG;
  const bool is_lo = n >= HPG;
  const int col_head = !active ? 0 : (is_lo ? 2 * HPG - 1 - n : n);
  const int hq = h0 + col_head;
  const bf16x8 zero8 = as_bf16x8(u32x4{0u, 0u, 0u, 0u});
  __shared__ __attribute__((aligned(16))) uint16_t prow[DV + 32 * (NRC > 0 ? NRC : 1)];
  __shared__ int32_t split_pages[PAGED ? kMaxPages : 1];   // paged: this split's page ids

  // The rows of this split are settled once the query loads are on their
  // way (they do not depend on the length), which takes a memory round trip
  // off the prologue.  The length is a scalar load through the constant
  // address space, requested here and waited for at first use.
  const int len_b = *(const __attribute__((address_space(4))) int32_t*)(a.lens + b);
  int L = 0, r0 = 0, r1 = 0;
  auto settle_rows = [&]() {
    L = len_b < 0 ? 0 : (len_b > a.t_max ? a.t_max : len_b);
    split_rows(L, a.S, a.split_rows, s, r0, r1);
    return r0 < r1 || s == 0;
  };
  auto write_empty = [&]() {                   // an empty split past the first: lse only
    if (tid < HPG) a.lse_part[((int64_t)b * a.H + h0 + tid) * a.S + s] = -INFINITY;
  };
  if (empty_slot && s > 0) {                   // bounded chunks: a split with no rows
    write_empty();
    return;
  }

  // ---- loads that do not depend on the length, oldest first: the current
  // token's rows (staged first, below), then the query.  Loads retire in
  // order, so waiting for them never waits for the tiles requested later.
  // (kept as loaded bits: converting them here would wait for them here)
  u32x4 pend_piece = {0u, 0u, 0u, 0u};
  uint32_t pend_kbits = 0u;
  double kfreq = 0.0;                          // the pair's RoPE frequency (kernel arguments)
  if (!GQA && a.v_new != nullptr) {
    if (tid < DV / 8)
      pend_piece = *(reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.v_new) + ((int64_t)b * a.G + g) * DV) + tid);
    if (tid < a.d_r / 2) {
      pend_kbits = *reinterpret_cast<const uint32_t*>(static_cast<const uint16_t*>(a.kr_new) + (int64_t)b * a.d_r + 2 * tid);
      kfreq = p.inv_freq[tid];
    }
  }
  // The query: raw bf16 (GQA baseline); pre-absorbed fp32 (q_abs, q_rot);
  // or, fused, the raw positional pair and the first round of q / M_h
  // chunks for this wave's first head.
  u32x4 xqg[GQA ? NC : 1];
  f32x4 xa[GQA ? 1 : NC][2];
  f32x4 xr[NRC > 0 ? NRC : 1][2];
  const int W = a.d_c + a.d_r;
  // Fused absorption, q~[i] = sum_k q[k] M_h[i][k]: M_h is read in whole
  // rows, 16 lanes of 16 bytes per row and 4 rows per load, so each load
  // covers whole cache lines (the MFMA operand order, 64 bytes of 16 rows
  // per load, took four times as long to arrive).  Each lane forms an
  // 8-term bf16 dot product with its piece of q, and a DPP sum over the
  // row's 16 lanes finishes the row.  Columns come in segments of 128, rows
  // in blocks of 4 AR: one load round per (segment, row block).  Loads are
  // unconditional, from clamped addresses (selecting a loaded value would
  // wait for it and for every load before it); pieces past d_c meet a
  // zeroed query piece.
  constexpr int ARB = DV / 4 / AR;             // row blocks per segment
  u32x4 am[FUSED ? AR : 1];
  u32x4 xqf = {0u, 0u, 0u, 0u};                // the query piece of the lane's columns
  const int nrounds = ((a.d_c + 127) / 128) * ARB;
  const int a_row = lane >> 4, a_col = 8 * (lane & 15);
  const int npair = a.d_r / 2;
  const int ptid = NT - 1 - tid;
  const bool has_pair = FUSED && ptid < HPG * npair;
  const int pair_h = npair > 0 ? ptid / npair : 0, pair_i = npair > 0 ? ptid % npair : 0;
  uint32_t rq_bits = 0u;                       // the raw positional pair (bf16 x 2)
  double qfreq = 0.0;
  auto load_round = [&](int hl, int ro) {      // the query piece and M_h pieces of one round
    const int h = h0 + hl;
    const int col = min((ro / ARB) * 128 + a_col, a.d_c - 8), rb = ro % ARB;
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) + ((int64_t)b * a.H + h) * W;
    const uint16_t* mh = static_cast<const uint16_t*>(a.m) + ((int64_t)h * DV + rb * AR * 4 + a_row) * a.d_c + col;
    xqf = *reinterpret_cast<const u32x4*>(qrow + col);
#pragma unroll
    for (int r = 0; r < AR; ++r) am[r] = *reinterpret_cast<const u32x4*>(mh + (int64_t)(4 * r) * a.d_c);
  };
  if constexpr (GQA) {
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) + ((int64_t)b * a.H + hq) * a.q_stride + 8 * qd;
#pragma unroll
    for (int c = 0; c < NC; ++c) xqg[c] = *reinterpret_cast<const u32x4*>(qrow + 32 * c);
  } else if constexpr (!FUSED) {
    const float* qa = a.q_abs + ((int64_t)b * a.H + hq) * DV + 8 * qd;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      xa[c][0] = *reinterpret_cast<const f32x4*>(qa + 32 * c);
      xa[c][1] = *reinterpret_cast<const f32x4*>(qa + 32 * c + 4);
    }
#pragma unroll
    for (int rc = 0; rc < NRC; ++rc) {
      const int j0 = min(32 * rc + 8 * qd, a.d_r - 8);    // lanes past d_r: any valid piece
      const float* qr = a.q_rot + ((int64_t)b * a.H + hq) * a.d_r + j0;
      xr[rc][0] = *reinterpret_cast<const f32x4*>(qr);
      xr[rc][1] = *reinterpret_cast<const f32x4*>(qr + 4);
    }
  } else {
    if (has_pair) {
      rq_bits = *reinterpret_cast<const uint32_t*>(
          static_cast<const uint16_t*>(a.q) + ((int64_t)b * a.H + h0 + pair_h) * W + a.d_c + 2 * pair_i);
      qfreq = p.inv_freq[pair_i];
    }
    if (w < HPG) load_round(w, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  request_args(a);
  if (!settle_rows()) {
    write_empty();
    return;
  }

  // Paged: the page ids of the split's rows [r0, r1), clamped into the pool
  // (an id outside it reads some page's data but never outside the pool).
  const int PR = PAGED ? a.page_rows : 1;
  const int pg0 = r0 / PR;
  if constexpr (PAGED) {
    const int npg = (r1 + PR - 1) / PR - pg0;
    const int32_t* bt = a.block_table + (int64_t)b * a.max_pages + pg0;
    for (int i = tid; i < npg; i += NT) {
      const int id = bt[i];
      split_pages[i] = id < 0 ? 0 : (id >= a.n_pages ? a.n_pages - 1 : id);
    }
    __syncthreads();
  }

  // With the current token's rows given, the split holding row L-1 takes
  // that row from them and streams only the rows before it from the cache.
  const bool pending = !GQA && a.v_new != nullptr && L > 0 && r0 <= L - 1 && L - 1 < r1;
  if (pending) r1 = L - 1;
  const int r1c = ((r1 + kLayoutRows - 1) / kLayoutRows) * kLayoutRows;

  // ---- streaming setup.  Rows are read through buffer descriptors that end
  // at the split's last layout tile: a tile past the end reads as zeros
  // without touching memory, so prefetches are issued unconditionally (the
  // wait counts stay static) and cost no traffic.  Each load is addressed as
  // a loop-invariant per-lane offset plus the tile base in a scalar
  // register.  Rows past the split inside its last layout tile may hold
  // never-written data; the tail tile zeroes them before use.
  const uint16_t* vbase = static_cast<const uint16_t*>(a.v) + ((int64_t)b * a.G + g) * a.t_max * DV;
  const uint16_t* kbase = static_cast<const uint16_t*>(a.kr) + (int64_t)b * a.t_max * a.d_r;
  const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(vbase), (short)0, r1c * DV * 2, kBufferWord3);
  const __amdgpu_buffer_rsrc_t kres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(kbase), (short)0, r1c * a.d_r * 2, kBufferWord3);
  const __amdgpu_buffer_rsrc_t kcres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(GQA ? static_cast<const void*>(static_cast<const uint16_t*>(a.k_gqa) +
                                                       ((int64_t)b * a.G + g) * a.t_max * DV)
                            : static_cast<const void*>(vbase)),
      (short)0, r1c * DV * 2, kBufferWord3);
  const int kpieces = a.d_r / 8;              // 16-byte pieces per key row
  const int v_lane = qd * 256 + n * 16;       // piece qd of row n (of a 32-column chunk)
  int k_lane[NRC > 0 ? NRC : 1];
#pragma unroll
  for (int rc = 0; rc < NRC; ++rc)            // lanes past d_r re-read a valid piece (weight 0)
    k_lane[rc] = min(4 * rc + qd, kpieces - 1) * 256 + n * 16;
  const int v_tile_bytes = 16 * DV * 2, k_tile_bytes = 16 * a.d_r * 2;

  const int ntiles = (r1 - r0 + kTileRows - 1) / kTileRows;
  const int my_tiles = ntiles > w ? (ntiles - w + NW - 1) / NW : 0;
  auto tile_row = [&](int j) { return r0 + (w + NW * j) * kTileRows; };
  // Paged: the descriptors of the page holding a tile (a tile never spans
  // pages: pages are whole multiples of 32 rows), ending at the split's last
  // layout tile like the contiguous ones; a tile past it gets empty ones.
  auto page_res = [&](int row0, __amdgpu_buffer_rsrc_t& vr, __amdgpu_buffer_rsrc_t& kr, int& lt) {
    const int pg = row0 / PR;
    const bool live = row0 < r1c;
    const int page = live ? __builtin_amdgcn_readfirstlane(split_pages[pg - pg0]) : 0;
    const int rows = live ? min(PR, r1c - pg * PR) : 0;
    const uint16_t* vp = static_cast<const uint16_t*>(a.v) + ((int64_t)page * a.G + g) * PR * DV;
    const uint16_t* kp = static_cast<const uint16_t*>(a.kr) + (int64_t)page * PR * a.d_r;
    vr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(vp), (short)0, rows * DV * 2, kBufferWord3);
    kr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(kp), (short)0, rows * a.d_r * 2, kBufferWord3);
    lt = (row0 - pg * PR) / kLayoutRows;
  };
  auto load_tile = [&](TileT& t, int row0) {
    int lt = row0 / kLayoutRows;               // first layout tile (uniform)
    __amdgpu_buffer_rsrc_t tv = vres, tk = kres;
    if constexpr (PAGED) page_res(row0, tv, tk, lt);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const int vsoff = (lt + hf) * v_tile_bytes;
      if constexpr (GQA) {                     // keys first: the scores need them first
#pragma unroll
        for (int c = 0; c < NC; ++c)
          t.kc[hf][c] = as_bf16x8(__builtin_amdgcn_raw_buffer_load_b128(kcres, v_lane + 1024 * c, vsoff, kAuxNT));
      }
#pragma unroll
      for (int c = 0; c < NC; ++c)
        t.v[hf][c] = as_bf16x8(__builtin_amdgcn_raw_buffer_load_b128(tv, v_lane + 1024 * c, vsoff, kAuxNT));
      const int ksoff = (lt + hf) * k_tile_bytes;
#pragma unroll
      for (int rc = 0; rc < NRC; ++rc)
        t.k[hf][rc] = as_bf16x8(__builtin_amdgcn_raw_buffer_load_b128(tk, k_lane[rc], ksoff, KR_STREAM ? kAuxNT : 0));
    }
  };
  TileT buf[DEPTH];
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d) {
    load_tile(buf[d], tile_row(d));
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- the current token's rows (Algorithm 1's append): wave 0 rotates
  // the positional pair (fp64 angle, one rounding, exactly as append_kernel
  // does), stages the row in LDS for the epilogue and stores it into the
  // caches.  This workgroup is the only reader of row L-1 of stream (b, g)
  // in this launch; the shared positional key is stored once, by group 0.
  // Other workgroups may load the layout tile holding it, but only as rows
  // past their split, which are zeroed.  Run while the query loads land
  // (pre-absorbed path) or after the absorption (fused path, whose M_h
  // round holds too many registers to overlap it).
  auto stage_current_row = [&]() {
    if (!(pending && w == 0)) return;
    // row L-1 of stream (b, g), or, paged, row (L-1) mod page_rows of its page
    int64_t vs = ((int64_t)b * a.G + g) * a.t_max * DV, ks = (int64_t)b * a.t_max * a.d_r;
    int crow = L - 1;
    if constexpr (PAGED) {
      const int page = split_pages[(L - 1) / PR - pg0];
      vs = ((int64_t)page * a.G + g) * PR * DV;
      ks = (int64_t)page * PR * a.d_r;
      crow = (L - 1) % PR;
    }
    uint16_t* vcache = static_cast<uint16_t*>(a.v) + vs;
    uint16_t* kcache = static_cast<uint16_t*>(a.kr) + ks;
    if (tid < DV / 8) {
      *(reinterpret_cast<u32x4*>(prow) + tid) = pend_piece;
      *reinterpret_cast<u32x4*>(vcache + tiled_off<uint16_t>(crow, 8 * tid, DV)) = pend_piece;
    }
    if (tid < 16 * NRC) {
      uint16_t y0b = 0, y1b = 0;
      if (tid < a.d_r / 2) {
        double y0, y1;
        rotate_pair(bf16_bits_to_f32(pend_kbits & 0xFFFFu), bf16_bits_to_f32(pend_kbits >> 16),
                    (double)(L - 1) * kfreq, y0, y1);
        y0b = f64_to_bf16_rne(y0);
        y1b = f64_to_bf16_rne(y1);
        if (g == 0) {
          const int64_t o = tiled_off<uint16_t>(crow, 2 * tid, a.d_r);
          kcache[o] = y0b;
          kcache[o + 1] = y1b;
        }
      }
      prow[DV + 2 * tid] = y0b;
      prow[DV + 2 * tid + 1] = y1b;
    }
  };

  // ---- the query as MFMA B operands: absorbed, rotated and scaled, each
  // head's values split into bf16 high and low columns.
  bf16x8 bq[NC];
  bf16x8 bk[NRC > 0 ? NRC : 1];
  if constexpr (GQA) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x[2 * j] = bf16_bits_to_f32(xqg[c][j] & 0xFFFFu) * a.scale_log2;
        x[2 * j + 1] = bf16_bits_to_f32(xqg[c][j] >> 16) * a.scale_log2;
      }
      bq[c] = active ? split_hi_lo(x, is_lo) : zero8;
    }
  } else if constexpr (!FUSED) {
    stage_current_row();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x[j] = xa[c][0][j] * a.scale_log2;
        x[4 + j] = xa[c][1][j] * a.scale_log2;
      }
      bq[c] = active ? split_hi_lo(x, is_lo) : zero8;
    }
#pragma unroll
    for (int rc = 0; rc < NRC; ++rc) {
      const bool in_range = 32 * rc + 8 * qd < a.d_r;
      float x[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x[j] = xr[rc][0][j] * a.scale_log2;
        x[4 + j] = xr[rc][1][j] * a.scale_log2;
      }
      bk[rc] = (active && in_range) ? split_hi_lo(x, is_lo) : zero8;
    }
  } else {
    // Fused absorption, wave w taking heads w, w+4, ...: each round's rows
    // are finished by a sum over their lanes and stored (first segment) or
    // added (later segments) by the row's first lane, pre-scaled.  The first
    // round was loaded above.
    float* qs = lds;                                  // [HPG][QS_STRIDE]
    float* qrs = lds + HPG * Cfg::QS_STRIDE;          // [HPG][QR_STRIDE]
    auto absorb_round = [&](int hl, int ro) {
      const int rb = ro % ARB;
      const u32x4 qv = (ro / ARB) * 128 + a_col < a.d_c ? xqf : u32x4{0u, 0u, 0u, 0u};
      float v[AR];
#pragma unroll
      for (int r = 0; r < AR; ++r) v[r] = dot8_bf16(am[r], qv);
#pragma unroll
      for (int r = 0; r < AR; ++r) v[r] = sum16(v[r]) * a.scale_log2;
      // every lane of a row's 16 writes the same value
      float* dst = qs + hl * Cfg::QS_STRIDE + rb * AR * 4 + a_row;
      if (ro < ARB) {
#pragma unroll
        for (int r = 0; r < AR; ++r) dst[4 * r] = v[r];
      } else {
#pragma unroll
        for (int r = 0; r < AR; ++r) dst[4 * r] += v[r];
      }
    };
    // the first round (loaded before the tiles) in straight-line code, so
    // its waits count only its own loads; then the rest
    if (w < HPG) absorb_round(w, 0);
    for (int hl = w; hl < HPG; hl += NW)
      for (int ro = hl == w ? 1 : 0; ro < nrounds; ++ro) {
        load_round(hl, ro);
        absorb_round(hl, ro);
      }
    stage_current_row();
    // rotate the positional query at position L-1 (fp64 angle, reduced
    // exactly, fp32 rotation); the padding past d_r is written as zeros in
    // the same phase, so one barrier covers both
    if (has_pair) {
      float y0, y1;
      rotate_query_pair(bf16_bits_to_f32(rq_bits & 0xFFFFu), bf16_bits_to_f32(rq_bits >> 16),
                        (double)(L > 0 ? L - 1 : 0) * qfreq, a.scale_log2, y0, y1);
      qrs[pair_h * Cfg::QR_STRIDE + 2 * pair_i] = y0;
      qrs[pair_h * Cfg::QR_STRIDE + 2 * pair_i + 1] = y1;
    }
    if constexpr (NRC > 0) {
      for (int idx = tid; idx < HPG * 32 * NRC; idx += NT) {
        const int j = idx % (32 * NRC);
        if (j >= a.d_r) qrs[(idx / (32 * NRC)) * Cfg::QR_STRIDE + j] = 0.f;
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const float* src = qs + col_head * Cfg::QS_STRIDE + 32 * c + 8 * qd;
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = src[j];
      bq[c] = active ? split_hi_lo(x, is_lo) : zero8;
    }
#pragma unroll
    for (int rc = 0; rc < NRC; ++rc) {
      const float* src = qrs + col_head * Cfg::QR_STRIDE + 32 * rc + 8 * qd;
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = src[j];
      bk[rc] = active ? split_hi_lo(x, is_lo) : zero8;
    }
  }

  // identity selectors for the V transpose: E_half[k][n] = (k == n + 16 half)
  bf16x8 esel[2];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    u32x4 u = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (8 * qd + j == n + 16 * half) u[j >> 1] |= 0x3F80u << (16 * (j & 1));
    esel[half] = as_bf16x8(u);
  }

  // ---- streaming loop
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 acc[NB];
#pragma unroll
  for (int ib = 0; ib < NB; ++ib) acc[ib] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto compute_tile = [&](TileT& t, int row0, int row_end) {
    if (row0 + kTileRows > row_end) {        // ragged tail: clear rows past the end
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const bool dead = row0 + 16 * hf + n >= row_end;
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
    // scores: rows 16*hf + 4*qd + jj of the tile, column n
    f32x4 sc[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      sc[hf] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < NC; ++c) sc[hf] = mfma16(GQA ? t.kc[hf][c] : t.v[hf][c], bq[c], sc[hf]);
#pragma unroll
      for (int rc = 0; rc < NRC; ++rc) sc[hf] = mfma16(t.k[hf][rc], bk[rc], sc[hf]);
    }
    float x[8];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const float v = sc[hf][jj];
        x[4 * hf + jj] = v + mirror<HPG>(v);   // hi + lo part of the same head
      }
    if (row0 + kTileRows > row_end) {        // ragged tail: rows past the end
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (row0 + 16 * (k >> 2) + 4 * qd + (k & 3) >= row_end) x[k] = -INFINITY;
    }
    float mt = x[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) mt = fmaxf(mt, x[k]);
    mt = max_over_rows(mt);
    const float m_new = fmaxf(m_run, mt);
    if (__ballot(m_new > m_run) != 0) {      // rescale only when a max grew
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int ib = 0; ib < NB; ++ib) acc[ib] *= alpha;
      m_run = m_new;
    }
    float pr[8];
    float psum = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      pr[k] = __builtin_amdgcn_exp2f(x[k] - m_run);
      psum += pr[k];
    }
    l_run += psum;
    const bf16x8 bp = active ? split_hi_lo(pr, is_lo) : zero8;
    // P.V: transpose each 16x16 block of V with an identity MFMA, then
    // accumulate O^T[i][n] over the tile's 32 rows.
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        const f32x4 t0 = mfma16(t.v[0][c], esel[half], z);
        const f32x4 t1 = mfma16(t.v[1][c], esel[half], z);
        bf16x8 a;
        const bf16x2 a01 = __builtin_convertvector((f32x2{t0[0], t0[1]}), bf16x2);
        const bf16x2 a23 = __builtin_convertvector((f32x2{t0[2], t0[3]}), bf16x2);
        const bf16x2 a45 = __builtin_convertvector((f32x2{t1[0], t1[1]}), bf16x2);
        const bf16x2 a67 = __builtin_convertvector((f32x2{t1[2], t1[3]}), bf16x2);
        a[0] = a01[0]; a[1] = a01[1]; a[2] = a23[0]; a[3] = a23[1];
        a[4] = a45[0]; a[5] = a45[1]; a[6] = a67[0]; a[7] = a67[1];
        acc[2 * c + half] = mfma16(a, bp, acc[2 * c + half]);
      }
  };

  // DEPTH-stage register pipeline: tile j+DEPTH-1 is requested before tile
  // j is consumed.  Every iteration issues the same loads, so the waits the
  // compiler places are exact; the scheduling barrier keeps each tile's
  // loads in issue order, so the oldest tile is always the first to land.
  for (int jt = 0; jt < my_tiles; jt += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const int j = jt + d;
      if (j >= my_tiles) break;
      load_tile(buf[(d + DEPTH - 1) % DEPTH], tile_row(j + DEPTH - 1));
      __builtin_amdgcn_sched_barrier(0);
      compute_tile(buf[d], tile_row(j), r1);
    }
  }

  // ---- the current token's row, staged in LDS by wave 0 in the prologue,
  // scored by wave 0 as a one-row tile
  if (pending && w == 0) {
    TileT t;
    const u32x4* pv = reinterpret_cast<const u32x4*>(prow);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      t.v[0][c] = n == 0 ? as_bf16x8(pv[4 * c + qd]) : zero8;
      t.v[1][c] = zero8;
    }
#pragma unroll
    for (int rc = 0; rc < NRC; ++rc) {
      t.k[0][rc] = n == 0 ? as_bf16x8(pv[DV / 8 + 4 * rc + qd]) : zero8;
      t.k[1][rc] = zero8;
    }
    compute_tile(t, L - 1, L);
  }

  // ---- merge the waves and write this split's partial
  l_run = sum_over_rows(l_run);
#pragma unroll
  for (int ib = 0; ib < NB; ++ib)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) acc[ib][jj] += mirror<HPG>(acc[ib][jj]);

  __syncthreads();   // the prologue's LDS is reused below
  constexpr int RS = DV + 2;                     // per-(wave, head) record: [m, l, o[DV]]
  float* red = lds;
  if (n < HPG) {
    float* rec = red + (w * HPG + n) * RS;
    if (qd == 0) {
      rec[0] = m_run;
      rec[1] = l_run;
    }
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) rec[2 + 16 * ib + 4 * qd + jj] = acc[ib][jj];
  }
  __syncthreads();
  for (int idx = tid; idx < HPG * DV; idx += NT) {
    const int hl = idx / DV, i = idx % DV;
    float mx = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) mx = fmaxf(mx, red[(ww * HPG + hl) * RS]);
    float o = 0.f, lsum = 0.f;
    if (mx != -INFINITY) {
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        const float* rec = red + (ww * HPG + hl) * RS;
        const float sc = rec[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(rec[0] - mx);
        lsum += rec[1] * sc;
        o += rec[2 + i] * sc;
      }
      o /= lsum;
    }
    const int64_t prow = ((int64_t)b * a.H + h0 + hl) * a.S + s;
    a.o_part[prow * DV + i] = o;
    if (i == 0) a.lse_part[prow] = mx == -INFINITY ? -INFINITY : (mx + log2f(lsum)) * kLn2;
  }
}

// ========================================================== decode (f32)
// fp32 storage on the fp32 matrix products (v_mfma 16x16x4 f32: full fp32
// multiply-adds), built like the bf16 kernel: a workgroup owns one
// (b, g, split), its waves take interleaved 16-row tiles and keep DEPTH of
// them in registers.  In the tiled layout a wave's 16-byte load gives lane
// (n, qd) = (lane % 16, lane / 16) four columns 4 qd + e of row n, so element
// e of every lane is the A operand of one product over columns
// {4 qd + e}, and the query's B operand is the same four entries of head n.
//   scores  S^T[t][n] += V[t][4 qd + e] q[n][4 qd + e]      e = 0..3 per chunk
//   P.V     O^T[i][n] += V^T[i][4 qd + j] P[4 qd + j][n]    j = 0..3 per block
// The scores come back with rows 4 qd + j in register j, the B operand of
// P.V as they are; V^T goes through LDS (a tile of the wave's own, rows
// padded by 16 bytes so that neither side conflicts), which moves bits and
// costs less than products with an identity would (4 of 16 x 16 x 4 per
// block).  NC and NRC are d_v and d_r in 16-column chunks, rounded up: pieces
// past either re-read a valid one, are zeroed and meet a zero query, and their
// outputs are not written.
// The matrix cores take 256 cycles per 16 x 16 block of a tile (9.8 TB/s of
// rows at 2.4 GHz), whatever the heads per group, so the kernel is bound by
// latency at the sizes fp32 is used at.  The kernel it replaced scored one
// row per lane on the vector units with every query entry read from LDS, and
// read each value row a second time for P.V.  Step times, then and now: B1
// T256 H8 G2 d 64/16 45.0 -> 9.6 us; B8 of up to 4096 rows, H16 G4 d 64/16,
// 87.2 -> 18.2 us; B32 T4096 H32 G8 d 128/16 (545 MB)
// 1051 -> 104 us, 5.2 TB/s.
constexpr int kF32MaxHpg = 8;
constexpr int kF32MaxDv = 256;
constexpr int kF32MaxDr = 64;
constexpr int kF32TileRows = 16;

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int NC, int NRC, int NW>
struct F32Cfg {
  static constexpr int PITCH = 16 * NC + 4;                  // floats per padded LDS row
  static constexpr int QR_PITCH = 16 * NRC + 4;
  static constexpr int DEPTH = NC <= 4 ? 4 : (NC <= 8 && NRC == 1 ? 3 : 2);
  static constexpr int AR = NC <= 4 ? 8 : 16;                // absorption: loads of four map rows per round
  static constexpr int LDS_PRO = kF32MaxHpg * (PITCH + QR_PITCH);
  static constexpr int LDS_TR = NW * 16 * PITCH;
  static constexpr int LDS_RED = NW * kF32MaxHpg * PITCH;    // per (wave, head): o, m, l
  static constexpr int LDS_A = LDS_PRO > LDS_TR ? LDS_PRO : LDS_TR;
  static constexpr int LDS_FLOATS = LDS_A > LDS_RED ? LDS_A : LDS_RED;
};

template <int NC, int NRC, int NW>
__global__ void __launch_bounds__(64 * NW, NW == kWaves && NC <= 8 ? 2 : 1)
    decode_f32_kernel(GVA_DECODE_HEAD_ARGS, DecodeParams p) {
  using Cfg = F32Cfg<NC, NRC, NW>;
  constexpr int NT = 64 * NW, DEPTH = Cfg::DEPTH, AR = Cfg::AR, PITCH = Cfg::PITCH, QRP = Cfg::QR_PITCH;
  const bool fused = (head_dims >> 26 & 1) != 0;
  DecodeArgs a = decode_args<true>(GVA_DECODE_HEAD_NAMES, p);
  if (!fused) {                                // the same two places carry the absorbed query
    a.q_abs = static_cast<const float*>(a.q);
    a.q_rot = static_cast<const float*>(a.m);
  }
  __shared__ __attribute__((aligned(16))) float lds[Cfg::LDS_FLOATS];
  __shared__ __attribute__((aligned(16))) float prow[16 * NC + 16 * NRC];   // the current token's row

  int b, s, g;
  bool empty_slot;
  if (!work_item(a, b, s, g, empty_slot)) return;   // grid padding
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, qd = lane >> 4;
  const int hpg = a.H / a.G, h0 = g * hpg;
  const int DV = a.d_v, DR = a.d_r;
  const int len_b = *(const __attribute__((address_space(4))) int32_t*)(a.lens + b);
  if (empty_slot && s > 0) {                   // bounded chunks: a split with no rows
    if (tid < hpg) a.lse_part[((int64_t)b * a.H + h0 + tid) * a.S + s] = -INFINITY;
    return;
  }

  // ---- loads that do not depend on the length: the current token's rows,
  // then the first round of the absorption
  f32x4 pend_piece = {0.f, 0.f, 0.f, 0.f};
  float pk0 = 0.f, pk1 = 0.f;
  double kfreq = 0.0;
  if (a.v_new != nullptr) {
    if (tid < DV / 4)
      pend_piece = *(reinterpret_cast<const f32x4*>(static_cast<const float*>(a.v_new) + ((int64_t)b * a.G + g) * DV) + tid);
    if (tid < DR / 2) {
      const float* kn = static_cast<const float*>(a.kr_new) + (int64_t)b * DR + 2 * tid;
      pk0 = kn[0];
      pk1 = kn[1];
      kfreq = p.inv_freq[tid];
    }
  }
  // Fused absorption: a job is 4 AR rows of one head's map, wave w taking
  // jobs w, w + NW, ...; a load covers four rows of 64 columns (16 lanes of
  // 16 bytes each), a round AR loads.  Rows that are not whole 16-byte
  // pieces (d_c not a multiple of 4) are read element by element.
  const int W = a.d_c + DR;
  const bool whole = (a.d_c & 3) == 0;
  const int per_head = (DV + 4 * AR - 1) / (4 * AR);
  const int njobs = fused ? hpg * per_head : 0;
  const int nseg = (a.d_c + 63) / 64;
  f32x4 am[AR], xq = {0.f, 0.f, 0.f, 0.f};
  auto load4 = [&](const float* row, int col) __attribute__((always_inline)) {
    if (whole) return *reinterpret_cast<const f32x4*>(row + min(col, a.d_c - 4));
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = row[min(col + e, a.d_c - 1)];
    return x;
  };
  auto load_round = [&](int job, int seg) __attribute__((always_inline)) {    // columns past d_c: valid ones, against zeros of the query
    const int hl = job / per_head, i0 = (job % per_head) * 4 * AR + qd;
    const int col = 64 * seg + 4 * n;
    xq = load4(static_cast<const float*>(a.q) + ((int64_t)b * a.H + h0 + hl) * W, col);
    const float* mh = static_cast<const float*>(a.m) + (int64_t)(h0 + hl) * DV * a.d_c;
#pragma unroll
    for (int r = 0; r < AR; ++r) am[r] = load4(mh + (int64_t)min(i0 + 4 * r, DV - 1) * a.d_c, col);
  };
  const int npair = DR / 2;
  const int ptid = NT - 1 - tid;
  const bool has_pair = fused && ptid < hpg * npair;
  const int pair_h = npair > 0 ? ptid / npair : 0, pair_i = npair > 0 ? ptid % npair : 0;
  float rq0 = 0.f, rq1 = 0.f;
  double qfreq = 0.0;
  if (has_pair) {
    const float* qp = static_cast<const float*>(a.q) + ((int64_t)b * a.H + h0 + pair_h) * W + a.d_c + 2 * pair_i;
    rq0 = qp[0];
    rq1 = qp[1];
    qfreq = p.inv_freq[pair_i];
  }
  if (w < njobs && nseg > 0) load_round(w, 0);
  __builtin_amdgcn_sched_barrier(0);
  request_args(a);

  const int L = len_b < 0 ? 0 : (len_b > a.t_max ? a.t_max : len_b);
  int r0, r1;
  split_rows(L, a.S, a.split_rows, s, r0, r1);
  if (r0 >= r1 && s > 0) {                     // an empty split past the first: lse only
    if (tid < hpg) a.lse_part[((int64_t)b * a.H + h0 + tid) * a.S + s] = -INFINITY;
    return;
  }
  const bool pending = a.v_new != nullptr && L > 0 && r0 <= L - 1 && L - 1 < r1;
  if (pending) r1 = L - 1;
  const int r1c = (r1 + kLayoutRows - 1) / kLayoutRows * kLayoutRows;

  // ---- streaming setup, as in the bf16 kernel: descriptors that end at the
  // split's last layout tile, so prefetches past it read zeros unconditionally
  const float* vbase = static_cast<const float*>(a.v) + ((int64_t)b * a.G + g) * a.t_max * DV;
  const float* kbase = static_cast<const float*>(a.kr) + (int64_t)b * a.t_max * DR;
  const __amdgpu_buffer_rsrc_t vres =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(vbase), (short)0, r1c * DV * 4, kBufferWord3);
  const __amdgpu_buffer_rsrc_t kres =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(kbase), (short)0, r1c * DR * 4, kBufferWord3);
  int v_lane[NC], k_lane[NRC];
#pragma unroll
  for (int c = 0; c < NC; ++c) v_lane[c] = min(4 * c + qd, DV / 4 - 1) * 256 + n * 16;
#pragma unroll
  for (int c = 0; c < NRC; ++c) k_lane[c] = max(min(4 * c + qd, DR / 4 - 1), 0) * 256 + n * 16;
  struct TileF {
    f32x4 v[NC], k[NRC];
  };
  const int ntiles = (r1 - r0 + kF32TileRows - 1) / kF32TileRows;
  const int my_tiles = ntiles > w ? (ntiles - w + NW - 1) / NW : 0;
  auto tile_row = [&](int j) { return r0 + (w + NW * j) * kF32TileRows; };
  auto load_tile = [&](TileF& t, int row0) __attribute__((always_inline)) {
    const int lt = row0 / kLayoutRows;
#pragma unroll
    for (int c = 0; c < NC; ++c)
      t.v[c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(vres, v_lane[c], lt * DV * 64, kAuxNT));
#pragma unroll
    for (int c = 0; c < NRC; ++c)
      t.k[c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(kres, k_lane[c], lt * DR * 64, 0));
  };
  TileF buf[DEPTH];
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d) {
    load_tile(buf[d], tile_row(d));
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- absorption (each lane's partial dots, summed over a row's 16 lanes)
  float* qs = lds;                             // [hpg][PITCH]
  float* qrs = lds + kF32MaxHpg * PITCH;       // [hpg][QRP]
  auto absorb_job = [&](int job, bool loaded) __attribute__((always_inline)) {
    const int hl = job / per_head, i0 = (job % per_head) * 4 * AR + qd;
    float v[AR];
#pragma unroll
    for (int r = 0; r < AR; ++r) v[r] = 0.f;
    for (int seg = 0; seg < nseg; ++seg) {
      if (!(loaded && seg == 0)) load_round(job, seg);
      f32x4 qv;
#pragma unroll
      for (int e = 0; e < 4; ++e) qv[e] = 64 * seg + 4 * n + e < a.d_c ? xq[e] : 0.f;
#pragma unroll
      for (int r = 0; r < AR; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[r] = fmaf(am[r][e], qv[e], v[r]);
    }
#pragma unroll
    for (int r = 0; r < AR; ++r) {
      v[r] = sum16(v[r]) * a.scale_log2;
      if (i0 + 4 * r < DV) qs[hl * PITCH + i0 + 4 * r] = v[r];
    }
  };
  if (w < njobs) absorb_job(w, true);
  for (int job = w + NW; job < njobs; job += NW) absorb_job(job, false);

  // ---- the current token's row: wave 0 rotates its positional pair (fp64,
  // rounded once, as append_kernel does), stores the row into the caches (it
  // is the only reader of row L-1 of the stream in this launch) and stages it
  if (pending && w == 0) {
    float* vcache = static_cast<float*>(a.v) + ((int64_t)b * a.G + g) * a.t_max * DV;
    if (tid < 4 * NC) *(reinterpret_cast<f32x4*>(prow) + tid) = pend_piece;   // zeros past d_v
    if (tid < DV / 4) *reinterpret_cast<f32x4*>(vcache + tiled_off<float>(L - 1, 4 * tid, DV)) = pend_piece;
    if (tid < 8 * NRC) {
      float y0f = 0.f, y1f = 0.f;
      if (tid < DR / 2) {
        double y0, y1;
        rotate_pair(pk0, pk1, (double)(L - 1) * kfreq, y0, y1);
        y0f = (float)y0;
        y1f = (float)y1;
        if (g == 0) {
          float* kcache = static_cast<float*>(a.kr) + (int64_t)b * a.t_max * DR + tiled_off<float>(L - 1, 2 * tid, DR);
          kcache[0] = y0f;
          kcache[1] = y1f;
        }
      }
      prow[16 * NC + 2 * tid] = y0f;
      prow[16 * NC + 2 * tid + 1] = y1f;
    }
  }
  if (has_pair) {
    double y0, y1;
    rotate_pair(rq0, rq1, (double)(L > 0 ? L - 1 : 0) * qfreq, y0, y1);
    qrs[pair_h * QRP + 2 * pair_i] = (float)(y0 * (double)a.scale_log2);
    qrs[pair_h * QRP + 2 * pair_i + 1] = (float)(y1 * (double)a.scale_log2);
  }
  __syncthreads();

  // ---- the query as B operands: lane (n, qd) holds entries 16 c + 4 qd .. + 3 of head n
  f32x4 bq[NC], bk[NRC];
  const bool active = n < hpg;
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int col = 16 * c + 4 * qd;
    bq[c] = zero4;
    if (active && col < DV)
      bq[c] = fused ? *reinterpret_cast<const f32x4*>(qs + n * PITCH + col)
                    : *reinterpret_cast<const f32x4*>(a.q_abs + ((int64_t)b * a.H + h0 + n) * DV + col) * a.scale_log2;
  }
#pragma unroll
  for (int c = 0; c < NRC; ++c) {
    const int col = 16 * c + 4 * qd;
    bk[c] = zero4;
    if (active && col < DR)
      bk[c] = fused ? *reinterpret_cast<const f32x4*>(qrs + n * QRP + col)
                    : *reinterpret_cast<const f32x4*>(a.q_rot + ((int64_t)b * a.H + h0 + n) * DR + col) * a.scale_log2;
  }
  __syncthreads();                             // the queries' LDS is the waves' transposition tiles from here on

  // the running maximum starts below every score but -inf (a row hidden from
  // the query): an exponential against it is 0, never -inf - -inf
  float m_run = -FLT_MAX, l_run = 0.f;
  f32x4 acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = zero4;
  float* const tr = lds + w * 16 * PITCH;
  const bool ragged = DV % 16 != 0 || DR % 16 != 0;   // the last chunks hold pieces past the row

  auto compute_tile = [&](TileF& t, int row0, int row_end) __attribute__((always_inline)) {
    const bool tail = row0 + kF32TileRows > row_end;
    // rows past the end may hold anything, and an infinity read again past the
    // row's width would meet the query's zero.  (One branch for both: with a
    // second one the d_v = 256 instance took 240 us where it takes 221, B100
    // T1024 H32 G4.)
    if (tail || ragged) {
      const bool dead = row0 + n >= row_end;
#pragma unroll
      for (int c = 0; c < NC; ++c) t.v[c] = dead || 16 * c + 4 * qd >= DV ? zero4 : t.v[c];
#pragma unroll
      for (int c = 0; c < NRC; ++c) t.k[c] = dead || 16 * c + 4 * qd >= DR ? zero4 : t.k[c];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) *reinterpret_cast<f32x4*>(tr + n * PITCH + 16 * c + 4 * qd) = t.v[c];
    f32x4 sc[2] = {zero4, zero4};
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) sc[e & 1] = mfma_f32(t.v[c][e], bq[c][e], sc[e & 1]);
#pragma unroll
    for (int c = 0; c < NRC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) sc[e & 1] = mfma_f32(t.k[c][e], bk[c][e], sc[e & 1]);
    float x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = sc[0][j] + sc[1][j];
      if (tail && row0 + 4 * qd + j >= row_end) x[j] = -INFINITY;
    }
    const float mt = max_over_rows(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
    const float m_new = fmaxf(m_run, mt);
    if (__ballot(m_new > m_run) != 0) {        // rescale only when a max grew
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] *= alpha;
      m_run = m_new;
    }
    float pr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pr[j] = __builtin_amdgcn_exp2f(x[j] - m_run);
      l_run += pr[j];
    }
    // the tile's rows, written above by the other lanes of this wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[c] = mfma_f32(tr[(4 * qd + j) * PITCH + 16 * c + n], pr[j], acc[c]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();           // the next tile's rows are written after these reads
  };

  for (int jt = 0; jt < my_tiles; jt += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      const int j = jt + d;
      if (j >= my_tiles) break;
      load_tile(buf[(d + DEPTH - 1) % DEPTH], tile_row(j + DEPTH - 1));
      __builtin_amdgcn_sched_barrier(0);
      compute_tile(buf[d], tile_row(j), r1);
    }
  }
  if (pending && w == 0) {                     // the current token's row, as a one-row tile
    TileF t;
#pragma unroll
    for (int c = 0; c < NC; ++c) t.v[c] = n == 0 ? *reinterpret_cast<const f32x4*>(prow + 16 * c + 4 * qd) : zero4;
#pragma unroll
    for (int c = 0; c < NRC; ++c)
      t.k[c] = n == 0 ? *reinterpret_cast<const f32x4*>(prow + 16 * NC + 16 * c + 4 * qd) : zero4;
    compute_tile(t, L - 1, L);
  }

  // ---- merge the waves and write this split's partial
  l_run = sum_over_rows(l_run);
  if (l_run == 0.f) m_run = -INFINITY;         // no row counted
  __syncthreads();                             // the transposition tiles are the records below
  if (active) {
    float* rec = lds + (w * kF32MaxHpg + n) * PITCH;
#pragma unroll
    for (int c = 0; c < NC; ++c) *reinterpret_cast<f32x4*>(rec + 16 * c + 4 * qd) = acc[c];
    if (qd == 0) {
      rec[16 * NC] = m_run;
      rec[16 * NC + 1] = l_run;
    }
  }
  __syncthreads();
  for (int idx = tid; idx < hpg * DV; idx += NT) {
    const int hl = idx / DV, i = idx % DV;
    float mx = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) mx = fmaxf(mx, lds[(ww * kF32MaxHpg + hl) * PITCH + 16 * NC]);
    float o = 0.f, lsum = 0.f;
    if (mx != -INFINITY) {
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        const float* rec = lds + (ww * kF32MaxHpg + hl) * PITCH;
        const float sc = rec[16 * NC] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(rec[16 * NC] - mx);
        lsum += rec[16 * NC + 1] * sc;
        o += rec[i] * sc;
      }
      o /= lsum;
    }
    const int64_t row = ((int64_t)b * a.H + h0 + hl) * a.S + s;
    a.o_part[row * DV + i] = o;
    if (i == 0) a.lse_part[row] = mx == -INFINITY ? -INFINITY : (mx + log2f(lsum)) * kLn2;
  }
}

// =============================================================== combine
// One wave per (b, h) row, lane = output element (up to 4 per lane).  A
// single pass keeps a running log-sum-exp and rescales the running sum;
// the split loads do not depend on each other, so they overlap.
// (Scalar arguments, all of them in registers before a wave starts: see
// GVA_DECODE_HEAD_ARGS.)
constexpr int kCombineMaxDv = 256;
constexpr long long kChunkItemsPerCu = 2;         // bounded chunks: chunks per CU
constexpr long long kMinChunkBytes = 128 << 10;   // bounded chunks: value bytes per chunk
constexpr long long kMinSplitStream = 192 << 10;  // even splits: a stream's value bytes worth splitting
constexpr long long kMinSplitBytes = 32 << 10;    // even splits: value bytes per split
constexpr long long kMaxEvenSplits = 16;

__global__ void __launch_bounds__(kThreads) combine_kernel(const float* o_part, const float* lse_part, float* o, float* lse,
                                                          int32_t rows, int32_t S, int32_t d_v) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (row >= rows) return;
  const float* lp = lse_part + (int64_t)row * S;
  const float* op = o_part + (int64_t)row * S * d_v;
  // the row's split LSEs, up to 4 per lane (S <= 256), and their maximum
  float l[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int s = lane + 64 * k;
    l[k] = s < S ? lp[s] : -INFINITY;
  }
  // The first kSpec splits' partials are requested with the LSEs, before it
  // is known which are empty (splits hold a sequence's rows from the front,
  // so the first ones are the likely non-empty ones): one memory round trip
  // less.  Empty splits' values are loaded but never used (selected away,
  // so whatever they hold cannot reach the output).
  constexpr int kSpec = 8;
  float v0[kSpec][4];
#pragma unroll
  for (int j = 0; j < kSpec; ++j)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = lane + 64 * u;
      v0[j][u] = (j < S && i < d_v) ? op[(int64_t)j * d_v + i] : 0.f;
    }
  float mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < 4; ++k) mx = fmaxf(mx, l[k]);
  mx = wave_max(mx);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  float z = 0.f;
  if (mx != -INFINITY) {
    float wk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      wk[k] = l[k] == -INFINITY ? 0.f : expf(l[k] - mx);
      z += wk[k];
    }
    z = wave_sum(z);
#pragma unroll
    for (int j = 0; j < kSpec; ++j) {
      if (j >= S) break;
      const float wj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wk[0]), j));
      const bool live = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l[0]), j)) != -INFINITY;
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = live ? fmaf(wj, v0[j][u], acc[u]) : acc[u];
    }
    // the remaining splits with rows, 8 at a time so their loads overlap
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (64 * k >= S) break;
      unsigned long long mask = __ballot(l[k] != -INFINITY);
      if (k == 0) mask &= ~((1ull << kSpec) - 1ull);
      while (mask != 0ull) {
        int sel[8];
        float wsel[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          sel[j] = -1;
          wsel[j] = 0.f;
          if (mask != 0ull) {
            const int bit = __builtin_ctzll(mask);
            mask &= mask - 1ull;
            sel[j] = 64 * k + bit;
            wsel[j] = __shfl(wk[k], bit, 64);
          }
        }
        float v[8][4];
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int i = lane + 64 * u;
            v[j][u] = (sel[j] >= 0 && i < d_v) ? op[(int64_t)sel[j] * d_v + i] : 0.f;
          }
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[u] = fmaf(wsel[j], v[j][u], acc[u]);
      }
    }
  }
  const float inv = z > 0.f ? 1.f / z : 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = lane + 64 * u;
    if (i < d_v) o[(int64_t)row * d_v + i] = acc[u] * inv;
  }
  if (lse != nullptr && lane == 0) lse[row] = mx == -INFINITY ? -INFINITY : mx + logf(z);
}

// At most kFewSplits splits: lanes n and n + 16 k hold split n's LSE, so the
// maximum and the sum over the splits are four DPP steps within 16 lanes
// (combine_kernel's two reductions go through LDS, about 0.3 us each), and the
// weights are read from their lanes.  The first kSpec partials are requested
// with the LSEs, as above; the others, all at once, when it is known which
// hold rows (an empty one re-reads the first partial instead).
// Step times: 350M shape, eight splits, 10.66 -> 9.34 us; B64 of 128 to 32K
// rows, H16 G2 d 128, up to sixteen splits, 46.6 -> 45.2 us.
constexpr int kFewSplits = 16;

__device__ __forceinline__ float max16(float x) {
  auto step = [](float v, auto ctrl) {
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, false)));
  };
  x = step(x, std::integral_constant<int, 0xB1>{});
  x = step(x, std::integral_constant<int, 0x1B>{});
  x = step(x, std::integral_constant<int, 0x141>{});
  return step(x, std::integral_constant<int, 0x140>{});
}

template <int U>
__global__ void __launch_bounds__(kThreads) combine_few_kernel(const float* o_part, const float* lse_part, float* o, float* lse,
                                                          int32_t rows, int32_t S, int32_t d_v) {
  const int lane = threadIdx.x & 63, n = lane & 15;
  const int row = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kWaves + (threadIdx.x >> 6)));
  if (row >= rows) return;
  const float* op = o_part + (int64_t)row * S * d_v;
  constexpr int kSpec = 8;
  const float l = n < S ? lse_part[(int64_t)row * S + n] : -INFINITY;
  float v[kSpec][U];
#pragma unroll
  for (int j = 0; j < kSpec; ++j)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = lane + 64 * u;
      v[j][u] = (j < S && i < d_v) ? op[(int64_t)j * d_v + i] : 0.f;
    }
  const float mx = fmaxf(max16(l), -INFINITY);
  const bool any = mx != -INFINITY;
  const unsigned live = any ? (unsigned)__ballot(l != -INFINITY) & 0xFFFFu : 0u;
  const float w = any && l != -INFINITY ? expf(l - mx) : 0.f;
  const float z = sum16(w);
  auto weight = [&](int j) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), j)); };
  float acc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) acc[u] = 0.f;
  auto add = [&](int j, const float (&x)[U]) {
    if (live >> j & 1)                         // an empty split's partial may hold anything
#pragma unroll
      for (int u = 0; u < U; ++u) acc[u] = fmaf(weight(j), x[u], acc[u]);
  };
  if (live >> kSpec) {                         // the further splits with rows
    float x[kFewSplits - kSpec][U];
#pragma unroll
    for (int j = kSpec; j < kFewSplits; ++j)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = lane + 64 * u;
        x[j - kSpec][u] = i < d_v ? op[(int64_t)((live >> j & 1) ? j : 0) * d_v + i] : 0.f;
      }
#pragma unroll
    for (int j = 0; j < kSpec; ++j) add(j, v[j]);
#pragma unroll
    for (int j = kSpec; j < kFewSplits; ++j) add(j, x[j - kSpec]);
  } else {
#pragma unroll
    for (int j = 0; j < kSpec; ++j) add(j, v[j]);
  }
  const float inv = z > 0.f ? 1.f / z : 0.f;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = lane + 64 * u;
    if (i < d_v) o[(int64_t)row * d_v + i] = acc[u] * inv;
  }
  if (lse != nullptr && lane == 0) lse[row] = mx == -INFINITY ? -INFINITY : mx + logf(z);
}

using DecodeFn = void (*)(GVA_DECODE_HEAD_ARGS, DecodeParams);

// Enqueues a decode launch; the leading arguments repeat those of p that the
// kernel's first instructions need.
void launch_decode(DecodeFn fn, long long grid, int threads, hipStream_t s, const DecodeParams& p, bool raw_query) {
  const DecodeArgs& a = p.a;
  const int dims = a.d_c | a.d_r << 10 | a.S << 17 | (raw_query ? 1 << 26 : 0) | (a.H / a.G) << 27;
  hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(threads), 0, s, a.lens, raw_query ? a.q : a.q_abs,
                     raw_query ? a.m : a.q_rot, a.v_new, a.kr_new, dims, a.B, a.G, a.split_rows, p);
}


template <int HPG, int DV, bool FUSED, bool PAGED>
DecodeFn pick_nrc(int nrc, bool kr_stream) {
  switch (nrc) {
    case 0: return decode_bf16_kernel<HPG, DV, 0, false, FUSED, PAGED>;
    case 1: return kr_stream ? decode_bf16_kernel<HPG, DV, 1, false, FUSED, PAGED, true>
                             : decode_bf16_kernel<HPG, DV, 1, false, FUSED, PAGED>;
    case 2: return kr_stream ? decode_bf16_kernel<HPG, DV, 2, false, FUSED, PAGED, true>
                             : decode_bf16_kernel<HPG, DV, 2, false, FUSED, PAGED>;
  }
  return nullptr;
}

template <int HPG, int DV>
DecodeFn pick_mode(int nrc, bool fused, bool paged, bool kr_stream) {
  if (paged) return fused ? pick_nrc<HPG, DV, true, true>(nrc, kr_stream) : pick_nrc<HPG, DV, false, true>(nrc, kr_stream);
  return fused ? pick_nrc<HPG, DV, true, false>(nrc, kr_stream) : pick_nrc<HPG, DV, false, false>(nrc, kr_stream);
}

template <int HPG>
DecodeFn pick_dv(int dv, int nrc, bool fused, bool paged, bool kr_stream) {
  switch (dv) {
    case 64: return pick_mode<HPG, 64>(nrc, fused, paged, kr_stream);
    case 128: return pick_mode<HPG, 128>(nrc, fused, paged, kr_stream);
  }
  return nullptr;
}

template <int DV>
DecodeFn pick_gqa_hpg(int hpg) {
  switch (hpg) {
    case 1: return decode_bf16_kernel<1, DV, 0, true, false, false>;
    case 2: return decode_bf16_kernel<2, DV, 0, true, false, false>;
    case 4: return decode_bf16_kernel<4, DV, 0, true, false, false>;
    case 8: return decode_bf16_kernel<8, DV, 0, true, false, false>;
  }
  return nullptr;
}

// Waves per GVA decode workgroup.  A launch with few workgroups leaves most
// CUs idle and is bound by each stream's chain of memory round trips, not
// by HBM: its workgroups take eight waves, so twice as many of each stream's
// tiles are in flight at once (one such workgroup per CU; sixteen waves
// would leave 128 registers per wave, too few for the tiles in flight).
// (The matched-GQA baseline, whose tiles carry a key row beside each value
// row, measured slower with eight waves at the 350M shape -- 14.5 against
// 13.2 us -- and keeps four.)
int decode_waves(long long grid, int n_cu) {
  return 2 * grid <= n_cu ? 8 : kWaves;
}

DecodeFn pick_gqa_decode(int hpg, int dv) {
  switch (dv) {
    case 64: return pick_gqa_hpg<64>(hpg);
    case 128: return pick_gqa_hpg<128>(hpg);
  }
  return nullptr;
}

// fused absorption, contiguous caches, NW waves (the few-workgroup launches)
template <int HPG, int DV, int NW>
DecodeFn pick_wide_nrc(int nrc) {
  switch (nrc) {
    case 0: return decode_bf16_kernel<HPG, DV, 0, false, true, false, false, NW>;
    case 1: return decode_bf16_kernel<HPG, DV, 1, false, true, false, false, NW>;
    case 2: return decode_bf16_kernel<HPG, DV, 2, false, true, false, false, NW>;
  }
  return nullptr;
}

template <int HPG>
DecodeFn pick_wide(int dv, int nrc, int nw) {
  switch (dv * 100 + nw) {
    case 6408: return pick_wide_nrc<HPG, 64, 8>(nrc);
    case 12808: return pick_wide_nrc<HPG, 128, 8>(nrc);
  }
  return nullptr;
}

DecodeFn pick_bf16_decode(int hpg, int dv, int nrc, bool fused, bool paged, bool kr_stream, int nw) {
  if (nw != kWaves) {
    if (!fused || paged) return nullptr;
    switch (hpg) {
      case 1: return pick_wide<1>(dv, nrc, nw);
      case 2: return pick_wide<2>(dv, nrc, nw);
      case 4: return pick_wide<4>(dv, nrc, nw);
      case 8: return pick_wide<8>(dv, nrc, nw);
    }
    return nullptr;
  }
  switch (hpg) {
    case 1: return pick_dv<1>(dv, nrc, fused, paged, kr_stream);
    case 2: return pick_dv<2>(dv, nrc, fused, paged, kr_stream);
    case 4: return pick_dv<4>(dv, nrc, fused, paged, kr_stream);
    case 8: return pick_dv<8>(dv, nrc, fused, paged, kr_stream);
  }
  return nullptr;
}

// The positional-key tiles are read by the G groups of a split through one
// L2, so they are normally cached.  With at least as many (sequence, group)
// streams as CUs, every L2 holds many sequences' keys at once and streaming
// them (non-temporal, like the value tiles) measured faster: B = 32, G = 8
// on 256 CUs gained 0.7-2.0 us per launch, while four long sequences
// (32 streams) lost 2.6-3 us.  Paged caches the same: 2.1-2.7 us per
// launch at B = 32, G = 8 with pages of 64 or 256 rows.
bool decode_kr_stream(const gva_dims* d) {
  return (long long)d->batch * d->n_groups >= device_cu_count();
}

template <int NC, int NW>
DecodeFn pick_f32_nrc(int d_r) {
  return d_r <= 16 ? decode_f32_kernel<NC, 1, NW> : (d_r <= 32 ? decode_f32_kernel<NC, 2, NW> : decode_f32_kernel<NC, 4, NW>);
}

// Waves per fp32 workgroup: eight while every CU has at most one workgroup
// (us per step, eight against four waves: B1 T2000 H8 G2 d 128 18.1 and 20.0;
// B32 T4096 H32 G8 d 128, 256 workgroups, 104 and 113; B16 T2000 H64 G8 45 and
// 54; the longest chains, B2 T8000 H8 G8 at 16 splits, lose 3%), four past
// that (B64 T1024 H16 G4, two per CU: 26.3 and 23.0).  Above d_v = 128 eight
// waves would not have the registers.
int f32_waves(const gva_dims* d, long long grid) {
  return d->d_v <= 128 && grid <= device_cu_count() ? 8 : kWaves;
}

DecodeFn pick_f32_decode(int d_v, int d_r, int nw) {
  if (d_v <= 64) return nw == kWaves ? pick_f32_nrc<4, kWaves>(d_r) : pick_f32_nrc<4, 8>(d_r);
  if (d_v <= 128) return nw == kWaves ? pick_f32_nrc<8, kWaves>(d_r) : pick_f32_nrc<8, 8>(d_r);
  return pick_f32_nrc<16, kWaves>(d_r);
}

// With launch = false every argument is checked and nothing is enqueued.
int absorb_impl(const gva_dims* dims, int n_per_seq, const void* q, const void* m, const int32_t* lens,
                float* q_abs, float* q_rot, void* stream, bool launch = true) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  if (n_per_seq < 1) return GVA_ERR_INVALID_ARG;
  if (!q || !m || !lens || !q_abs) return GVA_ERR_INVALID_ARG;
  if (dims->d_r > 0 && !q_rot) return GVA_ERR_INVALID_ARG;
  if (!aligned(q, 16) || !aligned(m, 16) || !aligned(lens, 4) || !aligned(q_abs, 16) ||
      (q_rot && !aligned(q_rot, 4)))
    return GVA_ERR_INVALID_ARG;
  if (dims->d_r / 2 > kMaxPairs) return GVA_ERR_UNSUPPORTED;
  const long long rows = (long long)dims->batch * n_per_seq;
  if (rows > (1LL << 20) || rows * dims->n_heads > 0x7FFFFFFFLL) return GVA_ERR_UNSUPPORTED;
  AbsorbParams p{};
  p.q = q;
  p.m = m;
  p.lens = lens;
  p.q_abs = q_abs;
  p.q_rot = q_rot;
  p.B = (int32_t)rows;
  p.H = dims->n_heads;
  p.d_v = dims->d_v;
  p.d_c = dims->d_c;
  p.d_r = dims->d_r;
  p.t_max = dims->t_max;
  p.n_per_seq = n_per_seq;
  // many rows (a prompt): each workgroup reuses M_h over 64 rows (32 from
  // 1024 rows on), which cuts the re-reads of M_h fourfold (twofold); a
  // decode batch keeps 16 rows per workgroup.  (2048 prompt rows at H = 16,
  // d = 64: 16.0 -> 10.3-11.1 us against one row block.)
  p.row_blocks = rows >= 2048 ? 4 : (rows >= 1024 ? 2 : 1);
  fill_inv_freq(dims, p.inv_freq);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (dims->dtype == GVA_DTYPE_BF16 && (dims->d_v % 16 != 0 || dims->d_c % 32 != 0 || dims->d_r % 8 != 0))
    return GVA_ERR_UNSUPPORTED;
  if (!launch) return GVA_OK;
  if (dims->dtype == GVA_DTYPE_BF16) {
    const long long rows_per_wg = 16LL * p.row_blocks;
    const dim3 grid(dims->n_heads, (unsigned)((rows + rows_per_wg - 1) / rows_per_wg));
    hipLaunchKernelGGL(absorb_bf16_kernel, grid, dim3(kThreads), 0, s, p);
  } else {
    hipLaunchKernelGGL(absorb_f32_kernel, dim3((unsigned)(rows * dims->n_heads)), dim3(128), 0, s, p);
  }
  return launch_status();
}

int append_impl(const gva_dims* dims, const gva_paging* paging, const int32_t* block_table, void* v_cache,
                void* kr_cache, const void* v_new, const void* kr_new, const int32_t* seq, const int32_t* pos,
                int32_t n_rows, void* stream) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  if (n_rows < 0) return GVA_ERR_INVALID_ARG;
  if (n_rows == 0) return GVA_OK;
  if (!v_cache || !v_new || !seq || !pos) return GVA_ERR_INVALID_ARG;
  if (dims->d_r > 0 && (!kr_cache || !kr_new)) return GVA_ERR_INVALID_ARG;
  if (!aligned(v_cache, 16) || !aligned(v_new, 16) || !aligned(seq, 4) || !aligned(pos, 4))
    return GVA_ERR_INVALID_ARG;
  if (dims->d_r > 0 && (!aligned(kr_cache, 16) || !aligned(kr_new, 4))) return GVA_ERR_INVALID_ARG;
  st = check_cache_layout(dims);
  if (st != GVA_OK) return st;
  AppendParams p{};
  p.v_cache = v_cache;
  p.kr_cache = kr_cache;
  p.v_new = v_new;
  p.kr_new = kr_new;
  p.seq = seq;
  p.pos = pos;
  p.B = dims->batch;
  p.G = dims->n_groups;
  p.t_max = dims->t_max;
  p.d_v = dims->d_v;
  p.d_r = dims->d_r;
  p.n_rows = n_rows;
  p.block_table = block_table;
  p.page_rows = paging ? paging->page_rows : 0;
  p.max_pages = paging ? paging->max_pages : 0;
  p.n_pages = paging ? paging->n_pages : 0;
  fill_inv_freq(dims, p.inv_freq);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const long long blocks = (n_rows + (long long)kAppendRows - 1) / kAppendRows;
  const int npc = dims->d_v / (int)(16 / elem_size(dims));
  const int kp = 8 * blocks * append_value_blocks(dims->n_groups, npc, 4) >= 3LL * device_cu_count() ? 4 : 1;
  const dim3 grid((unsigned)blocks,
                  (unsigned)(append_value_blocks(dims->n_groups, npc, kp) + append_pair_blocks(dims->d_r)));
  const auto fn = dims->dtype == GVA_DTYPE_BF16 ? (kp == 4 ? append_kernel<uint16_t, 4> : append_kernel<uint16_t, 1>)
                                                : (kp == 4 ? append_kernel<float, 4> : append_kernel<float, 1>);
  hipLaunchKernelGGL(fn, grid, dim3(kThreads), 0, s, p);
  return launch_status();
}

// A paging description consistent with dims: pages of whole 32-row tiles,
// a block-table row covering the capacity exactly, ids for at most
// kMaxPages pages per sequence.
int check_paging(const gva_dims* dims, const gva_paging* pg, const int32_t* block_table) {
  if (pg == nullptr || block_table == nullptr || !aligned(block_table, 4)) return GVA_ERR_INVALID_ARG;
  if (pg->page_rows < kTileRows || pg->page_rows % kTileRows != 0) return GVA_ERR_INVALID_ARG;
  if (pg->max_pages < 1 || pg->n_pages < 1) return GVA_ERR_INVALID_ARG;
  if ((long long)pg->max_pages * pg->page_rows != dims->t_max) return GVA_ERR_INVALID_ARG;
  if (pg->max_pages > kMaxPages) return GVA_ERR_UNSUPPORTED;
  if (dims->dtype != GVA_DTYPE_BF16) return GVA_ERR_UNSUPPORTED;
  return GVA_OK;
}

// The attention launch behind gva_decode_attention and, with paging given,
// gva_paged_decode_attention (v_cache / kr_cache are then the page pools).
int decode_attention_impl(const gva_dims* dims, const gva_paging* paging, const int32_t* block_table,
                          const void* q, const void* m, const float* q_abs, const float* q_rot,
                          void* v_cache, void* kr_cache, const int32_t* lens, const void* v_new,
                          const void* kr_new, int32_t num_splits, int32_t split_rows, float* o_part,
                          float* lse_part, void* stream, bool launch = true) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  if (num_splits < 1 || num_splits > GVA_MAX_SPLITS) return GVA_ERR_INVALID_ARG;
  if (split_rows < 0 || split_rows % kTileRows != 0) return GVA_ERR_INVALID_ARG;
  const bool fused = q != nullptr || m != nullptr;
  if (fused) {
    if (!q || !m || q_abs || q_rot) return GVA_ERR_INVALID_ARG;
    if (!aligned(q, 16) || !aligned(m, 16)) return GVA_ERR_INVALID_ARG;
  } else {
    if (!q_abs || (dims->d_r > 0 && !q_rot)) return GVA_ERR_INVALID_ARG;
    if (!aligned(q_abs, 16) || (q_rot && !aligned(q_rot, 16))) return GVA_ERR_INVALID_ARG;
  }
  if (!v_cache || !lens || !o_part || !lse_part) return GVA_ERR_INVALID_ARG;
  if (dims->d_r > 0 && !kr_cache) return GVA_ERR_INVALID_ARG;
  if (!aligned(v_cache, 16) || !aligned(lens, 4) || !aligned(o_part, 16) || !aligned(lse_part, 4) ||
      (dims->d_r > 0 && !aligned(kr_cache, 16)))
    return GVA_ERR_INVALID_ARG;
  if (!v_new && kr_new) return GVA_ERR_INVALID_ARG;          // the pending row comes whole
  if (v_new && (!aligned(v_new, 16) || (dims->d_r > 0 && (!kr_new || !aligned(kr_new, 4)))))
    return GVA_ERR_INVALID_ARG;
  st = check_cache_layout(dims);
  if (st != GVA_OK) return st;

  const int hpg = dims->n_heads / dims->n_groups;
  const long long n_items = decode_grid(dims, num_splits, split_rows);
  if (n_items > 0x7FFFFFFFLL) return GVA_ERR_UNSUPPORTED;

  DecodeParams p{};
  p.a.q = q;
  p.a.m = m;
  p.a.q_abs = q_abs;
  p.a.q_rot = q_rot;
  p.a.v = v_cache;
  p.a.kr = kr_cache;
  p.a.lens = lens;
  p.a.o_part = o_part;
  p.a.lse_part = lse_part;
  p.a.v_new = v_new;
  p.a.kr_new = kr_new;
  p.a.k_gqa = nullptr;
  p.a.q_stride = 0;
  p.a.B = dims->batch;
  p.a.H = dims->n_heads;
  p.a.G = dims->n_groups;
  p.a.d_v = dims->d_v;
  p.a.d_c = dims->d_c;
  p.a.d_r = dims->d_r;
  p.a.t_max = dims->t_max;
  p.a.S = num_splits;
  p.a.split_rows = split_rows;
  p.a.scale_log2 = scale_log2(dims);
  p.a.block_table = block_table;
  p.a.page_rows = paging ? paging->page_rows : 0;
  p.a.max_pages = paging ? paging->max_pages : 0;
  p.a.n_pages = paging ? paging->n_pages : 0;
  fill_inv_freq(dims, p.inv_freq);
  hipStream_t s = static_cast<hipStream_t>(stream);

  if (dims->dtype == GVA_DTYPE_BF16) {
    if (dims->d_c % 32 != 0 || dims->d_c > 512 || dims->d_r % 8 != 0 || dims->d_r > 64)
      return GVA_ERR_UNSUPPORTED;
    // the fused prologue absorbs at least one 32-column chunk of the query
    if (fused && dims->d_c == 0) return GVA_ERR_UNSUPPORTED;
    const int nrc = (dims->d_r + 31) / 32;
    const int nw = fused && paging == nullptr ? decode_waves(n_items, device_cu_count()) : kWaves;
    DecodeFn fn = pick_bf16_decode(hpg, dims->d_v, nrc, fused, paging != nullptr, decode_kr_stream(dims), nw);
    if (fn == nullptr) return GVA_ERR_UNSUPPORTED;
    if (!launch) return GVA_OK;
    launch_decode(fn, n_items, 64 * nw, s, p, fused);
  } else {
    if (paging != nullptr) return GVA_ERR_UNSUPPORTED;       // paged caches: bf16 only
    if (dims->d_v > kF32MaxDv || dims->d_c > 512 || dims->d_r > kF32MaxDr || hpg > kF32MaxHpg)
      return GVA_ERR_UNSUPPORTED;
    if (!launch) return GVA_OK;
    const int nw = f32_waves(dims, n_items);
    launch_decode(pick_f32_decode(dims->d_v, dims->d_r, nw), n_items, 64 * nw, s, p, fused);
  }
  return launch_status();
}

int combine_impl(const gva_dims* dims, const float* o_part, const float* lse_part, int32_t num_splits,
                 float* o, float* lse, void* stream, bool launch) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  if (num_splits < 1 || num_splits > GVA_MAX_SPLITS) return GVA_ERR_INVALID_ARG;
  if (!o_part || !lse_part || !o) return GVA_ERR_INVALID_ARG;
  if (!aligned(o_part, 4) || !aligned(lse_part, 4) || !aligned(o, 4) || (lse && !aligned(lse, 4)))
    return GVA_ERR_INVALID_ARG;
  if (dims->d_v > kCombineMaxDv) return GVA_ERR_UNSUPPORTED;
  if (!launch) return GVA_OK;
  const int rows = dims->batch * dims->n_heads;
  const dim3 grid((rows + kWaves - 1) / kWaves);
  const auto fn = num_splits > kFewSplits ? combine_kernel
                  : dims->d_v <= 64       ? combine_few_kernel<1>
                  : dims->d_v <= 128      ? combine_few_kernel<2>
                                          : combine_few_kernel<4>;
  hipLaunchKernelGGL(fn, grid, dim3(kThreads), 0, static_cast<hipStream_t>(stream), o_part, lse_part, o, lse, rows,
                     num_splits, dims->d_v);
  return launch_status();
}

// ---------------------------------------------------------- whole step
// One decode step in one call: the absorption (inside the attention launch,
// or its own launch, as gva_prefer_fused decides), the attention, and the
// combine when there are several splits.  The intermediate buffers -- the
// absorbed queries of the separate path and the split partials -- live in
// a workspace; with one split the attention writes o and lse directly.
constexpr size_t kWorkspaceAlign = 256;

struct StepLayout {
  bool fused;
  size_t q_abs, q_rot, o_part, lse_part;   // byte offsets into the workspace
  size_t bytes;                            // workspace bytes the step uses
};

inline size_t ws_round(size_t x) { return (x + kWorkspaceAlign - 1) / kWorkspaceAlign * kWorkspaceAlign; }

int step_layout(const gva_dims* d, int32_t num_splits, int32_t split_rows, StepLayout& L) {
  const int st = check_dims(d);
  if (st != GVA_OK) return st;
  if (num_splits < 1 || num_splits > GVA_MAX_SPLITS || split_rows < 0) return GVA_ERR_INVALID_ARG;
  L = StepLayout{};
  L.fused = gva_prefer_fused(d, num_splits, split_rows, 0) != 0;
  const size_t rows = (size_t)d->batch * (size_t)d->n_heads;
  size_t off = 0;
  if (!L.fused) {
    L.q_abs = off;
    off += ws_round(rows * (size_t)d->d_v * 4);
    L.q_rot = off;
    off += ws_round(rows * (size_t)d->d_r * 4);
  }
  if (num_splits > 1) {
    L.o_part = off;
    off += ws_round(rows * (size_t)num_splits * (size_t)d->d_v * 4);
    L.lse_part = off;
    off += ws_round(rows * (size_t)num_splits * 4);
  }
  L.bytes = off;
  return GVA_OK;
}

// The step's launches on workspace ws (L.bytes bytes, 256-byte aligned).
// Every launch is validated before the first is enqueued.
// With launch = false only the checks run.
int decode_step_impl(const gva_dims* dims, const void* q, const void* m, void* v_cache, void* kr_cache,
                     const int32_t* lens, const void* v_new, const void* kr_new, int32_t num_splits,
                     int32_t split_rows, char* ws, const StepLayout& L, float* o, float* lse, void* stream,
                     bool launch = true) {
  if (!q || !m || !o || !lse) return GVA_ERR_INVALID_ARG;
  const int S = num_splits;
  float* q_abs = L.fused ? nullptr : reinterpret_cast<float*>(ws + L.q_abs);
  float* q_rot = (L.fused || dims->d_r == 0) ? nullptr : reinterpret_cast<float*>(ws + L.q_rot);
  float* o_part = S > 1 ? reinterpret_cast<float*>(ws + L.o_part) : o;
  float* lse_part = S > 1 ? reinterpret_cast<float*>(ws + L.lse_part) : lse;
  const void* fq = L.fused ? q : nullptr;
  const void* fm = L.fused ? m : nullptr;
  for (int pass = 0; pass < (launch ? 2 : 1); ++pass) {   // pass 0 checks, pass 1 launches
    const bool go = pass == 1;
    int st = GVA_OK;
    if (!L.fused) st = absorb_impl(dims, 1, q, m, lens, q_abs, q_rot, stream, go);
    if (st == GVA_OK)
      st = decode_attention_impl(dims, nullptr, nullptr, fq, fm, q_abs, q_rot, v_cache, kr_cache, lens, v_new,
                                 kr_new, S, split_rows, o_part, lse_part, stream, go);
    if (st == GVA_OK && S > 1) st = combine_impl(dims, o_part, lse_part, S, o, lse, stream, go);
    if (st != GVA_OK) return st;
  }
  return GVA_OK;
}

}  // namespace

// ------------------------------------------------------- static scratch
// The workspace of gva_decode_step_static, for callers that cannot
// allocate: a file-scope device array, one copy on every GPU the library
// runs on, held until the process ends.  In host code `scratch` names a
// host-side stand-in, never the device memory: its device address is
// looked up once per device (hipGetSymbolAddress, with that device current)
// and only that address is passed to the kernels.
static __device__ __align__(256) unsigned char scratch[GVA_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_dev[kMaxDevices];   // per device: the address of its copy of scratch

int static_scratch(char** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GVA_ERR_HIP;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (scratch_dev[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return GVA_ERR_HIP;
    scratch_dev[dev] = ptr;
  }
  *out = static_cast<char*>(scratch_dev[dev]);
  return GVA_OK;
}

}  // namespace

extern "C" {


int gva_version(void) { return 20000; }

const char* gva_status_string(int status) {
  switch (status) {
    case GVA_OK: return "ok";
    case GVA_ERR_INVALID_ARG: return "invalid argument";
    case GVA_ERR_UNSUPPORTED: return "unsupported shape";
    case GVA_ERR_HIP: return "HIP runtime error";
    case GVA_ERR_SCRATCH: return "the step needs more than the static scratch buffer (GVA_STATIC_SCRATCH_BYTES)";
  }
  return "unknown status";
}

int gva_append_kv(const gva_dims* dims, void* v_cache, void* kr_cache, const void* v_new,
                  const void* kr_new, const int32_t* seq, const int32_t* pos, int32_t n_rows,
                  void* stream) {
  return append_impl(dims, nullptr, nullptr, v_cache, kr_cache, v_new, kr_new, seq, pos, n_rows, stream);
}

int gva_absorb_query(const gva_dims* dims, const void* q, const void* m, const int32_t* lens,
                     float* q_abs, float* q_rot, void* stream) {
  return absorb_impl(dims, 1, q, m, lens, q_abs, q_rot, stream);
}


int gva_decode_attention(const gva_dims* dims, const void* q, const void* m, const float* q_abs,
                         const float* q_rot, void* v_cache, void* kr_cache,
                         const int32_t* lens, const void* v_new, const void* kr_new,
                         int32_t num_splits, int32_t split_rows, float* o_part, float* lse_part,
                         void* stream) {
  return decode_attention_impl(dims, nullptr, nullptr, q, m, q_abs, q_rot, v_cache, kr_cache, lens, v_new,
                               kr_new, num_splits, split_rows, o_part, lse_part, stream);
}

int gva_paged_decode_attention(const gva_dims* dims, const gva_paging* paging, const void* q, const void* m,
                               const float* q_abs, const float* q_rot, void* v_pool, void* kr_pool,
                               const int32_t* block_table, const int32_t* lens, const void* v_new,
                               const void* kr_new, int32_t num_splits, int32_t split_rows, float* o_part,
                               float* lse_part, void* stream) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  st = check_paging(dims, paging, block_table);
  if (st != GVA_OK) return st;
  return decode_attention_impl(dims, paging, block_table, q, m, q_abs, q_rot, v_pool, kr_pool, lens, v_new,
                               kr_new, num_splits, split_rows, o_part, lse_part, stream);
}

int gva_paged_append_kv(const gva_dims* dims, const gva_paging* paging, void* v_pool, void* kr_pool,
                        const int32_t* block_table, const void* v_new, const void* kr_new, const int32_t* seq,
                        const int32_t* pos, int32_t n_rows, void* stream) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  st = check_paging(dims, paging, block_table);
  if (st != GVA_OK) return st;
  return append_impl(dims, paging, block_table, v_pool, kr_pool, v_new, kr_new, seq, pos, n_rows, stream);
}

int gva_gqa_decode_attention(const gva_dims* dims, const void* q, int32_t q_stride,
                             const void* k_cache, const void* v_cache, const int32_t* lens,
                             int32_t num_splits, int32_t split_rows, float* o_part, float* lse_part,
                             void* stream) {
  int st = check_dims(dims);
  if (st != GVA_OK) return st;
  if (num_splits < 1 || num_splits > GVA_MAX_SPLITS) return GVA_ERR_INVALID_ARG;
  if (split_rows < 0 || split_rows % kTileRows != 0) return GVA_ERR_INVALID_ARG;
  if (!q || !k_cache || !v_cache || !lens || !o_part || !lse_part) return GVA_ERR_INVALID_ARG;
  if (q_stride < dims->d_v) return GVA_ERR_INVALID_ARG;
  if (!aligned(q, 16) || !aligned(k_cache, 16) || !aligned(v_cache, 16) || !aligned(lens, 4) ||
      !aligned(o_part, 16) || !aligned(lse_part, 4))
    return GVA_ERR_INVALID_ARG;
  if (dims->dtype != GVA_DTYPE_BF16 || q_stride % 8 != 0) return GVA_ERR_UNSUPPORTED;
  if (dims->t_max % kLayoutRows != 0) return GVA_ERR_UNSUPPORTED;
  if ((double)dims->t_max * dims->d_v * 2.0 >= 2147483648.0 - 16777216.0) return GVA_ERR_UNSUPPORTED;
  const int hpg = dims->n_heads / dims->n_groups;
  const long long n_items = decode_grid(dims, num_splits, split_rows);
  if (n_items > 0x7FFFFFFFLL) return GVA_ERR_UNSUPPORTED;
  DecodeFn fn = pick_gqa_decode(hpg, dims->d_v);
  if (fn == nullptr) return GVA_ERR_UNSUPPORTED;

  DecodeParams p{};
  memset(&p, 0, sizeof(p));
  p.a.q = q;
  p.a.v = const_cast<void*>(v_cache);       // read only: the GQA kernel never appends
  p.a.k_gqa = k_cache;
  p.a.q_stride = q_stride;
  p.a.lens = lens;
  p.a.o_part = o_part;
  p.a.lse_part = lse_part;
  p.a.B = dims->batch;
  p.a.H = dims->n_heads;
  p.a.G = dims->n_groups;
  p.a.d_v = dims->d_v;
  p.a.d_c = dims->d_v;
  p.a.d_r = 0;
  p.a.t_max = dims->t_max;
  p.a.S = num_splits;
  p.a.split_rows = split_rows;
  const double sc = dims->scale > 0.0 ? dims->scale : 1.0 / sqrt((double)dims->d_v);
  p.a.scale_log2 = (float)(sc * kLog2e);
  launch_decode(fn, n_items, kThreads, static_cast<hipStream_t>(stream), p, true);
  return launch_status();
}

int gva_prefill_absorb(const gva_dims* dims, int32_t n_new, const void* q, const void* m,
                       const int32_t* lens, float* q_abs, float* q_rot, void* stream) {
  if (dims != nullptr && (n_new < 1 || n_new > dims->t_max)) return GVA_ERR_INVALID_ARG;
  return absorb_impl(dims, n_new, q, m, lens, q_abs, q_rot, stream);
}

int gva_combine(const gva_dims* dims, const float* o_part, const float* lse_part, int32_t num_splits,
                float* o, float* lse, void* stream) {
  return combine_impl(dims, o_part, lse_part, num_splits, o, lse, stream, true);
}

int gva_decode_workspace_size(const gva_dims* dims, int32_t num_splits, int32_t split_rows, size_t* bytes) {
  if (bytes == nullptr) return GVA_ERR_INVALID_ARG;
  StepLayout L;
  const int st = step_layout(dims, num_splits, split_rows, L);
  if (st != GVA_OK) return st;
  *bytes = L.bytes;
  return GVA_OK;
}

int gva_decode_step(const gva_dims* dims, const void* q, const void* m, void* v_cache, void* kr_cache,
                    const int32_t* lens, const void* v_new, const void* kr_new, int32_t num_splits,
                    int32_t split_rows, void* workspace, size_t workspace_bytes, float* o, float* lse,
                    void* stream) {
  StepLayout L;
  const int st = step_layout(dims, num_splits, split_rows, L);
  if (st != GVA_OK) return st;
  if (L.bytes > 0 && (workspace == nullptr || workspace_bytes < L.bytes || !aligned(workspace, kWorkspaceAlign)))
    return GVA_ERR_INVALID_ARG;
  return decode_step_impl(dims, q, m, v_cache, kr_cache, lens, v_new, kr_new, num_splits, split_rows,
                          static_cast<char*>(workspace), L, o, lse, stream);
}

int gva_decode_step_static(const gva_dims* dims, const void* q, const void* m, void* v_cache, void* kr_cache,
                           const int32_t* lens, const void* v_new, const void* kr_new, int32_t num_splits,
                           int32_t split_rows, float* o, float* lse, void* stream) {
  StepLayout L;
  int st = step_layout(dims, num_splits, split_rows, L);
  if (st != GVA_OK) return st;
  if (L.bytes > (size_t)GVA_STATIC_SCRATCH_BYTES) return GVA_ERR_SCRATCH;
  // every check before the first runtime call (the checks see a stand-in
  // workspace address, aligned like the buffer, that nothing dereferences);
  // then the device's scratch
  char* const stand_in = reinterpret_cast<char*>(kWorkspaceAlign);
  st = decode_step_impl(dims, q, m, v_cache, kr_cache, lens, v_new, kr_new, num_splits, split_rows, stand_in, L, o,
                        lse, stream, false);
  if (st != GVA_OK) return st;
  char* ws = nullptr;
  if (L.bytes > 0) {
    st = static_scratch(&ws);
    if (st != GVA_OK) return st;
  }
  return decode_step_impl(dims, q, m, v_cache, kr_cache, lens, v_new, kr_new, num_splits, split_rows, ws, L, o, lse,
                          stream);
}

int gva_prefer_fused(const gva_dims* dims, int32_t num_splits, int32_t split_rows, int32_t n_cu) {
  if (check_dims(dims) != GVA_OK || num_splits < 1 || split_rows < 0) return 0;
  if (n_cu <= 0) n_cu = device_cu_count();
  if (decode_grid(dims, num_splits, split_rows) <= 2LL * n_cu) return 1;
  // bounded chunks: each workgroup streams up to split_rows value rows
  // against the (H/G) d_c map rows of its absorption
  const long long map_rows = (long long)(dims->n_heads / dims->n_groups) * dims->d_c;
  return split_rows > 0 && split_rows >= map_rows ? 1 : 0;
}

int gva_pick_splits(const gva_dims* dims, int32_t max_len, int64_t total_len, int32_t n_cu,
                    int32_t* split_rows) {
  if (split_rows != nullptr) *split_rows = 0;
  if (check_dims(dims) != GVA_OK) return 1;
  if (n_cu <= 0) n_cu = device_cu_count();
  if (max_len <= 0 || max_len > dims->t_max) max_len = dims->t_max;
  const long long streams = (long long)dims->batch * dims->n_groups;
  if (total_len <= 0) total_len = (long long)dims->batch * max_len;
  const long long row_bytes = (long long)dims->d_v * (long long)elem_size(dims);
  const bool spread = 2 * total_len < (long long)dims->batch * max_len;
  // Few streams (at most a quarter of the CUs): even splits, one workgroup
  // per CU, whatever the spread of the lengths (bounded chunks measured
  // 4-30% slower there).
  const bool few_streams = 4 * streams <= n_cu;
  if (spread && split_rows != nullptr && !few_streams) {
    // Ragged lengths: bounded chunks, so every workgroup streams about the
    // same bytes whatever its sequence's length.  Chunks with rows number
    // at most stream_rows / c + streams (ceil(L / c) < L / c + 1);
    // c is chosen so that they fit the kChunkItemsPerCu resident
    // workgroups per CU, one dispatch round with no tail, when the streams
    // leave room for that; none shorter than kMinChunkBytes of value rows,
    // nor than the (H/G) d_c map rows a chunk's fused absorption reads.
    const long long stream_rows = total_len * dims->n_groups;
    const long long slots = kChunkItemsPerCu * n_cu;
    const long long room = slots - streams > slots / 2 ? slots - streams : slots / 2;
    long long c = (stream_rows + room - 1) / room;
    long long min_rows = (kMinChunkBytes + row_bytes - 1) / row_bytes;
    const long long map_rows = (long long)(dims->n_heads / dims->n_groups) * dims->d_c;
    if (min_rows < map_rows) min_rows = map_rows;
    if (c < min_rows) c = min_rows;
    c = (c + kTileRows - 1) / kTileRows * kTileRows;
    long long s = (max_len + c - 1) / c;
    if (s > GVA_MAX_SPLITS) {
      c = ((max_len + GVA_MAX_SPLITS - 1) / GVA_MAX_SPLITS + kTileRows - 1) / kTileRows * kTileRows;
      s = (max_len + c - 1) / c;
    }
    if (s > 1) {
      *split_rows = (int32_t)c;
      return (int)s;
    }
  }
  // Even splits.  A workgroup streams its rows at the pace of its own chain
  // of memory round trips, so a launch of fewer workgroups than CUs is
  // bound by that chain, not by HBM; splitting the streams over more CUs
  // shortens it, but adds the combine launch and a prologue per split
  // (~3.5 us).  So: one split while a stream holds less than
  // kMinSplitStream bytes of value rows; else enough splits to give each
  // CU one workgroup (one resident workgroup per CU already streams close
  // to the HBM ceiling), none shorter than kMinSplitBytes, at most
  // kMaxEvenSplits (more partials cost the combine more than they save).
  long long s = 1;
  const long long stream_bytes = (long long)max_len * row_bytes;
  if (stream_bytes >= kMinSplitStream) {
    s = (n_cu + streams - 1) / streams;
    if (s > stream_bytes / kMinSplitBytes) s = stream_bytes / kMinSplitBytes;
    if (s > kMaxEvenSplits) s = kMaxEvenSplits;
  }
  // Lengths spread widely (mean below half the longest) over many streams:
  // the longest sequences set the tail, so cut them finer -- where they are
  // split at all (below kMinSplitStream the combine costs more than a split
  // saves).  Few streams already give each CU one workgroup.
  if (spread && s > 1 && !few_streams) s *= 2;
  if (s < 1) s = 1;
  if (s > GVA_MAX_SPLITS) s = GVA_MAX_SPLITS;
  return (int)s;
}

}  // extern "C"
