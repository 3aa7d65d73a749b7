// conv_wgrad_tile.hip -- the fp32 filter gradient (see conv_igemm.hip) on
// tiles of 32, 64 or 128 filters x 128 taps, both operands straight from
// buffer loads into LDS.
//
// Serves fp32 layers whose filter and tap chunks are whole 16-byte vectors
// (K % 4 == 0, C % 4 == 0).  v_mfma_f32_32x32x2_f32 takes 64 cycles for 2,048
// multiply-adds, so a full tile is bound by the matrix cores and rows of
// padding cost in proportion: a layer of 32 filters on the 128-row tile spends
// three quarters of its time on zeros.  Small layers are bound by the few
// workgroups they make, so tile and splits of the reduction are chosen
// together by a model of the launch's time (wgrad_tile_plan).
#include "conv_common.h"

namespace singa {

namespace {

// BM filters x 128 taps, 4 waves in a WR x (4 / WR) grid, NS stages of 32
// reduction rows in LDS (two workgroups per CU).
template <int ID> struct WTile;
template <> struct WTile<0> { static constexpr int BM = 128, WR = 2, NS = 2; };
template <> struct WTile<1> { static constexpr int BM = 64, WR = 2, NS = 3; };
template <> struct WTile<2> { static constexpr int BM = 32, WR = 1, NS = 4; };
constexpr int WTILES = 3;
constexpr int kWRows[WTILES] = {128, 64, 32};
constexpr int WBN = 128, WBK = 32;

// NFAST: N % 32 == 0 and few output pixels: a K-tile holds 32 images at one
// output pixel; otherwise the reduction runs image by image.
// SEG: the workgroup sums pieces of kt_per_piece K-tiles and adds their sums
// in order, so that a few long splits lose no precision against many short
// ones.
template <int ID, bool NFAST, bool SEG>
__global__ __launch_bounds__(NT, 2) void conv_wgrad_tile_kernel(WgradArgs a) {
  typedef WTile<ID> D;
  constexpr int BMT = D::BM, NS = D::NS, WR = D::WR, WC = 4 / WR;
  constexpr int FM = BMT / (32 * WR), FN = WBN / (32 * WC);
  constexpr int ARB = BMT * 4, BRB = WBN * 4;                  // row bytes
  constexpr int ASL = ARB / 16, BSL = BRB / 16;                // 16-byte slots per row
  constexpr int ARI = 64 / ASL, BRI = 64 / BSL;                // rows per load instruction
  constexpr int AI = WBK / 4 / ARI, BI = WBK / 4 / BRI;        // load instructions per wave per K-tile
  constexpr int ATILE = WBK * ARB, STAGE = ATILE + WBK * BRB, LOADS = AI + BI;
  static_assert(AI * ARI * 4 == WBK && BI * BRI * 4 == WBK && AI > 0, "load split");
  static_assert(2 * NS * STAGE <= 163840, "two workgroups per CU");
  __shared__ __attribute__((aligned(16))) char smem[NS * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int split = L / a.tiles, tile = L - split * a.tiles;
  const int tm = tile / a.tiles_n, tn = tile - tm * a.tiles_n;
  const int m0 = tm * BMT, n0 = tn * WBN;
  const int kt_begin = split * a.kt_per_split;
  const int nk = min(a.nkt, kt_begin + a.kt_per_split) - kt_begin;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t dyr = make_rsrc(a.dy, a.dy_bytes);
  const int PQ = a.P * a.Q;
  const int ystride = PQ * a.M, xstride = a.H * a.W * a.C;

  // Chunk c of row r sits in slot c ^ (8 (r & 1)) (rows of 256 bytes or more;
  // 128-byte rows need none), so that a fragment read, 32 values of each of
  // two neighbouring rows, covers every bank once.  A lane's rows are of one
  // parity: every load instruction starts at an even row.
  const int arow = lane / ASL, brow = lane / BSL;
  const int i0 = m0 + 4 * ((lane % ASL) ^ (ASL > 8 ? 8 * (arow & 1) : 0));
  const int j0 = n0 + 4 * ((lane % BSL) ^ (8 * (brow & 1)));
  const bool aok = i0 < a.M, bok = j0 < a.Nn;
  const int jj = bok ? j0 : 0;
  const int rs = (int)fdiv((uint32_t)jj, a.dC);
  const int br = (int)fdiv((uint32_t)rs, a.dS), bs = rs - br * a.S;
  const int btap = (br * a.W + bs) * a.C + jj - rs * a.C;

  // row d of the K-tile starting at t0 -> (n, output pixel) and validity
  auto row_pix = [&](int t0, int d, int& n, int& pq) {
    if constexpr (NFAST) {
      const int kt = t0 / WBK;
      const int g = (int)fdiv((uint32_t)kt, a.dPQ);
      pq = kt - g * PQ;
      n = g * WBK + d;
      return true;
    } else {
      const int t = t0 + d;
      n = (int)fdiv((uint32_t)t, a.dPQ);
      pq = t - n * PQ;
      return t < a.T;
    }
  };
  // the loads of the k-th K-tile of this split (past its end: all out of range, no traffic)
  auto issue = [&](int k, char* St) {
    const bool live = k < nk;
    const int t0 = (kt_begin + (live ? k : 0)) * WBK;
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      const int d = (AI * wave + i) * ARI + arow;
      int n, pq;
      const bool ok = row_pix(t0, d, n, pq) & live & aok;
      ld_lds16(dyr, ok ? (uint32_t)(n * ystride + pq * a.M + i0) * 4u : OOB, St + (AI * wave + i) * ARI * ARB);
    }
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      const int d = (BI * wave + i) * BRI + brow;
      int n, pq;
      const bool in = row_pix(t0, d, n, pq);
      const int p = (int)fdiv((uint32_t)pq, a.dQ);
      const int h0 = p * a.sh - a.ph, w0 = (pq - p * a.Q) * a.sw - a.pw;
      const bool ok = in & live & bok & ((unsigned)(h0 + br) < (unsigned)a.H) & ((unsigned)(w0 + bs) < (unsigned)a.W);
      ld_lds16(xr, ok ? (uint32_t)(n * xstride + (h0 * a.W + w0) * a.C + btap) * 4u : OOB,
               St + ATILE + (BI * wave + i) * BRI * BRB);
    }
  };

  f32x16 acc[FM][FN], sum[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = sum[i][j][v] = 0.f;
  int left = a.kt_per_piece;  // SEG: K-tiles of the current piece still to run

  // fragment of the 2-row step kc: lane -> column (lane & 31) of a 32-column
  // block, row 2 kc + lane / 32
  const int wm = wave / WC, wn = wave % WC;
  const int li = lane & 31, lh = lane >> 5;
  int aaddr[FM], baddr[FN];
#pragma unroll
  for (int b = 0; b < FM; ++b) aaddr[b] = lh * ARB + (((wm * FM + b) ^ (ASL > 8 ? lh : 0)) * 32 + li) * 4;
#pragma unroll
  for (int b = 0; b < FN; ++b) baddr[b] = ATILE + lh * BRB + (((wn * FN + b) ^ lh) * 32 + li) * 4;
  // the bias column (tap index Nn) is loaded as an out-of-range zero and set
  // to 1 here; rows past the reduction's end hold dy = 0
  uint32_t ones[FN];
  bool bias_wave = false;
#pragma unroll
  for (int b = 0; b < FN; ++b) {
    const int cb = n0 + (wn * FN + b) * 32;
    ones[b] = (a.Ng > a.Nn && cb + li == a.Nn) ? 0x3f800000u : 0u;
    bias_wave |= a.Ng > a.Nn && cb <= a.Nn && a.Nn < cb + 32;
  }

#pragma unroll
  for (int s = 0; s < NS - 1; ++s) issue(s, smem + s * STAGE);
  int stage = 0;
  for (int k = 0; k < nk; ++k) {
    wait_vmcnt<(NS - 2) * LOADS>();  // tile k has landed for this thread
    block_barrier();                 // ... and for everyone; everyone is done with tile k-1
    const char* S = smem + stage * STAGE;
    issue(k + NS - 1, smem + (stage == 0 ? NS - 1 : stage - 1) * STAGE);
#pragma unroll
    for (int kc = 0; kc < WBK / 2; ++kc) {
      float fa[FM], fb[FN];
#pragma unroll
      for (int b = 0; b < FM; ++b) fa[b] = *(const float*)(S + aaddr[b] + 2 * kc * ARB);
#pragma unroll
      for (int b = 0; b < FN; ++b) fb[b] = *(const float*)(S + baddr[b] + 2 * kc * BRB);
      if (bias_wave) {
#pragma unroll
        for (int b = 0; b < FN; ++b) fb[b] = __uint_as_float(__float_as_uint(fb[b]) | ones[b]);
      }
#pragma unroll
      for (int bm = 0; bm < FM; ++bm)
#pragma unroll
        for (int bn = 0; bn < FN; ++bn)
          acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[bm], fb[bn], acc[bm][bn], 0, 0, 0);
    }
    stage = stage == NS - 1 ? 0 : stage + 1;
    if (SEG && (--left == 0 || k + 1 == nk)) {
      left = a.kt_per_piece;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            sum[i][j][v] += acc[i][j][v];
            acc[i][j][v] = 0.f;
          }
    }
  }
  if constexpr (SEG) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = sum[i][j];
  }
  wait_vmcnt<0>();  // the trailing all-OOB loads still write LDS

  const int row0 = m0 + wm * FM * 32, col0 = n0 + wn * FN * 32;
#pragma unroll
  for (int bn = 0; bn < FN; ++bn) {
    const int col = col0 + bn * 32 + li;
    if (col >= a.Ng) continue;
    const bool is_db = a.direct && col == a.Nn;
    float* __restrict__ base = a.direct ? (is_db ? a.db : a.out + col) : a.out + (size_t)split * a.M * a.ldp + col;
    const size_t stride = a.direct ? (is_db ? 1 : (size_t)a.Nn) : (size_t)a.ldp;
    const int accum = a.direct ? (is_db ? a.acc_db : a.acc_dw) : 0;
#pragma unroll
    for (int bm = 0; bm < FM; ++bm)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = row0 + bm * 32 + (v >> 2) * 8 + lh * 4 + (v & 3);
        if (row < a.M) {
          float* o = base + (size_t)row * stride;
          *o = accum ? *o + acc[bm][bn][v] : acc[bm][bn][v];
        }
      }
  }
}

// "conv_wgrad_kernel<f32,tile rows x tile columns,image fastest>"; the profiler's
// conv_wgrad_tile_kernel<tile, image fastest, several pieces>, tile as in kWRows
constexpr const char* kWNames[WTILES][2] = {
    {"conv_wgrad_kernel<f32,128x128,0>", "conv_wgrad_kernel<f32,128x128,1>"},
    {"conv_wgrad_kernel<f32,64x128,0>", "conv_wgrad_kernel<f32,64x128,1>"},
    {"conv_wgrad_kernel<f32,32x128,0>", "conv_wgrad_kernel<f32,32x128,1>"}};

template <int ID> void launch_wtile(const WgradArgs& a, const WgradTilePlan& p, hipStream_t st) {
  const dim3 grid(a.tiles * p.splits);
  const bool seg = a.kt_per_piece < a.kt_per_split;
  if (p.nfast && seg) hipLaunchKernelGGL((conv_wgrad_tile_kernel<ID, true, true>), grid, dim3(NT), 0, st, a);
  else if (p.nfast) hipLaunchKernelGGL((conv_wgrad_tile_kernel<ID, true, false>), grid, dim3(NT), 0, st, a);
  else if (seg) hipLaunchKernelGGL((conv_wgrad_tile_kernel<ID, false, true>), grid, dim3(NT), 0, st, a);
  else hipLaunchKernelGGL((conv_wgrad_tile_kernel<ID, false, false>), grid, dim3(NT), 0, st, a);
}

}  // namespace

int wgrad_tile_rows(int tile) { return kWRows[tile]; }

// Tile and splits by a model of the launch's time, in microseconds, like the
// forward's: a K-tile step of a workgroup alone on its CU and of a pair, a
// fixed time per workgroup, and the reduction of the partial tiles.  The
// constants are a least-squares fit to some 600 timed launches over 24 layers
// (filters 12 - 4,096, taps 5 - 5,185, reductions of 10 - 137,904); over these
// the choice is on average 1 % slower than the best one timed, 8 % at worst.
WgradTilePlan wgrad_tile_plan(long M, long Ng, long T, long max_splits, int pieces) {
  const int nkt = (int)((T + WBK - 1) / WBK);
  pieces = std::max(pieces, (nkt + F32_PIECE - 1) / F32_PIECE);
  if (const char* e = tuning_env("SINGA_WGRAD_TILE")) {
    int t = 0, s = 1;
    if (sscanf(e, "%d,%d", &t, &s) == 2) {
      const int per = (nkt + s - 1) / s;
      return WgradTilePlan{t, (nkt + per - 1) / per, pieces, false};
    }
  }
  const float mb = 1e-6f * (float)M * (float)((Ng + 63) / 64 * 64);
  WgradTilePlan best{0, 1, pieces, false};
  float best_us = 1e30f;
  for (int want : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256}) {
    if (want > 1 && nkt < 2 * want) break;
    const int per = (nkt + want - 1) / want, splits = (nkt + per - 1) / per;  // every split has a K-tile
    if (splits > 1 && splits > max_splits) break;
    for (int t = 0; t < WTILES; ++t) {
      const int bm = kWRows[t];
      const float rows = (float)bm;
      const int load = (int)(((M + bm - 1) / bm * ((Ng + WBN - 1) / WBN) * splits + 255) >> 8);  // workgroups per CU
      const float wg = 0.427f + 0.0125f * rows;
      float us = (load / 2) * (wg + 0.0331f * rows + per * (0.778f + 0.0241f * rows)) +
                 (load % 2) * (wg + per * (0.611f + 0.0141f * rows));
      if (splits > 1) us += 4.37f + 0.00216f * splits + 0.735f * mb * splits;
      if (us < best_us) {
        best_us = us;
        best = WgradTilePlan{t, splits, pieces, false};
      }
    }
  }
  return best;
}

hipError_t launch_conv_wgrad_tile(WgradArgs a, const WgradTilePlan& p, double flops, hipStream_t st) {
  a.kt_per_piece = (a.nkt + p.pieces - 1) / p.pieces;
  TraceScope ts(kWNames[p.tile][p.nfast], st, flops, WORK_FLOP);
  switch (p.tile) {
    case 0: launch_wtile<0>(a, p, st); break;
    case 1: launch_wtile<1>(a, p, st); break;
    default: launch_wtile<2>(a, p, st); break;
  }
  return hipGetLastError();
}

}  // namespace singa
