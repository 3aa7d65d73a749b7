// conv_fwd_tile.hip -- the forward GEMM (see conv_igemm.hip) on small and
// medium tiles, for both dtypes: 16-byte tap vectors of both operands go from
// buffer loads straight into LDS.
//
// Serves every forward / backward-data GEMM whose taps and filter rows are
// whole 16-byte vectors and that the 256-row bf16 kernel does not take: fp32,
// small batches, few filters.  What bounds these is less the matrix cores
// than the number of workgroups, the width of their loads and the wait for
// their operands, so the tile and the number of tap splits are chosen
// together (fwd_tile_plan), an operand row of a K-tile is a whole cache line,
// and two to five K-tiles are in LDS, one barrier per K-tile.  Against the
// 128 x 128 register-staged kernel for all of them (bf16 16900 x 384 x 3456:
// 69 -> 50 us, 907 TFLOP/s; 5408 x 384 x 2304: 36 -> 22; 46656 x 96 x 6400:
// 106 -> 72; fp32 25600 x 32 x 800: 69 -> 24; 5408 x 384 x 2304: 131 -> 96):
// 1.31x over 65 GEMMs.
#include "conv_common.h"

namespace singa {

namespace {

// Tile shapes: BM x BN outputs, NW waves in a WR x (NW / WR) grid, NS stages
// of K-tiles in LDS.  Rows are 128 bytes of a K-tile everywhere: with 64-byte
// rows (a deeper pipeline in the same LDS) every load fetches half a cache
// line and the same GEMMs ran 25-40 % slower (128 x 128, bf16, 16900 x 384 x
// 3456: 71 us with 64-byte rows in five stages, 52 with 128-byte rows in two).
template <int ID> struct TileDef;
template <> struct TileDef<0> { static constexpr int BM = 256, BN = 128, WR = 4, NS = 3, NW = 8; };
template <> struct TileDef<1> { static constexpr int BM = 192, BN = 128, WR = 2, NS = 3, NW = 8; };
template <> struct TileDef<2> { static constexpr int BM = 256, BN = 64, WR = 4, NS = 2, NW = 4; };
template <> struct TileDef<3> { static constexpr int BM = 128, BN = 128, WR = 2, NS = 2, NW = 4; };
template <> struct TileDef<4> { static constexpr int BM = 64, BN = 128, WR = 2, NS = 3, NW = 4; };
template <> struct TileDef<5> { static constexpr int BM = 128, BN = 64, WR = 2, NS = 3, NW = 4; };
template <> struct TileDef<6> { static constexpr int BM = 64, BN = 64, WR = 2, NS = 5, NW = 4; };
template <> struct TileDef<7> { static constexpr int BM = 128, BN = 32, WR = 4, NS = 4, NW = 4; };
template <> struct TileDef<8> { static constexpr int BM = 32, BN = 128, WR = 1, NS = 4, NW = 4; };
constexpr int TILES = 9;
constexpr int RB = 128;  // bytes of one operand row per K-tile
constexpr int kTileRows[TILES] = {256, 192, 256, 128, 64, 128, 64, 128, 32};
constexpr int kTileCols[TILES] = {128, 128, 64, 128, 128, 64, 64, 32, 128};
constexpr int kTileWaves[TILES] = {8, 8, 4, 4, 4, 4, 4, 4, 4};

// workgroups that share a CU's 160 KB of LDS
template <int ID>
constexpr int kWorkgroupsPerCu = TileDef<ID>::NS * (TileDef<ID>::BM + TileDef<ID>::BN) * RB * 2 <= 163840 ? 2 : 1;

// SEG: the workgroup runs several pieces of the tap range (kt_per_piece K-tiles
// each) and adds their sums in order, as the reduction of a split GEMM does.
template <typename T, int ID, bool SEG>
__global__ __launch_bounds__(64 * TileDef<ID>::NW, kWorkgroupsPerCu<ID>) void conv_fwd_tile_kernel(FwdArgs a) {
  typedef TileDef<ID> D;
  typedef typename Frag<T>::type FragT;
  constexpr uint32_t ES = sizeof(T);
  constexpr int VEC = 16 / (int)ES;
  constexpr int BMT = D::BM, BNT = D::BN, NS = D::NS;
  constexpr int LBK = RB / (int)ES;          // taps per K-tile
  constexpr int SL = RB / 16;                // 16-byte slots per row
  constexpr int RPI = 64 / SL;               // rows per load instruction
  constexpr int RPW = 256 / RB;              // rows per 256-byte bank window
  constexpr int NPAR = 2;                    // swizzles that a lane's rows of even and odd instructions see
  constexpr int NW = D::NW, WR = D::WR, WC = NW / WR;
  constexpr int FM = BMT / (32 * WR), FN = BNT / (32 * WC);
  constexpr int ABAND = BMT / NW, BBAND = BNT / NW;      // operand rows each wave loads
  constexpr int AI = ABAND / RPI, BI = BBAND / RPI;    // its load instructions per K-tile
  constexpr int ATILE = BMT * RB, STAGE = ATILE + BNT * RB, LOADS = AI + BI;
  constexpr int KS = RB / 32;                          // k-steps: a 32-byte chunk pair of every row
  static_assert(AI * RPI == ABAND && BI * RPI == BBAND && AI > 0 && BI > 0, "load bands");
  static_assert(FM * WR * 32 == BMT && FN * WC * 32 == BNT, "wave grid");
  static_assert((NS - 2) * LOADS < 64, "vmcnt range");
  constexpr int QPIT = 32 * FN * (int)ES + 16;         // row pitch of the epilogue's staging
  static_assert(NW * 32 * QPIT <= NS * STAGE, "staging fits the operand stages");
  __shared__ __attribute__((aligned(16))) char smem[NS * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int split = L / a.tiles, tile = L - split * a.tiles;
  const int tm = tile / a.tiles_n, tn = tile - tm * a.tiles_n;
  const int m0 = tm * BMT, n0 = tn * BNT;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);

  // Loader: instruction i of this wave fills rows RPI i .. RPI i + RPI - 1 of
  // its A / B band; this lane owns row RPI i + lane / SL, slot lane % SL,
  // which holds the row's tap chunk (lane % SL) ^ ((row / RPW) % SL), so that
  // a fragment read of 16 consecutive rows hits 16 distinct bank groups.
  const int lrow = lane / SL;
  int ca[NPAR], cb[NPAR];
#pragma unroll
  for (int p = 0; p < NPAR; ++p) {
    ca[p] = VEC * ((lane % SL) ^ (((ABAND * wave + RPI * p + lrow) / RPW) % SL));
    cb[p] = VEC * ((lane % SL) ^ (((BBAND * wave + RPI * p + lrow) / RPW) % SL));
  }
  int apix[AI], ah0[AI], aw0[AI];  // element offset of input pixel (n, h0, w0); window origin
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int m = m0 + ABAND * wave + RPI * i + lrow;
    if (m < a.M) {
      const int n = (int)fdiv((uint32_t)m, a.dPQ);
      const int pq = m - n * a.P * a.Q;
      const int p = (int)fdiv((uint32_t)pq, a.dQ);
      const int q = pq - p * a.Q;
      ah0[i] = p * a.sh - a.ph;
      aw0[i] = q * a.sw - a.pw;
      apix[i] = ((n * a.H + ah0[i]) * a.W + aw0[i]) * a.C;
    } else {
      ah0[i] = -(1 << 28);  // fails every bounds check
      aw0[i] = 0;
      apix[i] = 0;
    }
  }
  int brow[BI];  // element offset of the filter row, or -1
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    const int n = n0 + BBAND * wave + RPI * i + lrow;
    brow[i] = n < a.Nn ? n * a.Kg : -1;
  }

  const int nkt_all = (a.Kg + LBK - 1) / LBK;
  const int kt0 = split * a.kt_per_split;
  const int nkt = min(a.kt_per_split, nkt_all - kt0);  // K-tiles of this workgroup (>= 1)

  // The taps of K-tile kt: where the lane's chunks start in the filter row
  // and in the input window.  With whole K-tiles per tap (a.uni) tap and
  // channel slice are the same for every lane.
  struct Taps {
    int r[NPAR], s[NPAR], tap[NPAR];
    bool kin[NPAR];
    int kb;  // filter offset of the K-tile
  };
  auto taps = [&](int kt) {
    Taps t;
    const bool live = kt < nkt;
    const int k = kt0 + kt;
    if (a.uni) {
      const int hi = (int)fdiv((uint32_t)k, a.dU), lo = k - hi * (int)a.dU.d;
      const int rs = a.uni == 1 ? lo : hi, cs = a.uni == 1 ? hi : lo;
      const int r = (int)fdiv((uint32_t)rs, a.dS), s = rs - r * a.S;
      t.kb = rs * a.C + cs * LBK;
      const int base = (r * a.W + s) * a.C + cs * LBK;
#pragma unroll
      for (int p = 0; p < NPAR; ++p) {
        t.r[p] = r;
        t.s[p] = s;
        t.tap[p] = base + ca[p];
        t.kin[p] = live;
      }
    } else {
      t.kb = live ? k * LBK : a.Kg;
#pragma unroll
      for (int p = 0; p < NPAR; ++p) {
        const int kk = t.kb + ca[p];
        t.kin[p] = kk < a.Kg;
        const int rs = (int)fdiv((uint32_t)kk, a.dC);
        const int c = kk - rs * a.C;
        t.r[p] = (int)fdiv((uint32_t)rs, a.dS);
        t.s[p] = rs - t.r[p] * a.S;
        t.tap[p] = (t.r[p] * a.W + t.s[p]) * a.C + c;
      }
    }
    return t;
  };
  // slice j of KS of the loads of K-tile kt, whose taps are t (past the
  // split's end: all out of range, no traffic)
  auto issue = [&](const Taps& t, bool live, char* St, int j) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      if (i * KS / LOADS != j) continue;
      if (i < AI) {
        const int p = i & 1;
        const int h = ah0[i] + t.r[p], w = aw0[i] + t.s[p];
        const bool ok = t.kin[p] & ((unsigned)h < (unsigned)a.H) & ((unsigned)w < (unsigned)a.W);
        ld_lds16(xr, ok ? (uint32_t)(apix[i] + t.tap[p]) * ES : OOB, St + (ABAND * wave + RPI * i) * RB);
      } else {
        const int b = i - AI;
        const int kk = t.kb + cb[b & 1];
        const bool ok = live & (brow[b] >= 0) & (kk < a.Kg);
        ld_lds16(wr, ok ? (uint32_t)(brow[b] + kk) * ES : OOB, St + ATILE + (BBAND * wave + RPI * b) * RB);
      }
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

  const int wm = wave / WC, wn = wave % WC;
  const int li = lane & 31, lh = lane >> 5;
  // chunk 2 kc + lh of row r sits in slot (2 kc + lh) ^ ((r / RPW) % SL); every block starts at a multiple of 32 rows
  const int tsw = (lh ^ ((li / RPW) % SL)) << 4;
  const int aoff = (wm * FM * 32 + li) * RB, boff = ATILE + (wn * FN * 32 + li) * RB;

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
#pragma unroll
    for (int j = 0; j < KS; ++j) issue(taps(s), s < nkt, smem + s * STAGE, j);
  int stage = 0;
  for (int kt = 0; kt < nkt; ++kt) {
    wait_vmcnt<(NS - 2) * LOADS>();  // this thread's loads of tile kt have landed (later tiles' may be in flight)
    block_barrier();                 // ... and everyone's; everyone is also done with tile kt-1
    const char* S = smem + stage * STAGE;
    char* const Ns = smem + (stage == 0 ? NS - 1 : stage - 1) * STAGE;
    const Taps t = taps(kt + NS - 1);
#pragma unroll
    for (int kc = 0; kc < KS; ++kc) {
      FragT fa[FM], fb[FN];
#pragma unroll
      for (int b = 0; b < FM; ++b) fa[b] = *(const FragT*)(S + aoff + b * 32 * RB + ((32 * kc) ^ tsw));
#pragma unroll
      for (int b = 0; b < FN; ++b) fb[b] = *(const FragT*)(S + boff + b * 32 * RB + ((32 * kc) ^ tsw));
#pragma unroll
      for (int bm = 0; bm < FM; ++bm)
#pragma unroll
        for (int bn = 0; bn < FN; ++bn) {
          if constexpr (ES == 2) {
            acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[bm], fb[bn], acc[bm][bn], 0, 0, 0);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[bm][j], fb[bn][j], acc[bm][bn], 0, 0, 0);
          }
        }
      issue(t, kt + NS - 1 < nkt, Ns, kc);
    }
    stage = stage == NS - 1 ? 0 : stage + 1;
    if (SEG && (--left == 0 || kt + 1 == nkt)) {
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
  if (a.partial) {
    float* __restrict__ out = a.partial + (size_t)split * a.M * a.Nn;
#pragma unroll
    for (int bn = 0; bn < FN; ++bn) {
      const int col = col0 + bn * 32 + li;
      if (col >= a.Nn) continue;
#pragma unroll
      for (int bm = 0; bm < FM; ++bm)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = row0 + bm * 32 + (v >> 2) * 8 + lh * 4 + (v & 3);
          if (row < a.M) out[(size_t)row * a.Nn + col] = acc[bm][bn][v];
        }
    }
    return;
  }
  __syncthreads();  // every wave is done with the operand tiles
  const bool vec = a.Nn % VEC == 0 && (((uintptr_t)a.y | (uintptr_t)a.mask) % 16) == 0;
  if constexpr (NW * 32 * FM * QPIT <= NS * STAGE) {
    store_quadrant<T, FM, FN>(acc, smem + wave * 32 * FM * QPIT, lane, row0, col0, a.M, a.Nn, a.bias, a.relu, a.mask,
                              (T*)a.y, vec);
  } else {  // fp32 values of a whole quadrant exceed the stages: 32 rows at a time
    static_assert(FM <= 3, "staging passes");
    char* q = smem + wave * 32 * QPIT;
    store_quadrant<T, FM, FN, 0, 1>(acc, q, lane, row0, col0, a.M, a.Nn, a.bias, a.relu, a.mask, (T*)a.y, vec);
    store_quadrant<T, FM, FN, 1, 1>(acc, q, lane, row0 + 32, col0, a.M, a.Nn, a.bias, a.relu, a.mask, (T*)a.y, vec);
    if constexpr (FM > 2)
      store_quadrant<T, FM, FN, 2, 1>(acc, q, lane, row0 + 64, col0, a.M, a.Nn, a.bias, a.relu, a.mask, (T*)a.y, vec);
  }
}

// "conv_fwd_kernel<dtype,tile rows x tile columns,bwd>"; the profiler's
// conv_fwd_tile_kernel<dtype, tile, several pieces>, tile as in kTileRows
#define TILE_NAME(T, M, N, B) "conv_fwd_kernel<" T "," #M "x" #N "," #B ">"
#define TILE_NAMES(T, B) {TILE_NAME(T, 256, 128, B), TILE_NAME(T, 192, 128, B), TILE_NAME(T, 256, 64, B), TILE_NAME(T, 128, 128, B), TILE_NAME(T, 64, 128, B), TILE_NAME(T, 128, 64, B), TILE_NAME(T, 64, 64, B), TILE_NAME(T, 128, 32, B), TILE_NAME(T, 32, 128, B)}
constexpr const char* kTileNames[2][2][TILES] = {{TILE_NAMES("f32", 0), TILE_NAMES("f32", 1)},
                                                 {TILE_NAMES("bf16", 0), TILE_NAMES("bf16", 1)}};
#undef TILE_NAMES
#undef TILE_NAME

template <typename T, int ID> void launch_tile(const FwdArgs& a, const FwdTilePlan& p, hipStream_t st) {
  const dim3 grid(a.tiles * p.splits), block(64 * TileDef<ID>::NW);
  if (a.kt_per_piece < a.kt_per_split) hipLaunchKernelGGL((conv_fwd_tile_kernel<T, ID, true>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((conv_fwd_tile_kernel<T, ID, false>), grid, block, 0, st, a);
}

template <typename T> void launch_tile_id(const FwdArgs& a, const FwdTilePlan& p, hipStream_t st) {
  switch (p.tile) {
    case 0: launch_tile<T, 0>(a, p, st); break;
    case 1: launch_tile<T, 1>(a, p, st); break;
    case 2: launch_tile<T, 2>(a, p, st); break;
    case 3: launch_tile<T, 3>(a, p, st); break;
    case 4: launch_tile<T, 4>(a, p, st); break;
    case 5: launch_tile<T, 5>(a, p, st); break;
    case 6: launch_tile<T, 6>(a, p, st); break;
    case 7: launch_tile<T, 7>(a, p, st); break;
    default: launch_tile<T, 8>(a, p, st); break;
  }
}

// A dense layer on one to three rows (prediction of single images): each
// weight is used once or a few times, so the matrix cores have nothing to do
// and the weights' bytes and one launch are all there is.  A workgroup takes
// GEMV_COLS output columns and its four waves a quarter of the taps each (the
// 16-byte chunks q, q + 256, q + 512, ... of a row), so that even a few
// hundred columns make enough loads; a lane adds its products in fp32, the
// wave's lanes are added by a butterfly and the waves in order.  Against the
// tile kernel with split taps and its reduction: one row, 4096 x 4096 bf16
// 11.9 -> 7.4 us (4.5 TB/s).  At four rows the bf16 tiles are as fast on long
// reductions (4096 x 4096: 9.4 us, here 9.3) and far ahead on short ones (512
// taps, 9216 columns: 6.7 against 16.3); in fp32 long ones would still gain
// (4096 x 4096: 20.2 against 15.1).
constexpr int GEMV_COLS = 4, GEMV_ROWS = 3;

template <typename T> __device__ __forceinline__ void unpack_vec(const uint4& u, float* f);
template <> __device__ __forceinline__ void unpack_vec<bf16_t>(const uint4& u, float* f) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
template <> __device__ __forceinline__ void unpack_vec<float>(const uint4& u, float* f) {
  f[0] = __uint_as_float(u.x); f[1] = __uint_as_float(u.y); f[2] = __uint_as_float(u.z); f[3] = __uint_as_float(u.w);
}

template <typename T, int M>
__global__ __launch_bounds__(NT) void conv_fwd_gemv_kernel(FwdArgs a) {
  constexpr int VEC = 16 / (int)sizeof(T);
  constexpr uint32_t ES = sizeof(T);
  __shared__ float part[4][GEMV_COLS][M];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = blockIdx.x * GEMV_COLS;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);
  const int chunks = a.Kg / VEC;
  float acc[GEMV_COLS][M];
#pragma unroll
  for (int c = 0; c < GEMV_COLS; ++c)
#pragma unroll
    for (int m = 0; m < M; ++m) acc[c][m] = 0.f;
  constexpr int U = 2;  // chunks of every row in flight
  for (int q0 = tid; q0 < chunks; q0 += U * NT) {
    uint4 wv[U][GEMV_COLS], xv[U][M];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u * NT;
#pragma unroll
      for (int c = 0; c < GEMV_COLS; ++c)
        wv[u][c] = ld16(wr, (q < chunks && n0 + c < a.Nn) ? (uint32_t)((n0 + c) * a.Kg + q * VEC) * ES : OOB);
#pragma unroll
      for (int m = 0; m < M; ++m) xv[u][m] = ld16(xr, q < chunks ? (uint32_t)(m * a.Kg + q * VEC) * ES : OOB);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float xf[M][VEC];
#pragma unroll
      for (int m = 0; m < M; ++m) unpack_vec<T>(xv[u][m], xf[m]);
#pragma unroll
      for (int c = 0; c < GEMV_COLS; ++c) {
        float wf[VEC];
        unpack_vec<T>(wv[u][c], wf);
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[c][m] = fmaf(wf[e], xf[m][e], acc[c][m]);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < GEMV_COLS; ++c)
#pragma unroll
    for (int m = 0; m < M; ++m) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) acc[c][m] += __shfl_xor(acc[c][m], o, 64);
      if (lane == 0) part[wave][c][m] = acc[c][m];
    }
  __syncthreads();
  const int c = tid % GEMV_COLS, m = tid / GEMV_COLS, col = n0 + c;
  if (m < M && col < a.Nn) {
    float v = part[0][c][m] + part[1][c][m] + part[2][c][m] + part[3][c][m];
    if (a.bias) v += a.bias[col];
    if (a.relu) v = fmaxf(v, 0.f);
    const size_t o = (size_t)m * a.Nn + col;
    if (a.mask && !mask_pass<T>(a.mask, o)) v = 0.f;
    store_out<T>((T*)a.y + o, v);
  }
}

template <typename T> void launch_gemv(const FwdArgs& a, hipStream_t st) {
  const dim3 grid((a.Nn + GEMV_COLS - 1) / GEMV_COLS), block(NT);
  if (a.M == 1) hipLaunchKernelGGL((conv_fwd_gemv_kernel<T, 1>), grid, block, 0, st, a);
  else if (a.M == 2) hipLaunchKernelGGL((conv_fwd_gemv_kernel<T, 2>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((conv_fwd_gemv_kernel<T, 3>), grid, block, 0, st, a);
}

}  // namespace

// Tile and splits by a model of the launch's time, in microseconds.  A CU runs
// its workgroups one after another or, where two fit its LDS, in pairs; a
// workgroup takes a fixed time for its first loads and its epilogue and then
// one step per K-tile that grows with the tile's area (the matrix work) and
// its edge (the operand bytes); a split adds the reduction's launch and its
// partial sums' bytes.  The constants are least-squares fits to some 1,400
// timed launches of every tile and split count over 65 GEMMs (rows 5 -
// 186,624, columns 12 - 4,096, taps 4 - 9,216); over these the choice is on
// average 2 % slower than the best one timed, 14 % at worst.
// A bf16 GEMM's sum is taken in `segs` pieces whatever the tile, so that its
// results do not depend on the choice; its workgroups run all of them or one
// each.  An fp32 GEMM takes the split count that the model likes best; where
// that makes a workgroup's share of the taps longer than a piece, the
// workgroup sums it piece by piece (F32_PIECE).
FwdTilePlan fwd_tile_plan(long M, long Nn, long Kg, int dt, int segs, long max_splits) {
  const int lbk = RB / (int)dt_size(dt);
  const int nkt = (int)((Kg + lbk - 1) / lbk);
  if (dt != BF16) segs = std::max(segs, (nkt + F32_PIECE - 1) / F32_PIECE);
  if (const char* e = tuning_env("SINGA_FWD_TILE")) {
    int t = 0, s = 1;
    if (sscanf(e, "%d,%d", &t, &s) == 2) return FwdTilePlan{t, segs, dt == BF16 && s > 1 ? segs : s};
  }
  struct Model {
    float one0, one_area, one_edge;  // K-tile step of a workgroup alone on its CU
    float two0, two_area, two_edge;  // ... of a pair
    float big0, big_area;            // ... of eight waves
    float wg, wg_area, pair_area;    // per workgroup: its start, its outputs; more for the second of a pair
    float red0, red_mb, red_split;   // the reduction: per launch, per million partial sums, per split
  };
  static constexpr Model kModel[2] = {
      {0.174f, 1.14e-4f, 7.26e-4f, 0.334f, 2.01e-4f, 5.23e-4f, 0.307f, 1.07e-4f, 1.15f, 1.01e-4f, 1.53e-4f, 2.07f, 1.6f,
       0.04f},
      {0.128f, 1.96e-5f, 1.03e-3f, 0.152f, 1.73e-5f, 1.75e-3f, 0.374f, 1.24e-5f, 1.41f, 8.45e-5f, 9.12e-5f, 1.27f,
       1.13f, 0.173f}};
  const Model& m = kModel[dt == BF16];
  // split counts to try, each split with at least three K-tiles
  static constexpr int kSplits[8] = {1, 2, 3, 4, 6, 8, 12, 16};
  int per[8], splits[8], ns = 0;
  if (dt == BF16) {
    for (int want : {1, segs}) {
      if (want == 1 && ns) break;
      per[ns] = (nkt + want - 1) / want;
      splits[ns++] = want;
    }
  } else {
    for (int want : kSplits) {
      if (want > 1 && nkt < 3 * want) break;
      per[ns] = (nkt + want - 1) / want;
      splits[ns] = (nkt + per[ns] - 1) / per[ns];  // every split has a K-tile
      if (want > 1 && splits[ns] > max_splits) break;
      ++ns;
    }
  }
  const float mb = 1e-6f * (float)M * (float)Nn;
  FwdTilePlan best{0, 1, 1};
  float best_us = 1e30f;
  for (int t = 0; t < TILES; ++t) {
    // a tile of eight waves has its CU to itself: over fewer than eight K-tiles
    // its first loads and its epilogue stand uncovered (188,944 x 96 x 144:
    // 24.4 us, 20.9 with two workgroups of 128 x 128 on a CU)
    if (kTileWaves[t] == 8 && nkt < 8) continue;
    const int bm = kTileRows[t], bn = kTileCols[t];
    const int tiles = (int)((M + bm - 1) / bm) * (int)((Nn + bn - 1) / bn);
    const float area = (float)(bm * bn), edge = (float)(bm + bn);
    const float one = m.one0 + m.one_area * area + m.one_edge * edge;
    const float two = m.two0 + m.two_area * area + m.two_edge * edge, big = m.big0 + m.big_area * area;
    const float wg = m.wg + m.wg_area * area;
    for (int i = 0; i < ns; ++i) {
      const int load = (int)(((long)tiles * splits[i] + 255) >> 8);  // workgroups per CU
      float us = kTileWaves[t] == 8
                     ? load * (wg + per[i] * big)
                     : (load / 2) * (wg + m.pair_area * area + per[i] * two) + (load % 2) * (wg + per[i] * one);
      if (splits[i] > 1) us += m.red0 + (m.red_split + m.red_mb * mb) * splits[i];
      if (us < best_us) {
        best_us = us;
        best = FwdTilePlan{t, segs, splits[i]};
      }
    }
  }
  return best;
}

hipError_t launch_conv_fwd_tile(int dt, FwdArgs a, const FwdTilePlan& p, int bwd, double flops, hipStream_t st) {
  const int lbk = RB / (int)dt_size(dt);
  a.tiles_n = (a.Nn + kTileCols[p.tile] - 1) / kTileCols[p.tile];
  a.tiles = (a.M + kTileRows[p.tile] - 1) / kTileRows[p.tile] * a.tiles_n;
  const int nkt = (a.Kg + lbk - 1) / lbk;
  a.kt_per_split = (nkt + p.splits - 1) / p.splits;
  a.kt_per_piece = (nkt + p.segs - 1) / p.segs;
  // bf16: the taps in the filter row's order; fp32: taps fastest, so that
  // consecutive K-tiles read the same channels one tap apart and their
  // overlapping input rows meet in the caches
  a.uni = a.C % lbk != 0 ? 0 : dt == BF16 ? 2 : 1;
  a.dU = make_fastdiv((uint32_t)(a.uni == 2 ? a.C / lbk : a.RS));
  if (p.splits == 1) a.partial = nullptr;
  TraceScope ts(kTileNames[dt == BF16][bwd != 0][p.tile], st, flops, WORK_FLOP);
  if (dt == BF16) launch_tile_id<bf16_t>(a, p, st);
  else launch_tile_id<float>(a, p, st);
  return hipGetLastError();
}

// Short reductions leave most of a workgroup's lanes idle, and thousands of
// workgroups then cost more than the tiles' single round: a column takes this
// many bytes at least, by rows and columns.  In bf16 the line is where the
// tile kernel, timed beside this one on 8 - 9216 taps by 12 - 9216 columns,
// stops being faster (three rows, 4096 columns: 256 taps 5.0 us on tiles, 6.1
// here; 512 taps 6.6 and 6.1.  9216 columns: 16 taps 4.1 and 10.3, 4096 taps
// 19.6 and 15.4).  fp32 stays here longer, since this kernel's many short sums
// are nearer to 64 bits than a tile's one (64 taps 6.7e-8 and 1.5e-7): up to
// where the 128 x 128 kernel that had these layers first was faster (three
// rows, 9216 columns: 64 taps 8.3 us, 11.0 here and 5.3 on tiles; 128 taps
// 12.7 and 10.9).
bool fwd_gemv_ok(const ConvShape& s, int dt) {
  if (s.N > GEMV_ROWS || s.P != 1 || s.Q != 1 || s.ph != 0 || s.pw != 0 || s.R != s.H || s.S != s.W) return false;
  static constexpr int kLeast[2][GEMV_ROWS][4] = {{{0, 0, 0, 0}, {0, 0, 0, 256}, {0, 0, 0, 512}},
                                                  {{0, 0, 0, 1024}, {0, 256, 512, 4096}, {192, 512, 1024, 4096}}};
  const int cols = s.K <= 32 ? 0 : s.K <= 1024 ? 1 : s.K <= 4096 ? 2 : 3;
  return (long)s.R * s.S * s.C * (long)dt_size(dt) >= kLeast[dt == BF16][s.N - 1][cols];
}

hipError_t launch_conv_fwd_gemv(int dt, const FwdArgs& a, int bwd, double flops, hipStream_t st) {
  static const char* names[2][2] = {{"conv_fwd_kernel<f32,gemv,0>", "conv_fwd_kernel<f32,gemv,1>"},
                                    {"conv_fwd_kernel<bf16,gemv,0>", "conv_fwd_kernel<bf16,gemv,1>"}};
  TraceScope ts(names[dt == BF16][bwd != 0], st, flops, WORK_FLOP);
  if (dt == BF16) launch_gemv<bf16_t>(a, st);
  else launch_gemv<float>(a, st);
  return hipGetLastError();
}

}  // namespace singa
