// conv_common.h -- device code shared by the convolution GEMM kernels: buffer
// loads with out-of-range zeros, direct-to-LDS loads and their waits, the
// staged epilogue, and the arguments of the forward GEMM.
#pragma once

#include <cstdio>
#include <cstdlib>

#include "common.h"
#include "internal.h"

namespace singa {

namespace {

constexpr int NT = 256;

union V16 {
  uint4 u;
  float f[4];
  bf16_t h[8];
};

template <typename T> __device__ __forceinline__ void set_elem(V16& v, int j, T e);
template <> __device__ __forceinline__ void set_elem<float>(V16& v, int j, float e) { v.f[j] = e; }
template <> __device__ __forceinline__ void set_elem<bf16_t>(V16& v, int j, bf16_t e) { v.h[j] = e; }

template <typename T> __device__ __forceinline__ T one_elem();
template <> __device__ __forceinline__ float one_elem<float>() { return 1.f; }
template <> __device__ __forceinline__ bf16_t one_elem<bf16_t>() { return (bf16_t)0x3f80; }

template <typename T> __device__ __forceinline__ T zero_elem();
template <> __device__ __forceinline__ float zero_elem<float>() { return 0.f; }
template <> __device__ __forceinline__ bf16_t zero_elem<bf16_t>() { return (bf16_t)0; }

template <typename T> __device__ __forceinline__ void store_out(T* p, float v);
template <> __device__ __forceinline__ void store_out<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void store_out<bf16_t>(bf16_t* p, float v) { *p = f32_to_bf16(v); }

__device__ __forceinline__ float elem_f(float v) { return v; }
__device__ __forceinline__ float elem_f(bf16_t v) { return bf16_to_f32(v); }

// ReLU backward folded into an epilogue: keep v where the ReLU's output is > 0.
template <typename T> __device__ __forceinline__ bool mask_pass(const void* m, size_t i);
template <> __device__ __forceinline__ bool mask_pass<float>(const void* m, size_t i) {
  return ((const float*)m)[i] > 0.f;
}
template <> __device__ __forceinline__ bool mask_pass<bf16_t>(const void* m, size_t i) {
  return bf16_to_f32(((const bf16_t*)m)[i]) > 0.f;
}

// ------------------------------------------------------------ global loads
//
// Operands are read with raw buffer loads: a tap outside the input (padding,
// ragged tails) gets the offset OOB, past the end of every tensor, and the
// hardware returns zeros for it.  No branch, no select on the loaded data.
constexpr uint32_t OOB = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 ld16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ __forceinline__ uint2 ld8(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}
template <typename T> __device__ __forceinline__ T ld_elem(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <> __device__ __forceinline__ float ld_elem<float>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
template <> __device__ __forceinline__ bf16_t ld_elem<bf16_t>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return (bf16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0);
}

// Workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous
// run of tiles so neighbouring tiles (shared input rows, shared filters) meet
// in the same L2.
__device__ __forceinline__ int xcd_remap(int b, int G) {
  const int q = G >> 3, r = G & 7, x = b & 7, l = b >> 3;
  return x * q + min(x, r) + l;
}

// All-ones in the bits of each element of a 32-bit word that is > 0 (not
// NaN), zero elsewhere, from the bit patterns alone: with x = bits - 1 taken
// as a signed integer, an element is > 0 exactly when 0 <= x < bits(+inf).
// Integer arithmetic only, so a mask of many elements needs no condition
// registers.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

template <typename T> __device__ __forceinline__ uint32_t positive_bits(uint32_t w);
template <> __device__ __forceinline__ uint32_t positive_bits<bf16_t>(uint32_t w) {
  const int32_t xl = (int32_t)(w & 0xffffu) - 1, xh = (int32_t)(w >> 16) - 1;
  const uint32_t ml = (uint32_t)(((xl - 0x7f80) >> 31) & ~(xl >> 31)) & 0xffffu;
  const uint32_t mh = (uint32_t)(((xh - 0x7f80) >> 31) & ~(xh >> 31)) << 16;
  return ml | mh;
}
template <> __device__ __forceinline__ uint32_t positive_bits<float>(uint32_t w) {
  const uint32_t x = w - 1u;
  return (uint32_t)(((int32_t)(x - 0x7f800000u) >> 31) & ~((int32_t)x >> 31));
}

// ------------------------------------------------------------ epilogue
//
// y[row][col] = act(acc + bias[col]), optionally zeroed where mask <= 0, for
// row blocks B0 .. B0 + NB - 1 of one wave's (32 FM) x (32 FN) quadrant of
// the output tile (row0: the first row of block B0).  The accumulators hold
// one column per lane (rows 8 (v / 4) + 4 (lane / 32) + v % 4 of each 32 x 32
// block); they go through the wave's own LDS region as T so that the global
// stores (and the mask loads) are 16-byte vectors of consecutive columns.
// Needs (32 NB) * (32 FN * sizeof(T) + 16) bytes of LDS at `lds`; the caller
// has finished with the operand tiles there (barrier).  `vec`: y, mask and Nn
// allow 16-byte vectors; otherwise the staged values are stored one by one.
template <typename T, int FM, int FN, int B0 = 0, int NB = FM>
__device__ __forceinline__ void store_quadrant(const f32x16 (&acc)[FM][FN], char* lds, int lane, int row0, int col0,
                                               int M, int Nn, const float* bias, int relu, const void* mask,
                                               T* __restrict__ y, bool vec) {
  constexpr int ES = (int)sizeof(T);
  constexpr int COLS = FN * 32;
  constexpr int PIT = COLS * ES + 16;
  constexpr int VEC = 16 / ES;
  constexpr int CPR = COLS / VEC;    // 16-byte chunks per row
  constexpr int RPS = 64 / CPR;      // rows per pass of the wave (lanes past RPS * CPR idle)
  constexpr int PASSES = (NB * 32 + RPS - 1) / RPS;
  const int li = lane & 31, lh = lane >> 5;
  const int cc = lane % CPR, rr = lane / CPR;
  const int col = col0 + cc * VEC;
  const T* __restrict__ mk = (const T*)mask;
  // The mask vectors of every pass are requested before the values are
  // staged, so their latency overlaps the staging and each other (one load
  // waited for per pass would expose a memory latency per pass).
  uint4 mv[PASSES];
  if (vec && mk) {
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const int r = pass * RPS + rr;
      const int row = row0 + r;
      // every lane loads (element 0 stands in for rows and columns past the
      // end), so no load sits in a branch that the next must wait for
      const bool ok = rr < RPS && r < NB * 32 && row < M && col < Nn;
      mv[pass] = *(const uint4*)(mk + (ok ? (size_t)row * Nn + col : 0));
    }
  }
#pragma unroll
  for (int bn = 0; bn < FN; ++bn) {
    const int c = bn * 32 + li;
    const float bv = (bias && col0 + c < Nn) ? bias[col0 + c] : 0.f;
#pragma unroll
    for (int bm = B0; bm < B0 + NB; ++bm)
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        // rows r and r + 1 of column c
        float v0 = acc[bm][bn][v] + bv, v1 = acc[bm][bn][v + 1] + bv;
        if (relu) {
          v0 = fmaxf(v0, 0.f);
          v1 = fmaxf(v1, 0.f);
        }
        const int r = (bm - B0) * 32 + (v >> 2) * 8 + lh * 4 + (v & 3);
        if constexpr (sizeof(T) == 2) {
          // one conversion instruction rounds both (the per-element
          // software rounding costs about six VALU operations per value)
          const uint32_t p = f32x2_to_bf16x2(v0, v1);
          *(uint16_t*)(lds + r * PIT + c * ES) = (uint16_t)p;
          *(uint16_t*)(lds + (r + 1) * PIT + c * ES) = (uint16_t)(p >> 16);
        } else {
          store_out<T>((T*)(lds + r * PIT + c * ES), v0);
          store_out<T>((T*)(lds + (r + 1) * PIT + c * ES), v1);
        }
      }
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's LDS writes are done
  __builtin_amdgcn_wave_barrier();
  if (rr >= RPS) return;
  if (vec) {
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const int r = pass * RPS + rr;
      const int row = row0 + r;
      if (r >= NB * 32) break;
      uint4 val = *(const uint4*)(lds + r * PIT + cc * 16);
      if (row < M && col < Nn) {
        if (mk) {
          val.x &= positive_bits<T>(mv[pass].x);
          val.y &= positive_bits<T>(mv[pass].y);
          val.z &= positive_bits<T>(mv[pass].z);
          val.w &= positive_bits<T>(mv[pass].w);
        }
        // streamed past the caches' write allocation (measured 0.5-3 % faster
        // per layer, the consumers included)
        __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, val), (u32x4_t*)(y + (size_t)row * Nn + col));
      }
    }
  } else {
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const int r = pass * RPS + rr;
      const int row = row0 + r;
      if (r >= NB * 32) break;
      union { uint4 u; T e[VEC]; } val;
      val.u = *(const uint4*)(lds + r * PIT + cc * 16);
      if (row < M) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
          const int cj = col + j;
          if (cj < Nn) {
            const size_t o = (size_t)row * Nn + cj;
            T e = val.e[j];
            if (mk && !(elem_f(mk[o]) > 0.f)) e = T(0);
            y[o] = e;
          }
        }
      }
    }
  }
}

}  // namespace

// Arguments of the forward GEMM kernels (also backward-data on a flipped or
// transposed filter).
struct FwdArgs {
  const void* x;
  const void* w;
  const float* bias;
  void* y;
  uint32_t x_bytes, w_bytes;
  int M, Nn, Kg;
  int H, W, C, S, P, Q;
  int sh, sw, ph, pw;
  FastDiv dPQ, dQ, dC, dS;
  int relu;
  int tiles, tiles_n;
  float* partial;  // split-K: fp32 partial tiles [split][M][Nn] instead of y
  int kt_per_split;
  int kt_per_piece;  // the tile kernel: K-tiles summed in one go; the sums of pieces are added in order
  const void* mask;  // optional [M][Nn] tensor: an output is zeroed where mask <= 0
  // 256-row kernel: K-tile kt covers channels [cs BK, cs BK + BK) of tap
  // rs = kt mod RS, cs = kt div RS (taps fastest), instead of taps [kt BK,
  // kt BK + BK) in (r, s, c) order; needs C % BK == 0.
  int tap_major, RS;
  FastDiv dRS;
  // tile kernel: a K-tile of C % BK == 0 layers lies in one tap rs and one
  // channel slice cs; uni 1: taps fastest (k = cs RS + rs), 2: slices fastest
  // (k = rs (C / BK) + cs, the order of the filter row); dU divides by the
  // faster one's count.  0: a chunk's tap is computed lane by lane.
  int uni;
  FastDiv dU;
  // input patch (stride 1, tap-major): the padded input is Hp x Wp per image
  int patch, Hp, Wp;
  FastDiv dHp, dWp;
};

// Arguments of the filter-gradient kernels.  With a bias, the GEMM gets one more column, Ng = Nn + 1, whose operand is
// 1 for every reduction index: its results are db[k] = sum_t dy[t][k].
struct WgradArgs {
  const void* x;
  const void* dy;
  float* out;  // partial tiles [splits][M][Ng], or dw itself when direct
  float* db;   // direct: the bias gradient (column Nn); NULL without bias
  uint32_t x_bytes, dy_bytes;
  int M, Nn, Ng, T;  // M = K filters, Nn = R*S*C taps, Ng = Nn (+1 with bias), T = N*P*Q
  int ldp;           // row stride of the partial tiles: Ng rounded up to 64 (256-byte rows)
  int N, H, W, C, S, P, Q;
  int sh, sw, ph, pw;
  FastDiv dN, dPQ, dQ, dC, dS;
  int tiles, tiles_n, kt_per_split, nkt;
  int kt_per_piece;  // as in FwdArgs
  int direct, acc_dw, acc_db;
  int update;    // direct only: each element is applied to `u` (out / db: NULL, or where g is also stored)
  SgdTargets u;
};

// K-tiles (of 32 terms) that an fp32 tile kernel sums in one go.  A rounding
// error grows with the length of the running sum, so a split that is long
// because the chip is full anyway would cost precision against the many short
// ones of the 128 x 128 kernels; pieces of at most 256 terms do not, for 1 %
// of the time (32 x 13 x 13 x 256, 384 filters of 3 x 3, forward and backward:
// 291 -> 295 us; error against 64 bits 4.2e-7 -> 2.1e-7, with the 128 x 128
// kernels 2.5e-7 - 3.1e-7 by the inputs).
constexpr int F32_PIECE = 8;

// Tile and reduction splits of the fp32 tile kernel (conv_wgrad_tile.hip).
struct WgradTilePlan {
  int tile;    // index into the kernel's table of tiles
  int splits;  // > 1: partial tiles in WgradArgs::out
  int pieces;  // of the reduction, each summed in one go, the sums added in order (at least one to a split)
  bool nfast;  // a K-tile is 32 images at one output pixel
};
// max_splits: what the caller's workspace has room for.
WgradTilePlan wgrad_tile_plan(long M, long Ng, long T, long max_splits, int pieces);
int wgrad_tile_rows(int tile);
hipError_t launch_conv_wgrad_tile(WgradArgs a, const WgradTilePlan& p, double flops, hipStream_t st);

// Tile and tap splits of the direct-to-LDS tile kernel (conv_fwd_tile.hip)
// for a GEMM of M rows, Nn columns and Kg taps, whose operands are whole
// 16-byte vectors.
struct FwdTilePlan {
  int tile;    // index into the kernel's table of tiles
  int segs;    // pieces of the tap range, summed one by one and added in order
  int splits;  // workgroups over the taps (bf16: 1 or segs); > 1: fp32 partial tiles [split][M][Nn] in FwdArgs::partial
};
// segs: the pieces the tap range is summed in (fp32: at least); max_splits:
// what the workspace has room for (fp32; bf16 takes segs partial sums or none).
FwdTilePlan fwd_tile_plan(long M, long Nn, long Kg, int dt, int segs, long max_splits);
hipError_t launch_conv_fwd_tile(int dt, FwdArgs a, const FwdTilePlan& p, int bwd, double flops, hipStream_t st);
// A dense layer (P = Q = 1 and the window covers the whole input) of at most
// three rows and not too short a reduction, operands in whole 16-byte vectors:
// a matrix-vector kernel.
bool fwd_gemv_ok(const ConvShape& s, int dt);
hipError_t launch_conv_fwd_gemv(int dt, const FwdArgs& a, int bwd, double flops, hipStream_t st);

namespace {

// Operand load modes.  VEC16: 16-byte vectors of VEC taps (C % VEC == 0 for
// the input, Kg % VEC == 0 for the filter rows).  VEC8 (bf16 only): two 8-byte
// halves of 4 taps each, for channel counts that are a multiple of 4 but not
// of 8 (the first layer's colour channels padded to 4).  ELEM: one element at
// a time.
// BT16 (bf16 filter only): the filter is given transposed, w[tap][col] with
// the Nn columns contiguous (Nn % 8 == 0); 16-byte vectors of 8 columns go
// into LDS as tap-major rows and the MFMA fragments come from transposing
// reads.  Serves the dense backward-data, whose B operand is the weight
// matrix as stored, without a transposed copy.
constexpr int ELEM = 0, VEC8 = 1, VEC16 = 2, BT16 = 3;

typedef __attribute__((address_space(3))) void* lds_ptr;

// One 16-byte buffer load per lane into LDS slot (base + 16 * lane); base is
// wave-uniform.
__device__ __forceinline__ void ld_lds16(__amdgpu_buffer_rsrc_t r, uint32_t off, char* base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)base, 16, off, 0, 0, 0);
}

// The same load issued from inline assembly.  The compiler then does not
// know that the instruction writes LDS, so it adds no vmcnt wait in front of
// later LDS reads (it does so for the transpose reads, which would serialize
// every prefetch); the kernel orders the two itself with wait_vmcnt and a
// barrier.  M0 carries the LDS address; no other code of these kernels uses
// M0.
__device__ __forceinline__ void ld_lds16_asm(__amdgpu_buffer_rsrc_t r, uint32_t off, char* base) {
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)base;
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(__builtin_amdgcn_readfirstlane(lds)),
               "v"(off), "s"(r)
               : "memory");
}

// s_waitcnt vmcnt(n) (n < 64), leaving the other counters alone.
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Layout and split overrides for A/B measurements: read from the environment
// only in a library built with -DSINGA_TUNING.  The default build ignores the
// environment; its dispatch rules are the tested ones.
#ifdef SINGA_TUNING
inline const char* tuning_env(const char* name) { return getenv(name); }
#else
constexpr const char* tuning_env(const char*) { return nullptr; }
#endif

}  // namespace

}  // namespace singa
