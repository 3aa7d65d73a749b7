// conv_aux.hip -- the bandwidth-bound helpers around the convolution GEMMs:
//   * batched tiled transpose (flipped filter copies for backward-data, and the
//     filter transpose of a dense "fully connected" layer),
//   * direct gather backward-data for strides above one,
//   * bias-gradient column sums in a fixed order,
//   * NCHW <-> NHWC permutations for the NCHW entry points.
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace singa {

namespace {

template <typename T> __device__ __forceinline__ float ld_f(const T* p);
template <> __device__ __forceinline__ float ld_f<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float ld_f<bf16_t>(const bf16_t* p) { return bf16_to_f32(*p); }

template <typename T> __device__ __forceinline__ void st_f(T* p, float v);
template <> __device__ __forceinline__ void st_f<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void st_f<bf16_t>(bf16_t* p, float v) { *p = f32_to_bf16(v); }

// Batched transpose of a 64 x 64 tile through LDS.  VIN: rows of the input
// are read as 16-byte vectors (their length, stride and base allow it),
// otherwise element by element, 64 consecutive columns per wave; VOUT: the
// same for the rows written.  All loads of a tile are issued before the first
// is used: with a 32 x 32 tile of four loads a thread the permutations of a
// layer's activations between NCHW and NHWC moved 1.7-2 TB/s.  mask (optional,
// laid out like the output): an element is zeroed where mask <= 0.  flip 1:
// the batches go out in reverse order; 2: each batch's output rows do.
template <typename T, bool VIN, bool VOUT>
__global__ __launch_bounds__(256) void transpose_kernel(const T* __restrict__ in, T* __restrict__ out, int batch,
                                                        int rows, int cols, long in_bstride, long in_rstride,
                                                        long out_bstride, long out_rstride, int flip,
                                                        const T* __restrict__ mask) {
  constexpr int VEC = 16 / (int)sizeof(T);
  constexpr int TPR = 64 / VEC;   // threads per 64-element row of vectors
  constexpr int RPP = 256 / TPR;  // rows per pass
  __shared__ T tile[64][64 + 2];
  const int b = blockIdx.z;
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const T* src = in + (long)b * in_bstride;
  const long ob = (long)(flip == 1 ? batch - 1 - b : b) * out_bstride;
  const int tc = threadIdx.x % TPR, tr = threadIdx.x / TPR;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if constexpr (VIN) {
    union { uint4 u; T e[VEC]; } v[64 / RPP];
#pragma unroll
    for (int k = 0; k < 64 / RPP; ++k) {
      const int r = r0 + tr + k * RPP, c = c0 + tc * VEC;
      v[k].u = (r < rows && c < cols) ? *(const uint4*)(src + (long)r * in_rstride + c) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < 64 / RPP; ++k)
#pragma unroll
      for (int j = 0; j < VEC; ++j) tile[tr + k * RPP][tc * VEC + j] = v[k].e[j];
  } else {
    T v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int r = r0 + wave + 4 * k, c = c0 + lane;
      v[k] = (r < rows && c < cols) ? src[(long)r * in_rstride + c] : T(0);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) tile[wave + 4 * k][lane] = v[k];
  }
  __syncthreads();
  if constexpr (VOUT) {
#pragma unroll
    for (int k = 0; k < 64 / RPP; ++k) {
      const int c = c0 + tr + k * RPP, r = r0 + tc * VEC;  // output row c, output columns r .. r + VEC - 1
      if (c < cols && r < rows) {
        const long o = ob + (long)(flip == 2 ? cols - 1 - c : c) * out_rstride + r;
        union { uint4 u; T e[VEC]; } v;
#pragma unroll
        for (int j = 0; j < VEC; ++j) v.e[j] = tile[tc * VEC + j][tr + k * RPP];
        if (mask) {
          union { uint4 u; T e[VEC]; } m;
          m.u = *(const uint4*)(mask + o);
#pragma unroll
          for (int j = 0; j < VEC; ++j)
            if (!(ld_f<T>(&m.e[j]) > 0.f)) v.e[j] = T(0);
        }
        *(uint4*)(out + o) = v.u;
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int c = c0 + wave + 4 * k, r = r0 + lane;
      if (c < cols && r < rows) {
        const long o = ob + (long)(flip == 2 ? cols - 1 - c : c) * out_rstride + r;
        T v = tile[lane][wave + 4 * k];
        if (mask && !(ld_f<T>(mask + o) > 0.f)) v = T(0);
        out[o] = v;
      }
    }
  }
}

// dx[n,h,w,c] = sum over taps (r,s) whose output pixel (p,q) lands on a whole
// multiple of the stride, and over k, of w[k,r,s,c] * dy[n,p,q,k].
template <typename T>
__global__ __launch_bounds__(256) void bwd_data_direct_kernel(ConvShape s, const T* __restrict__ dy,
                                                              const T* __restrict__ w,
                                                              const T* __restrict__ mask, T* __restrict__ dx,
                                                              long total) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
    const int c = (int)(i % s.C);
    long t = i / s.C;
    const int x = (int)(t % s.W);
    t /= s.W;
    const int h = (int)(t % s.H);
    const int n = (int)(t / s.H);
    float acc = 0.f;
    for (int r = 0; r < s.R; ++r) {
      const int pn = h + s.ph - r;
      if (pn < 0 || pn % s.sh) continue;
      const int p = pn / s.sh;
      if (p >= s.P) continue;
      for (int q_s = 0; q_s < s.S; ++q_s) {
        const int qn = x + s.pw - q_s;
        if (qn < 0 || qn % s.sw) continue;
        const int q = qn / s.sw;
        if (q >= s.Q) continue;
        const T* dyr = dy + (((long)n * s.P + p) * s.Q + q) * s.K;
        const T* wr = w + ((long)r * s.S + q_s) * s.C + c;
        const long wk = (long)s.R * s.S * s.C;
        for (int k = 0; k < s.K; ++k) acc += ld_f<T>(wr + k * wk) * ld_f<T>(dyr + k);
      }
    }
    if (mask && !(ld_f<T>(mask + i) > 0.f)) acc = 0.f;
    st_f<T>(dx + i, acc);
  }
}

__global__ __launch_bounds__(256) void krsc_to_kcrs_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                           int K, int C, int RS, int accumulate) {
  const long total = (long)K * C * RS;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
    // i indexes the KCRS output
    const int rs = (int)(i % RS);
    const long kc = i / RS;
    const int c = (int)(kc % C);
    const int k = (int)(kc / C);
    const float v = in[((long)k * RS + rs) * C + c];
    out[i] = accumulate ? out[i] + v : v;
  }
}

// out[r][c] = in[r][c] for c < C, 0 for C <= c < Cp (Cp % 4 == 0), over two
// tensors in one launch (an input and its filter: a launch each, with another
// for the rows that an 8-row group left over, took longer than the work).
// A workgroup below `split` works on the first tensor, the others on the
// second; one thread per 4-channel chunk of an output row, stored as one vector.
template <typename T> struct PadSpan {
  const T* in;
  T* out;
  long rows;
};
template <typename T>
__global__ __launch_bounds__(256) void pad_channels_kernel(PadSpan<T> a, PadSpan<T> b, unsigned split, int C, int Cp) {
  typedef typename std::conditional<sizeof(T) == 2, uint2, uint4>::type V4;
  const bool first = blockIdx.x < split;
  const PadSpan<T> p = first ? a : b;
  const long blk = first ? blockIdx.x : blockIdx.x - split, nblk = first ? split : gridDim.x - split;
  const int nv = Cp / 4;
  const long total = p.rows * nv;
  for (long i = blk * blockDim.x + threadIdx.x; i < total; i += nblk * blockDim.x) {
    const long r = i / nv;
    const int c0 = (int)(i - r * nv) * 4;
    union { V4 u; T e[4]; } v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v.e[j] = (c0 + j < C) ? p.in[r * C + c0 + j] : (T)0;
    *(V4*)(p.out + r * Cp + c0) = v.u;
  }
}

// The same for C = 3, Cp = 4 (colour images): one thread per 8 rows, read as
// 3 (bf16) / 6 (fp32) 16-byte vectors and written as 4 / 8; the thread after
// the last whole group takes the rows left over one by one.
template <typename T>
__global__ __launch_bounds__(256) void pad_3to4_kernel(PadSpan<T> a, PadSpan<T> b, unsigned split) {
  constexpr int NI = 24 * (int)sizeof(T) / 16, NO = 32 * (int)sizeof(T) / 16;
  const bool first = blockIdx.x < split;
  const PadSpan<T> p = first ? a : b;
  const long blk = first ? blockIdx.x : blockIdx.x - split, nblk = first ? split : gridDim.x - split;
  const long groups = p.rows / 8;
  for (long i = blk * blockDim.x + threadIdx.x; i <= groups; i += nblk * blockDim.x) {
    if (i == groups) {
      for (long r = groups * 8; r < p.rows; ++r)
        for (int c = 0; c < 4; ++c) p.out[r * 4 + c] = c < 3 ? p.in[r * 3 + c] : T(0);
      break;
    }
    union { uint4 u[NI]; T e[24]; } s;
    union { uint4 u[NO]; T e[32]; } d;
    const uint4* src = (const uint4*)(p.in + i * 24);
#pragma unroll
    for (int k = 0; k < NI; ++k) s.u[k] = src[k];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      d.e[4 * q] = s.e[3 * q];
      d.e[4 * q + 1] = s.e[3 * q + 1];
      d.e[4 * q + 2] = s.e[3 * q + 2];
      d.e[4 * q + 3] = T(0);
    }
    uint4* dst = (uint4*)(p.out + i * 32);
#pragma unroll
    for (int k = 0; k < NO; ++k) dst[k] = d.u[k];
  }
}

// Space-to-depth rewrite of a strided convolution (stride sh x sw, padding
// ph, pw) as a stride-1 convolution without padding:
//   x'[n][h'][w'][(dh*sw + dw)*C + c] = x[n][sh*h' + dh - ph][sw*w' + dw - pw][c]  (0 outside x)
//   w'[k][r'][s'][(dh*sw + dw)*C + c] = w[k][sh*r' + dh][sw*s' + dw][c]           (0 past R, S)
// so that y[n][p][q][k] = sum over (r', s', c') of w'[k][r'][s'][c'] x'[n][p + r'][q + s'][c'].
// One thread per 16-byte chunk of x' (VEC channels of one rewritten pixel),
// 32-bit index math with precomputed divisors.
template <typename T>
__global__ __launch_bounds__(256) void space_to_depth_kernel(const T* __restrict__ x, T* __restrict__ xs, int H,
                                                             int W, int C, int Hs, int Ws, int sh, int sw, int ph,
                                                             int pw, FastDiv dJ, FastDiv dWs, FastDiv dHs, FastDiv dC,
                                                             FastDiv dSw, int total) {
  constexpr int VEC = 16 / (int)sizeof(T);
  const int J = (int)dJ.d;  // chunks per rewritten pixel
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int pix = (int)fdiv((uint32_t)i, dJ);
    const int j = i - pix * J;
    const int t = (int)fdiv((uint32_t)pix, dWs);
    const int wq = pix - t * Ws;
    const int n = (int)fdiv((uint32_t)t, dHs);
    const int hq = t - n * Hs;
    union { uint4 u; T e[VEC]; } v;
#pragma unroll
    for (int u = 0; u < VEC; ++u) {
      const int e = j * VEC + u;
      const int d = (int)fdiv((uint32_t)e, dC);
      const int c = e - d * C;
      const int dh = (int)fdiv((uint32_t)d, dSw);
      const int dw = d - dh * sw;
      const int h = sh * hq + dh - ph, w = sw * wq + dw - pw;
      const bool ok = (unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W;
      v.e[u] = ok ? x[((n * H + h) * W + w) * C + c] : T(0);
    }
    *(uint4*)(xs + (size_t)i * VEC) = v.u;
  }
}

// The same in bf16 where the sw * C elements of one input row that go into one
// rewritten pixel, a contiguous run in x and in x', are 24 bytes (3 colour
// channels at stride 4): one thread per run, read as the aligned words that
// hold it, shifted into place where it starts in the middle of one, and
// written as 8-byte words.  Runs that leave the image, or whose last word is
// not all inside the tensor, go element by element.  Against a thread per
// 16-byte chunk that gathers eight single elements: 256 x 227 x 227 x 3 43.0
// -> 35.5 us, 128 images 21.9 -> 16.0 (5.0 TB/s); fp32, whose elements are
// words already, measured no faster this way and keeps the gather.
__global__ __launch_bounds__(256) void space_to_depth_run_kernel(const bf16_t* __restrict__ x,
                                                                 bf16_t* __restrict__ xs, int H, int W, int C, int Hs,
                                                                 int Ws, int sh, int sw, int ph, int pw, FastDiv dSh,
                                                                 FastDiv dWs, FastDiv dHs, long elems, int total) {
  constexpr int E = 12, WORDS = E / 2;  // elements and 4-byte words of a run
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int pix = (int)fdiv((uint32_t)i, dSh);
    const int dh = i - pix * sh;
    const int t = (int)fdiv((uint32_t)pix, dWs);
    const int wq = pix - t * Ws;
    const int n = (int)fdiv((uint32_t)t, dHs);
    const int h = sh * (t - n * Hs) + dh - ph, w = sw * wq - pw;
    const long off = ((long)(n * H + h) * W + w) * C;  // first element of the run
    union { uint32_t d[WORDS]; bf16_t e[E]; } v;
    const bool row = (unsigned)h < (unsigned)H;
    const int odd = (int)(off & 1);
    if (row && w >= 0 && w + sw <= W && off + E + odd <= elems) {
      const uint32_t* __restrict__ p = (const uint32_t*)x + (off >> 1);
      uint32_t a[WORDS + 1];
#pragma unroll
      for (int k = 0; k < WORDS; ++k) a[k] = p[k];
      a[WORDS] = odd ? p[WORDS] : 0u;
#pragma unroll
      for (int k = 0; k < WORDS; ++k) v.d[k] = odd ? __builtin_amdgcn_alignbit(a[k + 1], a[k], 16) : a[k];
    } else {
#pragma unroll
      for (int u = 0; u < E; ++u) {
        const int wu = w + u / C;
        v.e[u] = (row && (unsigned)wu < (unsigned)W) ? x[off + u] : (bf16_t)0;
      }
    }
    uint2* dst = (uint2*)(xs + (size_t)i * E);
#pragma unroll
    for (int k = 0; k < WORDS / 2; ++k) dst[k] = make_uint2(v.d[2 * k], v.d[2 * k + 1]);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void filter_to_s2d_kernel(const T* __restrict__ w, T* __restrict__ ws, int R,
                                                            int S, int C, int Rs, int Ss, int sh, int sw,
                                                            int total) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int Cs = sh * sw * C;
    const int cs = i % Cs;
    int t = i / Cs;
    const int ss = t % Ss;
    t /= Ss;
    const int rs = t % Rs;
    const int k = t / Rs;
    const int c = cs % C, d = cs / C, dh = d / sw, dw = d % sw;
    const int r = sh * rs + dh, s = sw * ss + dw;
    ws[i] = (r < R && s < S) ? w[((k * R + r) * S + s) * C + c] : T(0);
  }
}

// dw[k][r][s][c] (+)= dws[k][r / sh][s / sw][((r % sh)*sw + s % sw)*C + c] (fp32 filter gradients).
__global__ __launch_bounds__(256) void s2d_to_filter_f32_kernel(const float* __restrict__ dws, float* __restrict__ dw,
                                                                int R, int S, int C, int Rs, int Ss, int sh, int sw,
                                                                int accumulate, int total) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int c = i % C;
    int t = i / C;
    const int s = t % S;
    t /= S;
    const int r = t % R;
    const int k = t / R;
    const int Cs = sh * sw * C;
    const float v = dws[((k * Rs + r / sh) * Ss + s / sw) * Cs + ((r % sh) * sw + s % sw) * C + c];
    dw[i] = accumulate ? dw[i] + v : v;
  }
}

// dx[n][h][w][c] = dxs[n][(h + ph) / sh][(w + pw) / sw][(((h + ph) % sh)*sw + (w + pw) % sw)*C + c]
// (0 where that position lies outside dxs: no output window reads it), then
// zeroed where mask <= 0 when a ReLU's output is given.
template <typename T>
__global__ __launch_bounds__(256) void depth_to_space_kernel(const T* __restrict__ dxs, const T* __restrict__ mask,
                                                             T* __restrict__ dx, FastDiv dC, FastDiv dW, FastDiv dH,
                                                             int H, int W, int C, int Hs, int Ws, int sh, int sw,
                                                             int ph, int pw, int total) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int t1 = (int)fdiv((uint32_t)i, dC);
    const int c = i - t1 * C;
    const int t2 = (int)fdiv((uint32_t)t1, dW);
    const int w = t1 - t2 * W;
    const int n = (int)fdiv((uint32_t)t2, dH);
    const int h = t2 - n * H;
    const int hq = (h + ph) / sh, wq = (w + pw) / sw;
    float v = 0.f;
    if (hq < Hs && wq < Ws) {
      const int Cs = sh * sw * C;
      v = ld_f<T>(dxs + ((n * Hs + hq) * Ws + wq) * Cs + (((h + ph) % sh) * sw + (w + pw) % sw) * C + c);
    }
    if (mask && !(ld_f<T>(mask + i) > 0.f)) v = 0.f;
    st_f<T>(dx + i, v);
  }
}

// out[r][c] (+)= in[r][c] for c < C: drops the zero-padded channels of an
// fp32 filter gradient computed on a channel-padded input.
__global__ __launch_bounds__(256) void unpad_channels_f32_kernel(const float* __restrict__ in,
                                                                 float* __restrict__ out, long rows, int Cp, int C,
                                                                 int accumulate) {
  const long total = rows * C;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
    const long r = i / C;
    const int c = (int)(i - r * C);
    const float v = in[r * Cp + c];
    out[i] = accumulate ? out[i] + v : v;
  }
}

unsigned grid_for(long total, int block = 256, long cap = 65536) {
  long g = (total + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

}  // namespace

template <typename T>
static void transpose(const void* in, void* out, int batch, int rows, int cols, long in_bstride, long in_rstride,
                      long out_bstride, long out_rstride, int flip, const void* mask, hipStream_t st) {
  constexpr long V = 16 / (long)sizeof(T);
  const bool vin = cols % V == 0 && in_rstride % V == 0 && in_bstride % V == 0 && (uintptr_t)in % 16 == 0;
  const bool vout = rows % V == 0 && out_rstride % V == 0 && out_bstride % V == 0 &&
                    (((uintptr_t)out | (uintptr_t)mask) % 16) == 0;
  const dim3 grid((cols + 63) / 64, (rows + 63) / 64, batch), block(256);
#define TRANSPOSE(I, O)                                                                                              \
  hipLaunchKernelGGL((transpose_kernel<T, I, O>), grid, block, 0, st, (const T*)in, (T*)out, batch, rows, cols,      \
                     in_bstride, in_rstride, out_bstride, out_rstride, flip, (const T*)mask)
  if (vin) { if (vout) TRANSPOSE(true, true); else TRANSPOSE(true, false); }
  else { if (vout) TRANSPOSE(false, true); else TRANSPOSE(false, false); }
#undef TRANSPOSE
}

hipError_t launch_transpose(int dt, const void* in, void* out, int batch, int rows, int cols, long in_bstride,
                            long in_rstride, long out_bstride, long out_rstride, int flip, hipStream_t st) {
  TraceScope ts("transpose_kernel", st, 2.0 * batch * (double)rows * cols * dt_size(dt), WORK_BYTE);
  if (dt == BF16)
    transpose<bf16_t>(in, out, batch, rows, cols, in_bstride, in_rstride, out_bstride, out_rstride, flip, nullptr, st);
  else
    transpose<float>(in, out, batch, rows, cols, in_bstride, in_rstride, out_bstride, out_rstride, flip, nullptr, st);
  return hipGetLastError();
}

hipError_t launch_conv_bwd_data_direct(int dt, const ConvShape& s, const void* dy, const void* w, void* dx,
                                       const void* mask, hipStream_t st) {
  const long total = (long)s.N * s.H * s.W * s.C;
  const unsigned g = grid_for(total);
  TraceScope ts("bwd_data_direct_kernel", st,
                2.0 * s.N * (double)s.P * s.Q * s.K * (double)s.C * s.R * s.S, WORK_FLOP);
  if (dt == BF16)
    hipLaunchKernelGGL(bwd_data_direct_kernel<bf16_t>, dim3(g), dim3(256), 0, st, s, (const bf16_t*)dy,
                       (const bf16_t*)w, (const bf16_t*)mask, (bf16_t*)dx, total);
  else
    hipLaunchKernelGGL(bwd_data_direct_kernel<float>, dim3(g), dim3(256), 0, st, s, (const float*)dy,
                       (const float*)w, (const float*)mask, (float*)dx, total);
  return hipGetLastError();
}

template <typename T>
static void pad_channels(const void* in, void* out, long rows, const void* in2, void* out2, long rows2, int C, int Cp,
                         hipStream_t st) {
  const PadSpan<T> a{(const T*)in, (T*)out, rows}, b{(const T*)in2, (T*)out2, rows2};
  const bool v = C == 3 && Cp == 4 && (((uintptr_t)in | (uintptr_t)out | (uintptr_t)in2 | (uintptr_t)out2) % 16) == 0;
  const long items = v ? rows / 8 + 1 : rows * (Cp / 4), items2 = v ? rows2 / 8 + 1 : rows2 * (Cp / 4);
  const unsigned split = grid_for(items), grid = split + (rows2 > 0 ? grid_for(items2) : 0);
  if (v) hipLaunchKernelGGL(pad_3to4_kernel<T>, dim3(grid), dim3(256), 0, st, a, b, split);
  else hipLaunchKernelGGL(pad_channels_kernel<T>, dim3(grid), dim3(256), 0, st, a, b, split, C, Cp);
}

hipError_t launch_pad_channels(int dt, const void* in, void* out, long rows, const void* in2, void* out2, long rows2,
                               int C, int Cp, hipStream_t st) {
  if (Cp % 4 != 0 || C > Cp) return hipErrorInvalidValue;
  TraceScope ts("pad_channels_kernel", st, (double)(rows + rows2) * (C + Cp) * dt_size(dt), WORK_BYTE);
  if (dt == BF16) pad_channels<bf16_t>(in, out, rows, in2, out2, rows2, C, Cp, st);
  else pad_channels<float>(in, out, rows, in2, out2, rows2, C, Cp, st);
  return hipGetLastError();
}

hipError_t launch_unpad_channels_f32(const float* in, float* out, long rows, int Cp, int C, int accumulate,
                                     hipStream_t st) {
  const long total = rows * C;
  TraceScope ts("unpad_channels_f32_kernel", st, (double)rows * (C * (accumulate ? 12.0 : 8.0)), WORK_BYTE);
  hipLaunchKernelGGL(unpad_channels_f32_kernel, dim3(grid_for(total)), dim3(256), 0, st, in, out, rows, Cp, C,
                     accumulate);
  return hipGetLastError();
}

hipError_t launch_space_to_depth(int dt, const ConvShape& s, const ConvShape& g, const void* x, void* xs,
                                 hipStream_t st) {
  const int vec = 16 / (int)dt_size(dt);
  if (g.C % vec != 0 || (uintptr_t)xs % 16 != 0) return hipErrorInvalidValue;  // callers guarantee both
  const int J = g.C / vec;
  const int total = g.N * g.H * g.W * J;
  TraceScope ts("space_to_depth_kernel", st,
                ((double)s.N * s.H * s.W * s.C + (double)g.N * g.H * g.W * g.C) * dt_size(dt), WORK_BYTE);
  // whole words only (3 channels at stride 4, in practice): the run's length is
  // the kernel's word count; other factors keep the gather
  if (dt == BF16 && s.sw * s.C == 12 && (uintptr_t)x % 4 == 0) {
    const int runs = g.N * g.H * g.W * s.sh;
    hipLaunchKernelGGL(space_to_depth_run_kernel, dim3(grid_for(runs)), dim3(256), 0, st, (const bf16_t*)x,
                       (bf16_t*)xs, s.H, s.W, s.C, g.H, g.W, s.sh, s.sw, s.ph, s.pw, make_fastdiv((uint32_t)s.sh),
                       make_fastdiv((uint32_t)g.W), make_fastdiv((uint32_t)g.H), (long)s.N * s.H * s.W * s.C, runs);
    return hipGetLastError();
  }
  const FastDiv dJ = make_fastdiv((uint32_t)J), dWs = make_fastdiv((uint32_t)g.W), dHs = make_fastdiv((uint32_t)g.H),
                dC = make_fastdiv((uint32_t)s.C), dSw = make_fastdiv((uint32_t)s.sw);
  if (dt == BF16)
    hipLaunchKernelGGL(space_to_depth_kernel<bf16_t>, dim3(grid_for(total)), dim3(256), 0, st, (const bf16_t*)x,
                       (bf16_t*)xs, s.H, s.W, s.C, g.H, g.W, s.sh, s.sw, s.ph, s.pw, dJ, dWs, dHs, dC, dSw, total);
  else
    hipLaunchKernelGGL(space_to_depth_kernel<float>, dim3(grid_for(total)), dim3(256), 0, st, (const float*)x,
                       (float*)xs, s.H, s.W, s.C, g.H, g.W, s.sh, s.sw, s.ph, s.pw, dJ, dWs, dHs, dC, dSw, total);
  return hipGetLastError();
}

hipError_t launch_filter_to_s2d(int dt, const ConvShape& s, const ConvShape& g, const void* w, void* ws,
                                hipStream_t st) {
  const int total = g.K * g.R * g.S * g.C;
  TraceScope ts("filter_to_s2d_kernel", st, (double)total * 2 * dt_size(dt), WORK_BYTE);
  if (dt == BF16)
    hipLaunchKernelGGL(filter_to_s2d_kernel<bf16_t>, dim3(grid_for(total)), dim3(256), 0, st, (const bf16_t*)w,
                       (bf16_t*)ws, s.R, s.S, s.C, g.R, g.S, s.sh, s.sw, total);
  else
    hipLaunchKernelGGL(filter_to_s2d_kernel<float>, dim3(grid_for(total)), dim3(256), 0, st, (const float*)w,
                       (float*)ws, s.R, s.S, s.C, g.R, g.S, s.sh, s.sw, total);
  return hipGetLastError();
}

hipError_t launch_s2d_to_filter_f32(const ConvShape& s, const ConvShape& g, const float* dws, float* dw,
                                    int accumulate, hipStream_t st) {
  const int total = s.K * s.R * s.S * s.C;
  TraceScope ts("s2d_to_filter_f32_kernel", st, (double)total * (accumulate ? 12.0 : 8.0), WORK_BYTE);
  hipLaunchKernelGGL(s2d_to_filter_f32_kernel, dim3(grid_for(total)), dim3(256), 0, st, dws, dw, s.R, s.S, s.C, g.R,
                     g.S, s.sh, s.sw, accumulate, total);
  return hipGetLastError();
}

hipError_t launch_depth_to_space(int dt, const ConvShape& s, const ConvShape& g, const void* dxs, const void* mask,
                                 void* dx, hipStream_t st) {
  const int total = s.N * s.H * s.W * s.C;
  TraceScope ts("depth_to_space_kernel", st, (double)total * (mask ? 3 : 2) * dt_size(dt), WORK_BYTE);
  const FastDiv dC = make_fastdiv((uint32_t)s.C), dW = make_fastdiv((uint32_t)s.W), dH = make_fastdiv((uint32_t)s.H);
  if (dt == BF16)
    hipLaunchKernelGGL(depth_to_space_kernel<bf16_t>, dim3(grid_for(total)), dim3(256), 0, st, (const bf16_t*)dxs,
                       (const bf16_t*)mask, (bf16_t*)dx, dC, dW, dH, s.H, s.W, s.C, g.H, g.W, s.sh, s.sw, s.ph, s.pw,
                       total);
  else
    hipLaunchKernelGGL(depth_to_space_kernel<float>, dim3(grid_for(total)), dim3(256), 0, st, (const float*)dxs,
                       (const float*)mask, (float*)dx, dC, dW, dH, s.H, s.W, s.C, g.H, g.W, s.sh, s.sw, s.ph, s.pw,
                       total);
  return hipGetLastError();
}

hipError_t launch_nchw_to_nhwc(int dt, const void* in, void* out, int N, int C, int H, int W, hipStream_t st) {
  const int HW = H * W;
  TraceScope ts("nchw_to_nhwc_kernel", st, 2.0 * N * (double)C * HW * dt_size(dt), WORK_BYTE);
  if (dt == BF16) transpose<bf16_t>(in, out, N, C, HW, (long)C * HW, HW, (long)C * HW, C, 0, nullptr, st);
  else transpose<float>(in, out, N, C, HW, (long)C * HW, HW, (long)C * HW, C, 0, nullptr, st);
  return hipGetLastError();
}

hipError_t launch_nhwc_to_nchw(int dt, const void* in, void* out, int N, int C, int H, int W, const void* mask,
                               hipStream_t st) {
  const int HW = H * W;
  TraceScope ts("nhwc_to_nchw_kernel", st, (mask ? 3.0 : 2.0) * N * (double)C * HW * dt_size(dt), WORK_BYTE);
  if (dt == BF16) transpose<bf16_t>(in, out, N, HW, C, (long)C * HW, C, (long)C * HW, HW, 0, mask, st);
  else transpose<float>(in, out, N, HW, C, (long)C * HW, C, (long)C * HW, HW, 0, mask, st);
  return hipGetLastError();
}

hipError_t launch_krsc_to_kcrs_f32(const float* in, float* out, int K, int C, int R, int S, int accumulate,
                                   hipStream_t st) {
  const long total = (long)K * C * R * S;
  TraceScope ts("krsc_to_kcrs_kernel", st, 4.0 * total * (accumulate ? 3 : 2), WORK_BYTE);
  hipLaunchKernelGGL(krsc_to_kcrs_kernel, dim3(grid_for(total)), dim3(256), 0, st, in, out, K, C, R * S,
                     accumulate);
  return hipGetLastError();
}

}  // namespace singa
