// LayerNorm forward and backward over rows of C channels (pre-LN blocks and
// the final norm, Figure 1). Statistics in fp32, biased variance, eps from the
// config. One wavefront per row; each lane owns channels {4*(lane + 64*i)..+3},
// read as 8-byte bf16 chunks.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace {

// Sum of two bf16 rows in fp32, rounded to bf16 (to nearest even): the
// residual connection's addition
DEV uint2 add_rows(uint2 r, uint2 a) {
  return make_uint2(pack2(lo_f(r.x) + lo_f(a.x), hi_f(r.x) + hi_f(a.x)),
                    pack2(lo_f(r.y) + lo_f(a.y), hi_f(r.y) + hi_f(a.y)));
}

// MAXCH: 4-channel chunks per lane, C <= 256*MAXCH. With SRC_RES the row is
// first formed as the residual sum x = bf16(res + x) (stored to xsum), and the
// normalisation then reads those rounded values, exactly as a separate
// addition followed by this kernel would. With SRC_SLICES the branch comes as
// fp32 slices of the projection before it (few rows: the product is split to
// fill the chip), x = bf16(sum + bias + res), so the split costs no launch of
// its own; w == nullptr then stops after xsum. xcopy (when not null) takes the
// row that is normalised as well.
constexpr int SRC_X = 0, SRC_RES = 1, SRC_SLICES = 2;
template <int MAXCH, int SRC = SRC_X>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const bf16_t* __restrict__ x, Slices sl,
                                                     const float* __restrict__ bias, const bf16_t* __restrict__ res,
                                                     bf16_t* __restrict__ xsum, const float* __restrict__ w,
                                                     const float* __restrict__ b, bf16_t* __restrict__ y,
                                                     float* __restrict__ mean_out, float* __restrict__ rstd_out,
                                                     int rows, int C, float eps, bf16_t* __restrict__ xcopy) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const bf16_t* xr = x + (size_t)row * C;
  // Every lane issues all its loads at once: chunks past C read the row's
  // last chunk (an in-range address) and are masked out of the arithmetic,
  // so no load waits behind a branch.
  uint2 xu[MAXCH], ru[MAXCH];
  float4 wv[MAXCH], bv[MAXCH];
#pragma unroll
  for (int i = 0; i < MAXCH; ++i) {
    const int c = min(4 * (lane + 64 * i), C - 4);
    if constexpr (SRC != SRC_SLICES) xu[i] = *reinterpret_cast<const uint2*>(xr + c);
    if constexpr (SRC != SRC_X) ru[i] = *reinterpret_cast<const uint2*>(res + (size_t)row * C + c);
    if (SRC != SRC_SLICES || w) {
      wv[i] = *reinterpret_cast<const float4*>(w + c);
      bv[i] = *reinterpret_cast<const float4*>(b + c);
    }
  }
  if constexpr (SRC == SRC_SLICES) {
    const float* sr = sl.p + (size_t)row * C;
#pragma unroll
    for (int i = 0; i < MAXCH; ++i) {
      const int c = min(4 * (lane + 64 * i), C - 4);
      const float4 t = sum_slices(sr + c, sl.n, (size_t)rows * C);
      const float4 bb = *reinterpret_cast<const float4*>(bias + c);
      xu[i] = make_uint2(pack2(t.x + bb.x + lo_f(ru[i].x), t.y + bb.y + hi_f(ru[i].x)),
                         pack2(t.z + bb.z + lo_f(ru[i].y), t.w + bb.w + hi_f(ru[i].y)));
    }
  }
  if constexpr (SRC != SRC_X) {
#pragma unroll
    for (int i = 0; i < MAXCH; ++i) {
      if constexpr (SRC == SRC_RES) xu[i] = add_rows(ru[i], xu[i]);
      const int c = 4 * (lane + 64 * i);
      if (c < C) *reinterpret_cast<uint2*>(xsum + (size_t)row * C + c) = xu[i];
    }
  }
  if (xcopy) {
#pragma unroll
    for (int i = 0; i < MAXCH; ++i) {
      const int c = 4 * (lane + 64 * i);
      if (c < C) *reinterpret_cast<uint2*>(xcopy + (size_t)row * C + c) = xu[i];
    }
  }
  if (SRC == SRC_SLICES && !w) return;
  float v[MAXCH][4];
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < MAXCH; ++i) {
    const bool in = 4 * (lane + 64 * i) < C;
    v[i][0] = in ? lo_f(xu[i].x) : 0.0f;
    v[i][1] = in ? hi_f(xu[i].x) : 0.0f;
    v[i][2] = in ? lo_f(xu[i].y) : 0.0f;
    v[i][3] = in ? hi_f(xu[i].y) : 0.0f;
    s += v[i][0] + v[i][1] + v[i][2] + v[i][3];
  }
  const float mean = wave_sum(s) / C;
  float q = 0.0f;
#pragma unroll
  for (int i = 0; i < MAXCH; ++i) {
    if (4 * (lane + 64 * i) < C)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float d = v[i][e] - mean;
        q += d * d;
      }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / C + eps);
  bf16_t* yr = y + (size_t)row * C;
#pragma unroll
  for (int i = 0; i < MAXCH; ++i) {
    int c = 4 * (lane + 64 * i);
    if (c < C) {
      float o0 = (v[i][0] - mean) * rstd * wv[i].x + bv[i].x;
      float o1 = (v[i][1] - mean) * rstd * wv[i].y + bv[i].y;
      float o2 = (v[i][2] - mean) * rstd * wv[i].z + bv[i].z;
      float o3 = (v[i][3] - mean) * rstd * wv[i].w + bv[i].w;
      *reinterpret_cast<uint2*>(yr + c) = make_uint2(pack2(o0, o1), pack2(o2, o3));
    }
  }
  if (lane == 0) {
    mean_out[row] = mean;
    rstd_out[row] = rstd;
  }
}

// dx = rstd * (g - mean(g) - xhat * mean(g * xhat)), g = dy * w; the result is
// added to the residual-stream gradient read from dres_in and written to
// dres_out (the two may be the same buffer: each row is read before it is
// written, by the same wave). Per-block sums of dy*xhat and dy.
// With SL the upstream gradient is the sum of fp32 slices of the product before
// it (few rows), taken unrounded.
template <int MAXCH, bool SL>
__global__ __launch_bounds__(256) void ln_bwd_kernel(const bf16_t* __restrict__ dy, Slices sl,
                                                     const bf16_t* __restrict__ x,
                                                     const float* __restrict__ mean_in,
                                                     const float* __restrict__ rstd_in, const float* __restrict__ w,
                                                     const bf16_t* dres_in, bf16_t* dres_out, int has_res,
                                                     float* __restrict__ part, int rows, int C) {
  __shared__ float red[4][MAXCH * 4 * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float aw[MAXCH][4], ab[MAXCH][4], ar[MAXCH][4], wr[MAXCH][4];
#pragma unroll
  for (int i = 0; i < MAXCH; ++i) {
    // chunks past C read an in-range address; their values are never used
    const int c = min(4 * (lane + 64 * i), C - 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) aw[i][e] = ab[i][e] = ar[i][e] = 0.0f;
    const float4 wv = *reinterpret_cast<const float4*>(w + c);
    wr[i][0] = wv.x; wr[i][1] = wv.y; wr[i][2] = wv.z; wr[i][3] = wv.w;
  }
  // Rows are software-pipelined: the next row's inputs (x, dy, the residual
  // gradient, mean, rstd) are loaded while the current row is reduced and
  // written, so each row costs one memory round trip, not two.
  using Dy = std::conditional_t<SL, float4, uint2>;   // four elements of dy
  uint2 xu[MAXCH], ru[MAXCH];
  Dy du[MAXCH];
  float mean = 0.0f, rstd = 0.0f;
  auto load_row = [&](int row, uint2 (&xl)[MAXCH], Dy (&dl)[MAXCH], uint2 (&rl)[MAXCH], float& ml, float& sdl) {
    ml = mean_in[row];
    sdl = rstd_in[row];
    const bf16_t* xr = x + (size_t)row * C;
    const bf16_t* dr = dy + (size_t)row * C;
    const bf16_t* rr = dres_in + (size_t)row * C;
    // all loads issued at once (no branch per chunk): chunks past C read the
    // row's last chunk and are never used
#pragma unroll
    for (int i = 0; i < MAXCH; ++i) {
      const int c = min(4 * (lane + 64 * i), C - 4);
      xl[i] = *reinterpret_cast<const uint2*>(xr + c);
      if constexpr (SL) dl[i] = sum_slices(sl.p + (size_t)row * C + c, sl.n, (size_t)rows * C);
      else dl[i] = *reinterpret_cast<const uint2*>(dr + c);
      rl[i] = has_res ? *reinterpret_cast<const uint2*>(rr + c) : make_uint2(0, 0);
    }
  };
  const int stride = gridDim.x * 4;
  int row = blockIdx.x * 4 + wave;
  if (row < rows) load_row(row, xu, du, ru, mean, rstd);
  for (; row < rows; row += stride) {
    uint2 xn[MAXCH], rn[MAXCH];
    Dy dn[MAXCH];
    float mean_n = 0.0f, rstd_n = 0.0f;
    if (row + stride < rows) load_row(row + stride, xn, dn, rn, mean_n, rstd_n);
    float xh[MAXCH][4], gg[MAXCH][4];
    float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int i = 0; i < MAXCH; ++i) {
      int c = 4 * (lane + 64 * i);
      if (c < C) {
        float xv[4] = {lo_f(xu[i].x), hi_f(xu[i].x), lo_f(xu[i].y), hi_f(xu[i].y)};
        float dv[4];
        if constexpr (SL) {
          dv[0] = du[i].x; dv[1] = du[i].y; dv[2] = du[i].z; dv[3] = du[i].w;
        } else {
          dv[0] = lo_f(du[i].x); dv[1] = hi_f(du[i].x); dv[2] = lo_f(du[i].y); dv[3] = hi_f(du[i].y);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          xh[i][e] = (xv[e] - mean) * rstd;
          gg[i][e] = dv[e] * wr[i][e];
          s1 += gg[i][e];
          s2 += gg[i][e] * xh[i][e];
          aw[i][e] += dv[e] * xh[i][e];
          ab[i][e] += dv[e];
        }
      }
    }
    const float gm = wave_sum(s1) / C, gxm = wave_sum(s2) / C;
    bf16_t* rr = dres_out + (size_t)row * C;
#pragma unroll
    for (int i = 0; i < MAXCH; ++i) {
      int c = 4 * (lane + 64 * i);
      if (c < C) {
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = rstd * (gg[i][e] - gm - xh[i][e] * gxm);
        if (has_res) {
          o[0] += lo_f(ru[i].x); o[1] += hi_f(ru[i].x); o[2] += lo_f(ru[i].y); o[3] += hi_f(ru[i].y);
        }
        const uint2 ou = make_uint2(pack2(o[0], o[1]), pack2(o[2], o[3]));
        *reinterpret_cast<uint2*>(rr + c) = ou;
        // the stored (rounded) values, so the sum matches what consumers read
        ar[i][0] += lo_f(ou.x); ar[i][1] += hi_f(ou.x); ar[i][2] += lo_f(ou.y); ar[i][3] += hi_f(ou.y);
      }
    }
#pragma unroll
    for (int i = 0; i < MAXCH; ++i) {
      xu[i] = xn[i];
      du[i] = dn[i];
      ru[i] = rn[i];
    }
    mean = mean_n;
    rstd = rstd_n;
  }
  // combine the four waves' partial sums in a fixed order; the block's row of
  // partials is [dw | db | column sum of the residual gradient], 3*C floats
  for (int pass = 0; pass < 3; ++pass) {
#pragma unroll
    for (int i = 0; i < MAXCH; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        red[wave][(i * 64 + lane) * 4 + e] = pass == 0 ? aw[i][e] : (pass == 1 ? ab[i][e] : ar[i][e]);
    __syncthreads();
    float* dst = part + (size_t)blockIdx.x * 3 * C + pass * C;
    for (int c = threadIdx.x; c < C; c += 256) {
      // channel c lives at chunk i = (c/4)/64, lane (c/4)%64, element c%4
      int cq = c >> 2, i = cq >> 6, l = cq & 63, e = c & 3;
      int k = (i * 64 + l) * 4 + e;
      dst[c] = red[0][k] + red[1][k] + red[2][k] + red[3][k];
    }
    __syncthreads();
  }
}

// the residual addition alone: out = bf16(res + x), 4 elements per thread
__global__ void residual_add_kernel(const bf16_t* __restrict__ res, const bf16_t* __restrict__ x,
                                    bf16_t* __restrict__ out, long n) {
  const long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= n) return;
  *reinterpret_cast<uint2*>(out + i) =
      add_rows(*reinterpret_cast<const uint2*>(res + i), *reinterpret_cast<const uint2*>(x + i));
}

template <int MAXCH>
hipError_t fwd_t(const bf16_t* x, const Slices& sl, const float* bias, const bf16_t* res, bf16_t* xsum, const float* w,
                 const float* b, bf16_t* y, float* mean, float* rstd, int rows, int C, float eps, hipStream_t s,
                 bf16_t* xcopy) {
  const dim3 grid((rows + 3) / 4), block(256);
  if (sl.n > 0)
    hipLaunchKernelGGL((ln_fwd_kernel<MAXCH, SRC_SLICES>), grid, block, 0, s, nullptr, sl, bias, res, xsum, w, b, y,
                       mean, rstd, rows, C, eps, xcopy);
  else if (res)
    hipLaunchKernelGGL((ln_fwd_kernel<MAXCH, SRC_RES>), grid, block, 0, s, x, sl, nullptr, res, xsum, w, b, y, mean,
                       rstd, rows, C, eps, xcopy);
  else
    hipLaunchKernelGGL((ln_fwd_kernel<MAXCH, SRC_X>), grid, block, 0, s, x, sl, nullptr, nullptr, nullptr, w, b, y,
                       mean, rstd, rows, C, eps, xcopy);
  return hipGetLastError();
}

hipError_t fwd(const bf16_t* x, const Slices& sl, const float* bias, const bf16_t* res, bf16_t* xsum, const float* w,
               const float* b, bf16_t* y, float* mean, float* rstd, int rows, int C, float eps, hipStream_t s,
               bf16_t* xcopy) {
  if (C <= 256) return fwd_t<1>(x, sl, bias, res, xsum, w, b, y, mean, rstd, rows, C, eps, s, xcopy);
  if (C <= 512) return fwd_t<2>(x, sl, bias, res, xsum, w, b, y, mean, rstd, rows, C, eps, s, xcopy);
  if (C <= 768) return fwd_t<3>(x, sl, bias, res, xsum, w, b, y, mean, rstd, rows, C, eps, s, xcopy);
  if (C <= 1024) return fwd_t<4>(x, sl, bias, res, xsum, w, b, y, mean, rstd, rows, C, eps, s, xcopy);
  if (C <= 2048) return fwd_t<8>(x, sl, bias, res, xsum, w, b, y, mean, rstd, rows, C, eps, s, xcopy);
  return hipErrorInvalidValue;
}

template <int MAXCH>
hipError_t bwd_t(const bf16_t* dy, const Slices& sl, const bf16_t* x, const float* mean, const float* rstd,
                 const float* w, const bf16_t* dres_in, bf16_t* dres_out, int has_res, float* part, int rows, int C,
                 hipStream_t s) {
  const dim3 grid(layernorm_bwd_blocks(rows)), block(256);
  if (sl.n > 0)
    hipLaunchKernelGGL((ln_bwd_kernel<MAXCH, true>), grid, block, 0, s, nullptr, sl, x, mean, rstd, w, dres_in,
                       dres_out, has_res, part, rows, C);
  else
    hipLaunchKernelGGL((ln_bwd_kernel<MAXCH, false>), grid, block, 0, s, dy, sl, x, mean, rstd, w, dres_in, dres_out,
                       has_res, part, rows, C);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_add_layernorm_fwd(const bf16_t* x, const bf16_t* res, bf16_t* xsum, const float* w, const float* b,
                                    bf16_t* y, float* mean, float* rstd, int rows, int C, float eps, hipStream_t s) {
  if (C % 4 || (res && !xsum)) return hipErrorInvalidValue;
  return fwd(x, {nullptr, 0}, nullptr, res, xsum, w, b, y, mean, rstd, rows, C, eps, s, nullptr);
}

hipError_t launch_slices_layernorm_fwd(const Slices& sl, const float* bias, const bf16_t* res, bf16_t* xsum,
                                       const float* w, const float* b, bf16_t* y, float* mean, float* rstd, int rows,
                                       int C, float eps, hipStream_t s, bf16_t* xcopy) {
  if (C % 4 || sl.n < 1 || !sl.p || !bias || !res || !xsum) return hipErrorInvalidValue;
  return fwd(nullptr, sl, bias, res, xsum, w, b, y, mean, rstd, rows, C, eps, s, xcopy);
}

hipError_t launch_layernorm_fwd(const bf16_t* x, const float* w, const float* b, bf16_t* y, float* mean,
                                float* rstd, int rows, int C, float eps, hipStream_t s, bf16_t* xcopy) {
  if (C % 4) return hipErrorInvalidValue;
  return fwd(x, {nullptr, 0}, nullptr, nullptr, nullptr, w, b, y, mean, rstd, rows, C, eps, s, xcopy);
}

hipError_t launch_residual_add(const bf16_t* res, const bf16_t* x, bf16_t* out, long n, hipStream_t s) {
  if (n % 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(residual_add_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, s, res, x, out, n);
  return hipGetLastError();
}

// Four waves per block, each block writing one row of partial sums. Many rows:
// 4 rows per wave and at most 768 blocks, three per CU, which is what the
// backward's registers (two rows' inputs in flight per wave) let stay
// resident at once. Fewer than 4096 rows: one row per wave up to 256 blocks,
// since a wave's rows follow one another (999 rows of 768: 7.7 -> 4.6 us).
int layernorm_bwd_blocks(int rows) {
  int n = std::max((rows + 15) / 16, std::min((rows + 3) / 4, 256));
  return n < 768 ? (n < 1 ? 1 : n) : 768;
}

hipError_t launch_layernorm_bwd(const bf16_t* dy, const Slices& sl, const bf16_t* x, const float* mean,
                                const float* rstd, const float* w, const bf16_t* dres_in, bf16_t* dres_out,
                                int has_res, float* part, int rows, int C, hipStream_t s) {
  if (C % 4) return hipErrorInvalidValue;
  if (C <= 256) return bwd_t<1>(dy, sl, x, mean, rstd, w, dres_in, dres_out, has_res, part, rows, C, s);
  if (C <= 512) return bwd_t<2>(dy, sl, x, mean, rstd, w, dres_in, dres_out, has_res, part, rows, C, s);
  if (C <= 768) return bwd_t<3>(dy, sl, x, mean, rstd, w, dres_in, dres_out, has_res, part, rows, C, s);
  if (C <= 1024) return bwd_t<4>(dy, sl, x, mean, rstd, w, dres_in, dres_out, has_res, part, rows, C, s);
  if (C <= 2048) return bwd_t<8>(dy, sl, x, mean, rstd, w, dres_in, dres_out, has_res, part, rows, C, s);
  return hipErrorInvalidValue;
}
