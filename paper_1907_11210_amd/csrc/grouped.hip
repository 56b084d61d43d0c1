// grouped.hip -- grouped and depthwise convolutions (section 3.2.3's depthwise
// case; PyTorch's groups): the direct kernels.
#include <algorithm>
#include <type_traits>

#include "device.hpp"
#include "kernels.hpp"

namespace huge2 {

// ---------------------------------------------------------------------------
// Grouped and depthwise convolutions (see GrArgs).
template <typename T>
__global__ __launch_bounds__(256) void grouped_kernel(GrArgs a, long long total) {
  const T* __restrict__ x = (const T*)a.x;
  const T* __restrict__ w = (const T*)a.w;
  const int cig = a.cin / a.groups, cog = a.cout / a.groups;
  for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long long)gridDim.x * blockDim.x) {
    long long t = idx;
    int k, oh, ow, n;
    if (a.nhwc) {
      k = (int)(t % a.cout);
      t /= a.cout;
      ow = (int)(t % a.wo);
      t /= a.wo;
      oh = (int)(t % a.ho);
      n = (int)(t / a.ho);
    } else {
      ow = (int)(t % a.wo);
      t /= a.wo;
      oh = (int)(t % a.ho);
      t /= a.ho;
      k = (int)(t % a.cout);
      n = (int)(t / a.cout);
    }
    const int g = k / cog, kg = k - g * cog, c0 = g * cig;
    float acc = 0.f;
    for (int m = 0; m < a.r; ++m) {
      int ih;
      if (a.transposed) {
        const int num = oh + a.pad_h - m * a.dil_h;  // = ih * stride_h on the phase's taps
        if (num < 0 || num % a.stride_h != 0) continue;
        ih = num / a.stride_h;
      } else {
        ih = oh * a.stride_h - a.pad_h + m * a.dil_h;
      }
      if (ih < 0 || ih >= a.h) continue;
      for (int q = 0; q < a.s; ++q) {
        int iw;
        if (a.transposed) {
          const int num = ow + a.pad_w - q * a.dil_w;
          if (num < 0 || num % a.stride_w != 0) continue;
          iw = num / a.stride_w;
        } else {
          iw = ow * a.stride_w - a.pad_w + q * a.dil_w;
        }
        if (iw < 0 || iw >= a.w_) continue;
        for (int ci = 0; ci < cig; ++ci) {
          const int c = c0 + ci;
          const size_t xi = a.nhwc ? (((size_t)n * a.h + ih) * a.w_ + iw) * a.cin + c
                                   : (((size_t)n * a.cin + c) * a.h + ih) * a.w_ + iw;
          const size_t wi = a.transposed ? (((size_t)c * cog + kg) * a.r + m) * a.s + q
                                         : (((size_t)k * cig + ci) * a.r + m) * a.s + q;
          acc = fmaf(to_f32(x[xi]), to_f32(w[wi]), acc);
        }
      }
    }
    const float v = activate(acc + (a.bias ? a.bias[k] : 0.f), a.act);
    if constexpr (std::is_same<T, uint16_t>::value)
      ((uint16_t*)a.y)[idx] = f32_to_bf16_rne(v);
    else
      ((float*)a.y)[idx] = v;
  }
}

hipError_t launch_grouped(const GrArgs& a, int dtype, hipStream_t stream) {
  const long long total = (long long)a.n * a.cout * a.ho * a.wo;
  const long long want = (total + 255) / 256;
  const int grid = (int)(want < 1048576 ? want : 1048576);
  if (total == 0) return hipSuccess;
  if (dtype == 1)
    hipLaunchKernelGGL(grouped_kernel<uint16_t>, dim3(grid), dim3(256), 0, stream, a, total);
  else
    hipLaunchKernelGGL(grouped_kernel<uint32_t>, dim3(grid), dim3(256), 0, stream, a, total);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Depthwise convolutions (see DwArgs): one input channel per output channel,
// so there is no contraction for the matrix cores and the bound is HBM (x
// once, y once).  The grouped kernel above reads one element per tap and
// output with 64-bit divisions in front: 114 us at 8 x 64 x 64 x 256 bf16 NHWC,
// 3x3, dilation 4 (0.29 TB/s of compulsory bytes).

// VEC channels as packed words, widened one channel at a time.
template <typename T, int VEC>
struct DwVec;
template <>
struct DwVec<uint16_t, 8> {
  uint4 v;
  __device__ __forceinline__ void load(const uint16_t* p) { v = *(const uint4*)p; }
  __device__ __forceinline__ float at(int e) const {
    const uint32_t u = e < 2 ? v.x : e < 4 ? v.y : e < 6 ? v.z : v.w;
    return __uint_as_float(e & 1 ? u & 0xffff0000u : u << 16);
  }
};
template <>
struct DwVec<uint32_t, 4> {
  uint4 v;
  __device__ __forceinline__ void load(const uint32_t* p) { v = *(const uint4*)p; }
  __device__ __forceinline__ float at(int e) const {
    return __uint_as_float(e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w);
  }
};
template <typename T>
struct DwVec<T, 1> {
  T v;
  __device__ __forceinline__ void load(const T* p) { v = *p; }
  __device__ __forceinline__ float at(int) const { return to_f32(v); }
};

template <typename T, int VEC>
__device__ __forceinline__ void dw_store(const DwArgs& a, size_t off, int k0, float (&acc)[VEC]) {
#pragma unroll
  for (int e = 0; e < VEC; ++e)
    acc[e] = activate(acc[e] + (a.bias ? a.bias[k0 + e] : 0.f), a.act);
  if constexpr (std::is_same<T, uint16_t>::value && VEC == 8) {
    *(uint4*)((uint16_t*)a.y + off) =
        make_uint4(pack_bf16x2_rne(acc[0], acc[1]), pack_bf16x2_rne(acc[2], acc[3]),
                   pack_bf16x2_rne(acc[4], acc[5]), pack_bf16x2_rne(acc[6], acc[7]));
  } else if constexpr (VEC == 4) {
    *(float4*)((float*)a.y + off) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  } else if constexpr (std::is_same<T, uint16_t>::value) {
    ((uint16_t*)a.y)[off] = f32_to_bf16_rne(acc[0]);
  } else {
    ((float*)a.y)[off] = acc[0];
  }
}

// Thread index -> image, row chain, column, first output channel.
struct DwPos {
  int img, chain, ow, k0;
};
__device__ __forceinline__ DwPos dw_index(const DwArgs& a, uint32_t idx) {
  const uint32_t t0 = fast_div(idx, a.mul[0], a.shift[0]);
  const int i0 = (int)(idx - t0 * a.dv[0]);
  const uint32_t t1 = fast_div(t0, a.mul[1], a.shift[1]);
  const int i1 = (int)(t0 - t1 * a.dv[1]);
  const uint32_t t2 = fast_div(t1, a.mul[2], a.shift[2]);
  const int i2 = (int)(t1 - t2 * a.dv[2]);
  DwPos p;
  p.img = (int)t2;
  p.chain = a.nhwc ? i2 : i1;
  p.ow = a.nhwc ? i1 : i0;
  p.k0 = a.nhwc ? i0 * a.vec : i2;
  return p;
}

// 3x3 conv.  A thread computes TR outputs of one column, rows oh0 + j * step,
// whose input rows lie dil_h apart: output j takes rows j * RATIO .. + 2 of
// the chain, so (TR - 1) * RATIO + 3 rows of three columns serve 9 TR
// products, each input loaded and widened once per chain.  All loads are
// issued up front at positions clamped into the input; products outside the
// input are skipped (not multiplied by zero), in the tap order of the grouped
// kernel, so the sums are the same bit for bit.  Blocks are mapped so that an
// XCD's run of neighbouring rows shares its L2.
template <typename T, int VEC, int TR, int RATIO>
__global__ __launch_bounds__(256) void depthwise3_kernel(DwArgs a) {
  constexpr int NR = (TR - 1) * RATIO + 3;
  const uint32_t idx = (uint32_t)xcd_remap(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  if (idx >= a.total) return;
  const DwPos at = dw_index(a, idx);
  const int img = at.img, chain = at.chain, ow = at.ow, k0 = at.k0;
  const int b = (int)fast_div((uint32_t)chain, a.mul[3], a.shift[3]);
  const int oh0 = b * TR * a.step + (chain - b * a.step);
  if (oh0 >= a.ho) return;
  const int ih0 = oh0 * a.stride_h - a.pad_h, iw0 = ow * a.stride_w - a.pad_w;
  const int xc = VEC == 1 ? (int)fast_div((uint32_t)k0, a.mul[4], a.shift[4]) : k0;
  // element strides of a row and a column of x
  const int xw = a.nhwc ? a.cin : 1, xh = a.w_ * xw;
  const T* const xp = (const T*)a.x + (a.nhwc ? (size_t)img * a.h * xh + xc
                                              : ((size_t)img * a.cin + xc) * a.h * xh);
  const T* const wp = (const T*)a.w + k0;
  bool cok[3];
  int coff[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int iw = iw0 + q * a.dil_w;
    cok[q] = (unsigned)iw < (unsigned)a.w_;
    coff[q] = min(max(iw, 0), a.w_ - 1) * xw;
  }
  DwVec<T, VEC> wv[9], xv[NR][3];
#pragma unroll
  for (int t = 0; t < 9; ++t) wv[t].load(wp + t * a.cout);
#pragma unroll
  for (int t = 0; t < NR; ++t) {
    const int row = min(max(ih0 + t * a.dil_h, 0), a.h - 1) * xh;
#pragma unroll
    for (int q = 0; q < 3; ++q) xv[t][q].load(xp + row + coff[q]);
  }
  float acc[TR][VEC];
#pragma unroll
  for (int j = 0; j < TR; ++j)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[j][e] = 0.f;
#pragma unroll
  for (int t = 0; t < NR; ++t) {
    if ((unsigned)(ih0 + t * a.dil_h) >= (unsigned)a.h) continue;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      if (!cok[q]) continue;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float v = xv[t][q].at(e);
#pragma unroll
        for (int j = 0; j < TR; ++j) {
          const int m = t - j * RATIO;
          if (m >= 0 && m < 3) acc[j][e] = fmaf(v, wv[3 * m + q].at(e), acc[j][e]);
        }
      }
    }
  }
  const size_t yw = a.nhwc ? a.cout : 1, yh = a.wo * yw;
  const size_t y0 = (a.nhwc ? (size_t)img * a.ho * yh + k0
                            : ((size_t)img * a.cout + k0) * a.ho * yh) + ow * yw;
#pragma unroll
  for (int j = 0; j < TR; ++j) {
    const int oh = oh0 + j * a.step;
    if (oh < a.ho) dw_store<T, VEC>(a, y0 + (size_t)oh * yh, k0, acc[j]);
  }
}

// Any kernel size, stride and dilation, conv or transposed conv: one output
// position of VEC channels per thread, over the taps that reach it.  A
// transposed output o sums the taps m of its phase, m = m0, m0 + mstep, ...
// with (o + pad - m * dil) divisible by the stride, reading input (o + pad -
// m * dil) / stride (section 3.1's sub-kernel of the phase).
template <typename T, int VEC>
__global__ __launch_bounds__(256) void depthwise_kernel(DwArgs a) {
  const uint32_t idx = (uint32_t)xcd_remap(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  if (idx >= a.total) return;
  const DwPos at = dw_index(a, idx);
  const int img = at.img, oh = at.chain, ow = at.ow, k0 = at.k0;
  const int xc = VEC == 1 ? (int)fast_div((uint32_t)k0, a.mul[4], a.shift[4]) : k0;
  const int xw = a.nhwc ? a.cin : 1, xh = a.w_ * xw;
  const T* const xp = (const T*)a.x + (a.nhwc ? (size_t)img * a.h * xh + xc
                                              : ((size_t)img * a.cin + xc) * a.h * xh);
  const T* const wp = (const T*)a.w + k0;
  int m0 = 0, q0 = 0, ih0 = oh * a.stride_h - a.pad_h, iw0 = ow * a.stride_w - a.pad_w;
  if (a.transposed) {
    // the phase's first tap: at most mstep candidates, the division exact there
    auto first = [](int v, int dil, int stride, int mstep, int r, uint32_t mul, uint32_t shift,
                    int* m, int* in) {
      const int lift = stride * dil;  // a multiple of the stride that makes v - m * dil positive
      for (*m = 0; *m < mstep; ++*m) {
        const int u = v - *m * dil + lift * mstep;
        const int d = (int)fast_div((uint32_t)u, mul, shift);
        if (d * stride == u) {
          *in = d - dil * mstep;
          return;
        }
      }
      *m = r;  // no tap reaches this phase
    };
    first(oh + a.pad_h, a.dil_h, a.stride_h, a.mstep_h, a.r, a.sh_mul, a.sh_shift, &m0, &ih0);
    first(ow + a.pad_w, a.dil_w, a.stride_w, a.mstep_w, a.s, a.sw_mul, a.sw_shift, &q0, &iw0);
  }
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
  for (int m = m0, ih = ih0; m < a.r; m += a.mstep_h, ih += a.istep_h) {
    if ((unsigned)ih >= (unsigned)a.h) continue;
#pragma unroll 4
    for (int q = q0, iw = iw0; q < a.s; q += a.mstep_w, iw += a.istep_w) {
      if ((unsigned)iw >= (unsigned)a.w_) continue;
      DwVec<T, VEC> xv, wv;
      xv.load(xp + (size_t)ih * xh + iw * xw);
      wv.load(wp + (size_t)(m * a.s + q) * a.cout);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] = fmaf(xv.at(e), wv.at(e), acc[e]);
    }
  }
  const size_t yw = a.nhwc ? a.cout : 1, yh = a.wo * yw;
  dw_store<T, VEC>(a, (a.nhwc ? (size_t)img * a.ho * yh + k0
                              : ((size_t)img * a.cout + k0) * a.ho * yh) + ow * yw + oh * yh,
                   k0, acc);
}

constexpr int kDwRowsVec = 4;   // outputs per thread of the 3x3 kernel, 16-byte channel pieces
constexpr int kDwRowsOne = 8;   // and one channel per thread
// Chains need outputs for this many whole ones (pieces; one channel), times the
// ratio: below, the kernel of one position per thread has more threads to hide
// its loads (3x3 on 3 x 52 x 37 x 64, stride 2, bf16 NHWC, 2.7 thousand chains: 7.5 us
// in chains, 6.0 without).  Chains' time in units of the other's, means of 400
// layers: one channel, stride 1, 1.0 to 1.1 up to 32 thousand, 0.85 to 64, 0.7 to 128,
// 0.4 beyond; stride 2 1.2 to 1.5, 1.14, 0.6, 0.7; pieces, stride 1, 1.0 to 1.1 up to 64
// thousand, then 0.8 and 0.7; stride 2 1.1 to 1.3 up to 128.
constexpr long long kDwChainsVec = 64 << 10, kDwChainsOne = 32 << 10;

bool depthwise_shape(DwArgs* a, int dtype, bool pieces) {
  const int full = dtype == 1 ? 8 : 4;
  a->mult = a->cout / a->cin;
  a->vec = pieces && a->nhwc && a->mult == 1 && a->cin % full == 0 ? full : 1;
  auto gcd = [](int p, int q) {
    while (q) {
      const int t = p % q;
      p = q;
      q = t;
    }
    return p;
  };
  const int gh = gcd(a->stride_h, a->dil_h), gw = gcd(a->stride_w, a->dil_w);
  a->step = a->dil_h / gh;
  a->ratio = a->stride_h / gh;
  if (a->transposed) {
    a->mstep_h = a->stride_h / gh;
    a->mstep_w = a->stride_w / gw;
    a->istep_h = -(a->dil_h / gh);
    a->istep_w = -(a->dil_w / gw);
  } else {
    a->mstep_h = a->mstep_w = 1;
    a->istep_h = a->dil_h;
    a->istep_w = a->dil_w;
  }
  const int tr = a->vec > 1 ? kDwRowsVec : kDwRowsOne;
  a->rows3 = !a->transposed && a->r == 3 && a->s == 3 && a->ratio <= 2;
  if (a->chains == 0 ||
      (a->chains < 0 && (long long)a->n * (a->cout / a->vec) * a->ho * a->wo / tr <
                            (a->vec > 1 ? kDwChainsVec : kDwChainsOne) * a->ratio))
    a->rows3 = 0;
  const long long chains =
      a->rows3 ? (long long)a->step * ((a->ho + (long long)tr * a->step - 1) / ((long long)tr * a->step))
               : a->ho;
  const long long groups = a->cout / a->vec;
  const long long total = (long long)a->n * groups * chains * a->wo;
  // indices, coordinates and the divisions' dividends stay below 2^31
  const long long reach =
      std::max({(long long)a->ho + a->pad_h + 2ll * a->stride_h * a->dil_h * a->mstep_h,
                (long long)a->wo + a->pad_w + 2ll * a->stride_w * a->dil_w * a->mstep_w,
                (long long)(a->ho + 2ll * tr * a->step) * a->stride_h + 3ll * tr * a->dil_h,
                (long long)a->cin * a->h * a->w_, (long long)a->cout * a->r * a->s});
  if (total >= (1ll << 31) - 256 || chains >= (1ll << 30) || reach >= (1ll << 30)) return false;
  a->total = (uint32_t)total;
  const uint32_t d[5] = {(uint32_t)(a->nhwc ? groups : a->wo), (uint32_t)(a->nhwc ? a->wo : chains),
                         (uint32_t)(a->nhwc ? chains : groups), (uint32_t)a->step,
                         (uint32_t)a->mult};
  for (int k = 0; k < 5; ++k) {
    a->dv[k] = d[k];
    division_magic(d[k], &a->mul[k], &a->shift[k]);
  }
  division_magic((uint32_t)a->stride_h, &a->sh_mul, &a->sh_shift);
  division_magic((uint32_t)a->stride_w, &a->sw_mul, &a->sw_shift);
  return true;
}

template <typename T, int VEC, int TR>
static void launch_depthwise_t(const DwArgs& a, hipStream_t stream) {
  const dim3 grid((a.total + 255u) / 256u), block(256);
  if (a.rows3 && a.ratio == 1)
    hipLaunchKernelGGL((depthwise3_kernel<T, VEC, TR, 1>), grid, block, 0, stream, a);
  else if (a.rows3)
    hipLaunchKernelGGL((depthwise3_kernel<T, VEC, TR, 2>), grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((depthwise_kernel<T, VEC>), grid, block, 0, stream, a);
}

hipError_t launch_depthwise(const DwArgs& a, int dtype, hipStream_t stream) {
  if (a.total == 0) return hipSuccess;
  if (dtype == 1) {
    if (a.vec == 8)
      launch_depthwise_t<uint16_t, 8, kDwRowsVec>(a, stream);
    else
      launch_depthwise_t<uint16_t, 1, kDwRowsOne>(a, stream);
  } else {
    if (a.vec == 4)
      launch_depthwise_t<uint32_t, 4, kDwRowsVec>(a, stream);
    else
      launch_depthwise_t<uint32_t, 1, kDwRowsOne>(a, stream);
  }
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(256) void pack_depthwise_kernel(const T* __restrict__ w,
                                                             T* __restrict__ wp, int cout,
                                                             int taps) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= cout) return;
  for (int t = blockIdx.y; t < taps; t += gridDim.y)
    wp[(size_t)t * cout + k] = w[(size_t)k * taps + t];
}

hipError_t launch_pack_depthwise(const void* w, void* wp, int dtype, int cout, int taps,
                                 hipStream_t stream) {
  const dim3 grid((cout + 255) / 256, std::min(taps, 1024));
  if (dtype == 1)
    hipLaunchKernelGGL(pack_depthwise_kernel<uint16_t>, grid, dim3(256), 0, stream,
                       (const uint16_t*)w, (uint16_t*)wp, cout, taps);
  else
    hipLaunchKernelGGL(pack_depthwise_kernel<uint32_t>, grid, dim3(256), 0, stream,
                       (const uint32_t*)w, (uint32_t*)wp, cout, taps);
  return hipGetLastError();
}

}  // namespace huge2
