// device.hpp -- device-side helpers shared by the kernel sources.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>

#include "kernels.hpp"

namespace huge2 {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }
constexpr int lcm3(int a, int b, int c) {
  return (a / gcd_c(a, b) * b) / gcd_c(a / gcd_c(a, b) * b, c) * c;
}
// f(integral_constant<int, u>) for u = 0 .. N-1, unrolled at compile time.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unroll_stages(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    unroll_stages<N, I + 1>(f);
  }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 16-byte store of output data that nothing in the kernel reads back, with
// the non-temporal (streaming) cache policy.
__device__ __forceinline__ void store_stream16(void* p, uint4 v) {
  const u32x4 t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, (u32x4*)p);
}

// Workgroups are dealt to the 8 XCDs round-robin (id mod 8).  Map them so
// that each XCD runs one contiguous run of the work list: neighbouring
// tiles share input rows and weight blocks, which then stay in that XCD's L2.
__device__ __forceinline__ int xcd_remap(int b, int g) {
  const int g8 = (g + 7) >> 3, r = g & 7, x = b & 7, y = b >> 3;
  if (r == 0 || x < r) return x * g8 + y;
  return r * g8 + (x - r) * (g8 - 1) + y;
}

// The epilogue's elementwise function (huge2_activation): 0 none, 1 max(v, 0),
// 2 tanh(v).  act is uniform over the launch.
__device__ __forceinline__ float activate(float v, int act) {
  return act == 1 ? fmaxf(v, 0.f) : act == 2 ? tanhf(v) : v;
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  // v_cvt_pk_bf16_f32: round to nearest even, NaN stays a (quiet) NaN
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// Two floats to bf16 (round to nearest even) in one 32-bit word, lo in the
// low half: one v_cvt_pk_bf16_f32 with both sources.
__device__ __forceinline__ uint32_t pack_bf16x2_rne(float lo, float hi) {
  typedef float f2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
  const f2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2_t));
}

__device__ __forceinline__ uint32_t fast_div(uint32_t v, uint32_t mul, uint32_t shift) {
  return (uint32_t)(((uint64_t)v * mul) >> shift);
}
template <typename T>
__device__ __forceinline__ float to_f32(T v) {
  if constexpr (std::is_same<T, uint16_t>::value)
    return __uint_as_float((uint32_t)v << 16);
  else
    return __uint_as_float(v);
}

// Decomposition of a segment pixel index into image, output and input coordinates.
struct PixelPos {
  int img, oh, ow, ih, iw;
};
// Bias entry of GEMM column ch (the 1x1-input product forms: bias_div
// columns per entry, or entries repeating every bias_mod columns).
__device__ __forceinline__ int bias_index(const GemmArgs& a, int ch) {
  const int bc = ch / a.bias_div;
  return a.bias_mod > 0 ? bc % a.bias_mod : bc;
}
__device__ __forceinline__ PixelPos pixel_pos(const SegDev& sg, const uint32_t* ptab, int m) {
  PixelPos p;
  uint32_t j = (uint32_t)m;
  if (sg.ptab >= 0) {
    const uint32_t img = fast_div(j, sg.div_mul[2], sg.div_shift[2]);
    const uint32_t e = ptab[sg.ptab + (int)(j - img * (uint32_t)sg.per_img)];
    p.img = (int)img;
    p.oh = (int)(e >> 16);
    p.ow = (int)(e & 0xffffu);
    p.ih = sg.in0_h + p.oh;
    p.iw = sg.in0_w + p.ow;
    return p;
  }
  uint32_t t = fast_div(j, sg.div_mul[0], sg.div_shift[0]);
  const int a_w = (int)(j - t * (uint32_t)sg.qn_w);
  j = t;
  t = fast_div(j, sg.div_mul[1], sg.div_shift[1]);
  const int a_h = (int)(j - t * (uint32_t)sg.qn_h);
  j = t;
  t = fast_div(j, sg.div_mul[2], sg.div_shift[2]);
  const uint32_t iph = j - t * (uint32_t)sg.nphase;
  p.img = (int)t;
  const uint32_t iph_h = fast_div(iph, sg.div_mul[3], sg.div_shift[3]);
  const int iph_w = (int)(iph - iph_h * (uint32_t)sg.nphase_w);
  const int qh = sg.q0_h + a_h, qw = sg.q0_w + a_w;
  p.oh = sg.phase0_h + (int)iph_h + sg.out_step_h * qh;
  p.ow = sg.phase0_w + iph_w + sg.out_step_w * qw;
  p.ih = sg.in0_h + sg.in_dphase_h * (int)iph_h + sg.in_step_h * qh;
  p.iw = sg.in0_w + sg.in_dphase_w * iph_w + sg.in_step_w * qw;
  return p;
}

// Epilogue: bias, rounding, and the scatter of a wave's TP x TC blocks of
// 32 x 32 results (pixels from pix0, output channels from ch0) to the
// interleaved output positions of their phase.  32x32 MFMA result layout:
// lane l holds column l % 32 and rows 8*(r/4) + 4*(l/32) + (r%4), r = 0..15.
// NCHW output puts pixels on the columns (a channel's stores coalesce along
// the lanes); NHWC output puts pixels on the rows.
// sb: bias by output channel (sb[ch], staged in LDS, zeros without bias):
// reading it from global memory between the stores would make every load
// wait for the stores issued before it.
template <bool BF16, bool NCHW_OUT, int TP, int TC>
__device__ __forceinline__ void store_tile(const GemmArgs& a, const SegDev& sg, int m_end, void* y,
                                           const f32x16 (&acc)[TP][TC], int pix0, int ch0,
                                           int lane, const float* sb) {
  const int hw_o = a.ho * a.wo;
  // the bias values are read from LDS up front: an LDS read between the
  // global stores would wait for its own latency element by element
  if constexpr (!NCHW_OUT) {
    float bv[TC];
#pragma unroll
    for (int j = 0; j < TC; ++j) {
      const int ch = ch0 + 32 * j + (lane & 31);
      bv[j] = ch < a.cout ? sb[ch] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < TP; ++i) {
      // the 16 rows' positions before their stores: a table lookup issued
      // behind stores would wait for them (the memory counter is in order)
      int pixr[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = pix0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const PixelPos p = pixel_pos(sg, a.ptab, m < m_end ? m : pix0);
        pixr[r] = m < m_end ? (p.img * a.ho + p.oh) * a.wo + p.ow : -1;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int pix = pixr[r];
        if (pix < 0) continue;
#pragma unroll
        for (int j = 0; j < TC; ++j) {
          const int ch = ch0 + 32 * j + (lane & 31);
          if (ch >= a.cout) continue;
          const float v = activate(acc[i][j][r] + bv[j], a.act);
          const size_t off = (size_t)pix * a.cout + ch;
          if constexpr (BF16)
            ((uint16_t*)y)[off] = f32_to_bf16_rne(v);
          else
            ((float*)y)[off] = v;
        }
      }
    }
  } else {
    size_t base[TP];
    bool ok[TP];
#pragma unroll
    for (int i = 0; i < TP; ++i) {
      const int m = pix0 + 32 * i + (lane & 31);
      ok[i] = m < m_end;
      const PixelPos p = pixel_pos(sg, a.ptab, ok[i] ? m : pix0);
      base[i] = (size_t)p.img * a.cout * hw_o + (size_t)p.oh * a.wo + p.ow;
    }
#pragma unroll
    for (int j = 0; j < TC; ++j) {
      float bv[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int ch = ch0 + 32 * j + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        bv[r] = ch < a.cout ? sb[ch] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < TP; ++i) {
        if (!ok[i]) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int ch = ch0 + 32 * j + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (ch >= a.cout) continue;
          const float v = activate(acc[i][j][r] + bv[r], a.act);
          const size_t off = base[i] + (size_t)ch * hw_o;
          if constexpr (BF16)
            ((uint16_t*)y)[off] = f32_to_bf16_rne(v);
          else
            ((float*)y)[off] = v;
        }
      }
    }
  }
}

// fp32 operands are multiplied by 2^24 before they are split into bf16 parts:
// the last bit of any float (2^-149 and up) then lies above bf16's smallest
// normal number and no part underflows.  Operands from 2^104 and sums from 2^76 to
// 2^80 are too large instead, and such sums are formed again (mfma_f32_step).
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-24f, kSumUnscale = 0x1p-48f;

// Eight floats, scaled, as three bf16 parts, x = x1 + x2 + x3: each part rounds
// what the ones before it left over, to nearest even, so with 8 bits a part the
// sum holds all 24, and part k is at most 2^-9k of x.
struct Split8 {
  uint4 p[3];
};
__device__ __forceinline__ Split8 split8(uint4 lo, uint4 hi) {
  const uint32_t u[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(u[e]) * kSplitScale;
  Split8 s;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      w[e] = pack_bf16x2_rne(v[2 * e], v[2 * e + 1]);
      if (k < 2) {
        v[2 * e] -= __uint_as_float(w[e] << 16);
        v[2 * e + 1] -= __uint_as_float(w[e] & 0xffff0000u);
      }
    }
    s.p[k] = make_uint4(w[0], w[1], w[2], w[3]);
  }
  return s;
}

// Weight of the three-part fp32 packing: the sum of its parts, which is exact,
// or, behind a NaN in the first plane, the bits in the other two.
__device__ __forceinline__ float join_weight(uint32_t h0, uint32_t h1, uint32_t h2) {
  if ((h0 & 0x7fffu) > 0x7f80u) return __uint_as_float(h1 << 16 | h2);
  return (__uint_as_float(h2 << 16) + __uint_as_float(h1 << 16) + __uint_as_float(h0 << 16)) *
         kSplitUnscale;
}
// The one at tap block byte slot_b, channel ch, input channel c.
__device__ __forceinline__ float split_weight(const char* wp, size_t plane_b, uint32_t slot_b,
                                              int cin_pad, int ch, int c) {
  const size_t at = slot_b + ((size_t)(ch >> 5) * (cin_pad >> 5) + (c >> 5)) * 2048u +
                    ((c >> 3) & 1) * 1024u + (((c >> 4) & 1) * 32 + (ch & 31)) * 16u + (c & 7) * 2u;
  uint32_t h[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) h[p] = *(const uint16_t*)(wp + p * plane_b + at);
  return join_weight(h[0], h[1], h[2]);
}

// Sums that the parts cannot give (an operand or a sum that is or becomes
// infinite, NaN) are formed again with the fp32 matrix instruction, a wave's
// whole tile at a time and without the pipeline of the ordinary path: 512 -> 256
// 4x4 on 64 x 8 x 8 takes 0.50 ms when every sum is one of them (0.09 when none
// is), and 0.37 with one infinite input.  One lane's term by term sums, 25.6 and
// 11.9 ms there, are left for NaN next to weights that are not finite, whose
// products with the zeros read outside the input must not count.
__device__ __forceinline__ bool finite(float v) { return fabsf(v) <= 3.402823466e38f; }

// acc += eight K elements per lane half of x rows times w rows, in fp32.
template <bool W_ROWS, int TP, int TC>
__device__ __forceinline__ void mfma_f32_step(f32x16 (&acc)[TP][TC], const float (&x)[TP][8],
                                              const float (&w)[TC][8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TC; ++j)
        acc[i][j] = W_ROWS ? __builtin_amdgcn_mfma_f32_32x32x2f32(w[j][e], x[i][e], acc[i][j], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][e], w[j][e], acc[i][j], 0, 0, 0);
}
__device__ __forceinline__ void unpack4(uint4 u, float* v) {
  v[0] = __uint_as_float(u.x);
  v[1] = __uint_as_float(u.y);
  v[2] = __uint_as_float(u.z);
  v[3] = __uint_as_float(u.w);
}
// A lane's eight weights of the three planes; true if all are finite.
__device__ __forceinline__ bool join_parts(const uint4 (&h)[3], float (&v)[8]) {
  bool all = true;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    uint32_t b[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const uint32_t u = e < 2 ? h[p].x : e < 4 ? h[p].y : e < 6 ? h[p].z : h[p].w;
      b[p] = e & 1 ? u >> 16 : u & 0xffffu;
    }
    v[e] = join_weight(b[0], b[1], b[2]);
    all &= finite(v[e]);
  }
  return all;
}

}  // namespace huge2
