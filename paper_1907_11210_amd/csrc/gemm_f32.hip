// gemm_f32.hip -- the fp32 phase GEMM on the bf16 matrix cores.
#include "device.hpp"
#include "kernels.hpp"

namespace huge2 {

// ---------------------------------------------------------------------------
// Phase GEMM, fp32.  The fp32 MFMA runs at a sixteenth of the bf16 rate, so
// every operand is split exactly into three bf16 parts (split8, which scales
// it first; the weights once, when packed) and six of the nine products are
// summed in fp32, the smallest first; the three left out stay below 2^-25 of the
// product, under the rounding of the sums.  A workgroup of KS groups of PW x CW
// waves computes a tile of 32 PW TP pixels x 32 CW TC output channels; a stage
// is 32 input channels of one tap.  The pixel rows (128 bytes of fp32) are loaded two stages ahead,
// split between the MFMAs of the stage before and kept in LDS as three planes
// of bf16 rows, double buffered; each wave reads its weight fragments straight
// from the lane-ordered planes.  Six MFMAs per fragment pair make the LDS and
// L2 traffic per MFMA a third of the bf16 form's.  K groups (KS = 2: two waves
// per SIMD where a compute unit gets one workgroup) take halves of the
// workgroup's stages; group 1's sums are added to group 0's through LDS.
//
// An operand that is or becomes infinite has no finite parts: a sum that comes
// out infinite or NaN is formed again (mfma_f32_step).
template <int PW, int CW, int TP, int TC, int KS, bool NCHW_OUT, bool AP>
__global__ __launch_bounds__(PW * CW * KS * 64, 2) void phase_gemm_f32_kernel(GemmArgs a) {
  constexpr int NTA = PW * CW * KS * 64, NT = PW * CW * 64;
  constexpr int BM = 32 * PW * TP, BN = 32 * CW * TC;
  constexpr int ROWB = 64 + 16;  // LDS row of one part: 32 channels and a pad for distinct banks
  constexpr int PLANE_B = BM * ROWB, STAGE_B = 3 * PLANE_B;
  constexpr int NROW = BM * 4 / NT;  // rows per thread, 32 bytes of each
  static_assert(BM * 4 % NT == 0, "whole loads per thread");
  constexpr int NREG = TP * TC * 16;
  constexpr int RED_B = PW * CW * NREG * 64 * 4;  // one K group's sums
  constexpr int SMEM_B = KS * 2 * STAGE_B > RED_B ? KS * 2 * STAGE_B : RED_B;
  constexpr uint32_t OOB = 0x80000000u;
  __shared__ __attribute__((aligned(16))) char smem_all[SMEM_B];
  __shared__ float s_bias[BN];

  const int wave_all = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63, grp = KS > 1 ? wave_all / (PW * CW) : 0;
  const int wave = wave_all - grp * (PW * CW);
  const int tid = (int)threadIdx.x - grp * NT;
  char* const smem = smem_all + grp * 2 * STAGE_B;
  const int half = lane >> 5, row32 = lane & 31;
  const int wp_i = wave % PW, wc_i = wave / PW;
  const int work = xcd_remap(blockIdx.x, gridDim.x);
  const WorkDev wk = a.works[work];
  const SegDev sg = a.segs[wk.seg];
  const uint32_t plane_b = a.wp_bytes / 3u;
  const uint32_t slot_bytes = plane_b / (uint32_t)a.nslots;
  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, a.x_bytes, 0x00020000);
  const char* const wbase = (const char*)a.wp[sg.plan];
  __amdgpu_buffer_rsrc_t wr[3];
#pragma unroll
  for (int p = 0; p < 3; ++p)
    wr[p] = __builtin_amdgcn_make_buffer_rsrc((void*)(wbase + (size_t)p * plane_b), 0, plane_b,
                                              0x00020000);

  // this thread's pixel rows: bytes [32 q, 32 q + 32) of rows tid / 4 + (NT / 4) i
  const int q = tid & 3;
  int p_ih[NROW], p_iw[NROW];
  uint32_t p_base[NROW];
#pragma unroll
  for (int i = 0; i < NROW; ++i) {
    const int m = min(wk.m0 + tid / 4 + (NT / 4) * i, wk.m1 - 1);
    const PixelPos p = pixel_pos(sg, a.ptab, m);
    p_ih[i] = p.ih;
    p_iw[i] = p.iw;
    p_base[i] = (((uint32_t)p.img * (uint32_t)a.h + (uint32_t)p.ih) * (uint32_t)a.w +
                 (uint32_t)p.iw) * (uint32_t)a.cin * 4u + 32u * q;
  }
  uint32_t w_off[TC];
#pragma unroll
  for (int j = 0; j < TC; ++j)
    w_off[j] = (uint32_t)((wk.n0 / 32 + wc_i * TC + j) * 32 * a.cin_pad * 2 + lane * 16);

  const float* const bias = a.bias[sg.plan];
  for (int t = threadIdx.x; t < BN; t += NTA)
    s_bias[t] = (bias && wk.n0 + t < a.cout) ? bias[bias_index(a, wk.n0 + t)] : 0.f;

  // stages (channel block outer, tap inner) of this workgroup's K slice and
  // of this group's share of it
  const int ntaps = wk.tap_count;
  const int cblocks = a.cin_pad / 32;
  const int tail_c = a.cin - (cblocks - 1) * 32;
  const int total = ntaps * cblocks;
  const int s_w0 = (int)((long long)wk.ks * total / a.ksplit);
  const int s_w1 = (int)((long long)(wk.ks + 1) * total / a.ksplit);
  const int per = (s_w1 - s_w0 + KS - 1) / KS;
  const int s_lo = min(s_w0 + grp * per, s_w1);
  const int nsteps = min(s_lo + per, s_w1) - s_lo;  // this group's; every group runs `per`

  struct Iter {
    int t, th, tw, cb;
  };
  Iter ia;
  ia.cb = ntaps > 0 ? s_lo / ntaps : 0;
  ia.t = s_lo - ia.cb * ntaps;
  ia.th = AP && ntaps > 0 ? ia.t / wk.ap_ntw : 0;
  ia.tw = AP ? ia.t - ia.th * wk.ap_ntw : 0;
  Iter ib = ia;
  // AP: every work's taps are a product of two progressions, stepped through
  // with selects only, so that a stage stays one block of straight-line code
  auto advance = [&](Iter& it) {
    const bool w = AP && it.tw + 1 == wk.ap_ntw, e = it.t + 1 == ntaps;
    it.th = e ? 0 : it.th + (w ? 1 : 0);
    it.tw = (w | e) ? 0 : it.tw + 1;
    it.t = e ? 0 : it.t + 1;
    it.cb = __builtin_amdgcn_readfirstlane(it.cb + (e ? 1 : 0));  // stays in a scalar register
  };
  auto tap_of = [&](const Iter& it, int* off_h, int* off_w, uint32_t* slot_b) {
    if constexpr (AP) {
      *off_h = wk.ap_off0_h + it.th * wk.ap_doff_h;
      *off_w = wk.ap_off0_w + it.tw * wk.ap_doff_w;
      *slot_b = (uint32_t)((wk.ap_kh0 + it.th * wk.ap_dkh) * a.ks + wk.ap_kw0 +
                           it.tw * wk.ap_dkw) * slot_bytes;
    } else {
      const TapDev tp = a.taps[wk.tap_begin + it.t];
      *off_h = tp.off_h;
      *off_w = tp.off_w;
      *slot_b = (uint32_t)tp.slot * slot_bytes;
    }
  };

  // two stages of rows (before the split) in flight; the weight fragments are
  // reloaded as soon as their last use is issued: a stage is 12 TP TC MFMAs of
  // 32 cycles, longer than a load takes
  uint4 ra[2][NROW][2];
  uint4 rb[2][3][TC];  // [16-channel step][part][channel block]
  // loads past this group's last stage return zeros (out-of-range offsets)
  auto load_a = [&](uint4 (&R)[NROW][2], bool valid) {
    int off_h, off_w;
    uint32_t slot_b;
    tap_of(ia, &off_h, &off_w, &slot_b);
    const int delta = (off_h * a.w + off_w) * a.cin * 4;
    const bool tail = ia.cb == cblocks - 1;
#pragma unroll
    for (int i = 0; i < NROW; ++i) {
      const int ih = p_ih[i] + off_h, iw = p_iw[i] + off_w;
      const bool in = valid & ((unsigned)ih < (unsigned)a.h) & ((unsigned)iw < (unsigned)a.w);
#pragma unroll
      for (int l = 0; l < 2; ++l) {
        const bool ok = in & !(tail && 8 * q + 4 * l >= tail_c);
        const uint32_t v = ok ? p_base[i] + (uint32_t)delta + 16u * l : OOB;
        R[i][l] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, v, (uint32_t)ia.cb * 128u, 0));
      }
    }
    advance(ia);
  };
  uint32_t b_at = 0;
  bool b_ok = false;
  auto begin_b = [&](bool valid) {  // the stage whose fragments load_b reads next
    int off_h, off_w;
    uint32_t slot_b;
    tap_of(ib, &off_h, &off_w, &slot_b);
    b_at = slot_b + (uint32_t)ib.cb * 2048u;
    b_ok = valid;
    advance(ib);
  };
  auto load_b = [&](int c) {
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int j = 0; j < TC; ++j)
        rb[c][p][j] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(wr[p], b_ok ? w_off[j] : OOB,
                                                         b_at + 1024u * c, 0));
  };
  auto store_a = [&](int buf, const uint4 (&R)[NROW][2]) {
#pragma unroll
    for (int i = 0; i < NROW; ++i) {
      const Split8 s = split8(R[i][0], R[i][1]);
      char* const at = smem + buf * STAGE_B + (tid / 4 + (NT / 4) * i) * ROWB + q * 16;
#pragma unroll
      for (int p = 0; p < 3; ++p) *(uint4*)(at + p * PLANE_B) = s.p[p];
    }
  };

  f32x16 acc[TP][TC];
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TC; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto read_f = [&](int buf, int c, uint4 (&f)[3][TP]) {
    const char* const at = smem + buf * STAGE_B + (wp_i * 32 * TP + row32) * ROWB +
                           pack_chunk_byte(c, half);
#pragma unroll
    for (int p = 2; p >= 0; --p)
#pragma unroll
      for (int i = 0; i < TP; ++i) f[p][i] = *(const uint4*)(at + p * PLANE_B + 32 * i * ROWB);
  };
  auto mfma_step = [&](const uint4 (&f)[3][TP], const uint4 (&w)[3][TC]) {
#pragma unroll
    for (int o = 2; o >= 0; --o)
#pragma unroll
      for (int p = 0; p <= o; ++p)
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
          for (int j = 0; j < TC; ++j) {
            const bf16x8 vp = __builtin_bit_cast(bf16x8, f[o - p][i]);
            const bf16x8 vc = __builtin_bit_cast(bf16x8, w[p][j]);
            acc[i][j] = NCHW_OUT
                            ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(vc, vp, acc[i][j], 0, 0, 0)
                            : __builtin_amdgcn_mfma_f32_32x32x16_bf16(vp, vc, acc[i][j], 0, 0, 0);
          }
  };

  // The order of a half stage: its loads, its LDS reads, then everything else
  // dealt between its MFMAs.
  auto deal = [&](auto loads_c) {
    __builtin_amdgcn_sched_group_barrier(0x020, decltype(loads_c)::value, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 3 * TP, 0);
    unroll_stages<6 * TP * TC>([&](auto) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // an MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);  // VALU
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // an LDS write
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // a load
    });
  };
  if (per > 0) {
    load_a(ra[0], 0 < nsteps);
    begin_b(0 < nsteps);
    load_b(0);
    load_b(1);
    load_a(ra[1], 1 < nsteps);
    store_a(0, ra[0]);
    __syncthreads();
    uint4 f0[3][TP], f1[3][TP];
    read_f(0, 0, f0);
    // At the top of stage s: LDS buffer s & 1 holds it, f0 its first
    // fragments, register buffer (s + 1) & 1 the rows of stage s + 1.  The one
    // barrier sits between the stage's two steps, so that every fragment is
    // read a step of MFMAs before its use; it separates the writes of stage
    // s + 1's rows from their first reads, and the last reads of a buffer (the
    // second step's, issued at the top) from the writes of the stage after.
    // Both halves are straight-line code in which the splitting, the address
    // arithmetic and the loads are dealt between the MFMAs (each leaves seven
    // issue slots free): the waves of a workgroup meet at the barrier every
    // stage, so work in front of the MFMAs would leave the matrix cores idle
    // on all SIMDs at once.  A stage past a group's last multiplies zeros.
    auto stage = [&](auto u_c, int s) {
      constexpr int u = decltype(u_c)::value;
      load_a(ra[u], s + 2 < nsteps);
      read_f(u, 1, f1);
      begin_b(s + 1 < nsteps);
      mfma_step(f0, rb[0]);
      store_a(u ^ 1, ra[u ^ 1]);
      load_b(0);
      deal(std::integral_constant<int, 2 * NROW>());
      __syncthreads();
      read_f(u ^ 1, 0, f0);
      mfma_step(f1, rb[1]);
      load_b(1);
      deal(std::integral_constant<int, 0>());
    };
    for (int s = 0; s < per; s += 2)
      unroll_stages<2>([&](auto u_c) { stage(u_c, s + decltype(u_c)::value); });
  }

  float* const red = (float*)smem_all + wave * (NREG * 64) + lane;
  if constexpr (KS > 1) {
    __syncthreads();
    if (grp == 1) {
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TC; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) red[((i * TC + j) * 16 + r) * 64] = acc[i][j][r];
    }
    __syncthreads();
    if (grp != 0) return;
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TC; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += red[((i * TC + j) * 16 + r) * 64];
  } else {
    __syncthreads();  // s_bias; every wave is done with the stage rows
  }

  const int pix0 = wk.m0 + wp_i * 32 * TP, ch0 = wk.n0 + wc_i * 32 * TC;
  float most[4] = {};  // (finite sums lie below 2^80: so does their total, about)
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TC; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[i][j][r] *= kSumUnscale;
        most[r & 3] += fabsf(acc[i][j][r]);
      }
  if (__builtin_expect(__any(!finite(most[0] + most[1] + (most[2] + most[3]))), 0)) {
    // the wave's own piece of LDS keeps the sums meanwhile
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TC; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          red[((i * TC + j) * 16 + r) * 64] = acc[i][j][r];
          acc[i][j][r] = 0.f;
        }
    PixelPos px[TP];
#pragma unroll
    for (int i = 0; i < TP; ++i) px[i] = pixel_pos(sg, a.ptab, min(pix0 + 32 * i + row32, wk.m1 - 1));
    bool w_fin = true;
    for (int s = s_w0; s < s_w1; ++s) {
      const int cb = s / ntaps;
      const TapDev tp = a.taps[wk.tap_begin + s - cb * ntaps];
      for (int c = 0; c < 2; ++c) {
        float xv[TP][8], wv[TC][8];
#pragma unroll
        for (int i = 0; i < TP; ++i) {
          const int ih = px[i].ih + tp.off_h, iw = px[i].iw + tp.off_w;
          const bool in = ((unsigned)ih < (unsigned)a.h) & ((unsigned)iw < (unsigned)a.w);
          const uint32_t at = ((uint32_t)px[i].img * (uint32_t)a.h + (uint32_t)ih) * (uint32_t)a.w + (uint32_t)iw;
#pragma unroll
          for (int l = 0; l < 2; ++l) {
            const int ch = 32 * cb + 16 * half + 8 * c + 4 * l;
            const uint32_t v = (in & (ch < a.cin)) ? (at * (uint32_t)a.cin + (uint32_t)ch) * 4u : OOB;
            unpack4(__builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, v, 0, 0)),
                    &xv[i][4 * l]);
          }
        }
#pragma unroll
        for (int j = 0; j < TC; ++j) {
          uint4 h[3];
#pragma unroll
          for (int p = 0; p < 3; ++p)
            h[p] = __builtin_bit_cast(
                uint4, __builtin_amdgcn_raw_buffer_load_b128(
                           wr[p], w_off[j], (uint32_t)tp.slot * slot_bytes + (uint32_t)cb * 2048u + 1024u * c, 0));
          w_fin &= join_parts(h, wv[j]);
        }
        mfma_f32_step<NCHW_OUT>(acc, xv, wv);
      }
    }
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TC; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float* const g = &red[((i * TC + j) * 16 + r) * 64];
          if (!finite(*g)) *g = acc[i][j][r];
        }
    // (until a sum is NaN, which it then stays)
    if (__any(!w_fin)) {
      for (int e = 0; e < NREG; ++e) {
        if (red[e * 64] == red[e * 64]) continue;
        const int i = e / (16 * TC), j = (e >> 4) % TC, r = e & 15;
        const int sub = 8 * (r >> 2) + 4 * half + (r & 3);
        const int m = pix0 + 32 * i + (NCHW_OUT ? row32 : sub);
        const int ch = ch0 + 32 * j + (NCHW_OUT ? sub : row32);
        if (m >= wk.m1 || ch >= a.cout) continue;
        const PixelPos p = pixel_pos(sg, a.ptab, m);
        float v = 0.f;
        for (int s = s_w0; s < s_w1 && v == v; ++s) {
          const int cb = s / ntaps;
          const TapDev tp = a.taps[wk.tap_begin + s - cb * ntaps];
          const int ih = p.ih + tp.off_h, iw = p.iw + tp.off_w;
          if ((unsigned)ih >= (unsigned)a.h || (unsigned)iw >= (unsigned)a.w) continue;
          const float* const xp = (const float*)a.x + (((size_t)p.img * a.h + ih) * a.w + iw) * a.cin;
          for (int c = 32 * cb; c < min(32 * cb + 32, a.cin); ++c)
            v = fmaf(xp[c], split_weight(wbase, plane_b, (uint32_t)tp.slot * slot_bytes, a.cin_pad, ch, c), v);
        }
        red[e * 64] = v;
      }
    }
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TC; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = red[((i * TC + j) * 16 + r) * 64];
  }
  void* const y = a.ksplit > 1 ? (void*)(a.part + (size_t)wk.ks * a.part_stride) : a.y[sg.plan];
  store_tile<false, NCHW_OUT, TP, TC>(a, sg, wk.m1, y, acc, pix0, ch0, lane, s_bias - wk.n0);
}

template <int PW, int CW, int TP, int TC, int KS>
static void launch_f32(const GemmArgs& a, bool nchw_out, hipStream_t stream) {
  const dim3 grid(a.n_works), block(PW * CW * KS * 64);
#define HUGE2_F32(N_, AP_)                                                                      \
  hipLaunchKernelGGL((phase_gemm_f32_kernel<PW, CW, TP, TC, KS, N_, AP_>), grid, block, 0, stream, a)
  if (a.all_ap) {
    if (nchw_out) HUGE2_F32(true, true); else HUGE2_F32(false, true);
  } else {
    if (nchw_out) HUGE2_F32(true, false); else HUGE2_F32(false, false);
  }
#undef HUGE2_F32
}

hipError_t launch_gemm_f32(const GemmArgs& a, int cfg, bool nchw_out, hipStream_t stream) {
  switch (cfg) {
    case TILE_F32_64x128_K2: launch_f32<1, 2, 2, 2, 2>(a, nchw_out, stream); break;
    case TILE_F32_128x128: launch_f32<2, 2, 2, 2, 1>(a, nchw_out, stream); break;
    case TILE_F32_128x64: launch_f32<2, 2, 2, 1, 1>(a, nchw_out, stream); break;
    case TILE_F32_128x32: launch_f32<4, 1, 1, 1, 1>(a, nchw_out, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace huge2
