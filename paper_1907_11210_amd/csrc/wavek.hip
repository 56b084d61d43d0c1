// wavek.hip -- the phase GEMM for short problems: every wave of a workgroup
// holds the whole tile and takes every eighth K stage.
#include "device.hpp"
#include "kernels.hpp"

namespace huge2 {

// ---------------------------------------------------------------------------
// Phase GEMM, wave-K form.  A workgroup of 8 waves computes a tile of 64
// pixels x 32 * TC output channels; K stage s (channel block outer, tap inner,
// 128 bytes of input channels) is wave s mod 8's alone.  Each wave loads its
// stage's pixel rows whole (8 lanes per 128-byte row), turns them into the
// MFMA lane layout through a piece of LDS of its own, multiplies them with
// weight fragments read straight from the lane-ordered packing, and the eight
// partial tiles are added through LDS in wave order at the end (a fixed order:
// bitwise reproducible).
// Why: a layer with few tiles is bound by the latency of its longest chain of
// stages, not by any rate.  With the stages dealt to the waves the chain is an
// eighth as long and nothing inside it meets a barrier.  The price is that no
// operand is shared between waves, twice the L2 traffic of the shared tiles,
// which is why large layers keep those (choose_cfg).
//
// fp32 runs on the bf16 matrix cores (16 times the fp32 rate): every operand
// is split exactly into three bf16 parts (split8, which scales it first) and
// six of the nine products are summed in fp32, leaving out the three that stay
// below 2^-25 of the product; weights are split once, when packed.  A sum that
// comes out infinite or NaN is formed again in plain fp32 (mfma_f32_step: an
// operand that is or becomes infinite has no finite parts).
constexpr int kWkWaves = 8;
// Up to two bf16 stages are one wave's: there is no chain to shorten, and one
// accumulator keeps the sum's order that of the shared tiles, bit for bit
// (100 -> 16384 channels, 64 rows: 10.9 us, 9.9 with a wave each, 12.1 on the 32 x
// 256 tile).
constexpr int kWkChain = 2;

template <bool F32, int TC, bool NCHW_OUT>
__global__ __launch_bounds__(kWkWaves * 64) void wavek_kernel(GemmArgs a) {
  constexpr int TP = 2, BM = 32 * TP, BN = 32 * TC;
  constexpr int NPL = F32 ? 3 : 1;     // bf16 parts per operand
  constexpr int ESZ = F32 ? 4 : 2;
  constexpr int KCH = F32 ? 2 : 4;     // 16-channel MFMA steps per stage
  constexpr int KC = 16 * KCH;         // channels per stage (128 bytes of input)
  constexpr int ROWB = 32 * KCH + 16;  // LDS row pitch (pad: distinct banks)
  constexpr int PLANE_B = BM * ROWB, WAVE_B = NPL * PLANE_B;
  constexpr int NREG = TP * TC * 16;
  constexpr int RED_B = kWkWaves * NREG * 64 * 4;
  constexpr int SMEM_B = RED_B > kWkWaves * WAVE_B ? RED_B : kWkWaves * WAVE_B;
  constexpr int LPR = F32 ? 4 : 8;     // lanes per pixel row (32 or 16 bytes each)
  constexpr int NROW = BM / (64 / LPR);  // rows per lane
  constexpr int NLD = F32 ? 2 : 1;     // 16-byte loads per row and lane
  constexpr uint32_t OOB = 0x80000000u;
  __shared__ __attribute__((aligned(16))) char smem[SMEM_B];
  __shared__ int4 s_row[BM];           // input byte offset, ih, iw, output offset (-1: none)
  __shared__ int4 s_taps[kMaxLdsTaps];
  __shared__ float s_bias[BN];
  __shared__ int s_bad;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, row32 = lane & 31;
  const int work = xcd_remap(blockIdx.x, gridDim.x);
  const WorkDev wk = a.works[work];
  const SegDev sg = a.segs[wk.seg];
  const int hw_o = a.ho * a.wo;
  const uint32_t slot_bytes = (uint32_t)a.cout_pad * (uint32_t)a.cin_pad * 2u;
  const int ntaps = wk.tap_count;
  const int cblocks = a.cin_pad / KC;
  const int nsteps = ntaps * cblocks;
  const int nwaves = min(nsteps, !F32 && nsteps <= kWkChain ? 1 : kWkWaves);  // that take stages
  const int tail_c = a.cin - (cblocks - 1) * KC;

  if (tid < BM) {
    const int m = min(wk.m0 + tid, wk.m1 - 1);
    const PixelPos p = pixel_pos(sg, a.ptab, m);
    const uint32_t base = (((uint32_t)p.img * (uint32_t)a.h + (uint32_t)p.ih) * (uint32_t)a.w +
                           (uint32_t)p.iw) * (uint32_t)a.cin * ESZ;
    const int out = NCHW_OUT ? p.img * a.cout * hw_o + p.oh * a.wo + p.ow
                             : ((p.img * a.ho + p.oh) * a.wo + p.ow) * a.cout;
    s_row[tid] = make_int4((int)base, p.ih, p.iw, wk.m0 + tid < wk.m1 ? out : -1);
  } else if (tid >= 128 && tid < 128 + ntaps) {
    const TapDev tp = a.taps[wk.tap_begin + tid - 128];
    s_taps[tid - 128] = make_int4((tp.off_h * a.w + tp.off_w) * a.cin * ESZ,
                                  (int)((uint32_t)tp.slot * slot_bytes), tp.off_h, tp.off_w);
  } else if (tid >= 256 && tid < 256 + BN) {
    const float* const bias = a.bias[sg.plan];
    const int t = tid - 256;
    s_bias[t] = (bias && wk.n0 + t < a.cout) ? bias[bias_index(a, wk.n0 + t)] : 0.f;
  }
  if (F32 && tid == 0) s_bad = 0;
  const uint32_t plane_b = a.wp_bytes / NPL;
  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, a.x_bytes, 0x00020000);
  const char* const wbase = (const char*)a.wp[sg.plan];
  // lane-ordered weights: 32-channel block n0 / 32 + j
  uint32_t w_off[TC];
#pragma unroll
  for (int j = 0; j < TC; ++j)
    w_off[j] = (uint32_t)((wk.n0 / 32 + j) * 32 * a.cin_pad * 2 + lane * 16);
  __syncthreads();

  const int chunk = lane % LPR, row0 = lane / LPR;
  int4 ri[NROW];
#pragma unroll
  for (int i = 0; i < NROW; ++i) ri[i] = s_row[row0 + (64 / LPR) * i];

  uint4 ra[NROW][NLD];
  uint4 rb[KCH][NPL][TC];
  struct Stage {
    int t, cb;
  };
  auto tap_at = [&](const Stage& st) {
    int4 ti = s_taps[st.t];
    ti.x = __builtin_amdgcn_readfirstlane(ti.x);
    ti.y = __builtin_amdgcn_readfirstlane(ti.y);
    ti.z = __builtin_amdgcn_readfirstlane(ti.z);
    ti.w = __builtin_amdgcn_readfirstlane(ti.w);
    return ti;
  };
  auto load_a = [&](const Stage& st, const int4& ti) {
    const bool tail = st.cb == cblocks - 1;
#pragma unroll
    for (int i = 0; i < NROW; ++i) {
      const int ih = ri[i].y + ti.z, iw = ri[i].z + ti.w;
      const bool in = ((unsigned)ih < (unsigned)a.h) & ((unsigned)iw < (unsigned)a.w);
#pragma unroll
      for (int l = 0; l < NLD; ++l) {
        const int piece = chunk * NLD + l;  // 16-byte piece of the row
        const bool ok = in & !(tail && piece * (16 / ESZ) >= tail_c);
        const uint32_t v = ok ? (uint32_t)ri[i].x + (uint32_t)ti.x + 16u * piece : OOB;
        ra[i][l] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, v, (uint32_t)st.cb * 128u, 0));
      }
    }
  };
  auto load_b = [&](const Stage& st, const int4& ti, int c) {
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl) {
      const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(wbase + (size_t)pl * plane_b), 0, plane_b, 0x00020000);
#pragma unroll
      for (int j = 0; j < TC; ++j)
        rb[c][pl][j] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(
                       wr, w_off[j],
                       (uint32_t)ti.y + (uint32_t)st.cb * (KCH * 1024u) + 1024u * c, 0));
    }
  };
  char* const mine = smem + wave * WAVE_B;
  auto store_a = [&]() {
#pragma unroll
    for (int i = 0; i < NROW; ++i) {
      char* const at = mine + (row0 + (64 / LPR) * i) * ROWB + chunk * 16;
      if constexpr (F32) {
        const Split8 s = split8(ra[i][0], ra[i][1]);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *(uint4*)(at + pl * PLANE_B) = s.p[pl];
      } else {
        *(uint4*)at = ra[i][0];
      }
    }
  };

  f32x16 acc[TP][TC];
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TC; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto mfma = [&](const uint4& x, const uint4& w, f32x16 c) {
    const bf16x8 vp = __builtin_bit_cast(bf16x8, x), vc = __builtin_bit_cast(bf16x8, w);
    return NCHW_OUT ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(vc, vp, c, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f32_32x32x16_bf16(vp, vc, c, 0, 0, 0);
  };

  Stage st{wave, 0};
  auto settle = [&](Stage& s) {
    while (s.t >= ntaps) {
      s.t -= ntaps;
      ++s.cb;
    }
  };
  if (wave < nwaves) {
    settle(st);
    const int4 ti = tap_at(st);
    load_a(st, ti);
#pragma unroll
    for (int c = 0; c < KCH; ++c) load_b(st, ti, c);
  }
  for (int s = wave < nwaves ? wave : nsteps; s < nsteps; s += nwaves) {
    store_a();
    // the piece of LDS is this wave's alone and its LDS accesses stay in
    // order: no barrier between the writes and the reads of other lanes
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const bool more = s + nwaves < nsteps;
    Stage nx{st.t + nwaves, st.cb};
    int4 ti = make_int4(0, 0, 0, 0);
    if (more) {
      settle(nx);
      ti = tap_at(nx);
      load_a(nx, ti);
    }
#pragma unroll
    for (int c = 0; c < KCH; ++c) {
      uint4 fa[NPL][TP];
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl)
#pragma unroll
        for (int i = 0; i < TP; ++i)
          fa[pl][i] = *(const uint4*)(mine + pl * PLANE_B + (32 * i + row32) * ROWB +
                                      pack_chunk_byte(c, half));
      // the smallest products first
#pragma unroll
      for (int o = NPL - 1; o >= 0; --o)
#pragma unroll
        for (int pl = 0; pl <= o; ++pl)
#pragma unroll
          for (int i = 0; i < TP; ++i)
#pragma unroll
            for (int j = 0; j < TC; ++j)
              acc[i][j] = mfma(fa[o - pl][i], rb[c][pl][j], acc[i][j]);
      if (more) load_b(nx, ti, c);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    st = nx;
  }

  // the eight partial tiles through LDS, [wave][register][lane]
  float* const red = (float*)smem;
  __syncthreads();  // every wave is done with its stage rows
  if (wave < nwaves) {
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TC; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          red[(wave * NREG + (i * TC + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    if constexpr (F32) {  // below 2^124 the eight add up to a finite sum
      float most[4] = {};
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TC; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) most[r & 3] += fabsf(acc[i][j][r]);
      if (!(most[0] + most[1] + (most[2] + most[3]) <= 0x1p124f)) s_bad = 1;
    }
  }
  __syncthreads();
  void* const y = a.y[sg.plan];
  // register rr = wave + 8 k of every lane's tile is this wave's to add and store
  auto total = [&](int k) {
    float v = 0.f;
    for (int p = 0; p < nwaves; ++p) v += red[(p * NREG + wave + kWkWaves * k) * 64 + lane];
    return v;
  };
  bool w_fin = true;
  auto store = [&](int k, float v) {
    const int rr = wave + kWkWaves * k, blk = rr >> 4, r = rr & 15;
    const int i = blk / TC, j = blk % TC;
    const int sub = 8 * (r >> 2) + 4 * half + (r & 3);  // 32x32 MFMA result rows
    const int px = 32 * i + (NCHW_OUT ? row32 : sub), ch = wk.n0 + 32 * j + (NCHW_OUT ? sub : row32);
    const int4 row = s_row[px];
    if (row.w < 0 || ch >= a.cout) return;
    if constexpr (F32) {
      if (!w_fin && v != v) {
        v = 0.f;
        for (int t = 0; t < ntaps && v == v; ++t) {  // a sum that is NaN stays so
          const int4 ti = s_taps[t];
          const int ih = row.y + ti.z, iw = row.z + ti.w;
          if ((unsigned)ih >= (unsigned)a.h || (unsigned)iw >= (unsigned)a.w) continue;
          const float* const xp = (const float*)((const char*)a.x + ((uint32_t)row.x + (uint32_t)ti.x));
          for (int c = 0; c < a.cin && v == v; ++c)
            v = fmaf(xp[c], split_weight(wbase, plane_b, (uint32_t)ti.y, a.cin_pad, ch, c), v);
        }
      }
    }
    v = activate(v + s_bias[ch - wk.n0], a.act);
    const size_t off = (size_t)row.w + (NCHW_OUT ? (size_t)ch * hw_o : (size_t)ch);
    if constexpr (F32)
      ((float*)y)[off] = v;
    else
      ((uint16_t*)y)[off] = f32_to_bf16_rne(v);
  };
  if (!F32 || __builtin_expect(s_bad == 0, 1)) {
#pragma unroll 2
    for (int k = 0; k < NREG / kWkWaves; ++k) store(k, F32 ? total(k) * kSumUnscale : total(k));
  } else if constexpr (F32) {
    float v[NREG / kWkWaves];
#pragma unroll
    for (int k = 0; k < NREG / kWkWaves; ++k) v[k] = total(k) * kSumUnscale;
    __syncthreads();  // no sum is read any more
#pragma unroll
    for (int i = 0; i < TP; ++i)
#pragma unroll
      for (int j = 0; j < TC; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    for (int s = wave; s < nsteps; s += kWkWaves) {
      const int cb = s / ntaps;
      const int4 ti = s_taps[s - cb * ntaps];
      for (int c = 0; c < 2; ++c) {
        float xv[TP][8], wv[TC][8];
#pragma unroll
        for (int i = 0; i < TP; ++i) {
          const int4 row = s_row[32 * i + row32];
          const int ih = row.y + ti.z, iw = row.z + ti.w;
          const bool in = ((unsigned)ih < (unsigned)a.h) & ((unsigned)iw < (unsigned)a.w);
#pragma unroll
          for (int l = 0; l < 2; ++l) {
            const int ch = 32 * cb + 16 * half + 8 * c + 4 * l;
            const uint32_t at = (in & (ch < a.cin)) ? (uint32_t)row.x + (uint32_t)ti.x + 4u * ch : OOB;
            unpack4(__builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, at, 0, 0)),
                    &xv[i][4 * l]);
          }
        }
#pragma unroll
        for (int j = 0; j < TC; ++j) {
          uint4 h[3];
#pragma unroll
          for (int pl = 0; pl < 3; ++pl)
            h[pl] = *(const uint4*)(wbase + (size_t)pl * plane_b + (uint32_t)ti.y +
                                    (uint32_t)cb * 2048u + 1024u * c + w_off[j]);
          w_fin &= join_parts(h, wv[j]);
        }
        mfma_f32_step<NCHW_OUT>(acc, xv, wv);
      }
    }
    if (wave < nwaves) {
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TC; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            red[(wave * NREG + (i * TC + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    }
    w_fin = __syncthreads_or(!w_fin) == 0;
#pragma unroll
    for (int k = 0; k < NREG / kWkWaves; ++k)
      if (!finite(v[k])) v[k] = total(k);
#pragma unroll
    for (int k = 0; k < NREG / kWkWaves; ++k) store(k, v[k]);
  }
}

hipError_t launch_wavek(const GemmArgs& a, int dtype, int bn, bool nchw_out, hipStream_t stream) {
  const dim3 grid(a.n_works), block(kWkWaves * 64);
#define HUGE2_WAVEK(F32_, TC_, N_) \
  hipLaunchKernelGGL((wavek_kernel<F32_, TC_, N_>), grid, block, 0, stream, a)
  if (dtype == 1) {
    if (bn == 64) {
      if (nchw_out) HUGE2_WAVEK(false, 2, true); else HUGE2_WAVEK(false, 2, false);
    } else {
      if (nchw_out) HUGE2_WAVEK(false, 1, true); else HUGE2_WAVEK(false, 1, false);
    }
  } else {
    if (bn == 64) {
      if (nchw_out) HUGE2_WAVEK(true, 2, true); else HUGE2_WAVEK(true, 2, false);
    } else {
      if (nchw_out) HUGE2_WAVEK(true, 1, true); else HUGE2_WAVEK(true, 1, false);
    }
  }
#undef HUGE2_WAVEK
  return hipGetLastError();
}

// fp32 weights to three bf16 parts, each plane in the lane order of the
// split-wave packing (blocks of 32 channels x 64 bytes of K): part k of plane
// k, slot, channel block, K block, [chunk < 2][lane < 64][8 channels].
__global__ __launch_bounds__(256) void pack_split_kernel(const float* __restrict__ w,
                                                         uint16_t* __restrict__ wp, bool transposed,
                                                         int cin, int cout, int r, int s,
                                                         int cin_pad, int cout_pad, long long total,
                                                         int prod_rs) {
  for (long long idx = (long long)blockIdx.x * 256 + threadIdx.x; idx < total;
       idx += (long long)gridDim.x * 256) {
    // idx walks a plane in its packed order: element e, lane, chunk, K block, ...
    long long t = idx;
    const int e = (int)(t & 7);
    const int lane = (int)(t >> 3) & 63, chunk = (int)(t >> 9) & 1;
    t >>= 10;
    const int kblocks = cin_pad / 32, nblocks = cout_pad / 32;
    const int kb = (int)(t % kblocks);
    t /= kblocks;
    const int nb = (int)(t % nblocks);
    const int slot = (int)(t / nblocks);
    const int k = nb * 32 + (lane & 31), c = kb * 32 + (lane >> 5) * 16 + chunk * 8 + e;
    float v = 0.f;
    if (k < cout && c < cin) {
      if (prod_rs > 0) {
        const int co = cout / prod_rs;
        v = w[((size_t)c * co + k % co) * prod_rs + k / co];
      } else {
        const size_t rs = (size_t)r * s;
        v = transposed ? w[((size_t)c * cout + k) * rs + slot] : w[((size_t)k * cin + c) * rs + slot];
      }
    }
    // a scaled weight that is or rounds to infinity, or is NaN, has no parts: a
    // NaN in the first plane has its sums formed again in fp32, and the other
    // two hold its bits (join_weight)
    const float vs = v * kSplitScale;
    uint16_t h0 = f32_to_bf16_rne(vs), h1, h2;
    if ((h0 & 0x7f80u) != 0x7f80u) {
      const float v1 = vs - __uint_as_float((uint32_t)h0 << 16);
      h1 = f32_to_bf16_rne(v1);
      h2 = f32_to_bf16_rne(v1 - __uint_as_float((uint32_t)h1 << 16));
    } else {
      h0 = 0x7fc0u;
      h1 = (uint16_t)(__float_as_uint(v) >> 16);
      h2 = (uint16_t)__float_as_uint(v);
    }
    wp[idx] = h0;
    wp[idx + total] = h1;
    wp[idx + 2 * total] = h2;
  }
}

hipError_t launch_pack_split(const void* w, void* wp, bool transposed, int cin, int cout, int r,
                             int s, int cin_pad, int cout_pad, int prod_rs, hipStream_t stream) {
  const long long total = (long long)r * s * cout_pad * cin_pad;
  if (total == 0) return hipSuccess;
  const long long blocks = (total + 255) / 256;
  hipLaunchKernelGGL(pack_split_kernel, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256),
                     0, stream, (const float*)w, (uint16_t*)wp, transposed, cin, cout, r, s, cin_pad,
                     cout_pad, total, prod_rs);
  return hipGetLastError();
}

}  // namespace huge2
