#pragma once
// Kernel template of family 1, DIRECT_F32, included by the per-MK units.
// Family 1, DIRECT_F32: direct convolution on the vector ALU, NCHW x,
// K x C x R x S w, NCHW y, fp32 throughout.
//
// A block computes a TK x TOH x TOW output tile of one image. Each thread
// owns MK consecutive output channels and MW output columns of one row. The
// reduction runs over input channels; with LDS staging it advances in chunks
// of CT channels whose input halo tile and filter slice are copied to LDS once
// and shared by the block. SPLIT > 1 gives each split a contiguous channel
// range and writes partial sums to a workspace that a second kernel adds in
// split order. Every output adds its terms channel by channel, taps in (r, s)
// order.
//
// Compile-time: MK, MW, LDS, UNR, the specialisation SPEC (1x1 s1/s2, 3x3 pad
// 1 s1/s2, filters of 5 or 7 columns with column stride 1 or 2 and no column
// dilation, generic) and ALT: without LDS, scalar filter loads where every wave
// lies inside one channel group; with LDS, the variant for chunks too deep for
// registers whose filter rows are whole 16-byte quads, or in the generic path
// the one for filter rows of four taps and more. Runtime: tiles, CT, SPLIT.
//
// What bounds it, and the layouts that follow. The operand traffic per
// multiply-add, not the multiply-adds: with one 4-byte LDS read per operand a
// 1x1 micro-tile issues two reads per multiply-add to an LDS that four SIMDs
// share, and a small grid waits out one latency after another.
//   * A thread's MW columns are consecutive (except in the generic path), so a
//     filter row reads one window of (MW - 1) * stride + S words, in 16-byte
//     pieces, instead of MW * S words one by one.
//   * The filter slice lies in LDS by channel groups, padded to distinct
//     banks, as [channel][tap][MK], so that a thread reads its MK values of a
//     tap at once. Rows of the halo are padded to the width their windows are
//     read in. A chunk that goes through registers costs one word per lane and
//     load either way; a deeper one is copied straight into LDS, where the
//     number of copies counts, so its slice keeps the order of global memory
//     and is copied 16 bytes per lane (1.12 times as fast over 165 such
//     schedules; 0.75 to 1.0 times over those that fit registers).
//   * Both from LDS and without it, a ring of load units (a filter row of one
//     channel, or four channels of a 1x1 filter) stays in flight: each unit's
//     registers are reloaded for a later one right after its multiply-adds.
// Measured on 80 sampled schedules of each ResNet-18 b1 layer and of three
// ragged ones (3x3, 5x5, 7x7), against strided columns, single-word reads and
// one step of loads at a time, summed: 99.4 to 59.5 ms on the whole GPU, 182.4
// to 118.9 ms on a quarter; a 5x5 layer of 37 channels (4 x 45 x 51 pixels, its
// best schedule) 52.1 to 33.9 us.
//
// Global reads are raw buffer loads with 32-bit offsets: an element outside
// the tensor (padding, a tile past the edge) gets an offset past the buffer,
// which the hardware reads as 0, word by word also for multi-word loads. A
// load then needs one offset register and no branch.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ct_internal.h"
#include "k_util.h"

namespace ct {

struct DirectArgs {
  int N, C, H, W, K, R, S, sh, sw, ph, pw, dh, dw;
  int OH, OW;
  int toh, tow, tk, ct;
  int tiles_w;
  int split, cps;
  int ih_t, iw_t;
  int threads, tp, cols;
  int vec_w;               // deep chunks: the filter slice is copied 16 bytes per lane
  float inv_wq;
  int deep_x, deep_w;      // deep chunks are copied plane by plane / slice by slice
  int pitch, wpc, ks, wt;  // LDS words: halo row, filter words per output channel and per group of MK, all groups
  // host-precomputed reciprocals of the staging and index divisors (see qdiv)
  float inv_plane, inv_pitch, inv_ks, inv_wpc, inv_tp, inv_cols;
  int64_t ny;
};

__host__ __device__ constexpr int spec_r(int spec) { return spec == 1 || spec == 2 ? 1 : (spec == 3 || spec == 4 ? 3 : 0); }

typedef float f32x2d __attribute__((ext_vector_type(2)));
typedef float f32x4d __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

// N words of LDS from p on, p a multiple of ALIGN words: 16- and 8-byte reads
// as far as ALIGN allows.
template <int N, int ALIGN>
__device__ __forceinline__ void lds_words(const float* p, float* v) {
  if constexpr (N >= 4 && ALIGN % 4 == 0) {
    const f32x4d q = *(const f32x4d*)p;
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    lds_words<N - 4, ALIGN>(p + 4, v + 4);
  } else if constexpr (N >= 2 && ALIGN % 2 == 0) {
    const f32x2d q = *(const f32x2d*)p;
    v[0] = q.x; v[1] = q.y;
    lds_words<N - 2, 2>(p + 2, v + 2);
  } else if constexpr (N >= 1) {
    v[0] = *p;
    lds_words<N - 1, 1>(p + 1, v + 1);
  }
}

template <int MK, int MW, bool LDS, int SPEC, int UNR, bool ALT>
__global__ void __launch_bounds__(direct_max_threads(MK * MW))
direct_f32_kernel(const float* __restrict__ x, const float* __restrict__ w, float* __restrict__ out,
                  DirectArgs a) {
  // RC: rows and columns of a fixed filter; SC: columns of the filter and STC
  // the column stride (the fixed filters have it as row stride too); 0: runtime
  constexpr int RC = spec_r(SPEC), SC = direct_spec_s(SPEC), STC = direct_spec_stride(SPEC);
  // columns of a thread: consecutive, or in the generic path TOW/MW apart
  constexpr bool CONSEC = STC != 0;
  const int R = RC ? RC : a.R, S = SC ? SC : a.S;
  const int sh = RC ? STC : a.sh, sw = STC ? STC : a.sw;
  const int dh = RC ? 1 : a.dh, dw = STC ? 1 : a.dw;
  const int ph = RC ? RC / 2 : a.ph, pw = RC ? RC / 2 : a.pw;
  const int RS = R * S;
  const int C = a.C, H = a.H, W = a.W, K = a.K;
  constexpr bool UNI = ALT && !LDS, DEEP = ALT && LDS && SPEC != 0;
  constexpr int kLimit = direct_max_threads(MK * MW) >= 1024 ? 128 : 256;  // registers per thread

  extern __shared__ __align__(16) float smem[];
  const int t = threadIdx.x;
  const int th = blockIdx.x / a.tiles_w, tw = blockIdx.x - th * a.tiles_w;
  const int k0 = blockIdx.y * a.tk;
  const int n = blockIdx.z / a.split, sp = blockIdx.z - n * a.split;
  const int oh0 = th * a.toh, ow0 = tw * a.tow;
  const int tki = qdiv(t, a.inv_tp), tpi = t - tki * a.tp;
  const int lr = qdiv(tpi, a.inv_cols), lc = tpi - lr * a.cols;
  const int oh = oh0 + lr;
  const int kbase = k0 + tki * MK;
  const int cj = CONSEC ? 1 : a.cols;               // distance of a thread's columns
  const int ow = ow0 + (CONSEC ? lc * MW : lc);     // its first one

  float acc[MK][MW];
#pragma unroll
  for (int i = 0; i < MK; ++i)
#pragma unroll
    for (int j = 0; j < MW; ++j) acc[i][j] = 0.f;

  const int c_begin = sp * a.cps * a.ct;
  const int c_end = min(C, c_begin + a.cps * a.ct);
  const int ih_org = oh0 * sh - ph, iw_org = ow0 * sw - pw;
  const float* xn = x + (int64_t)n * C * H * W;
  const int HW = H * W;

  if constexpr (LDS) {
    // LDS: the filter slice [TK/MK groups][KS], a group [MK][CT * R * S] as in
    // global memory or (TR) [CT][R * S][MK], then the halo [CT][IH][PITCH]
    constexpr bool TR = SPEC != 0 && !DEEP && MK > 1;
    const int wrow = TR ? 1 : a.wpc;  // words from one channel's filter row to the next one's
    const float* wsm = smem + tki * a.ks;
    float* xs = smem + (a.wt + 3) / 4 * 4;
    const int pitch = a.pitch, plane = a.ih_t * pitch;
    const float* xthr = xs + lr * sh * pitch + (CONSEC ? lc * MW : lc) * sw;

    // Units of the compute loop, and how many stay in flight (direct_regs)
    constexpr DirectRegs kHeld = direct_regs(MK, MW, SPEC);
    constexpr int NW = kHeld.x_words, WW = kHeld.w_words, D = kHeld.ring;
    constexpr int WA = MK % 4 == 0 ? 4 : MK;
    auto compute = [&](const int nc) __attribute__((always_inline)) {
      if constexpr (SC != 0) {
        constexpr int XA = MW * STC % 4 == 0 ? 4 : (MW * STC % 2 == 0 ? 2 : 1);
        auto load = [&](const float* xr, const float* wr, float* xv, float* wv) __attribute__((always_inline)) {
          if constexpr (SC == 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              if constexpr (STC == 1) {
                lds_words<MW, XA>(xr + q * plane, xv + q * MW);
              } else {
#pragma unroll
                for (int j = 0; j < MW; ++j) xv[q * MW + j] = xr[q * plane + 2 * j];
              }
            }
          } else {
            lds_words<NW, XA>(xr, xv);
          }
          if constexpr (TR) {
            lds_words<WW, WA>(wr, wv);
          } else {
#pragma unroll
            for (int i = 0; i < MK; ++i) lds_words<WW / MK, SC == 1 ? 4 : 1>(wr + i * wrow, wv + i * (WW / MK));
          }
        };
        auto macs = [&](const float* xv, const float* wv) __attribute__((always_inline)) {
          if constexpr (SC == 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int i = 0; i < MK; ++i)
#pragma unroll
                for (int j = 0; j < MW; ++j) acc[i][j] = fmaf(wv[TR ? q * MK + i : i * 4 + q], xv[q * MW + j], acc[i][j]);
          } else {
#pragma unroll
            for (int s = 0; s < SC; ++s)
#pragma unroll
              for (int i = 0; i < MK; ++i)
#pragma unroll
                for (int j = 0; j < MW; ++j) acc[i][j] = fmaf(wv[TR ? s * MK + i : i * SC + s], xv[j * STC + s], acc[i][j]);
          }
        };
        // units in order: the filter words are one run, the window moves by a
        // row or, after the last row, to the next channel
        const int NU = SC == 1 ? nc / 4 : nc * R;
        const int wstep = TR ? WW : WW / MK;
        const int xstep = SC == 1 ? 4 * plane : dh * pitch, xwrap = plane - (R - 1) * xstep;
        const float *xp = xthr, *wp = wsm;
        int r = 0;
        auto next = [&]() __attribute__((always_inline)) {
          wp += wstep;
          if constexpr (SC == 1) {
            xp += xstep;
          } else {
            const bool wrap = ++r == R;
            xp += wrap ? xwrap : xstep;
            r = wrap ? 0 : r;
          }
        };
        float xb[D][NW], wb[D][WW];
        if (NU >= D) {
#pragma unroll
          for (int d = 0; d < D; ++d) {
            load(xp, wp, xb[d], wb[d]);
            next();
            __builtin_amdgcn_sched_barrier(0);
          }
          for (int u = 2 * D; u <= NU; u += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
              macs(xb[d], wb[d]);
              __builtin_amdgcn_sched_barrier(0);
              load(xp, wp, xb[d], wb[d]);
              next();
              __builtin_amdgcn_sched_barrier(0);
            }
          }
#pragma unroll
          for (int d = 0; d < D; ++d) macs(xb[d], wb[d]);
        }
        const int rest = NU >= D ? NU % D : NU;
        for (int u = 0; u < rest; ++u) {
          load(xp, wp, xb[0], wb[0]);
          next();
          macs(xb[0], wb[0]);
        }
        if constexpr (SC == 1) {
          for (int c = nc & ~3; c < nc; ++c) {
            float xv[MW], wv[MK];
#pragma unroll
            for (int j = 0; j < MW; ++j) xv[j] = xthr[c * plane + j * STC];
#pragma unroll
            for (int i = 0; i < MK; ++i) wv[i] = wsm[TR ? c * MK + i : i * wrow + c];
#pragma unroll
            for (int i = 0; i < MK; ++i)
#pragma unroll
              for (int j = 0; j < MW; ++j) acc[i][j] = fmaf(wv[i], xv[j], acc[i][j]);
          }
        }
      } else {
        // ALT: the taps of a filter row in groups of G (by the unroll knob; 2 where four
        // taps of 8 channels exceed 128 registers), all of a group's reads before its
        // multiply-adds: a tap at a time waits out an LDS latency each. Shorter rows run
        // without, in kernels of their own: with both in one, their registers cost the
        // short rows 3 to 10 %. 80 sampled LDS schedules each of a 9 x 9, an 11 x 11 and
        // a 4 x 4 filter: 2924 to 2498 us, 3044 to 2856, 2935 to 2643.
        constexpr int G = ALT ? (UNR == 1 || (MK == 8 && kLimit == 128) ? 2 : 4) : 1, kUnr = ALT ? 1 : UNR;
        auto taps = [&](auto count, const float* xr, const float* wr) __attribute__((always_inline)) {
          constexpr int N = decltype(count)::value;
          float xv[N][MW], wv[N][MK];
#pragma unroll
          for (int u = 0; u < N; ++u) {
#pragma unroll
            for (int j = 0; j < MW; ++j) xv[u][j] = xr[j * cj * sw + u * dw];
#pragma unroll
            for (int i = 0; i < MK; ++i) wv[u][i] = wr[i * wrow + u];
          }
#pragma unroll
          for (int u = 0; u < N; ++u)
#pragma unroll
            for (int i = 0; i < MK; ++i)
#pragma unroll
              for (int j = 0; j < MW; ++j) acc[i][j] = fmaf(wv[u][i], xv[u][j], acc[i][j]);
        };
#pragma unroll kUnr
        for (int c = 0; c < nc; ++c) {
          const float* xr = xthr + c * plane;
          const float* wr = wsm + c * RS;
          for (int r = 0; r < R; ++r) {
            int s = 0;
            if constexpr (G > 1)
              for (; s + G <= S; s += G)
                taps(std::integral_constant<int, G>{}, xr + r * dh * pitch + s * dw, wr + r * S + s);
            for (; s < S; ++s) taps(std::integral_constant<int, 1>{}, xr + r * dh * pitch + s * dw, wr + r * S + s);
          }
        }
      }
    };

    // Byte offset of halo element `rem` of a channel's tile in that channel's
    // plane, and of filter element `rem` of a channel group in the group's
    // rows from the chunk's first channel on; kOob outside (also for padding
    // words). k_left: rows of w from the group's first one on.
    auto x_off = [&](const int rem) {
      const int hh = qdiv(rem, a.inv_pitch), ww = rem - hh * pitch;
      const int gh = ih_org + hh, gw = iw_org + ww;
      const bool ok = ww < a.iw_t && (unsigned)gh < (unsigned)H && (unsigned)gw < (unsigned)W;
      return ok ? (unsigned)(gh * W + gw) * 4 : kOob;
    };
    auto w_off = [&](const int rem, const int k_left) {
      int i, j;  // channel of the group, word of its (channel, tap) run
      if constexpr (TR) {
        j = rem / MK;
        i = rem % MK;
      } else {
        i = qdiv(rem, a.inv_wpc);
        j = rem - i * wrow;
      }
      return j < a.ct * RS && i < min(MK, k_left) ? (unsigned)(i * C * RS + j) * 4 : kOob;
    };
    // Element e of the filter region (wt words, whole rows of `threads`) and
    // of the halo region goes to LDS word e of that region. Where both together
    // take at most kMaxNs elements per thread, they go through registers: the next
    // chunk's loads are in flight during this chunk's MACs, so a block pays
    // one memory round trip per chunk only once. An element's offset depends
    // on the chunk only through its first channel cc, which moves the buffer's
    // base instead: the offsets are computed once, and a chunk's loads and
    // stores take no address arithmetic on lanes and no lane masks (both
    // regions are padded to whole rows of the block's threads; an element past
    // its region is loaded as 0). Channels of a last, partial chunk past nc
    // stage values that the MACs never read. kMaxNs is what fits beside the
    // accumulators and the units in flight (direct_regs).
    const int xt = a.ct * plane, wt = a.wt;
    auto rows = [&](const int words) { return __builtin_amdgcn_readfirstlane((words + a.threads - 1) / a.threads); };
    const int nsx = rows(xt), nsw = rows(wt), nst = nsw + nsx;
    auto rsrc_x = [&](const int cc) { return make_rsrc(xn + (int64_t)cc * HW, (int64_t)(C - cc) * HW * 4); };
    auto rsrc_w = [&](const int cc) { return make_rsrc(w + (int64_t)cc * RS, ((int64_t)K * C - cc) * RS * 4); };
    auto x_elem = [&](const int e) {
      const int c = qdiv(e, a.inv_plane);
      const unsigned o = x_off(e - c * plane);
      return e < xt && o != kOob ? o + (unsigned)c * HW * 4 : kOob;
    };
    auto w_elem = [&](const int e) {
      const int kg = qdiv(e, a.inv_ks);
      const unsigned o = w_off(e - kg * a.ks, kg * MK < a.tk ? K - k0 - kg * MK : 0);
      return o != kOob ? o + (unsigned)(k0 + kg * MK) * C * RS * 4 : kOob;
    };
    auto staged = [&](auto ns) __attribute__((always_inline)) {
      constexpr int NS = decltype(ns)::value;
      // rows past the last one repeat it: same element, same LDS word
      unsigned off[NS];
      float val[NS];
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int q = min(u, nst - 1);
        off[u] = q < nsw ? w_elem(t + q * a.threads) : x_elem(t + (q - nsw) * a.threads);
      }
      auto fetch = [&](const int cc) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rxc = rsrc_x(cc), rwc = rsrc_w(cc);
#pragma unroll
        for (int u = 0; u < NS; ++u) val[u] = bload1(min(u, nst - 1) < nsw ? rwc : rxc, off[u]);
      };
      float* xrow = xs - nsw * a.threads;
      fetch(c_begin);
      for (int cc = c_begin; cc < c_end; cc += a.ct) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
          const int q = min(u, nst - 1);
          (q < nsw ? smem : xrow)[q * a.threads + t] = val[u];
        }
        __syncthreads();
        if (cc + a.ct < c_end) fetch(cc + a.ct);
        compute(min(a.ct, c_end - cc));
        __syncthreads();  // the next chunk's stores overwrite the tiles
      }
    };
    constexpr int kMaxNs = kHeld.staged;
    const bool done = !DEEP && nst <= kMaxNs;
    if constexpr (!DEEP) {
      if (nst <= 2) {
        staged(std::integral_constant<int, 2>{});
      } else if (nst <= 4) {
        staged(std::integral_constant<int, 4>{});
      } else if (nst <= 6) {
        staged(std::integral_constant<int, 6>{});
      } else if constexpr (kMaxNs >= 8) {
        if (nst <= 8) {
          staged(std::integral_constant<int, 8>{});
        } else if constexpr (kMaxNs >= 12) {
          if (nst <= 12) {
            staged(std::integral_constant<int, 12>{});
          } else if constexpr (kMaxNs >= 16) {
            if (nst <= 16) {
              staged(std::integral_constant<int, 16>{});
            } else if constexpr (kMaxNs >= 24) {
              if (nst <= 24) staged(std::integral_constant<int, 24>{});
            }
          }
        }
    }
    }
    // Deeper chunks are copied straight into LDS by buffer loads, one per
    // word, thread t of copy j filling word j * threads + t (so a block of
    // fewer than 64 threads works too), every copy of the chunk in flight at
    // once, then one wait. A copy writes lane i of its wave at its LDS base +
    // i, so each wave's base is offset by 64 words per wave before it. Lanes
    // past the tile copy nothing. Where a channel's plane (a group's slice)
    // fills at least half of the rows of threads it takes, the copies go plane
    // by plane and only the scalar base moves between them: one offset per
    // lane, not one per copy (about 28 vector instructions). (Batches of 16
    // loads through registers instead took 1.2 times as long over the sampled
    // LDS schedules.) The loops over planes and groups are not unrolled: what
    // four copies at a time kept across chunks went through vector lanes, also
    // in the kernels that never come here (1600 sampled LDS schedules of
    // ResNet-18 and ragged layers: 58.3 ms, and 54.2 ms with one at a time and
    // the plan's bounds opaque).
    const int wbase = wave_id() * 64;
    // DEEP: the lane offsets of up to kPlan 16-byte filter copies and kPlan
    // halo copies are the same in every chunk and stay in registers: a chunk's
    // copies then take no vector instruction but themselves (lanes past a
    // region's end write zeros into its padding). kPlan is what fits beside the
    // accumulators and the units in flight, so that nothing goes to scratch.
    constexpr int kPlan = DEEP ? kHeld.plan : 1;
    unsigned pw[kPlan], px[kPlan];
    int npw = 0, npx = 0;
    const int gq = a.ks / 4, ng = min(a.tk / MK, (K - k0 + MK - 1) / MK);
    auto quad = [&](const int q) {  // byte offset of 16-byte quad q of a group's slice
      const int rq = wrow / 4, i = qdiv(q, a.inv_wq), j = q - i * rq;
      return i < MK ? ((unsigned)i * C * RS + 4 * j) * 4 : kOobQuad;
    };
    auto flat_quad = [&](const int e) {  // and of the whole filter region
      const int kg = qdiv(e, 4.f * a.inv_ks);
      const unsigned o = quad(e - kg * gq);
      return e < ng * gq && o != kOobQuad ? o + (unsigned)kg * MK * C * RS * 4 : kOobQuad;
    };
    if constexpr (DEEP) {
      npw = rows(ng * gq);
      npx = nsx;
      if (a.vec_w && npw <= kPlan && npx <= kPlan) {
#pragma unroll
        for (int u = 0; u < kPlan; ++u) {
          if (u < npw) pw[u] = flat_quad(u * a.threads + t);
          if (u < npx) px[u] = x_elem(u * a.threads + t);
        }
      } else {
        npw = 0;
      }
    }
    for (int cc = c_begin; cc < c_end && !done; cc += a.ct) {
      const int nc = min(a.ct, c_end - cc);
      if (DEEP && npw) {
        const __amdgpu_buffer_rsrc_t rw =
            make_rsrc(w + ((int64_t)k0 * C + cc) * RS, ((int64_t)(K - k0) * C - cc) * RS * 4), rx = rsrc_x(cc);
        // opaque here, so that the comparisons and LDS addresses are made where they
        // are used rather than kept in scalar registers, which do not suffice
        int cw = npw, cx = npx, row = a.threads;
        asm volatile("" : "+s"(cw), "+s"(cx), "+s"(row));
#pragma unroll
        for (int u0 = 0; u0 < kPlan; u0 += 4)
          if (u0 < cw) {
#pragma unroll
            for (int u = u0; u < u0 + 4 && u < kPlan; ++u)
              if (u < cw) copy16_to_lds(rw, smem + 4 * (u * row + wbase), pw[u]);
          }
#pragma unroll
        for (int u0 = 0; u0 < kPlan; u0 += 4)
          if (u0 < cx) {
#pragma unroll
            for (int u = u0; u < u0 + 4 && u < kPlan; ++u)
              if (u < cx) copy_to_lds(rx, xs + u * row + wbase, px[u]);
          }
      } else if (DEEP && a.vec_w) {
        const int64_t gstep = (int64_t)MK * C * RS;
        const float* base = w + ((int64_t)k0 * C + cc) * RS;
        const int64_t left = ((int64_t)(K - k0) * C - cc) * RS;
        if (a.deep_w) {
          for (int q0 = 0; q0 < gq; q0 += a.threads) {
            const unsigned off = quad(q0 + t);
            if (q0 + t < gq) {
#pragma unroll 1
              for (int kg = 0; kg < ng; ++kg)
                copy16_to_lds(make_rsrc(base + kg * gstep, (left - kg * gstep) * 4),
                              smem + kg * a.ks + 4 * (q0 + wbase), off);
            }
          }
        } else {
          const __amdgpu_buffer_rsrc_t r = make_rsrc(base, left * 4);
          for (int q0 = 0; q0 < ng * gq; q0 += a.threads)
            if (q0 + t < ng * gq) copy16_to_lds(r, smem + 4 * (q0 + wbase), flat_quad(q0 + t));
        }
      } else if (a.deep_w) {
        const int64_t gstep = (int64_t)MK * C * RS;
        for (int e0 = 0; e0 < a.ks; e0 += a.threads) {
          // (rows past K lie past the buffer: the group's first row moves its base)
          const unsigned off = w_off(e0 + t, MK);
          if (e0 + t < a.ks) {
            const float* base = w + ((int64_t)k0 * C + cc) * RS;
            int64_t left = ((int64_t)(K - k0) * C - cc) * RS;
            float* dst = smem + e0 + wbase;
#pragma unroll 1
            for (int kg = 0; kg < ng; ++kg) {
              copy_to_lds(make_rsrc(base, left * 4), dst, off);
              base += gstep;
              left -= gstep;
              dst += a.ks;
            }
          }
        }
      } else {
        const __amdgpu_buffer_rsrc_t rwc = rsrc_w(cc);
        for (int e0 = 0; e0 < wt; e0 += a.threads)
          if (e0 + t < wt) copy_to_lds(rwc, smem + e0 + wbase, w_elem(e0 + t));
      }
      if (DEEP && npw) {  // (copied above)
      } else if (a.deep_x) {
        for (int e0 = 0; e0 < plane; e0 += a.threads) {
          const unsigned off = x_off(e0 + t);
          if (e0 + t < plane) {
            const float* base = xn + (int64_t)cc * HW;
            float* dst = xs + e0 + wbase;
#pragma unroll 1
            for (int c = 0; c < nc; ++c) {
              copy_to_lds(make_rsrc(base, (int64_t)HW * 4), dst, off);
              base += HW;
              dst += plane;
            }
          }
        }
      } else {
        const __amdgpu_buffer_rsrc_t rxc = rsrc_x(cc);
        for (int e0 = 0; e0 < xt; e0 += a.threads)
          if (e0 + t < xt) copy_to_lds(rxc, xs + e0 + wbase, x_elem(e0 + t));
      }
      wait_copies();
      __syncthreads();
      compute(nc);
      __syncthreads();
    }
  } else if constexpr (RC != 0) {
    // Registers only, fixed filter. Row validity and the window's first column
    // are folded into one offset per filter row; a channel moves the buffer's
    // base. A window of several columns is read in 16-byte pieces from column
    // max(gw0, 0) on; at the left edge (gw0 = -1) it is shifted by one word,
    // and columns at or past W are cleared.
    constexpr int T = RC * RC;
    constexpr bool PT = RC == 3 && MW == 1;            // one resident offset per tap
    constexpr int NW = RC == 3 ? (MW - 1) * STC + 3 : MW;  // words of a unit's row
    unsigned xo[RC * (PT ? 3 : 1)];
    bool left = false, in[NW];
    {
      const int gw0 = ow * STC - RC / 2;
#pragma unroll
      for (int r = 0; r < RC; ++r) {
        const int gh = oh * STC - RC / 2 + r;
        const bool hok = (unsigned)gh < (unsigned)H && oh < a.OH;
        if constexpr (PT) {
#pragma unroll
          for (int s = 0; s < 3; ++s) {
            const int gw = gw0 + s;
            xo[r * 3 + s] = hok && (unsigned)gw < (unsigned)W ? (unsigned)(gh * W + gw) * 4 : kOob;
          }
        } else {
          xo[r] = hok && gw0 < W ? (unsigned)(gh * W + max(gw0, 0)) * 4 : kOob;
        }
      }
      left = gw0 < 0;
#pragma unroll
      for (int j = 0; j < NW; ++j) in[j] = gw0 + j < W;
    }
    auto xwords = [&](const __amdgpu_buffer_rsrc_t r, const int row, float* v) {
      if constexpr (PT) {
#pragma unroll
        for (int s = 0; s < 3; ++s) v[s] = bload1(r, xo[row * 3 + s]);
      } else if constexpr (RC == 1 && STC == 2) {
#pragma unroll
        for (int j = 0; j < MW; ++j) v[j] = bload1(r, xo[0] + j * 8u);
      } else {
        bload_words<NW>(r, xo[row], v);
      }
    };
    // the window of a filter row as the taps see it
    auto fix = [&](const float* q, float* v) {
#pragma unroll
      for (int j = 0; j < NW; ++j) v[j] = q[j];
      if constexpr (RC == 3 && !PT) {
#pragma unroll
        for (int j = 0; j < NW; ++j) v[j] = left ? (j ? q[j - 1] : 0.f) : q[j];
        // (columns 0 and 1 are inside for every stored output)
#pragma unroll
        for (int j = 2; j < NW; ++j) v[j] = in[j] ? v[j] : 0.f;
      }
    };
    auto rsrc_x = [&](const int c, const bool ok) { return make_rsrc(xn + (int64_t)c * HW, ok ? (int64_t)HW * 4 : 0); };
    auto rsrc_w = [&](const int c) { return make_rsrc(w + (int64_t)c * T, ((int64_t)K * C - c) * T * 4); };
    // (a channel past K reads row K-1: its sums are never stored)
    const int nch = c_end - c_begin;
    constexpr int kRegs = kLimit - MK * MW - 3 * RC - MK - 28;
    // UNI: every wave lies inside one channel group (TP a multiple of 64), so
    // the filter values are scalar loads, off the vector memory path, a unit
    // ahead of their use.
    const int kb = UNI ? __builtin_amdgcn_readfirstlane(kbase) : kbase;
    unsigned kofs[MK];
#pragma unroll
    for (int i = 0; i < MK; ++i) kofs[i] = (unsigned)(min(kb + i, K - 1) * C * T) * 4;
    if constexpr (RC == 3) {
      // unit (channel u of DC, filter row r)
      constexpr int U = NW + (UNI ? 0 : 3 * MK);
      constexpr int D0 = kRegs / (3 * U), D1 = 56 / (3 * ((PT ? 3 : (NW + 3) / 4) + (UNI ? 0 : MK)));
      constexpr int D2 = D0 < D1 ? D0 : D1, DC = D2 >= 4 ? 4 : (D2 >= 2 ? 2 : 1);
      float xq[DC][3][NW], ws[3 * MK];
      u32x3 wq[DC][3][MK];
      auto load = [&](const int c, const int r, float* xv, u32x3* wv) __attribute__((always_inline)) {
        xwords(rsrc_x(c_begin + c, true), r, xv);
        if constexpr (!UNI) {
          const __amdgpu_buffer_rsrc_t rw = rsrc_w(c_begin + c);
#pragma unroll
          for (int i = 0; i < MK; ++i) wv[i] = __builtin_amdgcn_raw_buffer_load_b96(rw, (int)(kofs[i] + r * 12u), 0, 0);
        }
      };
      // the scalar filter values of a unit (of the last channel past the range)
      auto scalars = [&](const int c, const int r, float* v) __attribute__((always_inline)) {
        const float* wc = w + (int64_t)min(c_begin + c, c_end - 1) * 9 + r * 3;
#pragma unroll
        for (int i = 0; i < MK; ++i)
#pragma unroll
          for (int s = 0; s < 3; ++s) v[i * 3 + s] = wc[(int64_t)min(kb + i, K - 1) * C * 9 + s];
      };
      auto macs = [&](const float* xr, const u32x3* wv) __attribute__((always_inline)) {
        float xv[NW];
        fix(xr, xv);
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int i = 0; i < MK; ++i) {
            const unsigned q = s == 0 ? wv[i].x : (s == 1 ? wv[i].y : wv[i].z);
            const float f = UNI ? ws[i * 3 + s] : __builtin_bit_cast(float, q);
#pragma unroll
            for (int j = 0; j < MW; ++j) acc[i][j] = fmaf(f, xv[j * STC + s], acc[i][j]);
          }
      };
      const int nfull = nch / DC * DC;
      if (nfull) {
#pragma unroll
        for (int u = 0; u < DC; ++u)
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            load(u, r, xq[u][r], wq[u][r]);
            __builtin_amdgcn_sched_barrier(0);
          }
        if constexpr (UNI) scalars(0, 0, ws);
        for (int c = 0; c + DC < nfull; c += DC) {
#pragma unroll
          for (int u = 0; u < DC; ++u)
#pragma unroll
            for (int r = 0; r < 3; ++r) {
              float wn[3 * MK];
              if constexpr (UNI) scalars(c + u + (r == 2), r == 2 ? 0 : r + 1, wn);
              macs(xq[u][r], wq[u][r]);
              __builtin_amdgcn_sched_barrier(0);
              load(c + u + DC, r, xq[u][r], wq[u][r]);
              __builtin_amdgcn_sched_barrier(0);
              if constexpr (UNI) {
#pragma unroll
                for (int q = 0; q < 3 * MK; ++q) ws[q] = wn[q];
              }
            }
        }
#pragma unroll
        for (int u = 0; u < DC; ++u)
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            if constexpr (UNI) {
              if (u + r) scalars(nfull - DC + u, r, ws);
            }
            macs(xq[u][r], wq[u][r]);
          }
      }
      for (int c = nfull; c < nch; ++c) {
#pragma unroll
        for (int r = 0; r < 3; ++r) load(c, r, xq[0][r], wq[0][r]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          if constexpr (UNI) scalars(c, r, ws);
          macs(xq[0][r], wq[0][r]);
        }
      }
    } else {
      // unit: four channels of the 1x1 filter
      constexpr int U = 4 * (MW + (UNI ? 0 : MK));
      constexpr int D0 = kRegs / U, D1 = 56 / (4 * (STC == 2 ? MW : 1) + (UNI ? 0 : MK));
      constexpr int D2 = D0 < D1 ? D0 : D1, DU = D2 >= 4 ? 4 : (D2 >= 2 ? 2 : 1);
      float xq[DU][4][MW], ws[4 * MK];
      u32x4 wq[DU][MK];
      auto load = [&](const int c, const int nq, float (*xv)[MW], u32x4* wv) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) xwords(rsrc_x(c_begin + c + q, q < nq), 0, xv[q]);
        if constexpr (!UNI) {
          const __amdgpu_buffer_rsrc_t rw = rsrc_w(c_begin + c);
#pragma unroll
          for (int i = 0; i < MK; ++i) wv[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)kofs[i], 0, 0);
        }
      };
      auto scalars = [&](const int c, float* v) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < MK; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) v[i * 4 + q] = w[(int64_t)min(kb + i, K - 1) * C + min(c_begin + c + q, c_end - 1)];
      };
      auto macs = [&](const int nq, float (*xv)[MW], const u32x4* wv) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (q >= nq) break;
#pragma unroll
          for (int i = 0; i < MK; ++i) {
            const unsigned g = q == 0 ? wv[i].x : (q == 1 ? wv[i].y : (q == 2 ? wv[i].z : wv[i].w));
            const float f = UNI ? ws[i * 4 + q] : __builtin_bit_cast(float, g);
#pragma unroll
            for (int j = 0; j < MW; ++j) acc[i][j] = fmaf(f, xv[q][j], acc[i][j]);
          }
        }
      };
      const int nfull = nch / (4 * DU) * (4 * DU);
      if (nfull) {
#pragma unroll
        for (int u = 0; u < DU; ++u) {
          load(4 * u, 4, xq[u], wq[u]);
          __builtin_amdgcn_sched_barrier(0);
        }
        for (int c = 0; c + 4 * DU < nfull; c += 4 * DU) {
#pragma unroll
          for (int u = 0; u < DU; ++u) {
            if constexpr (UNI) scalars(c + 4 * u, ws);
            macs(4, xq[u], wq[u]);
            __builtin_amdgcn_sched_barrier(0);
            load(c + 4 * (u + DU), 4, xq[u], wq[u]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
        for (int u = 0; u < DU; ++u) {
          if constexpr (UNI) scalars(nfull - 4 * (DU - u), ws);
          macs(4, xq[u], wq[u]);
        }
      }
      for (int c = nfull; c < nch; c += 4) {  // (a channel past the range loads no x and adds nothing)
        load(c, nch - c, xq[0], wq[0]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (UNI) scalars(c, ws);
        macs(nch - c, xq[0], wq[0]);
      }
    }
  } else if constexpr (SC != 0) {
    // Registers only, filters of SC columns: the ring's unit is a filter row of
    // one channel. The window's words are read one by one (any padding) at a
    // row plus a column offset; either part outside the image sends the sum
    // past the buffer.
    constexpr int NW = (MW - 1) * STC + SC;
    constexpr int U = NW + (UNI ? 0 : SC * MK), D0 = (kLimit - MK * MW - NW - MK - (UNI ? 60 : 40)) / U;
    constexpr int D1 = 56 / (NW + (UNI ? 0 : 2 * MK)), D2 = D0 < D1 ? D0 : D1, D = D2 < 1 ? 1 : (D2 > 4 ? 4 : D2);
    unsigned xo[NW], kofs[MK];
    const int kb = UNI ? __builtin_amdgcn_readfirstlane(kbase) : kbase;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      const int gw = ow * STC - pw + j;
      xo[j] = (unsigned)gw < (unsigned)W ? (unsigned)gw * 4 : kOob;
    }
#pragma unroll
    for (int i = 0; i < MK; ++i) kofs[i] = (unsigned)(min(kb + i, K - 1) * C * RS) * 4;
    const int gh0 = oh < a.OH ? oh * sh - ph : -R * dh;  // (every row outside)
    const int NU = (c_end - c_begin) * R;
    const int64_t wbytes = ((int64_t)K * C - c_begin) * RS * 4;
    float xq[D][NW], wq[D][SC * MK];
    auto load = [&](const int u, const int c, const int r, float* xv, float* wv) __attribute__((always_inline)) {
      const int gh = gh0 + r * dh;
      const unsigned ro = (unsigned)gh < (unsigned)H ? (unsigned)(gh * W) * 4 : kOob;
      const __amdgpu_buffer_rsrc_t rx = make_rsrc(xn + (int64_t)(c_begin + c) * HW, (int64_t)HW * 4);
#pragma unroll
      for (int j = 0; j < NW; ++j) xv[j] = bload1(rx, ro + xo[j]);
      if constexpr (!UNI) {
        const int64_t at = (int64_t)u * SC * 4;
        const __amdgpu_buffer_rsrc_t rw = make_rsrc(w + (int64_t)c_begin * RS + (int64_t)u * SC, wbytes - at);
#pragma unroll
        for (int i = 0; i < MK; ++i) bload_words<SC>(rw, kofs[i], wv + i * SC);
      }
    };
    auto macs = [&](const int u, const float* xv, const float* wv) __attribute__((always_inline)) {
      const float* wu = w + (int64_t)c_begin * RS + (int64_t)u * SC;
#pragma unroll
      for (int s = 0; s < SC; ++s)
#pragma unroll
        for (int i = 0; i < MK; ++i) {
          const float f = UNI ? wu[(int64_t)min(kb + i, K - 1) * C * RS + s] : wv[i * SC + s];
#pragma unroll
          for (int j = 0; j < MW; ++j) acc[i][j] = fmaf(f, xv[j * STC + s], acc[i][j]);
        }
    };
    int c = 0, r = 0;  // of the next unit to load
    auto next = [&]() __attribute__((always_inline)) {
      const bool wrap = ++r == R;
      c += wrap ? 1 : 0;
      r = wrap ? 0 : r;
    };
    int u = 0;
    if (NU >= D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        load(d, c, r, xq[d], wq[d]);
        next();
        __builtin_amdgcn_sched_barrier(0);
      }
      for (; u + 2 * D <= NU; u += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          macs(u + d, xq[d], wq[d]);
          __builtin_amdgcn_sched_barrier(0);
          load(u + D + d, c, r, xq[d], wq[d]);
          next();
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int d = 0; d < D; ++d) macs(u + d, xq[d], wq[d]);
      u += D;
    }
    for (; u < NU; ++u) {
      load(u, c, r, xq[0], wq[0]);
      next();
      macs(u, xq[0], wq[0]);
    }
  } else {
    // Registers only, any filter: one tap group at a time.
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(xn, (int64_t)C * HW * 4);
    auto direct = [&](const int kb) __attribute__((always_inline)) {
      // filter rows of this thread's channels; a channel past K reads row
      // K-1 (its sums are never stored)
      const float* wrow[MK];
#pragma unroll
      for (int i = 0; i < MK; ++i) wrow[i] = w + (int64_t)min(kb + i, K - 1) * C * RS;
#pragma unroll UNR
      for (int c = c_begin; c < c_end; ++c) {
        const int xo = c * HW;
        const int co = c * RS;
        for (int r = 0; r < R; ++r) {
          const int gh = oh * sh - ph + r * dh;
          const bool hok = (unsigned)gh < (unsigned)H && oh < a.OH;
          // the taps of a filter row go in groups of G, all of a group's
          // loads before its MACs (one memory round trip per group, not per
          // tap); taps past the row's end load and add nothing. G = 2 where
          // the launch bound leaves 128 registers and a tap loads 6 or more
          // values.
          constexpr int G = direct_max_threads(MK * MW) >= 1024 && MK + MW >= 6 ? 2 : 4;
          for (int s0 = 0; s0 < S; s0 += G) {
            float xv[G][MW], wv[G][MK];
#pragma unroll
            for (int u = 0; u < G; ++u) {
              if (u == 0 || s0 + u < S) {
                const int s = s0 + u;
#pragma unroll
                for (int j = 0; j < MW; ++j) {
                  const int gw = (ow + j * cj) * sw - pw + s * dw;
                  xv[u][j] = bload1(rx, hok && (unsigned)gw < (unsigned)W ? (unsigned)(xo + gh * W + gw) * 4 : kOob);
                }
#pragma unroll
                for (int i = 0; i < MK; ++i) wv[u][i] = wrow[i][co + r * S + s];
              }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < G; ++u) {
              if (u > 0 && s0 + u >= S) break;
#pragma unroll
              for (int i = 0; i < MK; ++i)
#pragma unroll
                for (int j = 0; j < MW; ++j) acc[i][j] = fmaf(wv[u][i], xv[u][j], acc[i][j]);
            }
          }
        }
      }
    };
    if ((a.tp & 63) == 0)
      direct(__builtin_amdgcn_readfirstlane(kbase));
    else
      direct(kbase);
  }

  if (oh >= a.OH) return;
  float* o = out + (int64_t)sp * a.ny + (((int64_t)n * K + kbase) * a.OH + oh) * a.OW + ow;
  const int64_t ohw = (int64_t)a.OH * a.OW;
#pragma unroll
  for (int i = 0; i < MK; ++i) {
    if (kbase + i >= K) break;
    float* oi = o + i * ohw;
    if constexpr (CONSEC && MW > 1) {
      if (ow + MW <= a.OW) {  // 8- or 16-byte stores (4-byte aligned ones are legal)
        if constexpr (MW == 4) {
          f32x4u q;
          q.x = acc[i][0]; q.y = acc[i][1]; q.z = acc[i][2]; q.w = acc[i][3];
          *(f32x4u*)oi = q;
        } else {
          f32x2u q;
          q.x = acc[i][0]; q.y = acc[i][1];
          *(f32x2u*)oi = q;
        }
        continue;
      }
    }
#pragma unroll
    for (int j = 0; j < MW; ++j)
      if (ow + j * cj < a.OW) oi[j * cj] = acc[i][j];
  }
}

using DirectFn = void (*)(const float*, const float*, float*, DirectArgs);


// The unroll knob is the generic paths' only; those without LDS have no ALT variant.
template <int MK, int MW, bool LDS, int SPEC>
static DirectFn pick_unr(int unr, bool alt) {
  if constexpr (SPEC != 0) {
    return alt ? (DirectFn)direct_f32_kernel<MK, MW, LDS, SPEC, 1, true>
               : (DirectFn)direct_f32_kernel<MK, MW, LDS, SPEC, 1, false>;
  } else {
    if (LDS && alt)
      return unr == 2 ? (DirectFn)direct_f32_kernel<MK, MW, LDS, SPEC, 2, LDS>
                      : (DirectFn)direct_f32_kernel<MK, MW, LDS, SPEC, 1, LDS>;
    return unr == 2 ? (DirectFn)direct_f32_kernel<MK, MW, LDS, SPEC, 2, false>
                    : (DirectFn)direct_f32_kernel<MK, MW, LDS, SPEC, 1, false>;
  }
}
template <int MK, int MW, bool LDS>
static DirectFn pick_spec(int spec, int unr, bool alt) {
  switch (spec) {
    case SPEC_1X1_S1: return pick_unr<MK, MW, LDS, 1>(unr, alt);
    case SPEC_1X1_S2: return pick_unr<MK, MW, LDS, 2>(unr, alt);
    case SPEC_3X3_S1: return pick_unr<MK, MW, LDS, 3>(unr, alt);
    case SPEC_3X3_S2: return pick_unr<MK, MW, LDS, 4>(unr, alt);
    case SPEC_ROW5_S1: return pick_unr<MK, MW, LDS, 5>(unr, alt);
    case SPEC_ROW5_S2: return pick_unr<MK, MW, LDS, 6>(unr, alt);
    case SPEC_ROW7_S1: return pick_unr<MK, MW, LDS, 7>(unr, alt);
    case SPEC_ROW7_S2: return pick_unr<MK, MW, LDS, 8>(unr, alt);
    default: return pick_unr<MK, MW, LDS, 0>(unr, alt);
  }
}
template <int MK, int MW>
static DirectFn pick_lds(int lds, int spec, int unr, bool alt) {
  return lds ? pick_spec<MK, MW, true>(spec, unr, alt) : pick_spec<MK, MW, false>(spec, unr, alt);
}
template <int MK>
DirectFn pick_mw(int mw, int lds, int spec, int unr, bool alt) {
  switch (mw) {
    case 1: return pick_lds<MK, 1>(lds, spec, unr, alt);
    case 2: return pick_lds<MK, 2>(lds, spec, unr, alt);
    default: return pick_lds<MK, 4>(lds, spec, unr, alt);
  }
}
}  // namespace ct
