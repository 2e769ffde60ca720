// Convolutional prediction (section 4.3's prediction workload on the paper's
// convolutional case) with the maps of several layers kept on chip: one
// workgroup takes a group of images of one variant through a segment of the
// net, layer by layer, from LDS to LDS.  A stage is a layer that produces a
// map on the matrix cores (the 3x3 stem or a pointwise layer) together with
// the 3x3 depthwise layer that reads it; the produced map itself never exists:
//   - a 32-pixel x 32-channel tile comes out of 32x32x16 bf16 MFMAs with lane l
//     holding channel l % 32 and 16 consecutive pixels of a row (the pixel a
//     tile row stands for is chosen so: tile row m is pixel 4 (m / 8) + m % 4 of
//     lane half (m / 4) % 2), biased, rectified and packed to bf16 pairs;
//   - the depthwise layer runs in those registers: a lane owns its channel's
//     taps and adds each produced row to the output rows it belongs to (dot2 for
//     two taps on an aligned pair, an fma for the third);
//   - its outputs, rounded to bf16, go to the next map in LDS ([pixel][channel],
//     two channels per write after an exchange between neighbouring lanes).
// Rows are dealt to the waves in ranges; a range recomputes the one or two
// produced rows it shares with its neighbour.  Maps wider than 16 pixels give
// each lane half one half of a row (the pixel across the middle comes by a
// lane exchange), narrower ones give the halves different row ranges.
// The layer-by-layer kernels moved every map through memory and re-read nine
// neighbours per depthwise output from LDS: 139 ms for 64 variants of the
// 32x32 net (stem 32, blocks 128 to 512) over 10,000 images, 66.2 ms here; 0.72
// and 0.10 ms for 6 variants of an 8x8 net over 600 images.  Bound by vector
// instructions: about 200 a lane for each 32 x 32 tile of a produced map
// (rectify and round 24, depthwise 50 to 100, its output 40, addresses), at two
// waves per SIMD, with the matrix cores busy an eighth of the time.  Per image
// of that net the three stages of the first segment take 15, 18 and 14 thousand
// cycles, the second segment 11 thousand.
// Loading the next group's images during the first stage instead of the last,
// and a stage's weights after instead of before the barrier, measured 69.4
// against 70.3 ms.  A stem that read its window rows from one copy of the
// image, elements at odd addresses included, took 19 thousand cycles for 15.
#include "gevo_cnn_fused.h"
#include "gevo_device.h"

namespace gevo {

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16_t seg_mma(u32x4_t a, u32x4_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                 0, 0, 0);
}

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_v, a), __builtin_bit_cast(bf16x2_v, b), c, false);
}
__device__ __forceinline__ float hi_f(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }
__device__ __forceinline__ float lo_f(uint32_t p) { return __uint_as_float(p << 16); }

// max(f, 0) of a value and its neighbour as a bf16 pair; NaN gives 0.  The
// median of (f, 0, largest float) is that in one instruction once rounded to
// bf16, which takes the largest float and infinity both to infinity (fmaxf
// takes two instructions, the first only quieting NaNs).
__device__ __forceinline__ float relu(float f) { return __builtin_amdgcn_fmed3f(f, 0.0f, 3.4028234663852886e38f); }
__device__ __forceinline__ uint32_t relu_pair(float a, float b) { return bf16x2(relu(a), relu(b)); }

// One channel's 3x3 taps: t01/t12 = bf16 pairs (w0, w1) and (w1, w2) of each
// row, f0/f2 = w0 and w2 of each row as floats.
struct Taps {
  uint32_t t01[3], t12[3];
  float f0[3], f2[3];
  float bias;
};

__device__ __forceinline__ Taps load_taps(const uint32_t* pairs, const float* bias, int C, int c) {
  uint32_t p[5];                                   // taps (0,1) (2,3) (4,5) (6,7) (8,-), tap 3 dy + dx
#pragma unroll
  for (int i = 0; i < 5; ++i) p[i] = pairs[i * C + c];
  Taps t;
  t.bias = bias[c];
  t.t01[0] = p[0];
  t.t12[0] = (p[0] >> 16) | (p[1] << 16);
  t.t01[1] = (p[1] >> 16) | (p[2] << 16);
  t.t12[1] = p[2];
  t.t01[2] = p[3];
  t.t12[2] = (p[3] >> 16) | (p[4] << 16);
  t.f0[0] = lo_f(p[0]); t.f2[0] = lo_f(p[1]);
  t.f0[1] = hi_f(p[1]); t.f2[1] = hi_f(p[2]);
  t.f0[2] = lo_f(p[3]); t.f2[2] = lo_f(p[4]);
  return t;
}

// A produced row of one lane: NP packed pixel pairs, the pixel left of the
// first and right of the last.
template <int NP> struct Row {
  uint32_t p[NP];
  float l, r;
};

// acc[xo] = from[xo] + row dy of the window of outputs xo, stride S (the fma
// first: it takes its addend from another register, dot2 adds in place)
template <int S, int NP, int NO, typename From>
__device__ __forceinline__ void dw_add(const Row<NP>& row, const Taps& t, int dy, float (&acc)[NO], From from) {
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const float left = j ? hi_f(row.p[j - 1]) : row.l;
    if constexpr (S == 2) {
      acc[j] = dot2(row.p[j], t.t12[dy], __builtin_fmaf(left, t.f0[dy], from(j)));
    } else {
      const float right = j + 1 < NP ? lo_f(row.p[j + 1]) : row.r;
      acc[2 * j] = dot2(row.p[j], t.t12[dy], __builtin_fmaf(left, t.f0[dy], from(2 * j)));
      acc[2 * j + 1] = dot2(row.p[j], t.t01[dy], __builtin_fmaf(right, t.f2[dy], from(2 * j + 1)));
    }
  }
}

// A range of q output rows.  next(rows) gives the lane's next RW produced
// rows, beginning RW == 2 && S == 2 ? two : one row(s) above the middle row of
// the first output's window; emit(k, acc) takes output row k.
template <int S, int RW, int NP, typename Next, typename Emit>
__device__ __forceinline__ void dw_rows(int q, const Taps& t, Next next, Emit emit) {
  constexpr int NO = S == 2 ? NP : 2 * NP;
  Row<NP> row[RW];
  float cur[NO];
  auto start = [&](int) { return t.bias; };
  auto go_on = [&](int j) { return cur[j]; };
  if constexpr (S == 2) {                          // rows 2 yo - 1 (odd), 2 yo (even), 2 yo + 1 (odd)
    next(row);
    dw_add<S>(row[RW - 1], t, 0, cur, start);
    for (int k = 0; k < q; ++k) {
      next(row);
      dw_add<S>(row[0], t, 1, cur, go_on);
      if constexpr (RW == 1) next(row);
      dw_add<S>(row[RW - 1], t, 2, cur, go_on);
      emit(k, cur);
      dw_add<S>(row[RW - 1], t, 0, cur, start);
    }
  } else {                                         // row y: last of output y - 1, middle of y, first of y + 1
    float nxt[NO];
    next(row);
    dw_add<S>(row[0], t, 0, nxt, start);
    auto middle = [&](const Row<NP>& r) {
      dw_add<S>(r, t, 1, cur, [&](int j) { return nxt[j]; });
      dw_add<S>(r, t, 0, nxt, start);
    };
    if constexpr (RW == 1) {
      next(row);
      middle(row[0]);
      for (int k = 0; k < q; ++k) {
        next(row);
        dw_add<S>(row[0], t, 2, cur, go_on);
        emit(k, cur);
        middle(row[0]);
      }
    } else {
      middle(row[1]);
      for (int k = 0; k < q; k += 2) {
        next(row);
        dw_add<S>(row[0], t, 2, cur, go_on);
        emit(k, cur);
        middle(row[0]);
        dw_add<S>(row[1], t, 2, cur, go_on);
        if (k + 1 < q) emit(k + 1, cur);
        middle(row[1]);
      }
    }
  }
}

// One stage for the group's images.  KS > 0: a pointwise producer with KS
// contraction steps whose input map is in LDS; KS == 0: the stem (a.st[0]).
template <int S, int WT, int KS>
__device__ __forceinline__ void stage_run(const CnnSegArgs& a, const CnnSegStage& st, char* smem, int v, int64_t img0,
                                          char* gout) {
  constexpr bool STEM = KS == 0;
  constexpr int NS = STEM ? 3 : KS;                // contraction steps
  constexpr int RW = WT == 8 ? 2 : 1, NP = WT == 8 ? 4 : 8, NO = S == 2 ? NP : 2 * NP;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  const int H = st.H, W = st.W, Ho = st.Ho, Wo = st.Wo, C = 32 * st.nct;
  const int wpc = 1 << st.wpc_log, q = st.q, parts = st.parts;
  // the pixel that this lane's row of an A operand stands for: lane half ah, run index ar
  const int ah = (l32 >> 2) & 1, ar = 4 * (l32 >> 3) + (l32 & 3);
  const int ax = WT == 32 ? 16 * ah + ar : WT == 16 ? ar : ar & 7, ary = WT == 8 ? ar >> 3 : 0;
  const int axc = ax < W ? ax : W - 1;
  // exchange of neighbouring channels: an even lane keeps the low halves, an odd one the high halves
  const uint32_t sel = (lane & 1) ? 0x03020706u : 0x05040100u;
  const bool wide = WT == 32;
  // stem: the slots of a step that are taps (the others read past the row of
  // the window and are masked)
  u32x4_t tmask{};
  if constexpr (STEM) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = 8 * lh + 2 * j;
      tmask[j] = (e < 3 * a.stem_c ? 0xffffu : 0u) | (e + 1 < 3 * a.stem_c ? 0xffff0000u : 0u);
    }
  }
  // a channel tile's weights, taps and biases
  u32x4_t w[NS];
  Taps taps;
  f32x16_t bc;                                     // the producer's bias in every accumulator row
  int c = 0;
  auto weights = [&](int ct) {
    const uint16_t* wp = st.wp + ((size_t)v * st.nct + ct) * NS * 512 + lane * 8;
#pragma unroll
    for (int s = 0; s < NS; ++s) w[s] = *reinterpret_cast<const u32x4_t*>(wp + s * 512);
    c = 32 * ct + l32;
    taps = load_taps(st.taps + (size_t)v * 5 * C, st.db + (size_t)v * C, C, c);
    const float b = st.pb[(size_t)v * C + c];
#pragma unroll
    for (int r = 0; r < 16; ++r) bc[r] = b;
  };
  const int ct0 = wave >> st.wpc_log;
  __syncthreads();                                 // the stage's input map is complete
  for (int ct = ct0; ct < st.nct; ct += kSegWaves >> st.wpc_log) {
    weights(ct);
    for (int img = 0, part = wave & (wpc - 1);; part += wpc) {
      while (part >= parts) { part -= parts; ++img; }
      if (img >= a.G) break;
      // output rows [r0 q, r0 q + q) of range r0 = part (wide) or 2 part + half
      const int ya0 = (wide ? part : 2 * part) * q, ya1 = wide ? ya0 : ya0 + q;
      if (ya0 >= Ho) continue;
      auto base_of = [&](int ya) { return S == 2 ? 2 * ya - RW : ya - 1; };   // first produced row
      const int b0 = base_of(ya0), b1 = base_of(ya1);
      const int ybA = (ah ? b1 : b0) + ary, ybD = lh ? b1 : b0, yoD = lh ? ya1 : ya0;
      const char* src = smem + (STEM ? 0 : st.in) + (size_t)img * st.img_in;
      // Three tiles are under way: one whose operands are being read from LDS,
      // one on the matrix cores, one in the depthwise layer.
      // (256 input channels hold too many weights for the first to be kept)
      constexpr bool DEEP = KS <= 8;
      u32x4_t op[DEEP ? NS : 1];
      auto load = [&](int t) {
        if constexpr (!DEEP) return;
        const int y = ybA + RW * t, yc = y < 0 ? 0 : (y < H ? y : H - 1);
        if constexpr (STEM) {
          // rows of the window, 16 elements each from the even or the odd copy
          int e = (yc * (W + 2) + axc) * a.stem_c;
#pragma unroll
          for (int s = 0; s < NS; ++s, e += (W + 2) * a.stem_c) {
            const uint32_t* im = reinterpret_cast<const uint32_t*>(src + seg_window(a.im, a.im2, e)) + 4 * lh;
#pragma unroll
            for (int j = 0; j < 4; ++j) op[s][j] = im[j];
          }
        } else {
          const char* ap = src + (yc * W + axc) * st.ps_in + 16 * lh;
#pragma unroll
          for (int s = 0; s < (DEEP ? NS : 0); ++s) op[s] = *reinterpret_cast<const u32x4_t*>(ap + 32 * s);
        }
      };
      auto multiply = [&](int t) {
        f32x16_t acc = bc;
        if constexpr (!DEEP) {
          const int y = ybA + RW * t, yc = y < 0 ? 0 : (y < H ? y : H - 1);
          const char* ap = src + (yc * W + axc) * st.ps_in + 16 * lh;
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            acc = seg_mma(*reinterpret_cast<const u32x4_t*>(ap + 32 * s), w[s], acc);
            if (s % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // at most four operands at a time
          }
          return acc;
        }
#pragma unroll
        for (int s = 0; s < (DEEP ? NS : 0); ++s)
          acc = seg_mma(STEM ? op[s] & tmask : op[s], w[s], acc);
        return acc;
      };
      load(0);
      f32x16_t ahead = multiply(0);
      load(1);
      int t = 0;
      auto next = [&](Row<NP> (&row)[RW]) {
        const f32x16_t acc = ahead;
        ahead = multiply(t + 1);
        load(t + 2);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
#pragma unroll
          for (int j = 0; j < NP; ++j) row[r].p[j] = relu_pair(acc[r * 2 * NP + 2 * j], acc[r * 2 * NP + 2 * j + 1]);
        }
        const int ya = b0 + RW * t, yb = b1 + RW * t;
        if (ya < 0 || yb < 0 || ya + RW > H || yb + RW > H) {   // rows outside the image are zero
          asm volatile("");                        // (a branch: seldom taken)
#pragma unroll
          for (int r = 0; r < RW; ++r) {
            const int yd = ybD + RW * t + r;
            const bool in = yd >= 0 && yd < H;
#pragma unroll
            for (int j = 0; j < NP; ++j) row[r].p[j] = in ? row[r].p[j] : 0u;
          }
        }
        if (W < WT) {                              // columns past the image are zero
          int w_ = W - (wide ? 16 * lh : 0);
          asm volatile("" : "+v"(w_));             // (the masks stay in here)
#pragma unroll
          for (int j = 0; j < NP; ++j) {
            const uint32_t m = (2 * j < w_ ? 0xffffu : 0u) | (2 * j + 1 < w_ ? 0xffff0000u : 0u);
#pragma unroll
            for (int r = 0; r < RW; ++r) row[r].p[j] &= m;
          }
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) {
          row[r].l = row[r].r = 0.0f;
          if constexpr (WT == 32) {
            // the pixel across the middle of the row: the upper half gets the
            // lower half's last pair, the lower half the upper half's first
            const auto sw = __builtin_amdgcn_permlane32_swap(row[r].p[0], row[r].p[NP - 1], false, false);
            row[r].l = lh ? hi_f(sw[0]) : 0.0f;
            if (S == 1) row[r].r = lh ? 0.0f : lo_f(sw[1]);
          }
        }
        ++t;
      };
      char* dst = gout ? gout + (size_t)img * st.img_out : smem + st.out + (size_t)img * st.img_out;
      const bool image_ok = !gout || img0 + img < a.n_test;
      auto emit = [&](int k, const float (&o)[NO]) {
        const int yo = yoD + k;
        const bool row_ok = k < q && yo < Ho && image_ok;
        const int xb = (wide ? lh * NO : 0) + (lane & 1);
        char* d = dst + ((size_t)yo * Wo + xb) * st.ps_out + (c & ~1) * 2;
#pragma unroll
        for (int i = 0; i < NO / 2; ++i) {
          const uint32_t own = relu_pair(o[2 * i], o[2 * i + 1]);
          const uint32_t nb = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
          const uint32_t val = __builtin_amdgcn_perm(nb, own, sel);
          if (row_ok && xb + 2 * i < Wo) *reinterpret_cast<uint32_t*>(d + 2 * i * st.ps_out) = val;
        }
      };
      dw_rows<S, RW, NP>(q, taps, next, emit);
    }
  }
}

template <int S, int WT>
__device__ __forceinline__ void stage_ks(const CnnSegArgs& a, const CnnSegStage& st, char* smem, int v, int64_t img0,
                                         char* gout) {
  switch (st.KS) {
    case 2: stage_run<S, WT, 2>(a, st, smem, v, img0, gout); break;
    case 4: stage_run<S, WT, 4>(a, st, smem, v, img0, gout); break;
    case 8: stage_run<S, WT, 8>(a, st, smem, v, img0, gout); break;
    default: stage_run<S, WT, 16>(a, st, smem, v, img0, gout);
  }
}

// Last pointwise layer and pooling: a lane's run of 16 pixels (lane half h of
// 32-pixel tile p: pixels 32 p + 16 h + 0..15 of the group's images laid end to
// end, each image's pixels padded to a multiple of 32 when it has more than
// 16, to t_run otherwise) is summed per image after rounding to bf16.
__device__ __forceinline__ void tail_run(const CnnSegArgs& a, const char* smem, int v, int64_t img0, int gi) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lh = lane >> 5, C = 32 * a.t_nct, HW = a.t_HW;
  const bool small = HW <= 16;
  const int tpi = (HW + 31) / 32;                              // tiles per image (large maps)
  const int ipr = small ? 16 / a.t_run : 0;                    // images per run (small maps)
  const int ntile = small ? (a.G + 2 * ipr - 1) / (2 * ipr) : a.G * tpi;
  const int ah = (l32 >> 2) & 1, ar = 4 * (l32 >> 3) + (l32 & 3);
  const float inv = 1.0f / (float)HW;
  for (int ct = wave; ct < a.t_nct; ct += kSegWaves) {
    const uint16_t* wp = a.t_wp + ((size_t)v * a.t_nct + ct) * a.t_KS * 512 + lane * 8;
    const int c = 32 * ct + l32;
    f32x16_t bc;
    {
      const float b = a.t_pb[(size_t)v * C + c];
#pragma unroll
      for (int r = 0; r < 16; ++r) bc[r] = b;
    }
    float sum = 0.0f;                                          // of the image in progress (large maps)
    for (int p0 = 0; p0 < ntile; p0 += 4) {
      // up to four tiles share each weight block
      const char* ap[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int p = p0 + u < ntile ? p0 + u : ntile - 1;
        int img, px;
        if (small) {
          img = (2 * p + ah) * ipr + ar / a.t_run;
          px = ar % a.t_run;
        } else {
          img = p / tpi;
          px = (p - img * tpi) * 32 + 16 * ah + ar;
        }
        img = img < a.G ? img : a.G - 1;
        px = px < HW ? px : HW - 1;
        ap[u] = smem + a.t_in + (size_t)img * a.t_img + px * a.t_ps + 16 * lh;
      }
      const int nu = ntile - p0 < 4 ? ntile - p0 : 4;
      f32x16_t acc[4] = {bc, bc, bc, bc};
      // eight steps' weights in flight while the eight before are used
      u32x4_t w[8], wn[8];
      auto fetch = [&](int s0, u32x4_t (&o)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          o[i] = *reinterpret_cast<const u32x4_t*>(wp + (size_t)(s0 + i < a.t_KS ? s0 + i : a.t_KS - 1) * 512);
      };
      fetch(0, w);
      for (int s0 = 0; s0 < a.t_KS; s0 += 8) {
        if (s0 + 8 < a.t_KS) fetch(s0 + 8, wn);
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (s0 + i < a.t_KS)
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (u < nu) acc[u] = seg_mma(*reinterpret_cast<const u32x4_t*>(ap[u] + 32 * (s0 + i)), w[i], acc[u]);
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = wn[i];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (u >= nu) continue;
        const int p = p0 + u;
        float f[16];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t pr = relu_pair(acc[u][2 * j], acc[u][2 * j + 1]);
          f[2 * j] = lo_f(pr);
          f[2 * j + 1] = hi_f(pr);
        }
        if (small) {
          float part = 0.0f;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int o = r & (a.t_run - 1);                   // t_run is a power of two
            if (o < HW) part += f[r];
            if (o == a.t_run - 1) {
              const int img = (2 * p + lh) * ipr + r / a.t_run;
              if (img < gi) a.pooled[a.pooled_vs * v + (size_t)(img0 + img) * C + c] = f32_to_bf16_bits(part * inv);
              part = 0.0f;
            }
          }
        } else {
          const int img = p / tpi, t = p - img * tpi, x0 = 32 * t + 16 * lh;
          float s = 0.0f;
#pragma unroll
          for (int r = 0; r < 16; ++r) s += x0 + r < HW ? f[r] : 0.0f;
          s += __shfl_xor(s, 32);
          sum = t == 0 ? s : sum + s;
          if (t == tpi - 1 && img < gi && lh == 0)
            a.pooled[a.pooled_vs * v + (size_t)(img0 + img) * C + c] = f32_to_bf16_bits(sum * inv);
        }
      }
    }
  }
}

}  // namespace

// One workgroup: a.per_wg groups of a.G images of one variant through the
// segment.  Its waves run at two per SIMD and the maps take most of a CU's LDS.
__global__ __launch_bounds__(64 * kSegWaves, 2) void k_cnn_seg(CnnSegArgs) {
  // the stages are indexed at run time: read from the kernel's argument
  // segment, where a copy by value would be indexed through scratch memory
  const CnnSegArgs& a = *(const CnnSegArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __align__(16) char smem[];
  // slot -> (variant, groups): neighbouring slots of an XCD share a variant's weights
  const int gx = gridDim.x, total = gx * gridDim.y, i0 = blockIdx.y * gx + blockIdx.x;
  const int j0 = total % 8 == 0 ? (i0 % 8) * (total / 8) + i0 / 8 : i0;
  const int v = j0 / gx, g0 = (j0 - v * gx) * a.per_wg;
  const int tid = threadIdx.x;
  // The group's padded images as bf16, one after the other in LDS, element i
  // of them by thread i % 512: read into registers (small images: during the
  // previous group's first stage), then written.
  constexpr int kPre = 8;
  const int W2 = a.W + 2, pitch = seg_pitch(a.H, a.W, a.stem_c), npad = a.stem_c ? pitch * a.G : 0;
  const bool ahead = npad <= kPre * 64 * kSegWaves;
  float pre[kPre];
  auto source = [&](int i) {                       // element i's place from the group's first pixel, ~0: border
    const int im = (int)__umulhi((uint32_t)i, a.pitch_magic), e = i - im * pitch;   // (the padding is a border)
    const int pix = a.stem_c == 1 ? e : (int)__umulhi((uint32_t)e, a.c_magic);   // (the magic of 1 does not fit)
    const int py = (int)__umulhi((uint32_t)pix, a.w2_magic), yy = py - 1, xx = pix - py * W2 - 1;
    return i < npad && yy >= 0 && yy < a.H && xx >= 0 && xx < a.W
               ? (uint32_t)(((im * a.H + yy) * a.W + xx) * a.stem_c + e - pix * a.stem_c) : ~0u;
  };
  auto fetch = [&](int g, int i0) {
    const int64_t first = a.img0 + (int64_t)g * a.G, left = a.n_test - first;
    const uint32_t have = (uint32_t)(left < a.G ? left : a.G) * (uint32_t)(a.H * a.W * a.stem_c);
    const float* x = a.x + (size_t)first * a.H * a.W * a.stem_c;
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
      const uint32_t f = source(i0 + u * 64 * kSegWaves + tid);
      pre[u] = f < have ? x[f] : 0.0f;
    }
  };
  auto store = [&](int i0) {
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
      const int i = i0 + u * 64 * kSegWaves + tid;
      const uint16_t h = f32_to_bf16_bits(pre[u]);
      if (i < npad) {
        reinterpret_cast<uint16_t*>(smem + a.im)[i] = h;
        reinterpret_cast<uint16_t*>(smem + a.im2)[i + 1] = h;
      }
    }
  };
  for (int g = g0; g < g0 + a.per_wg && g < a.groups; ++g) {
    const int64_t im0 = (int64_t)g * a.G;          // first image of the group within the launch
    const int64_t left = a.n_test - a.img0 - im0;
    const int gi = left < a.G ? (int)(left > 0 ? left : 0) : a.G;   // images of the group that exist
    __syncthreads();                               // the previous group's maps are read
    if (a.stem_c) {
      if (!ahead || g == g0) fetch(g, 0);
      store(0);
      for (int i0 = kPre * 64 * kSegWaves; i0 < npad; i0 += kPre * 64 * kSegWaves) {   // (images too large to hold)
        fetch(g, i0);
        store(i0);
      }
      if (ahead && g + 1 < g0 + a.per_wg && g + 1 < a.groups) fetch(g + 1, 0);   // arrives during the first stage
    } else {
      const int c8 = a.src_c / 8, n = a.src_px * c8 * gi;      // pieces of 16 bytes; the images are contiguous
      {
        const uint16_t* s = a.src + a.src_vs * v + (size_t)im0 * a.src_px * a.src_c;
        char* o = smem + a.src_off;
#pragma unroll 4
        for (int i = tid; i < n; i += 64 * kSegWaves) {
          const int px = (int)__umulhi((uint32_t)i, a.c8_magic);
          *reinterpret_cast<u32x4_t*>(o + px * a.src_ps + (i - px * c8) * 16) =
              *reinterpret_cast<const u32x4_t*>(s + (size_t)i * 8);
        }
      }
    }
    for (int k = 0; k < a.nst; ++k) {
      const CnnSegStage& st = a.st[k];
      char* gout = nullptr;
      if (k + 1 == a.nst && !a.tail)
        gout = reinterpret_cast<char*>(a.dst + a.dst_vs * v) + (size_t)im0 * st.img_out;
      const int64_t first = a.img0 + im0;
      if (k == 0 && a.stem_c) {
        if (st.S == 1) {
          if (st.wt == 32) stage_run<1, 32, 0>(a, st, smem, v, first, gout);
          else if (st.wt == 16) stage_run<1, 16, 0>(a, st, smem, v, first, gout);
          else stage_run<1, 8, 0>(a, st, smem, v, first, gout);
        } else {
          if (st.wt == 32) stage_run<2, 32, 0>(a, st, smem, v, first, gout);
          else if (st.wt == 16) stage_run<2, 16, 0>(a, st, smem, v, first, gout);
          else stage_run<2, 8, 0>(a, st, smem, v, first, gout);
        }
      } else if (st.S == 1) {
        if (st.wt == 32) stage_ks<1, 32>(a, st, smem, v, first, gout);
        else if (st.wt == 16) stage_ks<1, 16>(a, st, smem, v, first, gout);
        else stage_ks<1, 8>(a, st, smem, v, first, gout);
      } else {
        if (st.wt == 32) stage_ks<2, 32>(a, st, smem, v, first, gout);
        else if (st.wt == 16) stage_ks<2, 16>(a, st, smem, v, first, gout);
        else stage_ks<2, 8>(a, st, smem, v, first, gout);
      }
    }
    if (a.tail) {
      __syncthreads();
      tail_run(a, smem, v, im0, gi);
    }
  }
}

__global__ __launch_bounds__(256) void k_cnn_pack_op(const float* __restrict__ Wm, int Kp, int Np, int K, int KS, int run,
                                                     int P, uint16_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;      // ((v * nct + ct) * KS + s) * 64 + lane
  const int nct = Np / 32;
  if (i >= (int64_t)P * nct * KS * 64) return;
  const int lane = (int)(i & 63), s = (int)((i >> 6) % KS);
  const int64_t vt = (i >> 6) / KS;
  const int n = (int)(vt % nct) * 32 + (lane & 31), e0 = 8 * (lane >> 5);
  const float* w = Wm + (size_t)(vt / nct) * Np * Kp;
  uint32_t h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float f[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = e0 + 2 * j + u, k = s * run + e;
      f[u] = e < run && k < K ? w[((size_t)(k / 32) * Np + n) * 32 + k % 32] : 0.0f;
    }
    h[j] = bf16x2(f[0], f[1]);
  }
  *reinterpret_cast<uint4*>(out + i * 8) = make_uint4(h[0], h[1], h[2], h[3]);
}

hipError_t launch_cnn_seg(const CnnSegArgs& a, int P, hipStream_t s) {
  if (a.G < 1 || a.groups < 1 || a.per_wg < 1 || a.lds <= 0 || (size_t)a.lds > kSegLds - 256 || a.nst < 0 ||
      a.nst > kSegMaxStages || P < 1)
    return hipErrorInvalidValue;
  for (int k = 0; k < a.nst; ++k) {
    const CnnSegStage& t = a.st[k];
    const bool stem = k == 0 && a.stem_c;
    if ((t.S != 1 && t.S != 2) || (t.wt != 8 && t.wt != 16 && t.wt != 32) || t.W > t.wt || t.parts < 1 ||
        (stem ? t.KS != 3 : (t.KS != 2 && t.KS != 4 && t.KS != 8 && t.KS != 16)))
      return hipErrorInvalidValue;
  }
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_cnn_seg), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)(kSegLds - 256));
    attr = true;
  }
  hipLaunchKernelGGL(k_cnn_seg, dim3((a.groups + a.per_wg - 1) / a.per_wg, P), dim3(64 * kSegWaves), a.lds, s, a);
  return hipGetLastError();
}

hipError_t launch_cnn_pack_op(const float* Wm, int Kp, int Np, int K, int KS, int run, int P, uint16_t* out,
                              hipStream_t s) {
  if (Kp % 32 || Np % 32 || K > Kp || KS < 1 || run < 1 || run > 16 || KS * run < K) return hipErrorInvalidValue;
  const int64_t n = (int64_t)P * (Np / 32) * KS * 64;
  hipLaunchKernelGGL(k_cnn_pack_op, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Wm, Kp, Np, K, KS, run, P, out);
  return hipGetLastError();
}

}  // namespace gevo
