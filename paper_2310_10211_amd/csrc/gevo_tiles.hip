// Training and prediction kernels on tile-image operands (fully connected
// nets with hidden layers; section 6.2's SGD step, section 4.3's prediction).
//
// Every operand matrix is kept as 32 x 32 blocks in the order in which the
// matrix cores consume them: a block is [piece][lane][values], lane l holding
// row l % 32 and the contraction indexes crow(r, l) = 8 (r / 4) + 4 (l / 32) +
// r % 4, r = 0..15 (fp32: four 16-byte pieces of four values, bf16: two of
// eight).  A block is one wave's operand of a 32-deep contraction, read with
// contiguous 1 KiB loads (a row-major matrix costs one cache line per lane and
// load), and the order equals the accumulator order of a 32x32 MFMA (lane l:
// column l % 32, rows crow(r, l)), so a block that comes out of one product
// is stored, or fed to the next, without leaving its registers.
//   rows image  [row tile][input block][block]   lane = row,   contraction = inputs
//   cols image  [input block][row tile][block]   lane = input, contraction = rows
// The fp32 masters stay k-blocked ([Kp/32][Np][32]): lane l's 16-byte pieces
// of unit l % 32 are the same values in the same order.
//
// One SGD step: k_tile_out (logits, softmax cross-entropy, G_L and the
// gradient of the last hidden layer, per 32 batch rows), for three-layer nets
// k_tile_bwd, then per hidden layer k_tile_layer (weight gradient, masked
// update, next step's forward); the last hidden layer's launch also updates
// the output layer.
#include "gevo_internal.h"
#include "gevo_device.h"

#include <hip/hip_ext.h>
#include <math.h>

namespace gevo {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kBlk = 1024;               // values of a block
constexpr int kTP = 33;                  // row pitch (floats) of a transpose tile in LDS

// One 32 x 32 operand block: this lane's 16 values in crow order.
template <typename S> struct Blk;

template <> struct Blk<float> {
  f32x4_t q[4];
  __device__ __forceinline__ static Blk load(const float* p, int lane) {
    Blk b;
#pragma unroll
    for (int i = 0; i < 4; ++i) b.q[i] = *reinterpret_cast<const f32x4_t*>(p + i * 256 + lane * 4);
    return b;
  }
  __device__ __forceinline__ static Blk pack(const float (&f)[16]) {
    Blk b;
#pragma unroll
    for (int r = 0; r < 16; ++r) b.q[r >> 2][r & 3] = f[r];
    return b;
  }
  __device__ __forceinline__ void store(float* p, int lane) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4_t*>(p + i * 256 + lane * 4) = q[i];
  }
  __device__ __forceinline__ float val(int r) const { return q[r >> 2][r & 3]; }
  // offset of value r of lane l in a block
  __host__ __device__ static int off(int r, int l) { return (r >> 2) * 256 + l * 4 + (r & 3); }
};

template <> struct Blk<uint16_t> {
  u32x4_t q[2];
  __device__ __forceinline__ static Blk load(const uint16_t* p, int lane) {
    Blk b;
#pragma unroll
    for (int i = 0; i < 2; ++i) b.q[i] = *reinterpret_cast<const u32x4_t*>(p + i * 512 + lane * 8);
    return b;
  }
  __device__ __forceinline__ static Blk pack(const float (&f)[16]) {
    uint32_t h[8];
    to_bf16x2(f, h);
    Blk b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b.q[i >> 2][i & 3] = h[i];
    return b;
  }
  __device__ __forceinline__ void store(uint16_t* p, int lane) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) *reinterpret_cast<u32x4_t*>(p + i * 512 + lane * 8) = q[i];
  }
  __device__ __forceinline__ float val(int r) const {
    const uint32_t h = q[r >> 3][(r >> 1) & 3];
    return __uint_as_float((r & 1) ? h & 0xffff0000u : h << 16);
  }
  __host__ __device__ static int off(int r, int l) { return (r >> 3) * 512 + l * 8 + (r & 7); }
};

__device__ __forceinline__ f32x16_t blk_mma(const Blk<float>& a, const Blk<float>& b, f32x16_t c) {
#pragma unroll
  for (int r = 0; r < 16; ++r) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.q[r >> 2][r & 3], b.q[r >> 2][r & 3], c, 0, 0, 0);
  return c;
}

// Two independent products with their MFMAs alternating: a chain on one sum
// waits out each result (10% of the fp32 rate with one wave per SIMD).
__device__ __forceinline__ void blk_mma2(const Blk<float>& a0, const Blk<float>& b0, f32x16_t& c0, const Blk<float>& a1,
                                         const Blk<float>& b1, f32x16_t& c1) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.q[r >> 2][r & 3], b0.q[r >> 2][r & 3], c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.q[r >> 2][r & 3], b1.q[r >> 2][r & 3], c1, 0, 0, 0);
  }
}

__device__ __forceinline__ f32x16_t mma_bf16(u32x4_t a, u32x4_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                 0, 0, 0);
}
__device__ __forceinline__ f32x16_t blk_mma(const Blk<uint16_t>& a, const Blk<uint16_t>& b, f32x16_t c) {
  return mma_bf16(a.q[1], b.q[1], mma_bf16(a.q[0], b.q[0], c));
}
__device__ __forceinline__ void blk_mma2(const Blk<uint16_t>& a0, const Blk<uint16_t>& b0, f32x16_t& c0,
                                         const Blk<uint16_t>& a1, const Blk<uint16_t>& b1, f32x16_t& c1) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    c0 = mma_bf16(a0.q[i], b0.q[i], c0);
    c1 = mma_bf16(a1.q[i], b1.q[i], c1);
  }
}

// this lane's 16 values of a k-blocked fp32 master tile [32 units][32 inputs] (unit = lane % 32)
__device__ __forceinline__ void load_w(const float* tile, int lane, f32x4_t (&w)[4]) {
  const float* p = tile + (lane & 31) * 32 + 4 * (lane >> 5);
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = *reinterpret_cast<const f32x4_t*>(p + 8 * q);
}

// masked SGD step of the tile: w = keep ? fl(w - fl(lr d)) : +0, stored in place
__device__ __forceinline__ void update_w(float* tile, int lane, const f32x4_t (&w)[4], uint32_t mask, float lr,
                                         const f32x16_t& d, float (&wn)[16]) {
  float* p = tile + (lane & 31) * 32 + 4 * (lane >> 5);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const bool keep = (mask >> crow(r, lane)) & 1u;
    wn[r] = keep ? __fsub_rn(w[r >> 2][r & 3], __fmul_rn(lr, d[r])) : 0.0f;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<f32x4_t*>(p + 8 * q) = f32x4_t{wn[4 * q], wn[4 * q + 1], wn[4 * q + 2], wn[4 * q + 3]};
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// A wave's 32 x 32 values (lane = column l32, rows crow(r)) turned over
// through its LDS tile: lane = row l32, columns crow(r).
__device__ __forceinline__ void transpose16(float* tile, int lane, const float (&f)[16], float (&t)[16]) {
  const int l32 = lane & 31;
#pragma unroll
  for (int r = 0; r < 16; ++r) tile[crow(r, lane) * kTP + l32] = f[r];
  wave_sync();
#pragma unroll
  for (int r = 0; r < 16; ++r) t[r] = tile[l32 * kTP + crow(r, lane)];
  wave_sync();
}

}  // namespace

// ------------------------------------------------------------ hidden layer
// Workgroup (NT unit tiles of 32, variant v), NW waves: four, one per SIMD with
// the whole register file, or eight; wave j takes the input blocks j, j + NW,
// ...  For
// each block the wave forms, per unit tile,
//   dW[k][n] = sum_b A[b][k] G[b][n]            (A from the cols image, G from LDS)
// in accumulator order, applies the masked update to its 16 master values and
// feeds the new values straight to the next step's forward
//   Z[n][b] += sum_k W[n][k] X[b][k]            (X from the rows image)
// The waves' partial Z are summed through LDS in wave order; bias and ReLU
// follow, and the tile is written as both images.  With a.WL one wave also
// updates the output layer's input columns of these tiles (dW_L = G_L^T A over
// the step that just ended), and workgroup 0 its biases and the loss totals.
// fp32 is bound by the fp32 matrix cores (64 clocks per MFMA), which one wave
// per SIMD keeps busy when its operands arrive ahead of use and its MFMAs
// alternate between two sums; with two waves per SIMD the waves' loads and
// MFMAs got in each other's way (a probe of this loop: 512 workgroups 276 us
// two to a CU, 205 us one after the other).  NT = 2 halves the operand bytes.
// 64 variants of 784-256-10, batch 128: 75 us per launch, 88 TFLOP/s, where a
// kernel that read row-major operands a cache line per lane, one 32-unit tile
// of whole inputs per workgroup, took 133 us; the MFMAs alone are 43 us, 48
// with 25 input blocks on four waves.  4 variants of 784-128-10, batch 32:
// 16 us from 45.
template <int BT, int NT, int NW>
struct TileLayerLds {
  static constexpr int NTILE = NT * BT;                    // 32 x 32 output tiles
  static constexpr int TR = NTILE < 8 ? NTILE : 8;         // tiles per reduction round
  static constexpr size_t gs = (size_t)NTILE * kBlk * 4;
  static constexpr size_t red = (size_t)(NW - 1) * TR * kBlk * 4;
  static constexpr size_t tiles = gs > red ? gs : red;
  static constexpr size_t bytes = tiles + (size_t)TR * 32 * kTP * 4;
};

template <typename S, int BT, int NT, int NW, bool UPD, bool FWD>
__global__ __launch_bounds__(64 * NW, 1) void k_tile_layer(TileLayerArgs<S> a) {
  typedef TileLayerLds<BT, NT, NW> Ly;
  typedef Blk<S> B;
  using O = Op<S>;
  extern __shared__ __align__(16) char smem[];
  __shared__ float bias_l[32 * NT];
  S* gs = reinterpret_cast<S*>(smem);                      // [NT][BT] blocks of G (lane = unit, contraction = batch)
  float* red = reinterpret_cast<float*>(smem);             // after the loop: [NW - 1][TR][16][64]
  float* tiles = reinterpret_cast<float*>(smem + Ly::tiles);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31;
  const int nt = blockIdx.x * NT, v = blockIdx.y, n0 = nt * 32;
  const uint64_t vt0 = vt_now();
  if (a.wout && n0 >= (int)a.wout[v]) {                    // every unit of the tiles removed
    vt_add_wg(a.vtime, v, vt0);
    return;
  }
  const int KB = a.Kp / 32, NB = a.Np / 32;
  float* Wv = a.Wm + (size_t)v * a.Np * a.Kp + (size_t)n0 * 32;
  const uint32_t* mk = a.mask + ((size_t)v * a.Np + n0 + l32) * KB;
  const float lrv = UPD ? a.lr[v] : 0.0f;
  // This wave's blocks are j0, j0 + NW, ... of an order that starts at another
  // block in each workgroup of an XCD (workgroup i runs on XCD i % 8), so
  // they do not all ask the L2 for the same lines at once.
  const int j0 = (wave + blockIdx.x + v) % NW, base = (int)((v * gridDim.x + blockIdx.x) >> 3) % KB;
  const int cnt = (KB - j0 + NW - 1) / NW;                 // may be 0
  auto block_of = [&](int i) {
    const int j = j0 + NW * i + base;
    return j < KB ? j : j - KB;
  };
  const S* Ac = UPD ? a.Acols + v * a.ac_vs : nullptr;
  const S* Xr = FWD ? a.Xrows + v * a.xr_vs : nullptr;
  // Operand blocks of an input block in order of use, cols (update) then rows
  // (forward), go through the matrix cores U at a time; two groups are in
  // flight while one is multiplied.
  constexpr int U = NT > 1 || BT == 1 ? 1 : 2;
  constexpr int NG = (BT + U - 1) / U;                     // groups per phase (the last may be short)
  constexpr int PH = (UPD ? 1 : 0) + (FWD ? 1 : 0), NGT = PH * NG;
  struct Grp { B b[U]; };
  auto load_group = [&](int kb, int g) {
    Grp x;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool up = UPD && g < NG;
      const int i = (up || !UPD ? g : g - NG) * U + u;
      x.b[u] = up ? B::load(Ac + ((size_t)kb * BT + (i < BT ? i : 0)) * kBlk, lane)
                  : B::load(Xr + ((size_t)(i < BT ? i : 0) * KB + kb) * kBlk, lane);
    }
    return x;
  };
  auto load_master = [&](int kb, f32x4_t (&w)[NT][4], uint32_t (&mw)[NT]) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      load_w(Wv + ((size_t)kb * a.Np + 32 * n) * 32, lane, w[n]);
      mw[n] = UPD ? mk[(size_t)32 * n * KB + kb] : 0u;
    }
  };
  f32x4_t w[NT][4];
  uint32_t mw[NT];
  const int kb0 = cnt > 0 ? block_of(0) : 0;               // waves without a block load one and leave it
  load_master(kb0, w, mw);
  Grp xa = load_group(kb0, 0), xb = load_group(NGT > 1 ? kb0 : block_of(cnt > 1 ? 1 : 0) % KB, 1 % NGT);
  if constexpr (UPD) {
    const S* G = a.G + ((size_t)v * NB + nt) * BT * kBlk;
    constexpr int PER = 16 / (int)sizeof(S);
    for (int i = tid * PER; i < NT * BT * kBlk; i += 64 * NW * PER)
      *reinterpret_cast<uint4*>(gs + i) = *reinterpret_cast<const uint4*>(G + i);
    __syncthreads();
    // bias gradients: eight lanes per unit, fixed-order reduction
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      if (tid >= 256) break;
      const int nl = tid >> 3, lh = tid & 1, g = (tid >> 1) & 3;
      float s = 0.0f;
#pragma unroll
      for (int bt = 0; bt < BT; ++bt)
#pragma unroll
        for (int i = 0; i < 4; ++i) s += O::to_f32(gs[(n * BT + bt) * kBlk + B::off(4 * g + i, 32 * lh + nl)]);
      s += __shfl_xor(s, 1);
      s += __shfl_xor(s, 2);
      s += __shfl_xor(s, 4);
      if ((tid & 7) == 0) {
        const size_t bi = (size_t)v * a.Np + n0 + 32 * n + nl;
        const float bo = a.bias[bi];
        const bool bk = (a.bmask[(size_t)v * NB + nt + n] >> nl) & 1u;
        const float bn = bk ? __fsub_rn(bo, __fmul_rn(lrv, s)) : 0.0f;
        a.bias[bi] = bn;
        bias_l[32 * n + nl] = bn;
      }
    }
    if (a.WL) {
      if (j0 == NW - 1) {                                  // the wave with the fewest blocks
#pragma unroll 1
        for (int n = 0; n < NT; ++n) {
          float* tile = a.WL + ((size_t)v * NB + nt + n) * kBlk;
          f32x4_t wl[4];
          load_w(tile, lane, wl);
          const uint32_t ml = a.maskL[((size_t)v * 32 + l32) * NB + nt + n];
          f32x16_t d = zero16();
#pragma unroll
          for (int bt = 0; bt < BT; ++bt)
            d = blk_mma(B::load(a.Hcols + (((size_t)v * NB + nt + n) * BT + bt) * kBlk, lane),
                        B::load(a.GL + ((size_t)v * BT + bt) * kBlk, lane), d);
          float wn[16];
          update_w(tile, lane, wl, ml, a.lrL[v], d, wn);
        }
      }
      if (nt == 0 && tid < 32) {
        float db = 0.0f;
        for (int t = 0; t < BT; ++t) db += a.opdb[((size_t)v * BT + t) * 32 + tid];
        const float bo = a.biasL[(size_t)v * 32 + tid];
        const bool bk = (a.bmaskL[v] >> tid) & 1u;
        a.biasL[(size_t)v * 32 + tid] = bk ? __fsub_rn(bo, __fmul_rn(a.lrL[v], db)) : 0.0f;
      }
      if (nt == 0 && tid == 64) {
        double t = 0.0;
        unsigned int cc = 0;
        for (int u = 0; u < BT; ++u) { t += a.opce[(size_t)v * BT + u]; cc += a.opcorr[(size_t)v * BT + u]; }
        a.ce_acc[v] += t;
        a.correct_acc[v] += cc;
      }
    }
  } else if (tid < 32 * NT) {
    bias_l[tid] = a.bias[(size_t)v * a.Np + n0 + tid];
  }

  f32x16_t z[NT][FWD ? BT : 1];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int t = 0; t < (FWD ? BT : 1); ++t) z[n][t] = zero16();
  // The next block's master words are loaded between update and forward; the
  // fences keep the loads where they are issued.
  for (int i = 0; i < cnt; ++i) {
    const int kb = block_of(i), kn = block_of(i + 1 < cnt ? i + 1 : i);   // past the end: unused re-reads
    Grp x[NGT + 2];
    x[0] = xa;
    x[1] = xb;
    auto ahead = [&](int g) {                              // group g + 2, of this block or the ones after it
      const int e = g + 2;
      x[e] = load_group(e < NGT ? kb : e < 2 * NGT ? kn : block_of(i + 2 < cnt ? i + 2 : cnt - 1), e % NGT);
      __builtin_amdgcn_sched_barrier(0);
    };
    B wb[NT];
    if constexpr (UPD) {
      f32x16_t d[2];
      d[0] = zero16();
      d[1] = zero16();
      B ga[NG + 1], gb[NG + 1];                            // G of group g, read from LDS a group ahead
      auto load_g = [&](int g) {
        ga[g] = B::load(gs + U * g * kBlk, lane);
        if (NT == 2) gb[g] = B::load(gs + (BT + g) * kBlk, lane);
        else if (U == 2 && 2 * g + 1 < BT) gb[g] = B::load(gs + (2 * g + 1) * kBlk, lane);
      };
      load_g(0);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + 1 < NG) load_g(g + 1);
        ahead(g);
        if constexpr (NT == 2) blk_mma2(x[g].b[0], ga[g], d[0], x[g].b[0], gb[g], d[1]);
        else if (U == 2 && 2 * g + 1 < BT) blk_mma2(x[g].b[0], ga[g], d[0], x[g].b[U - 1], gb[g], d[1]);
        else d[0] = blk_mma(x[g].b[0], ga[g], d[0]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (NT == 1 && U == 2) d[0] += d[1];
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        float wn[16];
        update_w(Wv + ((size_t)kb * a.Np + 32 * n) * 32, lane, w[n], mw[n], lrv, d[n], wn);
        wb[n] = B::pack(wn);
      }
    } else {
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        float wn[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) wn[r] = w[n][r >> 2][r & 3];
        wb[n] = B::pack(wn);
      }
    }
    load_master(kn, w, mw);
    if constexpr (FWD) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int j = g + (UPD ? NG : 0);
        ahead(j);
        if constexpr (NT == 2) blk_mma2(wb[0], x[j].b[0], z[0][g], wb[NT - 1], x[j].b[0], z[NT - 1][g]);
        else if (U == 2 && 2 * g + 1 < BT) blk_mma2(wb[0], x[j].b[0], z[0][(U * g) % BT], wb[0], x[j].b[U - 1], z[0][(U * g + 1) % BT]);
        else z[0][U * g] = blk_mma(wb[0], x[j].b[0], z[0][U * g]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    xa = x[NGT];
    xb = x[NGT + 1];
  }
  if constexpr (FWD) {
#pragma unroll
    for (int r0 = 0; r0 < Ly::NTILE; r0 += Ly::TR) {
      __syncthreads();                                     // G (first round) or the previous round is read
#pragma unroll
      for (int tt = 0; tt < Ly::TR; ++tt) {
        const int e = r0 + tt, own = tt % NW;
        if (e >= Ly::NTILE) continue;
        if (wave != own) {
          float* dst = red + ((wave < own ? wave : wave - 1) * Ly::TR + tt) * kBlk + lane;
#pragma unroll
          for (int r = 0; r < 16; ++r) dst[r * 64] = z[e / BT][e % BT][r];
        }
      }
      __syncthreads();
#pragma unroll
      for (int tt = 0; tt < Ly::TR; ++tt) {
        const int e = r0 + tt, own = tt % NW;
        if (e >= Ly::NTILE) continue;
        if (wave == own) {
          const int n = e / BT, t = e % BT;
          float f[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) f[r] = 0.0f;
#pragma unroll
          for (int p = 0; p < NW; ++p) {                   // partial sums in wave order
            if (p == own) {
#pragma unroll
              for (int r = 0; r < 16; ++r) f[r] += z[n][t][r];
            } else {
              const float* src = red + ((p < own ? p : p - 1) * Ly::TR + tt) * kBlk + lane;
#pragma unroll
              for (int r = 0; r < 16; ++r) f[r] += src[r * 64];
            }
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float zz = f[r] + bias_l[32 * n + crow(r, lane)];
            f[r] = zz > 0.0f ? zz : 0.0f;
          }
          B::pack(f).store(a.Orows + (((size_t)v * BT + t) * NB + nt + n) * kBlk, lane);
          float ft[16];
          transpose16(tiles + tt * 32 * kTP, lane, f, ft);
          B::pack(ft).store(a.Ocols + (((size_t)v * NB + nt + n) * BT + t) * kBlk, lane);
        }
      }
    }
  }
  vt_add_wg(a.vtime, v, vt0);
}

// ------------------------------------------------------------ output layer
namespace {

// Softmax cross-entropy of one row held by the lane pair (l, l ^ 32): z[r] is
// the logit of class crow(r, lane).  Lowest index on argmax ties, a NaN logit
// is a miss and makes the loss NaN.
__device__ __forceinline__ void row_softmax(const float (&z)[16], int C, int y, int lane, float (&ex)[16], float& sm,
                                            float& ce, bool& hit) {
  float m = -INFINITY, bv = -INFINITY;
  int bi = 64, nanl = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int c = crow(r, lane);
    if (c < C) {
      m = fmaxf(m, z[r]);
      if (z[r] != z[r]) nanl = 1;
      else if (z[r] > bv) { bv = z[r]; bi = c; }
    }
  }
  m = fmaxf(m, __shfl_xor(m, 32));
  nanl |= __shfl_xor(nanl, 32);
  const float ov = __shfl_xor(bv, 32);
  const int oi = __shfl_xor(bi, 32);
  if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  float sl = 0.0f, zy = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int c = crow(r, lane);
    ex[r] = c < C ? expf(z[r] - m) : 0.0f;
    sl += ex[r];
    if (c == y) zy = z[r];
  }
  sm = sl + __shfl_xor(sl, 32);
  zy += __shfl_xor(zy, 32);                                // exactly one lane of the pair holds class y
  ce = (logf(sm) + m) - zy;
  if (nanl) ce = NAN;
  hit = !nanl && bi == y;
}

}  // namespace

// Training, one workgroup per (32 batch rows rt, variant v), four waves:
// logits (classes x rows, the input blocks dealt to the waves, partial sums
// added in wave order by every wave), softmax, G_L = (p - y) scale; then the
// waves form the last hidden layer's gradient per 32 inputs,
//   G[b][n] = (sum_c G_L[b][c] W_L[c][n]) [A[b][n] > 0],
// with pre-update weights read transposed (one 128-byte line per class).  G_L,
// its class sums, the loss and the hits go to memory for the layer launch
// that updates W_L.  Bound by the latency of its dependent steps, so every
// operand of a wave's first input block is loaded at the start.
template <typename S>
__global__ __launch_bounds__(256) void k_tile_out(TileOutArgs<S> a) {
  typedef Blk<S> B;
  constexpr int NW = 4;
  __shared__ float red[NW][16][64];
  __shared__ float tile[32 * kTP];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31;
  const int rt = blockIdx.x, v = blockIdx.y;
  const uint64_t vt0 = vt_now();
  const int NB = a.Kp / 32, BT = a.Bp / 32;
  const float* WL = a.WL + (size_t)v * NB * kBlk;
  auto rows_at = [&](int nb) { return (((size_t)v * BT + rt) * NB + nb) * kBlk; };
  auto cols_at = [&](int nb) { return (((size_t)v * NB + nb) * BT + rt) * kBlk; };
  auto load_wt = [&](int nb, float (&wt)[16]) {            // lane = input, contraction = classes
#pragma unroll
    for (int r = 0; r < 16; ++r) wt[r] = WL[(size_t)nb * kBlk + crow(r, lane) * 32 + l32];
  };
  const int y = a.labels[rt * 32 + l32];
  const int nb0 = wave < NB ? wave : 0;                    // waves without a block load block 0 and leave it
  f32x4_t w4[4];
  load_w(WL + (size_t)nb0 * kBlk, lane, w4);
  B hr = B::load(a.Arows + rows_at(nb0), lane);
  float bias[16], wt[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) bias[r] = a.bias[(size_t)v * 32 + crow(r, lane)];
  load_wt(nb0, wt);
  B hc = B::load(a.Acols + cols_at(nb0), lane);
  const B hr0 = hr;
  f32x16_t acc = zero16();
  for (int nb = wave; nb < NB; nb += NW) {
    if (nb != wave) {
      load_w(WL + (size_t)nb * kBlk, lane, w4);
      hr = B::load(a.Arows + rows_at(nb), lane);
    }
    float wf[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) wf[r] = w4[r >> 2][r & 3];
    acc = blk_mma(B::pack(wf), hr, acc);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
  __syncthreads();
  float z[16], ex[16], g[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float s = red[0][r][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[w][r][lane];
    z[r] = s + bias[r];
  }
  float sm, ce;
  bool hit;
  row_softmax(z, a.C, y, lane, ex, sm, ce, hit);
  const bool rvalid = y >= 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int c = crow(r, lane);
    const float sc = a.gscale ? a.gscale[((size_t)v * a.Bp + rt * 32 + l32) * 32 + c] : a.scale;
    g[r] = (c < a.C && rvalid) ? (ex[r] / sm - (c == y ? 1.0f : 0.0f)) * sc : 0.0f;
  }
  const B gb = B::pack(g);                                 // lane = row, contraction = classes
  for (int nb = wave; nb < NB; nb += NW) {
    if (nb != wave) {
      load_wt(nb, wt);
      hc = B::load(a.Acols + cols_at(nb), lane);
    }
    const B wb = B::pack(wt);
    {
      const f32x16_t d = blk_mma(gb, wb, zero16());        // rows = batch, columns = inputs
      float f[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) f[r] = hc.val(r) > 0.0f ? d[r] : 0.0f;
      B::pack(f).store(a.Gcols + cols_at(nb), lane);
    }
    if (a.Grows) {
      const B h = nb == wave ? hr0 : B::load(a.Arows + rows_at(nb), lane);
      const f32x16_t d = blk_mma(wb, gb, zero16());        // rows = inputs, columns = batch
      float f[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) f[r] = h.val(r) > 0.0f ? d[r] : 0.0f;
      B::pack(f).store(a.Grows + rows_at(nb), lane);
    }
  }
  if (wave == NW - 1) {                                    // the wave with the fewest input blocks
    float gt[16];
    transpose16(tile, lane, g, gt);                        // lane = class, rows crow(r)
    B::pack(gt).store(a.GL + ((size_t)v * BT + rt) * kBlk, lane);
    float db = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) db += gt[r];
    db += __shfl_xor(db, 32);
    if (lane < 32) a.opdb[((size_t)v * BT + rt) * 32 + lane] = db;
    double ce_sum = (lane < 32 && rvalid) ? (double)ce : 0.0;
    unsigned int corr = (lane < 32 && rvalid && hit) ? 1u : 0u;
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) {
      ce_sum += __shfl_xor(ce_sum, off);
      corr += __shfl_xor(corr, off);
    }
    if (lane == 0) { a.opce[(size_t)v * BT + rt] = ce_sum; a.opcorr[(size_t)v * BT + rt] = corr; }
  }
  vt_add_wg(a.vtime, v, vt0);
}

// Prediction, one workgroup per (256 rows, variant), a row tile per wave.
template <typename S>
__global__ __launch_bounds__(512) void k_tile_pred_out(TileOutArgs<S> a) {
  typedef Blk<S> B;
  __shared__ double red_ce[8];
  __shared__ unsigned int red_corr[8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31;
  const int chunk = blockIdx.x, v = blockIdx.y;
  const uint64_t vt0 = vt_now();
  const int NB = a.Kp / 32, rt = chunk * 8 + wave;
  const float* WL = a.WL + (size_t)v * NB * kBlk;
  const S* Ar = a.Arows + v * a.ar_vs + (size_t)rt * NB * kBlk;
  f32x16_t acc = zero16();
  for (int nb = 0; nb < NB; ++nb) {
    f32x4_t w4[4];
    load_w(WL + (size_t)nb * kBlk, lane, w4);
    float wf[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) wf[r] = w4[r >> 2][r & 3];
    acc = blk_mma(B::pack(wf), B::load(Ar + (size_t)nb * kBlk, lane), acc);
  }
  const int y = a.labels[rt * 32 + l32];
  float z[16], ex[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = acc[r] + a.bias[(size_t)v * 32 + crow(r, lane)];
  float sm, ce;
  bool hit;
  row_softmax(z, a.C, y, lane, ex, sm, ce, hit);
  double ce_sum = (lane < 32 && y >= 0) ? (double)ce : 0.0;
  unsigned int corr = (lane < 32 && y >= 0 && hit) ? 1u : 0u;
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) {
    ce_sum += __shfl_xor(ce_sum, off);
    corr += __shfl_xor(corr, off);
  }
  if (lane == 0) { red_ce[wave] = ce_sum; red_corr[wave] = corr; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    unsigned int cc = 0;
    for (int w = 0; w < 8; ++w) { t += red_ce[w]; cc += red_corr[w]; }
    a.part_ce[(size_t)v * a.n_chunks_total + a.chunk0 + chunk] = t;
    a.part_correct[(size_t)v * a.n_chunks_total + a.chunk0 + chunk] = cc;
  }
  vt_add_wg(a.vtime, v, vt0);
}

// ------------------------------------------------------- hidden backward
// G_{l-1}[b][k] = (sum_n G_l[b][n] W_l[n][k]) [A_{l-1}[b][k] > 0], one 32 x 32
// tile (inputs kt, rows bt) per wave; W read transposed from the master.
template <typename S>
__global__ __launch_bounds__(256) void k_tile_bwd(TileBwdArgs<S> a) {
  typedef Blk<S> B;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31;
  const int v = blockIdx.y, KB = a.Kp / 32, NB = a.Np / 32, BT = a.Bp / 32;
  const uint64_t vt0 = vt_now();
  const int t = blockIdx.x * 4 + wave;
  if (t >= KB * BT) return;
  const int kt = t / BT, bt = t % BT;
  const float* W = a.Wm + (size_t)v * a.Kp * a.Np + (size_t)kt * a.Np * 32;
  const S* G = a.Grows + ((size_t)v * BT + bt) * NB * kBlk;
  const size_t ci = (((size_t)v * KB + kt) * BT + bt) * kBlk;
  const B h = B::load(a.Acols + ci, lane);
  f32x16_t d = zero16();
  for (int nb = 0; nb < NB; ++nb) {
    float wt[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) wt[r] = W[((size_t)nb * 32 + crow(r, lane)) * 32 + l32];
    d = blk_mma(B::load(G + (size_t)nb * kBlk, lane), B::pack(wt), d);
  }
  float f[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) f[r] = h.val(r) > 0.0f ? d[r] : 0.0f;
  B::pack(f).store(a.Gcols + ci, lane);
  vt_add_wg(a.vtime, v, vt0);
}

// ------------------------------------------------------- prediction forward
// O = relu(X W + b) over R rows: a wave (one per SIMD, the whole register
// file) takes NT unit tiles and RT row tiles; the four waves of a workgroup
// take neighbouring unit tiles of the same rows, which meet in the L1.
// Operands come straight from L2, two row blocks and one input block of
// weights ahead of their use: per input block 4 (NT + RT) KiB for 16 NT RT
// MFMAs.  The launcher picks the tile by the rounds its waves take.  2,048
// rows, 64 variants, 784 -> 256 in fp32: 386 us per launch (136 TFLOP/s), 693
// with two waves per SIMD.
template <typename S, int NT, int RT>
__global__ __launch_bounds__(256, 1) void k_tile_fwd(TileFwdArgs<S> a) {
  typedef Blk<S> B;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nt = (blockIdx.x * 4 + wave) * NT, rt0 = blockIdx.y * RT, v = blockIdx.z;
  const uint64_t vt0 = vt_now();
  const int KB = a.Kp / 32, NB = a.Np / 32, NRT = a.R / 32;
  if (nt >= NB) return;
  const float* Wv = a.Wm + (size_t)v * a.Np * a.Kp;
  const float* Wt[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) Wt[n] = Wv + (size_t)(nt + n < NB ? nt + n : nt) * kBlk;   // past the end: unused
  const S* X = a.Xrows + v * a.xr_vs;
  auto load_x = [&](int t, int kb) {                       // rows past the end: the last tile's, unused
    return B::load(X + ((size_t)(rt0 + t < NRT ? rt0 + t : NRT - 1) * KB + kb) * kBlk, lane);
  };
  f32x16_t z[NT][RT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int t = 0; t < RT; ++t) z[n][t] = zero16();
  f32x4_t w[NT][4];
#pragma unroll
  for (int n = 0; n < NT; ++n) load_w(Wt[n], lane, w[n]);
  B xa = load_x(0, 0), xb = RT > 1 ? load_x(1 % RT, 0) : load_x(0, KB > 1 ? 1 : 0);
  for (int kb = 0; kb < KB; ++kb) {
    const int k1 = kb + 1 < KB ? kb + 1 : kb, k2 = kb + 2 < KB ? kb + 2 : k1;   // past the end: unused re-reads
    B wb[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      float wf[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) wf[r] = w[n][r >> 2][r & 3];
      wb[n] = B::pack(wf);
      load_w(Wt[n] + (size_t)k1 * a.Np * 32, lane, w[n]);
    }
    B x[RT + 2];
    x[0] = xa;
    x[1] = xb;
    constexpr int U = NT > 1 || RT == 1 ? 1 : 2;
#pragma unroll
    for (int t = 0; t < RT; t += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int g = t + u + 2;
        x[g] = load_x(g % RT, g < RT ? kb : g < 2 * RT ? k1 : k2);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (NT == 2) blk_mma2(wb[0], x[t], z[0][t], wb[NT - 1], x[t], z[NT - 1][t]);
      else if constexpr (U == 2) blk_mma2(wb[0], x[t], z[0][t], wb[0], x[t + 1], z[0][(t + 1) % RT]);
      else z[0][t] = blk_mma(wb[0], x[t], z[0][t]);
      __builtin_amdgcn_sched_barrier(0);
    }
    xa = x[RT];
    xb = x[RT + 1];
  }
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    if (nt + n >= NB) continue;
    float bias[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) bias[r] = a.bias[(size_t)v * a.Np + (nt + n) * 32 + crow(r, lane)];
#pragma unroll
    for (int t = 0; t < RT; ++t)
      if (rt0 + t < NRT) {
        float f[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float zz = z[n][t][r] + bias[r];
          f[r] = zz > 0.0f ? zz : 0.0f;
        }
        B::pack(f).store(a.Orows + v * a.or_vs + ((size_t)(rt0 + t) * NB + nt + n) * kBlk, lane);
      }
  }
  vt_add_wg(a.vtime, v, vt0);
}

// ------------------------------------------------------------ data movement
// Rows of the dataset in the epoch's order as images: rows [t][row tile][kb],
// cols [t][kb][row tile] (nullable), zero past d0 and past the step's rows;
// labels [t][Bp] (-1 for padding).  One workgroup per block.
template <typename S>
__global__ __launch_bounds__(256) void k_tile_gather(GatherArgs a) {
  using O = Op<S>;
  typedef Blk<S> B;
  __shared__ float tile[32 * kTP];
  const int rt = blockIdx.x, kb = blockIdx.y, t = blockIdx.z, KB = a.Kp / 32, NRT = a.Bp / 32;
  const int tid = threadIdx.x, k = tid & 31;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rl = (tid >> 5) + 8 * i, b = rt * 32 + rl;
    const int64_t r = (int64_t)t * a.B + b;
    const bool valid = b < a.B && r < a.n;
    const int64_t src = valid ? (a.perm ? (int64_t)a.perm[r] : r) : 0;
    tile[rl * kTP + k] = (valid && kb * 32 + k < a.d0) ? a.X[src * a.d0 + kb * 32 + k] : 0.0f;
    if (kb == 0 && k == 0) a.labels[(size_t)t * a.Bp + b] = valid ? a.y[src] : -1;
  }
  __syncthreads();
  S* rows = reinterpret_cast<S*>(a.rows) + (((size_t)t * NRT + rt) * KB + kb) * kBlk;
  S* cols = a.cols ? reinterpret_cast<S*>(a.cols) + (((size_t)t * KB + kb) * NRT + rt) * kBlk : nullptr;
  // thread: lane l of the block and one group of four values r = 4 g + i
  const int l = tid & 63, g = tid >> 6, l32 = l & 31;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = crow(4 * g + i, l);
    rows[B::off(4 * g + i, l)] = O::from_f32(tile[l32 * kTP + c]);
    if (cols) cols[B::off(4 * g + i, l)] = O::from_f32(tile[c * kTP + l32]);
  }
}

// ---------------------------------------------------------------- launchers
template <typename S, int BT, int NT, int NW, bool UPD, bool FWD>
static hipError_t launch_tl(const TileLayerArgs<S>& a, int P, hipStream_t s, const LaunchEv& ev) {
  static bool attr = false;
  const size_t lds = TileLayerLds<BT, NT, NW>::bytes;
  if (!attr) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tile_layer<S, BT, NT, NW, UPD, FWD>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr = true;
  }
  hipExtLaunchKernelGGL((k_tile_layer<S, BT, NT, NW, UPD, FWD>), dim3(a.Np / 32 / NT, P), dim3(64 * NW), lds, s,
                        ev.start, ev.stop, 0, a);
  return hipGetLastError();
}

template <typename S, int BT, int NT, int NW>
static hipError_t launch_tl_uf(const TileLayerArgs<S>& a, int P, bool upd, bool fwd, hipStream_t s, const LaunchEv& ev) {
  if (upd && fwd) return launch_tl<S, BT, NT, NW, true, true>(a, P, s, ev);
  if (upd) return launch_tl<S, BT, NT, NW, true, false>(a, P, s, ev);
  return launch_tl<S, BT, NT, NW, false, true>(a, P, s, ev);
}

template <typename S, int BT>
static hipError_t launch_tl_mode(const TileLayerArgs<S>& a, int P, bool upd, bool fwd, hipStream_t s, const LaunchEv& ev) {
  // two unit tiles per workgroup once that still gives every CU a workgroup
  // (eight row tiles of two unit tiles would not fit the registers)
  const int NB = a.Np / 32;
  if constexpr (BT < 8)
    if (NB % 2 == 0 && (int64_t)P * (NB / 2) >= 256) return launch_tl_uf<S, BT, 2, 4>(a, P, upd, fwd, s, ev);
  // Eight waves where the chip has a workgroup per CU at most and a wave's
  // chain of blocks, not the matrix cores, is the time: in bf16 up to 128 rows
  // (an epoch of 24 variants of 784-300-100-10, batch 100: 2.75 ms with four
  // waves, 2.66 with eight; 16 of 784-512-10, batch 64: 0.99 and 0.90), in fp32
  // one row tile (4 of 784-128-10, batch 32: 1.59 and 1.53; with two row tiles,
  // 16 of 784-300-100-10, 3.56 and 4.04, with four 1.3 and 1.9).
  if constexpr (BT == 1 || (BT <= 4 && sizeof(S) == 2))
    if ((int64_t)P * NB <= 256) return launch_tl_uf<S, BT, 1, 8>(a, P, upd, fwd, s, ev);
  return launch_tl_uf<S, BT, 1, 4>(a, P, upd, fwd, s, ev);
}

template <typename S>
hipError_t launch_tile_layer(const TileLayerArgs<S>& a, int P, bool upd, bool fwd, hipStream_t s, const LaunchEv& ev) {
  if (a.Kp % 32 || a.Np % 32 || a.Bp % 32 || a.Kp <= 0 || a.Np <= 0 || a.Bp < 32 || a.Bp > 256 || !(upd || fwd))
    return hipErrorInvalidValue;
  switch (a.Bp / 32) {
    case 1: return launch_tl_mode<S, 1>(a, P, upd, fwd, s, ev);
    case 2: return launch_tl_mode<S, 2>(a, P, upd, fwd, s, ev);
    case 3: return launch_tl_mode<S, 3>(a, P, upd, fwd, s, ev);
    case 4: return launch_tl_mode<S, 4>(a, P, upd, fwd, s, ev);
    case 5: return launch_tl_mode<S, 5>(a, P, upd, fwd, s, ev);
    case 6: return launch_tl_mode<S, 6>(a, P, upd, fwd, s, ev);
    case 7: return launch_tl_mode<S, 7>(a, P, upd, fwd, s, ev);
    default: return launch_tl_mode<S, 8>(a, P, upd, fwd, s, ev);
  }
}

template <typename S>
hipError_t launch_tile_out(const TileOutArgs<S>& a, int P, hipStream_t s, const LaunchEv& ev) {
  if (a.Kp % 32 || a.Bp % 32 || a.Kp <= 0 || a.Bp <= 0) return hipErrorInvalidValue;
  hipExtLaunchKernelGGL(k_tile_out<S>, dim3(a.Bp / 32, P), dim3(256), 0, s, ev.start, ev.stop, 0, a);
  return hipGetLastError();
}

template <typename S>
hipError_t launch_tile_pred_out(const TileOutArgs<S>& a, int rows, int P, hipStream_t s, const LaunchEv& ev) {
  if (a.Kp % 32 || a.Kp <= 0 || rows <= 0 || rows % 256) return hipErrorInvalidValue;
  hipExtLaunchKernelGGL(k_tile_pred_out<S>, dim3(rows / 256, P), dim3(512), 0, s, ev.start, ev.stop, 0, a);
  return hipGetLastError();
}

template <typename S>
hipError_t launch_tile_bwd(const TileBwdArgs<S>& a, int P, hipStream_t s, const LaunchEv& ev) {
  if (a.Kp % 32 || a.Np % 32 || a.Bp % 32 || a.Kp <= 0 || a.Np <= 0 || a.Bp <= 0) return hipErrorInvalidValue;
  const int tiles = (a.Kp / 32) * (a.Bp / 32);
  hipExtLaunchKernelGGL(k_tile_bwd<S>, dim3((tiles + 3) / 4, P), dim3(256), 0, s, ev.start, ev.stop, 0, a);
  return hipGetLastError();
}

template <typename S, int NT, int RT>
static hipError_t launch_tf(const TileFwdArgs<S>& a, int P, hipStream_t s, const LaunchEv& ev) {
  const dim3 grid((a.Np / 32 + 4 * NT - 1) / (4 * NT), (a.R / 32 + RT - 1) / RT, P);
  hipExtLaunchKernelGGL((k_tile_fwd<S, NT, RT>), grid, dim3(256), 0, s, ev.start, ev.stop, 0, a);
  return hipGetLastError();
}

template <typename S>
hipError_t launch_tile_fwd(const TileFwdArgs<S>& a, int P, hipStream_t s, const LaunchEv& ev) {
  if (a.Kp % 32 || a.Np % 32 || a.R % 32 || a.Kp <= 0 || a.Np <= 0 || a.R <= 0) return hipErrorInvalidValue;
  // Rounds of 256 workgroups (one per CU) times the products of a wave, with
  // one product's worth for the operands that a smaller tile loads more often.
  // ms per prediction by this rule, and with (2, 8), (2, 4), (1, 4), (1, 2) and (1, 1)
  // for every launch: 64 variants of 784-256-10, 10,000 rows 2.09 (2.08, 2.11, 3.57,
  // 4.08, 3.20); 4 of 784-128-10, 512 rows 0.035 (0.199, 0.111, 0.067, 0.045, 0.035); 128
  // of 784-256-10, 250 rows 0.139 (0.223, 0.136, 0.198, 0.219, 0.188); 256 of 784-32-10,
  // 2,048 rows 0.375 (1.49, 1.52, 0.38, 0.42, 0.37).  It is furthest off where two
  // tiles cost nearly the same: 32 of 784-512-256-10, 3,000 rows 0.91 (0.95, 0.86, ...).
  const int64_t NB = a.Np / 32, NRT = a.R / 32;
  auto cost = [&](int nt, int rt) {
    const int64_t wg = (NB + 4 * nt - 1) / (4 * nt) * ((NRT + rt - 1) / rt) * P;
    return (wg + 255) / 256 * (nt * rt + 1);
  };
  const int64_t c[5] = {cost(2, 8), cost(2, 4), cost(1, 4), cost(1, 2), cost(1, 1)};
  int best = 0;
  for (int i = 1; i < 5; ++i)
    if (c[i] < c[best]) best = i;
  switch (best) {
    case 0: return launch_tf<S, 2, 8>(a, P, s, ev);
    case 1: return launch_tf<S, 2, 4>(a, P, s, ev);
    case 2: return launch_tf<S, 1, 4>(a, P, s, ev);
    case 3: return launch_tf<S, 1, 2>(a, P, s, ev);
    default: return launch_tf<S, 1, 1>(a, P, s, ev);
  }
}

template <typename S>
hipError_t launch_tile_gather(const GatherArgs& a, hipStream_t s, const LaunchEv& ev) {
  if (a.Kp % 32 || a.Bp % 32) return hipErrorInvalidValue;
  hipExtLaunchKernelGGL(k_tile_gather<S>, dim3(a.Bp / 32, a.Kp / 32, a.T), dim3(256), 0, s, ev.start, ev.stop, 0, a);
  return hipGetLastError();
}

template hipError_t launch_tile_layer<float>(const TileLayerArgs<float>&, int, bool, bool, hipStream_t, const LaunchEv&);
template hipError_t launch_tile_out<float>(const TileOutArgs<float>&, int, hipStream_t, const LaunchEv&);
template hipError_t launch_tile_pred_out<float>(const TileOutArgs<float>&, int, int, hipStream_t, const LaunchEv&);
template hipError_t launch_tile_bwd<float>(const TileBwdArgs<float>&, int, hipStream_t, const LaunchEv&);
template hipError_t launch_tile_fwd<float>(const TileFwdArgs<float>&, int, hipStream_t, const LaunchEv&);
template hipError_t launch_tile_gather<float>(const GatherArgs&, hipStream_t, const LaunchEv&);
// bf16: training only
template hipError_t launch_tile_layer<uint16_t>(const TileLayerArgs<uint16_t>&, int, bool, bool, hipStream_t,
                                                const LaunchEv&);
template hipError_t launch_tile_out<uint16_t>(const TileOutArgs<uint16_t>&, int, hipStream_t, const LaunchEv&);
template hipError_t launch_tile_bwd<uint16_t>(const TileBwdArgs<uint16_t>&, int, hipStream_t, const LaunchEv&);
template hipError_t launch_tile_gather<uint16_t>(const GatherArgs&, hipStream_t, const LaunchEv&);

}  // namespace gevo
