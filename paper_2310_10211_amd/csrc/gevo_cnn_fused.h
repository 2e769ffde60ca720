// Convolutional prediction in whole segments: arguments and launcher of
// gevo_cnn_fused.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace gevo {

constexpr int kSegWaves = 8;                      // waves per workgroup
constexpr size_t kSegLds = 160 * 1024;            // LDS of a CU
constexpr int kSegMaxStages = 4;

// The stem's images in LDS: each is (H + 2) x (W + 2) x C bf16 elements with a
// zero border, padded to an even count, so that every image of a group begins
// on a dword whatever H, W and C are (with 7x7x1 or 15x15x3 back to back, every
// second image's windows would be read through misaligned dwords).
constexpr int seg_pitch(int H, int W, int C) { return ((H + 2) * (W + 2) * C + 1) / 2 * 2; }   // elements

// A window row starts at any element e of its image and is read in dwords: at
// even e from the images at byte im, at odd e from their copy at im2, which lies
// one element further on.  (Bytes from the image's first; e >= 0.)
constexpr int seg_window(int im, int im2, int e) { return ((e & 1) ? im2 : im) + 4 * ((e + 1) >> 1); }

// A producing layer (the stem, or a pointwise layer) and the depthwise layer
// after it, from one map in LDS to the next (LDS or, for the segment's last
// stage without a tail, global memory).
struct CnnSegStage {
  int S, KS, nct;                                 // depthwise stride, 16-deep contraction steps (stem: one per
                                                  // row of taps), 32-channel tiles
  int H, W, Ho, Wo;                               // the producer's map, the depthwise output
  int wt;                                         // pixels per tile row: 8, 16 or 32 (W rounded up)
  int parts, q;                                   // row ranges per image (and lane half, wt < 32), rows of a range
  int wpc_log;                                    // log2 of the waves per channel tile
  int in, out;                                    // LDS byte offsets of the maps of the group's images
  int img_in, img_out;                            // bytes per image map
  int ps_in, ps_out;                              // bytes per pixel
  const uint16_t* wp;                             // packed producer weights [P][nct][KS][64][8]
  const float* pb;                                // producer biases [P][32 nct]
  const uint32_t* taps; const float* db;          // depthwise tap pairs [P][5][32 nct], biases [P][32 nct]
};

struct CnnSegArgs {
  int G, groups, per_wg;                          // images per group, groups per variant, groups per workgroup
  // source: the images (stem_c > 0) or a map [v][image][pixels][channels] in global memory
  int stem_c;                                     // input channels of the stem, 0: no stem
  const float* x; int64_t img0, n_test; int H, W; // images; first of the launch, one past its last
  uint32_t w2_magic, pitch_magic, c_magic;        // ceil(2^32 / d) for d = W + 2, seg_pitch(H, W, C), C
  int im, im2;                                    // LDS byte offsets of the padded bf16 images and their copy
                                                  // one element further on
  const uint16_t* src; size_t src_vs;             // source map, elements per variant
  int src_px, src_c, src_off, src_ps;             // pixels, channels; LDS offset, bytes per pixel
  uint32_t c8_magic;                              // ceil(2^32 / (src_c / 8))
  int nst;
  CnnSegStage st[kSegMaxStages];
  uint16_t* dst; size_t dst_vs;                   // last stage's output in global memory (no tail)
  // tail: last pointwise layer and global average pooling
  int tail, t_KS, t_nct, t_HW, t_run, t_in, t_img, t_ps;   // t_run: pixels of a lane's run that belong to one image
  const uint16_t* t_wp; const float* t_pb;
  uint16_t* pooled; size_t pooled_vs;             // [v][image][32 t_nct]
  int lds;                                        // bytes
};

// Depthwise strides 1 and 2, contraction steps 3 (stem) or 2, 4, 8, 16.
hipError_t launch_cnn_seg(const CnnSegArgs& a, int P, hipStream_t s);
// bf16 copy of a weight tensor in the segment kernel's operand order:
// out[v][n / 32][s][lane][8], lane l holding column n = 32 i + l % 32 and
// slots e = 8 (l / 32) + 0..7 of step s: row k = s run + e for e < run, zero
// past it and past K (run 16: the rows in order; the stem's run is one row of
// taps, 3 C)
hipError_t launch_cnn_pack_op(const float* Wm, int Kp, int Np, int K, int KS, int run, int P, uint16_t* out,
                              hipStream_t s);

}  // namespace gevo
