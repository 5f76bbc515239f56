// conv_lat.hip -- which layers run conv_mfma_lat_kernel, and its launch.
#include <stdio.h>
#include <string.h>

#include "conv_lat.h"

namespace qc {
namespace mfma {

namespace {

// 32 x 32 output tiles and (tap, 64-channel) k-steps of a layer.
int64_t lat_tiles(const ConvArgs& a) {
  const int64_t units = (int64_t)a.n * (a.pool ? (int64_t)(a.ho / 2) * (a.wo / 2) : (int64_t)a.ho * a.wo);
  return ((units * (a.pool ? 4 : 1) + 31) / 32) * ceil_div(a.cout, 32);
}
int lat_steps(const ConvArgs& a) { return a.kh * a.kw * ceil_div(a.cw, 2); }

// Channel tiles and waves per block.  One channel tile while that leaves few
// blocks or little work; two (half the reads of the input words per product)
// from about 320 tiles on when a tile is long enough: at 2 bits 512 x 7 x 7
// batch 16 (400 tiles of 72 steps) 7.9 against 6.1 us, 256 x 14 x 14 batch 16
// (784 of 36) 6.8 against 5.7, but 128 x 28 x 28 batch 4 (392 of 18) 3.7
// against 3.8 and with an fp32 output 5.3 against 5.4.
void lat_shape(const ConvArgs& a, int* nt, int* sk) {
  const int64_t tiles = lat_tiles(a), steps = lat_steps(a);
  *nt = tiles > 320 && tiles * steps > 10000 ? 2 : 1;
  *sk = *nt == 2 || steps >= 64 ? 8 : 4;  // 512 x 7 x 7 batch 1: 5.6 us with 4 waves, 5.3 with 8
}

bool lat_plan(const ConvArgs& a, int nt, MfmaArgs* m) {
  memset(m, 0, sizeof(*m));
  m->c = a;
  m->ksteps = ceil_div(a.cw, 2);
  m->wx = a.w_fp4;
  const int64_t wxb = (int64_t)a.kh * a.kw * m->ksteps * a.cop * 32;
  const int64_t ab = (int64_t)a.n * a.h * a.w * a.cw * act_words(a.a_bits) * 4;
  if (wxb >= ((int64_t)1 << 30) || ab >= ((int64_t)1 << 30)) return false;
  m->wx_bytes = (int)wxb;
  m->act_bytes = (int)ab;
  m->pool = a.pool;
  m->uw = a.pool ? a.wo / 2 : a.wo;
  m->upi = (a.pool ? a.ho / 2 : a.ho) * m->uw;
  if (m->upi < 1) return false;
  m->units_pb = a.pool ? 8 : 32;
  const int64_t units = (int64_t)a.n * m->upi;
  // exact fast divisions: dividend * divisor < 2^32 (dividends up to a tile past the end)
  if ((units + 32) * m->upi >= ((int64_t)1 << 32) || (int64_t)m->upi * m->uw >= ((int64_t)1 << 32)) return false;
  m->fd_upi = make_fastdiv((uint32_t)m->upi);
  m->fd_uw = make_fastdiv((uint32_t)m->uw);
  m->tiles_px = (int)((units + m->units_pb - 1) / m->units_pb);
  m->tiles_co = ceil_div(a.cout, 32 * nt);
  m->inv = 1.0f / (float)(1 << a.shift);
  m->othr = thr_unclamped(a.othr);
  const int64_t ob = (int64_t)a.n * a.cout * m->upi * 4;
  if (a.mode != QCONV_EPI_BN_PACK && ob > OFF_NONE) return false;
  m->out_bytes = a.mode == QCONV_EPI_BN_PACK ? 0 : (int)ob;
  return true;
}

template <int PA, int NT, int SK>
int launch_shape(const MfmaArgs& m, hipStream_t s) {
  const dim3 grid((unsigned)(m.tiles_px * m.tiles_co));
  const size_t lds = (size_t)NT * 4 * SK * 1024;
  if (m.c.pool)
    conv_mfma_lat_kernel<PA, NT, SK, 1><<<grid, 64 * SK, lds, s>>>(m);
  else
    conv_mfma_lat_kernel<PA, NT, SK, 0><<<grid, 64 * SK, lds, s>>>(m);
  return hip_status();
}

template <int PA>
int launch_pa(const MfmaArgs& m, int nt, int sk, hipStream_t s) {
  if (nt == 2) return launch_shape<PA, 2, 8>(m, s);
  if (sk == 8) return launch_shape<PA, 1, 8>(m, s);
  return launch_shape<PA, 1, 4>(m, s);
}

}  // namespace

// Layers of at most 1024 tiles and 40000 tile steps: with more, the blocks'
// repeated expansion of the input words costs more than the latency chain it
// replaces.  At 2 bits, this kernel against the one that would run instead:
// 784 tiles of 36 steps (256 x 14 x 14 batch 16, residual and packed copy) 9.1
// against 9.7 us, 784 of 9 (64 x 56 x 56 batch 4, the same) 7.7 against 8.2;
// 1568 of 18 (128 x 28 x 28 batch 16) 12.5 against 10.1, 1568 of 36 (256 -> 512
// / 2 batch 64, packed) 11.3 against 10.7.  Only with fp4 operands and where
// the LDS-staged kernel serves the layer too.  Unpacked outputs of 3-bit inputs,
// whose expansion is the longest, up to 512 tiles where a tile has more than 9
// steps (128 -> 128, 14 x 14: 392 tiles 5.4 against 7.0 us, 588 7.4 against 7.2,
// 784 7.9 against 7.3; packed 5.2 against 7.3).  Int32 and scaled outputs, whose
// epilogue hides least of it, up to 768 tiles where a tile has 9 to 17 steps and
// the split-K shape's 64 channels are used (64 -> 64 int32: 13 x 13 782 tiles 0.93
// of its speed, 898 0.88, 38 x 38 904 0.90, 28 x 28 784 1.00, 56 x 56 784 1.03;
// 32 -> 32 13 x 13 999 1.38; with batch norm 1.00 to 1.26).
bool lat_applies(const ConvArgs& a) {
  if (a.mfma_op != OP_FP4 || a.stride > 2 || a.kh > 16 || a.kw > 16 || a.n < 1) return false;
  const int64_t tiles = lat_tiles(a);
  if (tiles < 1 || tiles > 1024 || tiles * lat_steps(a) > 40000) return false;
  if (a.a_bits == 3 && tiles > 512 && lat_steps(a) > 9 && !a.pool && a.mode != QCONV_EPI_BN_PACK) return false;
  if ((a.mode == QCONV_EPI_INT32 || a.mode == QCONV_EPI_SCALE_F32) && !a.pool && tiles > 768 && a.kreal > 256 &&
      lat_steps(a) >= 9 && lat_steps(a) < 18 && (a.cout - 1) % 64 >= 32)
    return false;
  MfmaArgs m;
  return lat_plan(a, 1, &m);
}

// Whether AUTO prefers it to the XNOR kernel (contractions of up to 256
// values).  It does except for int32 outputs of 1-bit weights in one or two
// k-steps, where the XNOR kernel is as fast from about 768 tiles on (128 -> 256,
// 28 x 28 / 2, 784 tiles: XNOR 6.1 us, this kernel 6.5; 592 tiles 6.0 and 5.3;
// with batch norm 784 tiles 7.0 and 6.6, with 2-bit weights 7.1 and 6.5, and
// 256 -> 256, four k-steps, 14 x 14, 784 tiles 7.0 and 6.6).
bool lat_beats_xnor(const ConvArgs& a) {
  if (!lat_applies(a)) return false;
  return !(a.mode == QCONV_EPI_INT32 && a.w_bits == 1 && lat_steps(a) <= 2 && lat_tiles(a) > 768);
}

int lat_kernel_name(const ConvArgs& a, char* buf, int len) {
  int nt, sk;
  lat_shape(a, &nt, &sk);
  return snprintf(buf, (size_t)len, "conv_mfma_lat_kernel<%d, %d, %d, %d>", act_words(a.a_bits), nt, sk, a.pool ? 1 : 0);
}

int launch_conv_lat(const ConvArgs& a, hipStream_t s) {
  int nt, sk;
  lat_shape(a, &nt, &sk);
  MfmaArgs m;
  if (!lat_plan(a, nt, &m)) return QCONV_EUNSUPPORTED;
  const int pa = act_words(a.a_bits);
  if (pa == 1) return launch_pa<1>(m, nt, sk, s);
  if (pa == 2) return launch_pa<2>(m, nt, sk, s);
  return launch_pa<4>(m, nt, sk, s);
}

}  // namespace mfma
}  // namespace qc
