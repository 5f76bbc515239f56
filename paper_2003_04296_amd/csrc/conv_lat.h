#pragma once
// conv_lat.h -- the fp4 layer product for layers of few output tiles, whose
// time is one chain of latencies rather than matrix work or bandwidth: the
// caches of the XCDs hold nothing at a launch, so every first read of a
// weight or an input word takes most of a microsecond, and a block of the
// LDS-staged kernel makes such reads one after another (halo, weights two
// k-steps ahead, parameters, residual).
//
// Here a block has one output tile of 32 pixels x 32 NT channels and SK
// waves that split its (tap, k-step) range; a wave issues the reads of up to
// D of its k-steps back to back before it waits once.  A lane reads the packed
// word of its own pixel for each step (taps outside the image at an offset
// past the buffer's end: 0 = Q(0)) and expands it into its operand fragment
// in registers, so there is no input tile in LDS, no barrier before the
// products and no index arithmetic beyond one offset per tap.  The partial
// tiles are summed through LDS in pieces of 4 accumulator registers, a
// piece to a wave, so that the epilogue is spread over the block's waves as
// well; its parameters and residual values are read under the products.
//
// Orientation: pixels as the A operand.  Register 4q + i of lane l holds
// channel l % 32 of row 8q + 4 (l / 32) + i: piece q is four consecutive
// pixels per lane (a 16-byte NCHW store), or one pooling window (rows in the
// order of conv_mfma.h), and the packed words are wave ballots.
//
// Measured (2 bits, back to back; the split-K shape of conv_mfma_kernel
// before it): ResNet-18's layers at batch 1, 64 channels 56 x 56 packed 6.8 ->
// 3.4 us, 256 x 14 x 14 with residual and packed copy 8.9 -> 4.6, 512 x 7 x 7
// 9.6 -> 5.3, the 1 x 1 / 2 shortcuts (XNOR kernel) 7.0-7.6 -> 3.4; batch 16,
// 512 x 7 x 7 9.9 -> 6.1; ConvNet's two fully connected layers at batch 256
// 15.4 -> 7.7 and 6.7 -> 3.6.
#include "conv_mfma.h"

namespace qc {
namespace mfma {

// k-steps whose reads are in flight together (6 the same, 9 slower: the code
// of the steps past a wave's range costs more than a second round saves)
constexpr int LAT_D = 5;

// The packed words of one piece of the epilogue: four rows (or one window) of 32
// channels per half-wave.  z: this lane's output values; u0: the tile's first
// unit; q: the piece; co32: its first channel; total: units of the layer.
template <int POOL, int OB>
__device__ __forceinline__ void lat_pack(const MfmaArgs& m, const float (&z)[4], int u0, int q, int co32, int total,
                                         int lane) {
  constexpr int P = planes_of(OB);
  const ConvArgs& a = m.c;
  uint32_t pw[P];
#pragma unroll
  for (int p = 0; p < P; ++p) pw[p] = 0u;
  int unit;
  bool ok;
  if constexpr (POOL) {
    // windows u0 + q (lanes 0-31) and u0 + 4 + q (lanes 32-63)
    uint64_t bl[P];
    plane_ballots<OB>(z[0], true, m.othr, bl);
#pragma unroll
    for (int p = 0; p < P; ++p) pw[p] = (lane & 1) ? (uint32_t)(bl[p] >> 32) : (uint32_t)bl[p];
    unit = u0 + q + 4 * (lane & 1);
    ok = lane < 2;
  } else {
    uint64_t bl[4][P];
#pragma unroll
    for (int i = 0; i < 4; ++i) plane_ballots<OB>(z[i], true, m.othr, bl[i]);
#pragma unroll
    for (int p = 0; p < P; ++p)
      pw[p] = writelanes8<0, 1, 2, 3, 4, 5, 6, 7>(
          pw[p], (uint32_t)bl[0][p], (uint32_t)bl[1][p], (uint32_t)bl[2][p], (uint32_t)bl[3][p],
          (uint32_t)(bl[0][p] >> 32), (uint32_t)(bl[1][p] >> 32), (uint32_t)(bl[2][p] >> 32),
          (uint32_t)(bl[3][p] >> 32));
    unit = u0 + 8 * q + lane;
    ok = lane < 8;
  }
  if (co32 + 32 > a.cout) {  // uniform: channels past the last one are 0 in every plane
    const uint32_t valid = (1u << (a.cout - co32)) - 1u;
#pragma unroll
    for (int p = 0; p < P; ++p) pw[p] &= valid;
  }
  if (ok && unit < total) store_words<P>(a.out_packed + ((int64_t)unit * a.out_cw + (co32 >> 5)) * P, pw);
}

template <int PA, int NT, int SK, int POOL>
__global__ __launch_bounds__(64 * SK) void conv_mfma_lat_kernel(const MfmaArgs m) {
  // one tile of 32 rows a block: two measured slower at every size
  constexpr int PIECES = NT * 4, PPW = (PIECES + SK - 1) / SK, D = LAT_D;
  constexpr int TU = POOL ? 8 : 32;  // units per block
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  const ConvArgs& a = m.c;
  const int tid = threadIdx.x, lane = tid & 63, wk = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, r32 = lane & 31;
  const int pt = (int)blockIdx.x / m.tiles_co;
  const int co_blk = ((int)blockIdx.x - pt * m.tiles_co) * (32 * NT);
  const int total = a.n * m.upi;

  // the pixel of this lane's row: byte offset of its first tap's word (this
  // lane's k-half; may lie before the tensor) and the taps inside the image
  const int apix = a.cw * PA * 4;  // bytes per pixel
  const int unit = POOL ? 8 * pt + 4 * ((r32 >> 2) & 1) + (r32 >> 3) : 32 * pt + r32;
  const int uimg = (int)fdiv((uint32_t)unit, m.fd_upi);
  const int uu = unit - uimg * m.upi;
  const int uy = (int)fdiv((uint32_t)uu, m.fd_uw);
  const int ux = uu - uy * m.uw;
  const int iy = (POOL ? 2 * uy + ((r32 >> 1) & 1) : uy) * a.stride - a.pad;
  const int ix = (POOL ? 2 * ux + (r32 & 1) : ux) * a.stride - a.pad;
  const int base = ((uimg * a.h + iy) * a.w + ix) * apix + g * (PA * 4);
  const uint32_t rmask = unit < total ? tap_mask(iy, a.h, a.kh) : 0u;
  const uint32_t cmask = tap_mask(ix, a.w, a.kw);
  const __amdgpu_buffer_rsrc_t arsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)a.act, (short)0, m.act_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t brsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)m.wx, (short)0, m.wx_bytes, 0x00020000);
  const int bvoff = (co_blk + r32) * 32 + g * 16;
  const int bstride = a.cop * 32;

  // this wave's steps
  const int nall = a.kh * a.kw * m.ksteps;
  const int sbeg = (nall * wk) / SK, send = (nall * (wk + 1)) / SK;
  int step = sbeg;
  const int tap0 = sbeg / m.ksteps;
  int ks = sbeg - tap0 * m.ksteps, ky = tap0 / a.kw, kx = tap0 - (tap0 / a.kw) * a.kw;
  int voff;
  auto tap_offsets = [&]() __attribute__((always_inline)) {
    const int to = (ky * a.w + kx) * apix;
    voff = ((rmask >> ky) & (cmask >> kx) & 1u) ? base + to : OFF_NONE;
  };
  tap_offsets();
  uint32_t ra[D][PA];
  v4i rb[D][NT];
  auto issue = [&](auto DD) __attribute__((always_inline)) {
    constexpr int d = decltype(DD)::value;
    const int ao = ks * (2 * PA * 4), bo = step * bstride;
    load_words<PA>(arsrc, voff, ao, ra[d]);
#pragma unroll
    for (int j = 0; j < NT; ++j)
      rb[d][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(brsrc, bvoff + j * 1024, bo, 0));
    ++step;
    if (++ks == m.ksteps) {  // uniform
      ks = 0;
      if (++kx == a.kw) {
        kx = 0;
        ++ky;
      }
      tap_offsets();
    }
  };
  v16f acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.0f;
  auto consume = [&](auto DD) __attribute__((always_inline)) {
    constexpr int d = decltype(DD)::value;
    uint32_t o[4];
    expand_fp4_word<PA>(ra[d], 0xFFFFFFFFu, o);
    const v4i A = {(int)o[0], (int)o[1], (int)o[2], (int)o[3]};
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = mfma<OP_FP4>(A, rb[d][j], acc[j]);
  };
  int left = send - sbeg;
  Unroll<0, D>::run([&](auto dd) {
    if (decltype(dd)::value < left) issue(dd);
  });

  // this wave's pieces of the epilogue: parameters and residual, read under
  // the products
  const bool bn = a.mode == QCONV_EPI_BN_F32 || a.mode == QCONV_EPI_BN_PACK;
  const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(bn ? a.bn_k : a.scale), (short)0, a.mode == QCONV_EPI_INT32 ? 0 : a.cout * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t prsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)a.bn_b, (short)0, bn ? a.cout * 4 : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rrsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)a.residual, (short)0, a.residual_on ? m.out_bytes : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc(a.out, (short)0, m.out_bytes, 0x00020000);
  constexpr int NV = POOL ? 1 : 4;  // output values of a piece per lane
  float kv[PPW], bv[PPW], rv[PPW][4];
  int oo[PPW][NV];  // byte offsets of the outputs
#pragma unroll
  for (int k = 0; k < PPW; ++k) {
    const int pc = wk + SK * k;  // piece: channel tile pc / 4, rows pc % 4
    const int tj = pc >> 2, q = pc & 3;
    const int co = co_blk + 32 * tj + r32;
    const int cvo = co < a.cout ? co * 4 : OFF_NONE;
    kv[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(krsrc, cvo, 0, 0));
    bv[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(prsrc, cvo, 0, 0));
    const int u = pt * TU + (POOL ? q + 4 * g : 8 * q + 4 * g);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      oo[k][i] = OFF_NONE;
      rv[k][i] = 0.0f;
    }
    if (a.mode != QCONV_EPI_BN_PACK) {  // uniform
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int img = (int)fdiv((uint32_t)(u + i), m.fd_upi);
        const bool ok = u + i < total && co < a.cout;
        oo[k][i] = ok ? ((img * a.cout + co) * m.upi + (u + i - img * m.upi)) * 4 : OFF_NONE;
        rv[k][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rrsrc, oo[k][i], 0, 0));
      }
    }
  }

  // products, D steps at a time
  while (left > 0) {
    Unroll<0, D>::run([&](auto dd) {
      if (decltype(dd)::value < left) consume(dd);
    });
    left -= D;
    Unroll<0, D>::run([&](auto dd) {
      if (decltype(dd)::value < left) issue(dd);
    });
  }

  // partial tiles through LDS: [piece][wave][lane]
  typedef float e4 __attribute__((ext_vector_type(4)));
  e4* red = reinterpret_cast<e4*>(lds_raw);
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const e4 t = {acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
      red[((j * 4 + q) * SK + wk) * 64 + lane] = t;
    }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < PPW; ++k) {
    const int pc = wk + SK * k;
    if (pc >= PIECES) break;  // uniform
    const int tj = pc >> 2, q = pc & 3;
    const int co32 = co_blk + 32 * tj;
    if (co32 >= a.cout) continue;  // uniform
    e4 s = red[(pc * SK) * 64 + lane];
#pragma unroll
    for (int w = 1; w < SK; ++w) s += red[(pc * SK + w) * 64 + lane];
    float z[4];
    if constexpr (POOL) {
      z[0] = fmaxf(fmaxf(s.x, s.y), fmaxf(s.z, s.w));
      z[1] = z[2] = z[3] = 0.0f;
    } else {
      z[0] = s.x;
      z[1] = s.y;
      z[2] = s.z;
      z[3] = s.w;
    }
    if (a.mode == QCONV_EPI_INT32) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
        __builtin_amdgcn_raw_buffer_store_b32((uint32_t)(int)z[i], orsrc, oo[k][i], 0, 0);
      continue;
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const float v = z[i] * m.inv;
      z[i] = a.mode == QCONV_EPI_SCALE_F32 ? kv[k] * v : fmaf(kv[k], v, bv[k]);
    }
    if (a.mode != QCONV_EPI_BN_PACK) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        if (a.residual_on) z[i] = z[i] + rv[k][i];
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(z[i]), orsrc, oo[k][i], 0, 0);
      }
    }
    if (a.out_packed) {
      const int u0 = pt * TU;
      if (a.out_bits == 1) lat_pack<POOL, 1>(m, z, u0, q, co32, total, lane);
      else if (a.out_bits == 2) lat_pack<POOL, 2>(m, z, u0, q, co32, total, lane);
      else lat_pack<POOL, 3>(m, z, u0, q, co32, total, lane);
    }
  }
}

}  // namespace mfma
}  // namespace qc
