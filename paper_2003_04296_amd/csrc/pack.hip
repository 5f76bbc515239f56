// pack.hip -- quantize-and-pack kernels (Sec. III-C, Eq. 20 with the
// quantizers of Eqs. 4, 21, 22).
//
// Activations: fp32 NCHW -> bitplanes [n][h][w][cw][P] (HBM-bound: 4 bytes
// read per channel, P/8 bytes written).
//
// 16-bit inputs: fp32 NCHW -> fp16 [n][h][w][cw * 32] (round to nearest
// even; channels past c are +0).
//
// Weights: fp32 OIHW -> per-channel scale s_c = mean|W_c| (double, storage
// order) -> thresholds scaled by s_c -> bitplanes [kh][kw][cw][cout_pad][P],
// then the int8, fp4 and fp16 matrix-core operand copies of the same codes.
#include "qconv_internal.h"

namespace qc {

namespace {

// Channels of a 32-channel word that exist, given how many remain (>= 1).
__device__ __forceinline__ uint32_t chan_mask(int remaining) {
  return remaining >= 32 ? 0xFFFFFFFFu : ((1u << remaining) - 1u);
}

// Activations: a unit is one 32-channel word of `run` (64, or the pixels of as
// many whole images as fit in 64) consecutive pixels, counted over all images,
// computed by one wave with a pixel per lane: each channel is read as one run
// of 256 bytes, 16 channels in flight before the first compare.  A block holds
// `group` words of `sub` runs, one wave per unit, in LDS and writes each
// pixel's as one run; where they are all of its words the block's whole output
// is one run.
// Bound by reading fp32 from HBM.  Inputs in cache / not, 2 bits: 256 x 64 x 56 x
// 56 32.9 / 42.2 us, 256 x 512 x 8 x 8 5.4 / 9.1, where waves that looped over
// whole pixel runs of one image took 33.1 / 42.7 and 8.3 / 15.4; 900 x 300 x 9 x
// 9 at 3 bits 21.1 / 25.0, where they branched per compare and took 43.5 / 58.8.
// In a loop whose convolution has just left 134 or 205 MB of writes, whose
// write-back shares HBM, the first at 3 bits takes 58.6 us and 256 x 128 x 32 x
// 32 at 2 bits 28.9 (22.7 / 28.6).  Two or four pixels per lane (8- and 16-byte loads)
// and 8 or 32 channels in flight measured the same or slower.
// Compares are gathered from the highest channel down, word = 2 word + bit
// (one v_addc per compare).  With t0 >= 0, x > t0 is the sign of a nonzero
// level; the one-hot planes are combined per word.
template <int BITS>
struct WordBits {
  static constexpr int NC = BITS == 1 ? 1 : (BITS == 2 ? 2 : 4);
  uint32_t w[NC];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < NC; ++i) w[i] = 0u;
  }
  __device__ __forceinline__ void push(float x, const Thr& t) {
    if constexpr (BITS == 1) {
      w[0] = w[0] + w[0] + (x > 0.0f ? 1u : 0u);
    } else {
      const float ax = fabsf(x);
      w[0] = w[0] + w[0] + (x > t.t0 ? 1u : 0u);
      w[1] = w[1] + w[1] + (!(ax <= t.t0) ? 1u : 0u);
      if constexpr (BITS == 3) {
        w[2] = w[2] + w[2] + (!(ax <= t.t1) ? 1u : 0u);
        w[3] = w[3] + w[3] + (!(ax <= t.t2) ? 1u : 0u);
      }
    }
  }
  // plane words of the channels in `valid`
  __device__ __forceinline__ void planes(uint32_t valid, uint32_t* pl) const {
    pl[0] = w[0] & valid;
    if constexpr (BITS == 2) pl[1] = w[1] & valid;
    if constexpr (BITS == 3) {
      pl[1] = w[3] & valid;
      pl[2] = w[2] & ~w[3] & valid;
      pl[3] = w[1] & ~w[2] & valid;
    }
  }
};

// LDS word of packed word i of the block's run: one spare word per 32 keeps
// lanes whose pixels lie a multiple of 32 words apart in different banks.
__device__ __forceinline__ int tile_slot(int i) { return i + (i >> 5); }

template <int BITS>
__global__ __launch_bounds__(1024) void pack_act_lds_kernel(const float* __restrict__ x, int c, int hw, int cwn,
                                                            int groups, int group, int npix, int sub, int run,
                                                            Thr t, int vec_out, uint32_t* __restrict__ out) {
  constexpr int P = planes_of(BITS);
  extern __shared__ uint32_t tile[];  // [sub * run][gw][P], padded by tile_slot
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int pb = blockIdx.x, cw0 = 0;  // run of pixels, first word
  if (groups > 1) {
    // the groups of a run on one XCD (blocks go to the 8 XCDs in turn), whose
    // L2 then joins their pieces of a pixel's words; past the last run: exit
    const int k = pb >> 3, q = k / groups;
    cw0 = (k - q * groups) * group;
    pb = q * 8 + (pb & 7);
    if (pb * sub * run >= npix) return;
  }
  const int gw = min(cwn - cw0, group);  // this block's words per pixel
  const int pix0 = pb * sub * run;
  const int sb = wave / gw, cwl = wave - sb * gw;
  if (sb < sub) {
    const int pl0 = sb * run + min(lane, run - 1);  // pixel of the block (lanes past a run: its last one again)
    const int pix = min(pix0 + pl0, npix - 1);      // past the end: the last pixel, never written
    const int b = (int)((uint32_t)pix / (uint32_t)hw);
    const int c0 = (cw0 + cwl) * 32, nch = min(32, c - c0);
    const float* src = x + ((int64_t)b * c + c0) * hw + (pix - b * hw);
    WordBits<BITS> wb;
    wb.clear();
    // NB channels from j0 up, every load issued before the first value is waited for
    auto read = [&](auto NBC, int j0) __attribute__((always_inline)) {
      constexpr int NB = decltype(NBC)::value;
      float v[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) v[j] = src[(int64_t)min(j0 + j, nch - 1) * hw];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = NB - 1; j >= 0; --j) wb.push(v[j], t);
    };
    if (nch == 32) {
      read(std::integral_constant<int, 16>{}, 16);
      read(std::integral_constant<int, 16>{}, 0);
    } else {
      for (int j0 = (nch - 1) & ~3; j0 >= 0; j0 -= 4) read(std::integral_constant<int, 4>{}, j0);
    }
    uint32_t pl[P];
    wb.planes(chan_mask(nch), pl);
#pragma unroll
    for (int p = 0; p < P; ++p) tile[tile_slot((pl0 * gw + cwl) * P + p)] = pl[p];
  }
  __syncthreads();
  const int nwords = min(sub * run, npix - pix0) * gw * P;
  if (groups > 1) {
    uint32_t* dst = out + ((int64_t)pix0 * cwn + cw0) * P;
    for (int i = threadIdx.x; i < nwords; i += blockDim.x) {
      const int px = i / (gw * P);
      dst[(int64_t)px * cwn * P + (i - px * gw * P)] = tile[tile_slot(i)];
    }
    return;
  }
  uint32_t* dst = out + (int64_t)pix0 * cwn * P;
  int done = 0;
  if (vec_out) {
    for (int i = threadIdx.x * 4; i + 3 < nwords; i += blockDim.x * 4) {
      const uint32_t* s = tile + tile_slot(i);
      *reinterpret_cast<uint4*>(dst + i) = make_uint4(s[0], s[1], s[2], s[3]);
    }
    done = nwords & ~3;
  }
  for (int i = done + threadIdx.x; i < nwords; i += blockDim.x) dst[i] = tile[tile_slot(i)];
}

// The same for maps of a few pixels (fully connected inputs): lanes along the
// channels, a plane's two words of a 64-channel unit are one wave ballot.  A
// wave takes U units.
template <int BITS>
__global__ __launch_bounds__(256) void pack_act_chan_kernel(const float* __restrict__ x, int c, int hw, int cwn,
                                                            uint32_t units, Thr t, uint32_t* __restrict__ out) {
  constexpr int P = planes_of(BITS), U = 4;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t pairs = (cwn + 1) / 2;
  const uint32_t u0 = (blockIdx.x * 4 + wave) * U;
  float v[U];
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const uint32_t u = min(u0 + k, units - 1);
    const uint32_t pix = u / pairs, b = pix / (uint32_t)hw;
    const int ch = min((int)(u - pix * pairs) * 64 + lane, c - 1);
    v[k] = x[((int64_t)b * c + ch) * hw + (pix - b * hw)];
  }
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const uint32_t u = u0 + k;
    if (u >= units) break;
    const uint32_t pix = u / pairs;
    const int pr = (int)(u - pix * pairs);
    uint64_t bl[P];
    plane_ballots<BITS>(v[k], pr * 64 + lane < c, t, bl);
    const int cw = 2 * pr + lane;
    if (lane < 2 && cw < cwn) {
#pragma unroll
      for (int p = 0; p < P; ++p)
        out[((int64_t)pix * cwn + cw) * P + p] = lane ? (uint32_t)(bl[p] >> 32) : (uint32_t)bl[p];
    }
  }
}

__global__ __launch_bounds__(256) void pack_act_f16_kernel(const float* __restrict__ x, int c, int hw, int cwn,
                                                           int64_t total, uint32_t* __restrict__ out) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= total) return;
  const int pix = (int)(tid % hw);
  const int64_t r = tid / hw;
  const int cw = (int)(r % cwn);
  const int64_t b = r / cwn;
  const int c0 = cw * 32;
  const int nch = min(32, c - c0);
  const float* src = x + (b * c + c0) * (int64_t)hw + pix;
  uint32_t h[16];
  if (nch == 32) {
#pragma unroll
    for (int j = 0; j < 16; ++j)
      h[j] = f16_bits(src[(int64_t)(2 * j) * hw]) | (f16_bits(src[(int64_t)(2 * j + 1) * hw]) << 16);
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const uint32_t lo = 2 * j < nch ? f16_bits(src[(int64_t)(2 * j) * hw]) : 0u;
      const uint32_t hi = 2 * j + 1 < nch ? f16_bits(src[(int64_t)(2 * j + 1) * hw]) : 0u;
      h[j] = lo | (hi << 16);
    }
  }
  uint4* dst = reinterpret_cast<uint4*>(out + ((b * hw + pix) * cwn + cw) * 16);
#pragma unroll
  for (int q = 0; q < 4; ++q) dst[q] = make_uint4(h[4 * q], h[4 * q + 1], h[4 * q + 2], h[4 * q + 3]);
}

// The same through LDS: a block owns `sub` x 64 consecutive pixels (over all
// images) x `group` words, one wave per word of 64 pixels with all its channels'
// loads in flight, and writes each pixel's words as one run.  The direct kernel
// above stores 16 bytes per lane 64 bytes and more apart.  Bound by HBM.
// In the loop of an a16w1 layer 256 x 128 x 32 x 32 takes 42.4 us; inputs in
// cache / not, against the direct kernel, it takes 30.1 / 39.3 us (34.2 / 46.6),
// 256 x 64 x 56 x 56 52.2 / 57.9 (61.3 / 67.6); 4 x 128 x 32 x 32, too few blocks,
// 3.7 in cache (3.0).
__global__ __launch_bounds__(512) void pack_act_f16_lds_kernel(const float* __restrict__ x, int c, int hw, int cwn,
                                                               int groups, int group, int sub, int npix,
                                                               uint4* __restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) uint32_t tile[];  // [sub * 64][16 gw + 4]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pb = groups == 1 ? blockIdx.x : blockIdx.x / groups;
  const int cw0 = (blockIdx.x - pb * groups) * group;
  const int gw = min(cwn - cw0, group);
  const int pitch = gw * 16 + 4;  // 4 words of padding: lanes' 16-byte writes fall in different banks
  const int pix0 = pb * sub * 64;
  const int sb = wave / gw, cwl = wave - sb * gw;
  if (sb < sub) {
    const int pl0 = sb * 64 + lane;
    const int pix = min(pix0 + pl0, npix - 1);
    const int b = (int)((uint32_t)pix / (uint32_t)hw);
    const int c0 = (cw0 + cwl) * 32, nch = min(32, c - c0);
    const float* src = x + ((int64_t)b * c + c0) * hw + (pix - b * hw);
    float v[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) v[j] = src[(int64_t)min(j, nch - 1) * hw];
    __builtin_amdgcn_sched_barrier(0);  // every load is issued before the first value is waited for
    uint4* dst = reinterpret_cast<uint4*>(tile + pl0 * pitch + cwl * 16);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 8 * q + 2 * e;
        const uint32_t lo = j < nch ? f16_bits(v[j]) : 0u, hi = j + 1 < nch ? f16_bits(v[j + 1]) : 0u;
        h[e] = lo | (hi << 16);
      }
      dst[q] = make_uint4(h[0], h[1], h[2], h[3]);
    }
  }
  __syncthreads();
  const int row = gw * 4, n4 = min(sub * 64, npix - pix0) * row;
  uint4* dst = out + ((int64_t)pix0 * cwn + cw0) * 4;
  for (int i = threadIdx.x; i < n4; i += blockDim.x) {
    const int px = i / row, r = i - px * row;
    dst[(int64_t)px * cwn * 4 + r] = *reinterpret_cast<const uint4*>(tile + px * pitch + r * 4);
  }
}

// s_c = (float)(sum_k |W_ck| / K), the sum in double in storage order.
// s_c = mean |W_c| (Eq. 20's scale of a channel's weights), one block per
// output channel.  The sum is taken in double in a fixed order, so the
// result does not depend on the launch: thread j adds |w_i| for i = j,
// j + 256, ... in turn (coalesced reads, up to 32 loads in flight), then the
// 256 partial sums are added pairwise: lanes exchange with lane l ^ 1, l ^ 2,
// ... l ^ 32 (every lane of a pair forms the same sum, IEEE addition being
// commutative), and the four wave sums are added (w0 + w1) + (w2 + w3).  One
// rounding to float at the end.
__global__ __launch_bounds__(256) void weight_scale_kernel(const float* __restrict__ w, int k,
                                                          float* __restrict__ scale) {
  __shared__ double wsum[4];
  const int co = blockIdx.x;
  const float* p = w + (int64_t)co * k;
  double acc = 0.0;
  constexpr int B = 32;
  for (int i0 = threadIdx.x; i0 < k; i0 += 256 * B) {
    // unguarded loads (indices clamped into the channel) so that all of them
    // issue before the first addition; only in-range values are added
    float v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) v[u] = p[min(i0 + 256 * u, k - 1)];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const double t = fabs((double)v[u]);
      if (i0 + 256 * u < k) acc += t;
    }
  }
#pragma unroll
  for (int m = 1; m < 64; m *= 2) acc = acc + __shfl_xor(acc, m);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) scale[co] = (float)(((wsum[0] + wsum[1]) + (wsum[2] + wsum[3])) / (double)k);
}

template <int BITS>
__global__ __launch_bounds__(256) void pack_weight_kernel(const float* __restrict__ w, int cout,
                                                          int cin, int kh, int kw, int cwn,
                                                          int cop, Thr base,
                                                          const float* __restrict__ scale,
                                                          uint32_t* __restrict__ out) {
  constexpr int P = planes_of(BITS);
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)kh * kw * cwn * cop;
  if (tid >= total) return;
  const int co = (int)(tid % cop);
  int64_t r = tid / cop;
  const int cw = (int)(r % cwn);
  r /= cwn;
  const int x = (int)(r % kw);
  const int y = (int)(r / kw);
  uint32_t word[P];
#pragma unroll
  for (int p = 0; p < P; ++p) word[p] = 0u;
  if (co < cout) {
    Thr t = {0.0f, 0.0f, 0.0f};
    if constexpr (BITS > 1) {
      const double s = (double)scale[co];
      t.t0 = (float)((double)base.t0 * s);
      t.t1 = (float)((double)base.t1 * s);
      t.t2 = (float)((double)base.t2 * s);
    }
    const int c0 = cw * 32;
    const int nch = min(32, cin - c0);
    for (int j = 0; j < nch; ++j) {
      const float v = w[(((int64_t)co * cin + c0 + j) * kh + y) * kw + x];
      const uint32_t pl = quant_planes<BITS>(v, t);
#pragma unroll
      for (int p = 0; p < P; ++p) word[p] |= ((pl >> p) & 1u) << j;
    }
  }
  uint32_t* dst = out + tid * P;
#pragma unroll
  for (int p = 0; p < P; ++p) dst[p] = word[p];
}

// Matrix-core operand copies of packed weights: one thread per
// (tap, word, output channel) for int8 (32 bytes), per (tap, word pair,
// output channel) for fp4 (32 bytes = 64 nibbles), per (tap, 16-channel
// k-step, output channel) for fp16 (32 bytes = 16 halves).  Channels past
// cin and padding output channels get code 0 (a 1-bit sign plane alone
// would read as -1 there).
template <int P>
__global__ __launch_bounds__(256) void expand_weight_kernel(const uint32_t* __restrict__ planes,
                                                            int taps, int cwn, int cout, int cop, int cin,
                                                            uint8_t* __restrict__ w_i8,
                                                            uint8_t* __restrict__ w_fp4,
                                                            uint8_t* __restrict__ w_f16) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int cwp = (cwn + 1) / 2;
  const int64_t n_i8 = (int64_t)taps * cwn * cop;
  const int64_t n_fp4 = (int64_t)taps * cwp * cop;
  const int64_t n_f16 = (int64_t)taps * 2 * cwn * cop;
  if (tid >= n_i8 + n_fp4 && tid < n_i8 + n_fp4 + n_f16) {
    const int64_t u = tid - n_i8 - n_fp4;
    const int co = (int)(u % cop);
    const int64_t r = u / cop;
    const int ks = (int)(r % (2 * cwn));
    const int tap = (int)(r / (2 * cwn));
    const int cw = ks >> 1, half = ks & 1;
    const uint32_t* src = planes + (((int64_t)tap * cwn + cw) * cop + co) * P;
    const uint32_t valid = co < cout ? chan_mask(cin - cw * 32) : 0u;
    uint32_t pl[P];
#pragma unroll
    for (int p = 0; p < P; ++p) pl[p] = src[p];
    uint32_t o[8];
    expand_i8_word<P>(pl, valid, o);
    uint32_t hv[8];  // channels 16 half .. 16 half + 15 as fp16 pairs
#pragma unroll
    for (int q = 0; q < 4; ++q) i8_word_to_f16(o[4 * half + q], &hv[2 * q], &hv[2 * q + 1]);
    uint4* dst = reinterpret_cast<uint4*>(w_f16 + u * 32);
    dst[0] = make_uint4(hv[0], hv[1], hv[2], hv[3]);
    dst[1] = make_uint4(hv[4], hv[5], hv[6], hv[7]);
  } else if (tid < n_i8) {
    const int co = (int)(tid % cop);
    const int64_t r = tid / cop;
    const int cw = (int)(r % cwn);
    const int tap = (int)(r / cwn);
    const uint32_t* src = planes + (((int64_t)tap * cwn + cw) * cop + co) * P;
    const uint32_t valid = co < cout ? chan_mask(cin - cw * 32) : 0u;
    uint32_t pl[P];
#pragma unroll
    for (int p = 0; p < P; ++p) pl[p] = src[p];
    uint32_t o[8];
    expand_i8_word<P>(pl, valid, o);
    uint4* dst = reinterpret_cast<uint4*>(w_i8 + tid * 32);
    dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
    dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
  } else if (tid < n_i8 + n_fp4) {
    const int64_t u = tid - n_i8;
    const int co = (int)(u % cop);
    const int64_t r = u / cop;
    const int kp = (int)(r % cwp);
    const int tap = (int)(r / cwp);
    uint32_t o[8];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int cw = 2 * kp + half;
      uint32_t pl[P];
      uint32_t valid = 0u;
#pragma unroll
      for (int p = 0; p < P; ++p) pl[p] = 0u;
      if (cw < cwn) {
        const uint32_t* src = planes + (((int64_t)tap * cwn + cw) * cop + co) * P;
#pragma unroll
        for (int p = 0; p < P; ++p) pl[p] = src[p];
        valid = co < cout ? chan_mask(cin - cw * 32) : 0u;
      }
      expand_fp4_word<P>(pl, valid, o + 4 * half);
    }
    uint4* dst = reinterpret_cast<uint4*>(w_fp4 + u * 32);
    dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
    dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
  }
}

// The planes and every operand copy in one pass over the weights: a block
// owns CO output channels x 64 input channels, whose taps are one contiguous
// run per output channel.  A wave reads whole runs (row by row, V weights per
// lane, eight rows in flight), so a lane's (channel, tap) places are the same
// for every row; the plane bits go to LDS as a byte per weight, ordered
// [output channel][tap][word] with channel 8 b + k of a word in byte b of u32
// k, so that a thread builds a plane word of one (tap, word, output channel)
// as the OR of its eight u32, masked and shifted by k.  Lanes run along the
// output channels there, so every copy leaves in runs of 32 CO bytes.  Bound
// by HBM (4 bytes read, 3.5 + P / 8 written per weight).  With the scales,
// 2432 x 512 x 3 x 3 at 2 bits: 27.2 us, where a gather of single weights 36
// bytes apart (pack_weight_kernel) and a second pass over its planes
// (expand_weight_kernel) took 69.2; those two remain for kernels of more taps
// than fit in LDS.
constexpr int PWT_MAX_TAPS = 25;
__host__ __device__ constexpr int pwt_pitch(int taps) { return 64 * taps + 16; }  // LDS bytes per output channel

template <int BITS, int CO, int V>
__global__ __launch_bounds__(256) void pack_weight_tile_kernel(
    const float* __restrict__ w, int cout, int cin, int taps, FastDiv fd_taps, int cwn, int cop, Thr base,
    const float* __restrict__ scale, uint32_t* __restrict__ out, uint8_t* __restrict__ w_i8,
    uint8_t* __restrict__ w_fp4, uint8_t* __restrict__ w_f16) {
  constexpr int P = planes_of(BITS), R = CO / 4;  // rows per wave
  extern __shared__ __attribute__((aligned(16))) uint8_t codes[];  // [CO][pitch]
  __shared__ float thr[3][CO];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pairs = (cwn + 1) / 2;
  const int kp = blockIdx.x % pairs, co0 = (blockIdx.x / pairs) * CO;
  const int c0 = kp * 64, nch = min(64, cin - c0);
  const int nco = min(CO, cout - co0);  // <= 0: padding rows only
  const int pitch = pwt_pitch(taps);
  if (threadIdx.x < CO) {
    // the same rounding as pack_weight_kernel
    const double s = (double)scale[min(co0 + (int)threadIdx.x, cout - 1)];
    thr[0][threadIdx.x] = (float)((double)base.t0 * s);
    thr[1][threadIdx.x] = (float)((double)base.t1 * s);
    thr[2][threadIdx.x] = (float)((double)base.t2 * s);
  }
  if (nch < 64)  // uniform: channels past the last one are 0 in every plane
    for (int i = threadIdx.x; i < CO * pitch / 16; i += 256)
      reinterpret_cast<uint4*>(codes)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  const int len = nch * taps;
  const float* src = w + ((int64_t)co0 * cin + c0) * taps;
  const int64_t rs = (int64_t)cin * taps;
  if (nco > 0) {
    for (int e0 = 0; e0 < len; e0 += 64 * V) {
      const int e = e0 + lane * V;
      const bool ok = e < len;  // V = 4: len is a multiple of 4
      const int el = ok ? e : 0;
      float v[R][V];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float* s = src + min(wave + 4 * r, nco - 1) * rs + el;
        if constexpr (V == 4) {
          const float4 f = *reinterpret_cast<const float4*>(s);
          v[r][0] = f.x;
          v[r][1] = f.y;
          v[r][2] = f.z;
          v[r][3] = f.w;
        } else {
          v[r][0] = *s;
        }
      }
      int off[V];
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const int c = (int)fdiv((uint32_t)(el + i), fd_taps), tap = el + i - c * taps;
        off[i] = tap * 64 + (c & 32) + (c & 7) * 4 + ((c >> 3) & 3);
      }
      if (ok) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int row = wave + 4 * r;
          const float t0 = thr[0][row], t1 = thr[1][row], t2 = thr[2][row];
          uint8_t* d = codes + row * pitch;
#pragma unroll
          for (int i = 0; i < V; ++i) {
            // plane bits of a weight: quant_planes in its order of compares
            // (without branches), so that weights meet thresholds that are
            // not finite as there: s_c is data, and a NaN or infinite weight
            // makes NaN ones (a NaN compares false: not <= it, so beyond it)
            const float x = v[r][i];
            uint32_t b = x > 0.0f ? 1u : 0u;
            if constexpr (BITS > 1) {
              const float ax = fabsf(x);
              if constexpr (BITS == 2) b |= 2u;
              else b |= ax <= t1 ? 8u : (ax <= t2 ? 4u : 2u);
              if (ax <= t0) b = 0u;
            }
            d[off[i]] = (uint8_t)b;
          }
        }
      }
    }
  }
  __syncthreads();
  for (int u = threadIdx.x; u < 2 * CO * taps; u += 256) {
    const int col = u & (CO - 1), h = (u / CO) & 1, tap = u / (2 * CO);
    const int co = co0 + col, cw = 2 * kp + h;
    const uint4* cp = reinterpret_cast<const uint4*>(codes + col * pitch + tap * 64 + 32 * h);
    const uint4 x0 = cp[0], x1 = cp[1];
    const uint32_t x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
    const bool in = col < nco && cw < cwn;
    const uint32_t valid = in ? chan_mask(cin - cw * 32) : 0u;
    uint32_t pl[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      uint32_t o = 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k) o |= ((x[k] >> p) & 0x01010101u) << k;
      pl[p] = in ? o : 0u;
    }
    uint32_t f4[4];
    expand_fp4_word<P>(pl, valid, f4);
    *reinterpret_cast<uint4*>(w_fp4 + (((int64_t)tap * pairs + kp) * cop + co) * 32 + 16 * h) =
        make_uint4(f4[0], f4[1], f4[2], f4[3]);
    if (cw >= cwn) continue;
    const int64_t rec = ((int64_t)tap * cwn + cw) * cop + co;
#pragma unroll
    for (int p = 0; p < P; ++p) out[rec * P + p] = pl[p];
    uint32_t o[8];
    expand_i8_word<P>(pl, valid, o);
    uint4* d8 = reinterpret_cast<uint4*>(w_i8 + rec * 32);
    d8[0] = make_uint4(o[0], o[1], o[2], o[3]);
    d8[1] = make_uint4(o[4], o[5], o[6], o[7]);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      uint32_t hv[8];
#pragma unroll
      for (int q = 0; q < 4; ++q) i8_word_to_f16(o[4 * half + q], &hv[2 * q], &hv[2 * q + 1]);
      uint4* df = reinterpret_cast<uint4*>(w_f16 + (((int64_t)tap * 2 * cwn + 2 * cw + half) * cop + co) * 32);
      df[0] = make_uint4(hv[0], hv[1], hv[2], hv[3]);
      df[1] = make_uint4(hv[4], hv[5], hv[6], hv[7]);
    }
  }
}

template <int BITS, int CO, int V>
void pack_weight_tiles(const float* w, int cout, int cin, int taps, Thr base, const float* scale, uint32_t* out,
                       uint8_t* w_i8, uint8_t* w_fp4, uint8_t* w_f16, hipStream_t s) {
  const int cwn = ceil_div(cin, 32), cop = cout_pad(cout);
  const dim3 g((unsigned)(ceil_div(cwn, 2) * (cop / CO)));
  pack_weight_tile_kernel<BITS, CO, V><<<g, 256, (size_t)CO * pwt_pitch(taps), s>>>(
      w, cout, cin, taps, make_fastdiv((uint32_t)taps), cwn, cop, base, scale, out, w_i8, w_fp4, w_f16);
}

// 16-bit weights (Table I rows with 1..3-bit inputs and 16-bit weights):
// fp32 OIHW -> fp16 [kh][kw][2 cw][cout_pad][16 halves], the layout of the
// fp16 operand copy, rounded to nearest even; channels past cin and padding
// output channels are +0.  One thread per 32-byte record.
__global__ __launch_bounds__(256) void pack_weight_f16_kernel(const float* __restrict__ w, int cout, int cin,
                                                              int kh, int kw, int cwn, int cop,
                                                              uint32_t* __restrict__ out) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)kh * kw * 2 * cwn * cop;
  if (tid >= total) return;
  const int co = (int)(tid % cop);
  const int64_t r = tid / cop;
  const int ks = (int)(r % (2 * cwn));
  const int tap = (int)(r / (2 * cwn));
  const int y = tap / kw, x = tap - (tap / kw) * kw;
  uint32_t hv[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    uint32_t pair = 0u;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int ci = 16 * ks + 2 * q + e;
      if (co < cout && ci < cin) pair |= f16_bits(w[(((int64_t)co * cin + ci) * kh + y) * kw + x]) << (16 * e);
    }
    hv[q] = pair;
  }
  uint4* dst = reinterpret_cast<uint4*>(out + tid * 8);
  dst[0] = make_uint4(hv[0], hv[1], hv[2], hv[3]);
  dst[1] = make_uint4(hv[4], hv[5], hv[6], hv[7]);
}

}  // namespace

// Lanes along the pixels where a wave's 64 pixels span at most five images (a
// channel is then read in runs of 64 bytes and more), on smaller maps from 4
// pixels on where that still fills the chip, and from 2 on up to 8 channels,
// which leave most lanes along them idle; else along the channels.  Both at 1 bit,
// pixels / channels: 256 x 512 x 3 x 5 3.5 / 10.9 us, 16 x 512 x 3 x 5 3.6 /
// 2.6, 1024 x 128 x 2 x 4 2.9 / 4.2, 64 x 512 x 3 x 3 3.9 / 2.9, 16384 x 32 x 1
// x 7 5.1 / 13.6, 1024 x 512 x 2 x 2 5.9 / 5.4, 65536 x 64 x 1 x 1 10.8 / 8.4,
// 256 x 1024 x 1 x 1 29.7 / 2.5; 2000 x 3 x 2 x 2 3.0 / 3.6, 141 x 8 x 3 x 4 3.0
// / 3.2, 141 x 16 x 3 x 4 3.4 / 3.2.
bool pack_act_by_pixel(int n, int c, int h, int w) {
  const int64_t hw = (int64_t)h * w, npix = n * hw, pairs = npix * ceil_div(ceil_div(c, 32), 2);
  return npix < ((int64_t)1 << 31) - 1024 &&
         (hw >= 16 || (hw >= 2 && c <= 8) || (hw >= 8 && pairs >= 8192) || (hw >= 4 && pairs >= 65536));
}

int launch_pack_act(const float* x, int n, int c, int h, int w, int bits, Thr t, uint32_t* out,
                    hipStream_t s) {
  const int hw = h * w;
  const int cwn = ceil_div(c, 32);
  const int64_t npix = (int64_t)n * hw;
  if (npix == 0) return QCONV_OK;
  if (pack_act_by_pixel(n, c, h, w)) {
    // How many words (group) and runs (sub) a block takes.  At 1 bit, inputs in
    // cache / not, against one block per 64 pixels of an image:
    // - Maps of 16 to 63 pixels that do not divide 64: runs of whole images,
    //   which are then read from a few whole cache lines where a run of 64
    //   pixels reads parts of lines of two images, in groups of four words: 935
    //   x 512 x 7 x 7 15.7 / 19.3 us (15.6 / 21.5; runs of 64 23.7 / 25.0), 512
    //   x 640 x 7 x 7 11.7 / 14.0 (12.6 / 19.6; 17.0 / 18.0), 675 x 256 x 6 x 6
    //   5.1 / 7.0 (5.8 / 9.2; 6.4 / 8.0).  (The limit keeps a launch of such
    //   runs, up to 64 lanes for 33 pixels, below 2^32 threads.)
    // - Larger maps whose planes are not whole runs of 64 bytes: two words of
    //   four consecutive runs, which share the cache lines at their ends, where
    //   that leaves one wave per SIMD: 195 x 512 x 11 x 11 at 2 bits 11.7 / 13.7
    //   (13.8 / 17.9; all 16 words of one run 14.7 / 16.0), 900 x 128 x 9 x 9
    //   8.8 / 11.0 (11.3 / 11.9; 11.7 / 12.0).
    // - Else up to 16 words all of a pixel's, with one wave per word of a run
    //   while the tensor has fewer runs than four per CU, else at least four
    //   waves, and two runs (8 to 16 waves) for 4 to 8 words where it has more
    //   than eight per CU (256 x 128 x 32 x 32 25.9 -> 24.9 us).
    // - More words, and maps below 16 pixels, whose runs are few: groups of
    //   four.  32 x 640 x 32 x 32 13.5 / 16.0 us (13.5 / 18.1; groups of 16
    //   15.9 / 20.0), 64 x 544 x 28 x 28 19.5 / 22.3 (22.4 / 25.2; 27.7 / 30.4),
    //   128 x 1024 x 14 x 14 21.2 / 23.5 (24.2 / 27.7; 25.2 / 27.1); 256 x 512 x
    //   3 x 5 3.5 (5.2; 6.6).
    const int run = hw >= 16 && hw < 64 && npix * cwn < ((int64_t)1 << 31) ? 64 / hw * hw : 64;
    const int64_t runs = npix / run;
    int group = cwn, sub = 1;
    if (hw < 16) group = cwn < 4 ? cwn : 4;
    else if (cwn < 4) sub = runs < 1024 ? 1 : ceil_div(4, cwn);
    else if (run < 64) group = 4;
    else if (cwn > 16) group = 4, sub = 2;
    else if (hw % 16 && runs * cwn >= 1024) group = 2, sub = 4;
    else if (cwn <= 8 && runs >= 2048) sub = 2;
    const int groups = ceil_div(cwn, group);
    const int64_t blocks = (npix + sub * run - 1) / (sub * run);
    const dim3 g((unsigned)(groups == 1 ? blocks : (blocks + 7) / 8 * 8 * groups));
    const int threads = 64 * sub * group;
    const size_t words = (size_t)sub * run * group * planes_of(bits);
    const size_t lds = (words + words / 32) * sizeof(uint32_t);
    // every block's output starts on 16 bytes
    const int vec_out = ((uintptr_t)out & 15u) == 0 && (sub * run * cwn * planes_of(bits)) % 4 == 0;
#define QC_PACK(B) \
  pack_act_lds_kernel<B><<<g, threads, lds, s>>>(x, c, hw, cwn, groups, group, (int)npix, sub, run, t, vec_out, out)
    if (bits == 1) QC_PACK(1);
    else if (bits == 2) QC_PACK(2);
    else QC_PACK(3);
#undef QC_PACK
    return hip_status();
  }
  // images in runs whose grids stay below 2^31 threads (16 per unit; a launch
  // takes fewer than 2^32) and whose unit indices fit 32 bits: one launch
  // below 2^27 units
  const int64_t upi = (int64_t)hw * ceil_div(cwn, 2), limit = (int64_t)1 << 27;
  const int per = (int)(upi < limit ? (limit / upi < n ? limit / upi : n) : 1);
  for (int i = 0; i < n;) {
    const int m = n - i < per ? n - i : per;
    const uint32_t units = (uint32_t)(m * upi);
    const dim3 grid((unsigned)(((int64_t)units + 15) / 16));
    const float* xi = x + (int64_t)i * c * hw;
    uint32_t* oi = out + (int64_t)i * hw * cwn * planes_of(bits);
    switch (bits) {
      case 1: pack_act_chan_kernel<1><<<grid, 256, 0, s>>>(xi, c, hw, cwn, units, t, oi); break;
      case 2: pack_act_chan_kernel<2><<<grid, 256, 0, s>>>(xi, c, hw, cwn, units, t, oi); break;
      default: pack_act_chan_kernel<3><<<grid, 256, 0, s>>>(xi, c, hw, cwn, units, t, oi); break;
    }
    const int rc = hip_status();
    if (rc) return rc;
    i += m;
  }
  return QCONV_OK;
}

int launch_pack_act_f16(const float* x, int n, int c, int h, int w, uint32_t* out, hipStream_t s) {
  const int hw = h * w;
  const int cwn = ceil_div(c, 32);
  const int64_t npix = (int64_t)n * hw, total = npix * cwn;
  if (total == 0) return QCONV_OK;
  // through LDS where lanes run along the pixels and every CU gets four waves
  if (hw >= 16 && npix < ((int64_t)1 << 31) - 1024 && total >= 64 * 1024) {
    // up to eight words of one run of 64 pixels; of maps whose planes are not
    // whole runs of 64 bytes two words (or all three) of two consecutive runs or
    // a single one of four, which share the cache lines at their ends (451 x 256 x 6 x 6 6.4 / 7.5 us,
    // the direct kernel 6.4 / 8.9, eight words 7.3 / 8.0; 416 x 32 x 44 x 47 27.2
    // / 32.9, 29.1 / 36.2, one run 31.6 / 33.8)
    const bool shared = hw % 16 != 0;
    const int group = shared ? (cwn <= 3 ? cwn : 2) : (cwn < 8 ? cwn : 8), sub = shared ? (cwn == 1 ? 4 : 2) : 1;
    const int groups = ceil_div(cwn, group);
    const dim3 g((unsigned)((npix + sub * 64 - 1) / (sub * 64) * groups));
    pack_act_f16_lds_kernel<<<g, 64 * group * sub, (size_t)sub * 64 * (group * 16 + 4) * sizeof(uint32_t), s>>>(
        x, c, hw, cwn, groups, group, sub, (int)npix, reinterpret_cast<uint4*>(out));
    return hip_status();
  }
  pack_act_f16_kernel<<<dim3((unsigned)((total + 255) / 256)), 256, 0, s>>>(x, c, hw, cwn, total, out);
  return hip_status();
}

int launch_pack_weight_f16(const float* w, int cout, int cin, int kh, int kw, uint32_t* out, float* scale,
                           hipStream_t s) {
  weight_scale_kernel<<<cout, 256, 0, s>>>(w, cin * kh * kw, scale);
  const int cwn = ceil_div(cin, 32);
  const int64_t total = (int64_t)kh * kw * 2 * cwn * cout_pad(cout);
  pack_weight_f16_kernel<<<dim3((unsigned)((total + 255) / 256)), 256, 0, s>>>(w, cout, cin, kh, kw, cwn,
                                                                                cout_pad(cout), out);
  return hip_status();
}

int launch_pack_weight(const float* w, int cout, int cin, int kh, int kw, int bits,
                       const float* base_thr, uint32_t* out, float* scale, hipStream_t s) {
  const int k = cin * kh * kw;
  weight_scale_kernel<<<cout, 256, 0, s>>>(w, k, scale);
  const int cwn = ceil_div(cin, 32);
  const int cop = cout_pad(cout);
  const int taps = kh * kw;
  Thr b = {base_thr[0], base_thr[1], base_thr[2]};
  uint8_t* w_i8 = reinterpret_cast<uint8_t*>(out) + wbytes_planes(cout, cin, kh, kw, bits);
  uint8_t* w_fp4 = w_i8 + wbytes_i8(cout, cin, kh, kw);
  uint8_t* w_f16 = w_fp4 + wbytes_fp4(cout, cin, kh, kw);
  if (taps <= PWT_MAX_TAPS) {
    // 16-byte loads where every run starts on 16 bytes; 32 output channels
    // per block where that gives every CU two blocks, else 8
    const bool vec = ((int64_t)cin * taps) % 4 == 0 && ((uintptr_t)w & 15u) == 0;
    const bool wide = ceil_div(cwn, 2) * (cop / 32) >= 512;
#define QC_PWT(B)                                                                                              \
  do {                                                                                                         \
    if (wide && vec) pack_weight_tiles<B, 32, 4>(w, cout, cin, taps, b, scale, out, w_i8, w_fp4, w_f16, s);    \
    else if (wide) pack_weight_tiles<B, 32, 1>(w, cout, cin, taps, b, scale, out, w_i8, w_fp4, w_f16, s);      \
    else if (vec) pack_weight_tiles<B, 8, 4>(w, cout, cin, taps, b, scale, out, w_i8, w_fp4, w_f16, s);        \
    else pack_weight_tiles<B, 8, 1>(w, cout, cin, taps, b, scale, out, w_i8, w_fp4, w_f16, s);                 \
  } while (0)
    if (bits == 1) QC_PWT(1);
    else if (bits == 2) QC_PWT(2);
    else QC_PWT(3);
#undef QC_PWT
    return hip_status();
  }
  const int64_t total = (int64_t)taps * cwn * cop;
  const dim3 grid((unsigned)((total + 255) / 256));
  switch (bits) {
    case 1: pack_weight_kernel<1><<<grid, 256, 0, s>>>(w, cout, cin, kh, kw, cwn, cop, b, scale, out); break;
    case 2: pack_weight_kernel<2><<<grid, 256, 0, s>>>(w, cout, cin, kh, kw, cwn, cop, b, scale, out); break;
    default: pack_weight_kernel<3><<<grid, 256, 0, s>>>(w, cout, cin, kh, kw, cwn, cop, b, scale, out); break;
  }
  const int64_t items =
      (int64_t)taps * cwn * cop + (int64_t)taps * ((cwn + 1) / 2) * cop + (int64_t)taps * 2 * cwn * cop;
  const dim3 g2((unsigned)((items + 255) / 256));
  switch (bits) {
    case 1: expand_weight_kernel<1><<<g2, 256, 0, s>>>(out, taps, cwn, cout, cop, cin, w_i8, w_fp4, w_f16); break;
    case 2: expand_weight_kernel<2><<<g2, 256, 0, s>>>(out, taps, cwn, cout, cop, cin, w_i8, w_fp4, w_f16); break;
    default: expand_weight_kernel<4><<<g2, 256, 0, s>>>(out, taps, cwn, cout, cop, cin, w_i8, w_fp4, w_f16); break;
  }
  return hip_status();
}

}  // namespace qc
