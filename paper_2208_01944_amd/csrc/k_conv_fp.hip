// Grouped B-bit convolution: B = 2, 3, 4 on the FP4 / FP6 matrix cores, 6- and
// 8-bit codes (B = 8 below) on int8.
//
// Per group the layer is D[k][m] = sum_K W[k][K] X[K][m] (Eq. 1), k an output
// channel, m an output pixel, K = (ky, kx, c), in K-blocks of 64 codes of one
// tap: one v_mfma_scale_f32_32x32x64_f8f6f4 per 32 channels x 32 pixels.
//
//  * B = 2: codes as E2M1 c / 2 (the code is the bit pattern), weights w / 2;
//    accumulator t / 4.
//  * B = 3, 4: E2M3, c / 8 for a code c in 0..15 is the pattern c itself (0..7
//    subnormal, 8..15 with exponent field 1), w / 8 is the pattern |w| with the
//    sign in bit 5; accumulator t / 64.
//  Products are exact multiples of 1/4 (1/64) and the fp32 accumulator holds
//  every partial sum exactly while |t| + |bias| + qmax |res_mult| < 2^24.
//
//  * B = 8 (also 6-bit codes, stored as bytes): x - 128 as int8 (the top bit
//    flipped), two v_mfma_i32_32x32x32_i8 a K-block, accumulators starting at
//    bias + 128 sum(w), which also restores taps outside the image (their code
//    0 reads as -128); requant in fp64.
//
// Any channel count: K-blocks and channel blocks are padded with zero weights,
// so what an operand load brings in past the end of a row (the row's padding,
// the next row, zeros past the tensor) is multiplied by zero; padded output
// channels have scale 0, give code 0 (the row's padding bits) and only words
// inside the row are stored.
//
// Requant: the accumulator starts at bias, u = t + bias (+ res_mult code), and
// one fma with rounding towards minus infinity gives RD(x), x = u M 2^-sh +
// 1/2.  Integers are representable, so floor(RD(x)) = floor(x): the definition,
// for every shift (M < 2^24).  Layers with a channel past those bounds (M up to
// 2^31, bias up to 2^30) take the wide builds: the accumulator starts at 0, u is
// an int32 (B = 8: formed in fp64) and the same fma in fp64 holds for every u and
// M the interface admits (both below 2^53).  14x14, 256 channels, G = 4, batch
// 128, 2-bit: 38.5 us against 34.7 for 15-bit multipliers (119 with the int64
// requant of the int8 kernels, which took such layers); 4-bit with a shortcut
// 58.5 against 50.3 (145); 14x14, 1024 channels, batch 8, 2-bit 26.7 against 24.8
// (67 ms on the direct kernel, as the filter passes the int8 kernels' LDS).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "codes.h"
#include "conv_common.h"
#include "palq_internal.h"

namespace palq {

namespace {

// ------------------------------------------------------------ per-width facts
template <int B>
struct FpT {
  static constexpr int SLAB = B == 2 ? 1024 : B == 8 ? 2048 : 1536;  // weight bytes of (K-block, 32 channels)
  static constexpr int PPX = B == 2 ? 1 : B == 8 ? 4 : 2;  // 16-byte LDS pieces of a pixel's K-block
  static constexpr int XB = 8 * B;                         // its bytes in memory
  static constexpr int CHS = 4 * B;                        // bytes of a lane half's 32 codes
  static constexpr int L = B == 2 ? 2 : B == 8 ? 0 : 6;    // the accumulator is 2^-L t
  static constexpr int J = B == 8 ? 2 : 1;                 // MFMAs (operands) of a K-block
  using Acc = typename std::conditional<B == 8, v16i, v16f>::type;
};

// K order of a lane's 32 codes: field f of the operand holds code fp_code(f).
// B = 2: nibble n (word q = n / 8, position j = n % 8) is code 16 (q >> 1) +
// 2 j + (q & 1): a word's even (odd) codes are its bit pairs masked in place
// (after one shift).  B = 3: kPerm3, B = 4: kPerm4 (act_fp6_4).
__host__ __device__ inline int fp_code(int B, int f) {
  constexpr int kPerm3[16] = {0, 3, 6, 9, 12, 15, 2, 5, 8, 11, 14, 1, 4, 7, 10, 13};
  constexpr int kPerm4[16] = {0, 1, 3, 4, 6, 7, 9, 10, 12, 13, 15, 8, 2, 11, 5, 14};
  if (B == 2) return 16 * (f >> 4) + 2 * (f & 7) + ((f >> 3) & 1);
  return (f & 16) + (B == 3 ? kPerm3[f & 15] : kPerm4[f & 15]);
}

// A lane's 32 codes as the MFMA operand.
__device__ __forceinline__ v8i act_fp4(uint32_t x, uint32_t y) {
  const uint32_t m = 0x33333333u;
  const v4i b = {(int)(x & m), (int)((x >> 2) & m), (int)(y & m), (int)((y >> 2) & m)};
  return __builtin_shufflevector(b, b, 0, 1, 2, 3, -1, -1, -1, -1);
}
// 3-bit chunk (low words 0, 1, bit-2 word): word 3 u + d = low word u masked
// to its fields' code pairs, or'ed with the bit-2 word rotated so that bit 2
// of those codes lands two bits above its pair.
__device__ __forceinline__ v8i act_fp6_3(uint32_t lo0, uint32_t lo1, uint32_t hi) {
  const uint32_t r0 = __builtin_amdgcn_alignbit(hi, hi, 30), r1 = __builtin_amdgcn_alignbit(hi, hi, 31);
  v8i d;
  d[0] = (int)((lo0 & 0xC30C30C3u) | (r0 & 0x04104104u));
  d[1] = (int)((lo0 & 0x30C30C30u) | (r0 & 0x41041041u));
  d[2] = (int)((lo0 & 0x0C30C30Cu) | (r0 & 0x10410410u));
  d[3] = (int)((lo1 & 0xC30C30C3u) | (r1 & 0x04104104u));
  d[4] = (int)((lo1 & 0x30C30C30u) | (r1 & 0x41041041u));
  d[5] = (int)((lo1 & 0x0C30C30Cu) | (r1 & 0x10410410u));
  d[6] = d[7] = 0;
  return d;
}
// Two words of nibbles (codes 0-7 in w, 8-15 in v) to 16 six-bit fields: a
// nibble at bit 4 j meets a field at bit 6 f after a shift by 0 or by 2, so
// three words come from masks of w, v and w << 2, (v:w) >> 30.
__device__ __forceinline__ void nib6(uint32_t w, uint32_t v, int *d) {
  const uint32_t s = __builtin_amdgcn_alignbit(v, w, 30);                       // v << 2 | w >> 30
  d[0] = (int)((w & 0x0F00F00Fu) | ((w << 2) & 0xC03C03C0u));                  // w0 w1 w3 w4 w6 w7 (low half)
  d[1] = (int)((v & 0xF00F00F0u) | (s & 0x03C03C03u));                         // w7 (high half) v1 v2 v4 v5 v7
  d[2] = (int)((w & 0x00F00F00u) | (s & 0x3C03C03Cu));                         // v0 w2 v3 w5 v6
}
__device__ __forceinline__ v8i act_fp6_4(v4i x) {
  int d[6];
  nib6((uint32_t)x[0], (uint32_t)x[1], d);
  nib6((uint32_t)x[2], (uint32_t)x[3], d + 3);
  return v8i{d[0], d[1], d[2], d[3], d[4], d[5], 0, 0};
}
template <int B>
__device__ __forceinline__ v8i act_fp(v4i x) {
  static_assert(B != 8, "FP4 and FP6 operands");
  if constexpr (B == 2) return act_fp4((uint32_t)x[0], (uint32_t)x[1]);
  else if constexpr (B == 3) return act_fp6_3((uint32_t)x[0], (uint32_t)x[1], (uint32_t)x[2]);
  else return act_fp6_4(x);
}
template <int B>
__device__ __forceinline__ v8i wt_fp(v4i a, v2i b) {
  if constexpr (B == 2) return __builtin_shufflevector(a, a, 0, 1, 2, 3, -1, -1, -1, -1);
  else return v8i{a[0], a[1], a[2], a[3], b[0], b[1], 0, 0};
}
__device__ __forceinline__ v4i flip_i8(v4i x) {
  const int m = (int)0x80808080u;
  return v4i{x[0] ^ m, x[1] ^ m, x[2] ^ m, x[3] ^ m};
}
template <int B>
__device__ __forceinline__ v16f mfma_fp(v8i a, v8i b, v16f c) {
  constexpr int F = B == 2 ? 4 : 2;  // E2M1 / E2M3
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, F, F, 0, 0, 0, 0);
}

// Constants of 64 channels, one 1 KB block: [scale 64][bias 64][res_mult
// 64][unused 64] floats in accumulator units, or (B = 8 and the wide builds)
// [M 2^-sh 64] doubles, [bias 64][res_mult 64] int32 (B = 8: bias + 128 sum(w)).
constexpr int kCstBlock = 1024;

// The requant of a build.  kBase: fp32, B = 8: fp64 on an int32 u.  kFp4: the
// 2-bit form by FP4 conversions (requant_z).  kWide: any parameters.
enum Ep { kBase, kFp4, kWide };

// ------------------------------------------------------------ prepare
// One launch per layer (B = 8: wsum_i8_kernel before it).  Workgroup 0: the
// requant constants (zero for padded channels; B < 8: of the base builds, then
// of the wide ones) and two flags: bad[0], some channel is outside the base
// builds' bounds; bad[1], some shift exceeds 21 (requant_z).  The others: weight
// slabs, one lane operand (16 or 24 bytes) per thread, [G][coutp /
// 32][kb_total][SLAB]; E2M3 slabs hold bytes 0-15 of every lane, then bytes
// 16-23.  Projection K-blocks of source group g hold the projection filter of
// its destination group (g + s) mod G.
struct PrepArgs {
  const uint8_t *w, *pw;
  const int32_t *mult, *shift, *bias, *res_mult;
  int32_t G, cout, coutp, taps, cin, pcin, cpb, km, kb, shuffle, res_max;
  int64_t row, prow;  // packed bytes of a tap's row of the filter and of a projection row
  int64_t acc_bound;
  uint8_t *wp;
  float *cst;     // B < 8: constants of the base builds
  uint8_t *wide;  // constants of the wide builds and of B = 8
  int32_t *bad;
  int32_t w_bits;
  int32_t *wsum;  // B = 8: 128 sum(w) per channel
};

// 128 times the sum of each output channel's weights (the projection's of the
// destination group included), one wave per channel.
__global__ __launch_bounds__(256) void wsum_i8_kernel(PrepArgs a) {
  const int c = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  if (c >= a.G * a.cout) return;
  const int g = c / a.cout, k = c - g * a.cout, sh = 8 - a.w_bits;
  int32_t sum = 0;
  const int8_t *w = (const int8_t *)(a.w + (int64_t)c * a.taps * a.row);
  for (int tap = 0; tap < a.taps; ++tap)
    for (int i = lane; i < a.cin; i += 64) sum += (int32_t)(int8_t)(w[tap * a.row + i] << sh) >> sh;
  if (a.pw) {
    const int8_t *p = (const int8_t *)(a.pw + ((int64_t)((g + a.shuffle) % a.G) * a.cout + k) * a.prow);
    for (int i = lane; i < a.pcin; i += 64) sum += (int32_t)(int8_t)(p[i] << sh) >> sh;
  }
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) a.wsum[c] = 128 * sum;
}

template <int B>
__global__ __launch_bounds__(512) void conv_fp_prep_kernel(PrepArgs a) {
  if (blockIdx.x == 0) {
    __shared__ int any_bad, any_wide;
    if (threadIdx.x == 0) any_bad = any_wide = 0;
    __syncthreads();
    int bad = 0, wide = 0;
    for (int i = threadIdx.x; i < a.G * a.coutp; i += 512) {
      const int g = i / a.coutp, k = i - g * a.coutp;
      double s = 0.0;
      float sc = 0.0f, b = 0.0f, rm = 0.0f;
      int32_t bw = 0, rw = 0;
      if (k < a.cout) {
        const int c = g * a.cout + k;
        const int64_t m = a.mult[c], bi = a.bias ? a.bias[c] : 0, r = a.res_mult ? a.res_mult[c] : 0;
        const int sh = a.shift[c];
        const int64_t lim = (int64_t)1 << (B == 8 ? 31 : 24);
        const int64_t umax = a.acc_bound + (bi < 0 ? -bi : bi) + (r < 0 ? -r : r) * a.res_max;
        s = ldexp((double)m, -sh);
        bw = (int32_t)((uint32_t)bi + (B == 8 ? (uint32_t)a.wsum[c] : 0u));
        rw = (int32_t)r;
        if (umax >= lim || (B != 8 && (sh < 1 || sh > 62 || m <= -lim || m >= lim))) {
          bad = 1;
        } else if constexpr (B != 8) {
          if (sh > 21) wide = 1;
          sc = ldexpf((float)m, FpT<B>::L - sh);
          b = ldexpf((float)bi, -FpT<B>::L);
          rm = ldexpf((float)r, -FpT<B>::L);
        }
      }
      uint8_t *wb = a.wide + (int64_t)(i >> 6) * kCstBlock;
      ((double *)wb)[i & 63] = s;
      ((int32_t *)wb)[128 + (i & 63)] = bw;
      ((int32_t *)wb)[192 + (i & 63)] = rw;
      if constexpr (B == 8) continue;
      float *blk = a.cst + (int64_t)(i >> 6) * 256 + (i & 63);
      blk[0] = sc;
      blk[64] = b;
      blk[128] = rm;
      blk[192] = 0.0f;
    }
    if (bad) atomicOr(&any_bad, 1);
    if (wide) atomicOr(&any_wide, 1);
    __syncthreads();
    if (threadIdx.x == 0) {
      a.bad[0] = any_bad;
      a.bad[1] = any_wide;
    }
    return;
  }
  const int64_t t = (int64_t)(blockIdx.x - 1) * 512 + threadIdx.x;
  const int nc32 = a.coutp / 32;
  if (t >= (int64_t)a.G * nc32 * a.kb * 64 * FpT<B>::J) return;
  const int lane = (int)(t & 63), half = lane >> 5;
  const int jj = (int)(t >> 6) % FpT<B>::J;  // operand of the K-block
  const int rest = (int)(t >> 6) / FpT<B>::J;
  const int r2 = rest / a.kb, kb = rest - r2 * a.kb;
  const int g = r2 / nc32, k = (r2 - g * nc32) * 32 + (lane & 31);
  const bool main = kb < a.km;
  const int tap = main ? kb / a.cpb : 0;
  if constexpr (B == 8) {
    // codes 32 half + 16 jj .. + 15 of the K-block, sign-extended from w_bits
    const int c0 = 64 * (main ? kb - tap * a.cpb : kb - a.km) + 32 * half + 16 * jj;
    const int n = min(16, (main ? a.cin : a.pcin) - c0);
    const uint8_t *row = main ? a.w + (((int64_t)g * a.cout + k) * a.taps + tap) * a.row
                              : a.pw + ((int64_t)((g + a.shuffle) % a.G) * a.cout + k) * a.prow;
    const int sh = 8 - a.w_bits;
    uint32_t o[4] = {0, 0, 0, 0};
    if (k < a.cout)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (e < n) o[e >> 2] |= (uint32_t)(uint8_t)((int32_t)(int8_t)(row[c0 + e] << sh) >> sh) << (8 * (e & 3));
    *(uint4 *)(a.wp + (int64_t)rest * FpT<B>::SLAB + (jj * 64 + lane) * 16) = make_uint4(o[0], o[1], o[2], o[3]);
    return;
  }
  const int c0 = 64 * (main ? kb - tap * a.cpb : kb - a.km) + 32 * half;  // first code of the lane
  const int n = min(32, (main ? a.cin : a.pcin) - c0);                     // its codes inside the row
  uint32_t u[4] = {0, 0, 0, 0};
  if (k < a.cout && n > 0) {
    const uint8_t *row = main ? a.w + (((int64_t)g * a.cout + k) * a.taps + tap) * a.row
                              : a.pw + ((int64_t)((g + a.shuffle) % a.G) * a.cout + k) * a.prow;
    const uint32_t *p = (const uint32_t *)(row + (int64_t)(c0 / 32) * FpT<B>::CHS);
    constexpr int PER = B == 3 ? 16 : 32 / B;  // codes of a word (B = 3: of its low words)
#pragma unroll
    for (int q = 0; q < B; ++q)
      if (B == 3 || q * PER < n) u[q] = p[q];
  }
  uint32_t o[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int f = 0; f < 32; ++f) {
    const int j = fp_code(B, f);
    uint32_t v;
    if constexpr (B == 3) v = ((u[j >> 4] >> (2 * (j & 15))) & 3u) | (((u[2] >> b3_hi_pos(j)) & 1u) << 2);
    else v = (u[j * B / 32] >> ((j * B) & 31)) & ((1u << B) - 1u);
    if (j >= n) v = 0;
    if constexpr (B == 2) {
      o[f >> 3] |= ((0x9A10u >> (4 * v)) & 15u) << (4 * (f & 7));  // 0, 1, -2, -1 -> 0, 0.5, -1, -0.5
    } else {
      const int w = sext(v, B);
      const uint32_t e = w < 0 ? (uint32_t)(-w) | 0x20u : (uint32_t)w;
      const int bit = 6 * f;
      o[bit >> 5] |= e << (bit & 31);
      if ((bit & 31) > 26) o[(bit >> 5) + 1] |= e >> (32 - (bit & 31));
    }
  }
  uint8_t *slab = a.wp + (int64_t)rest * FpT<B>::SLAB;
  *(uint4 *)(slab + lane * 16) = make_uint4(o[0], o[1], o[2], o[3]);
  if constexpr (B != 2) *(uint2 *)(slab + 1024 + lane * 8) = make_uint2(o[4], o[5]);
}

// ------------------------------------------------------------ kernel arguments
struct FpArgs {
  const uint8_t *in, *wp, *res, *proj;
  uint8_t *out;
  const float *cst;
  const int32_t *bad;  // the prepare kernel's flags
  int32_t fast;        // bad[1] is known to be clear
  int32_t gated;       // one of the two launches of a one-off call: base builds leave if bad[0], wide ones unless
  int32_t *dump;
  uint32_t in_bytes, w_bytes, res_bytes, proj_bytes, cst_bytes;
  int32_t in_pix, in_gs, res_pix, res_gs, proj_pix, proj_gs, out_pix, out_gs;  // bytes, < 2^30
  const int32_t *wsum;                      // B = 8: 128 sum(w) per channel (DUMP)
  int32_t out_words;                        // words of an output row
  int32_t M, h, w, stride, pad, kh, kw;     // M: output pixels; h, w: the input's
  int32_t hw_out, wo;
  int32_t ph, pw, pstride;                  // projection input
  int32_t cpb, km, kb;                      // K-blocks per tap, of the main taps, in all
  int32_t G, shuffle, cout, coutp, out_bits;
  uint32_t rowpat;                          // bit ky kw of every filter row
  FastDiv d_hw, d_wo, d_cpb, d_kw;
  // tile order: pixel chunks of cl tiles (the last: llen), per chunk the
  // (group, channel block) combos, per combo the chunk's pixel tiles
  int32_t ncb, ncombo, nchunk, cl, llen, tiles;
  FastDiv d_chunk, d_cl, d_llen, d_ncb;
};

struct TileId { int pt, cbk, g; };
// Workgroup i runs on XCD i mod 8, which takes one contiguous range of the
// tile order: an XCD's L2 then fetches a chunk's input lines once for all
// groups, or (one chunk) holds a few combos' weights.  False: no tile.
__device__ __forceinline__ bool tile_of(const FpArgs &a, TileId &id) {
  const int x = (int)(blockIdx.x & 7), j = (int)(blockIdx.x >> 3);
  const int q = a.tiles >> 3, r = a.tiles & 7;
  if (j >= q + (x < r ? 1 : 0)) return false;
  const uint32_t t = (uint32_t)(x * q + min(x, r) + j);
  const uint32_t c = a.d_chunk.div(t);
  const uint32_t rem = t - c * a.d_chunk.d;
  const bool last = (int)c == a.nchunk - 1;
  const uint32_t combo = last ? a.d_llen.div(rem) : a.d_cl.div(rem);
  id.pt = (int)(c * a.cl + rem - combo * (uint32_t)(last ? a.llen : a.cl));
  id.g = (int)a.d_ncb.div(combo);
  id.cbk = (int)combo - id.g * a.ncb;
  return true;
}

// Geometry of output pixel m: byte offset of tap (0, 0) (may be negative), the
// taps outside the image (every bit for a pixel past the end, bits past the
// taps set) and the projection's pixel offset (kOob past the end).
struct PixelGeo { int off0; uint32_t out_mask; uint32_t poff; };
template <bool PROJ>
__device__ __forceinline__ PixelGeo pixel_geo(const FpArgs &a, int m) {
  const bool valid = m < a.M;
  const uint32_t mm = valid ? (uint32_t)m : 0u;
  const int n = (int)a.d_hw.div(mm);
  const int rem = (int)mm - n * a.hw_out;
  const int oy = (int)a.d_wo.div((uint32_t)rem), ox = rem - oy * a.wo;
  const int iy0 = oy * a.stride - a.pad, ix0 = ox * a.stride - a.pad;
  PixelGeo p;
  p.off0 = ((n * a.h + iy0) * a.w + ix0) * a.in_pix;
  // bits [lo, hi) of one row (kw <= 32 bits) and of the row pattern
  const int xlo = max(0, -ix0), xhi = max(xlo, min(a.kw, a.w - ix0));
  const int ylo = max(0, -iy0), yhi = max(ylo, min(a.kh, a.h - iy0));
  auto below = [](int b) __attribute__((always_inline)) { return (uint32_t)(((uint64_t)1 << min(b, 32)) - 1u); };
  const uint32_t cols = below(min(xhi, 32)) & ~below(min(xlo, 32));
  const uint32_t rows = a.rowpat & below(min(yhi, 32) * a.kw) & ~below(min(ylo, 32) * a.kw);
  p.out_mask = valid ? ~(cols * rows) : 0xffffffffu;
  p.poff = kOob;
  if constexpr (PROJ)
    if (valid) p.poff = (uint32_t)(((n * a.ph + oy * a.pstride) * a.pw + ox * a.pstride) * a.proj_pix);
  return p;
}

// 16 bytes per lane from the buffer into LDS at `dst` (uniform) + 16 lane.  In
// asm, so that the compiler does not order its LDS reads after these loads:
// the ring's own waits and barriers do (the loads have no register results).
// m0 is set in the same statement and named as overwritten.
__device__ __forceinline__ void dma16(v4i rsrc, uint32_t dst, uint32_t voff, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(dst), "v"(voff), "s"(rsrc), "s"(soff)
               : "m0");
}
__device__ __forceinline__ v4i rsrc4(const void *base, uint32_t bytes) {
  const uint64_t p = (uint64_t)base;
  return v4i{(int)(uint32_t)p, (int)((uint32_t)(p >> 32) & 0xffffu), (int)bytes, 0x00020000};
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Wait until at most N of this wave's loads are in flight and all of its LDS
// reads are done, then meet the workgroup.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// Requant of one quad of channels: code = min(floor(u sc + 1/2), qmax), zero
// below (the conversion truncates and takes negative values to 0).  Runs with
// fp32 rounding towards minus infinity (see the top of the file).
__device__ __forceinline__ uint32_t requant_rd(float u, float sc, uint32_t qmax) {
  const float y = __builtin_fmaf(u, sc, 0.5f);
  uint32_t q;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(q) : "v"(y));
  return min(q, qmax);
}
// The same in fp64, s = M 2^-sh.
__device__ __forceinline__ uint32_t requant_f64(double u, double s, uint32_t qmax) {
  const double d = __builtin_fma(u, s, 0.5);
  uint32_t q;
  asm("v_cvt_u32_f64 %0, %1" : "=v"(q) : "v"(d));
  return min(q, qmax);
}
// Every later fp32 and fp64 operation that depends on a value passed through
// here rounds towards minus infinity (asm volatile statements keep their order).
__device__ __forceinline__ void set_round_down() {
  asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 4), 10");
}

// The 2-bit requant of two channels at once, for shifts up to 21: with v = u M
// 2^-sh, z = clamp((v + 2^-22) / 4) to [0, 1] is one fma, and the conversion to
// FP4 (rounding to nearest even whatever the mode, scale 1/2) gives the nibble
// RNE(4 z), 4 for z = 1.  The sum v + 2^-22 moves every tie v = k + 1/2 (k <=
// 2) above it and is representable there; values below it are at most k + 1/2
// - 2^-21, stay at most k + 1/2 - 2^-22 and round to k.  So the nibble is
// floor(v + 1/2) clamped to [0, 4], and fp4_codes takes 4 to 3.
__device__ __forceinline__ float requant_z(float u, float sc, float o) {
  float z;
  asm("v_fma_f32 %0, %1, %2, %3 clamp" : "=v"(z) : "v"(u), "v"(sc), "v"(o));
  return z;
}
__device__ __forceinline__ uint32_t fp4_codes(uint32_t w) { return w - ((w >> 2) & 0x11111111u); }

// Four shortcut codes of channels 8 qi + 4 half .. + 3 of a 32-channel block
// held in c (B = 2: two words; 3: the chunk; 4: four words).
template <int B, typename V>
__device__ __forceinline__ void quad_codes(const uint32_t *c, int qi, int half, V out[4]) {
  uint32_t v, hi = 0;
  if constexpr (B == 2 || B == 3) {
    v = c[qi >> 1] >> (16 * (qi & 1) + 8 * half);
    if constexpr (B == 3) hi = c[2] >> (16 * (qi & 1) + 8 * half + (qi >> 1));
  } else {
    v = c[qi] >> (16 * half);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t q;
    if constexpr (B == 3) q = ((v >> (2 * e)) & 3u) | (((hi >> (2 * e)) & 1u) << 2);
    else q = (v >> (B * e)) & ((1u << B) - 1u);
    out[e] = (V)q;
  }
}

// ------------------------------------------------------------ tile kernel
// A workgroup computes TN = 64 WN channels x TM = 32 PB WM pixels of one group;
// wave (wn, wm) owns 2 x PB blocks of 32 x 32.  A ring of S LDS stages, each of
// KPS K-blocks (weight slabs, then the pixels' packed codes), is filled with
// 16-byte LDS loads S - 1 stages ahead of the MFMAs, one barrier per stage.
//
// What bounds it: the fetch path into LDS and the latency of a stage.  Counters
// of the 14x14, 256-channel 2-bit layer (G = 4, batch 128), cycles per CU: MFMAs 28k
// and LDS reads 23k, but the vector memory data unit busy for 58k of 64k with
// one 16-byte piece of a 64-byte pixel row per lane, as each piece takes a
// line of its own; 40k of 55k with a pixel's four pieces in neighbouring lanes
// (PAIR: 43k vector L1 accesses -> 24k).  With the stages of four that it allows
// ResNet-18 G = 4 2-bit at batch 64 went 417 -> 386 us, ResNet-50 at batch 128
// 1123 -> 1086, the 3-bit layer with a shortcut 56.4 -> 52.8; the 2-bit layer
// above stayed (31.5, 31.7), latency-bound.  Deeper rings (three and four stages
// of two K-blocks) measured equal or slower.  The prologue has no loops
// and no dependent loads before the first fetch (constants arrive by the same LDS
// loads), a K-block's position is decoded with two multiplies instead of carried
// state, the in-image test is three VALU instructions, and a stage's LDS reads are
// in flight while the next fetch is issued.
// MODE 0: no shortcut, 1: identity, 2: projection (more K-blocks).
template <int B, int PB, int WN, int WM, int KPS>
struct FpCfg {
  using T = FpT<B>;
  static constexpr int NT = WN * WM * 64;
  static constexpr int TN = 64 * WN, TM = 32 * PB * WM;
  static constexpr int W1 = TN / 32 * T::SLAB, X1 = TM * 16 * T::PPX;
  static constexpr int WST = KPS * W1, XST = KPS * X1, SST = WST + XST;
  static constexpr int WP = WST / 16, XP = XST / 16;
  static_assert(WP % 64 == 0 && XP % 64 == 0 && (XP / KPS) % 64 == 0, "whole waves of pieces");
  static constexpr int WL = (WP + NT - 1) / NT, XL = (XP + NT - 1) / NT;
  // loads wave w issues per stage: the waves below `full` one more
  static constexpr int loads(int w) {
    int n = 0;
    for (int i = 0; i < WL; ++i) n += 64 * w + i * NT < WP ? 1 : 0;
    for (int i = 0; i < XL; ++i) n += 64 * w + i * NT < XP ? 1 : 0;
    return n;
  }
  static constexpr int LMAX = loads(0), LMIN = loads(NT / 64 - 1);
  static constexpr int full() {
    int w = 0;
    while (w < NT / 64 && loads(w) == LMAX) ++w;
    for (int i = w; i < NT / 64; ++i)
      if (loads(i) != LMIN) return -1;
    return w;
  }
  static_assert(full() > 0, "at most two load counts");
  static constexpr int RP = TM * (B == 2 ? TN / 64 : B == 8 ? TN / 16 : TN / 32);  // 16-byte shortcut pieces
};

// PAIR (K-blocks per tap a multiple of KPS): a stage's pieces are ordered by
// pixel, so that neighbouring lanes fetch a pixel's adjacent pieces from one
// line; a pixel's NP pieces are swizzled so that 16 consecutive pixels' 16-byte
// reads of one piece meet all banks.  2-bit lanes read eight bytes of a piece, so
// half of the banks idle: two conflict cycles per MFMA on the layers without a
// shortcut (SQ_LDS_BANK_CONFLICT / SQ_INSTS_MFMA), swizzled or not.
template <int NP>
__device__ __forceinline__ int piece_swizzle(int pixel) { return (pixel / (16 / NP)) & (NP - 1); }
template <int B, int PB, int WN, int WM, int MODE, bool DUMP, int KPS, int S, int EP, bool PAIR>
__device__ __forceinline__ void conv_fp_tile(const FpArgs &a) {
  static_assert(!DUMP || EP == kWide, "one build with the dump, for every layer");
  using C = FpCfg<B, PB, WN, WM, KPS>;
  using T = FpT<B>;
  constexpr int NT = C::NT, TN = C::TN, TM = C::TM, CB = 2;
  constexpr int RING = S * C::SST;
  constexpr int CST = TN / 64 * 1024;
  // the shortcut's codes: a buffer of their own, or (where that would cost a
  // workgroup per CU) the free slot of the last stage
  constexpr bool LATE = MODE == 1 && S == 2 && KPS == 4;
  static_assert(!LATE || C::RP * 16 <= C::SST, "a free slot during the last stage");
  constexpr int RSB = MODE == 1 && !LATE ? C::RP * 16 : 0;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[RING + CST + RSB];

  if (a.gated && (a.bad[0] != 0) != (EP == kWide)) return;
  TileId id;
  if (!tile_of(a, id)) return;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int wn = wave / WM, wm = wave % WM;
  const int g = id.g, gd = g + a.shuffle < a.G ? g + a.shuffle : g + a.shuffle - a.G;
  const int m0 = id.pt * TM;

  const v4i r_w = rsrc4(a.wp, a.w_bytes), r_in = rsrc4(a.in, a.in_bytes);
  const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
  // constants, then the shortcut's codes: before stage 0, whose wait covers them
  if (wave < TN / 64)
    dma16(rsrc4(a.cst, a.cst_bytes), base + RING + wave * 1024, (uint32_t)(lane * 16),
          (uint32_t)(((g * a.coutp + id.cbk * TN) / 64 + wave) * 1024));
  auto fetch_res = [&](int at) __attribute__((always_inline)) {
    const v4i r_res = rsrc4(a.res, a.res_bytes);
    constexpr int CBY = B == 2 || B == 8 ? 16 : T::CHS;  // bytes of a piece's channels in the row
#pragma unroll
    for (int i = 0; i < (C::RP + NT - 1) / NT; ++i)
      if (64 * wave + i * NT < C::RP) {
        const int q = tid + i * NT, cc = q / TM, m = m0 + q % TM;
        const uint32_t vo = m < a.M ? (uint32_t)(m * a.res_pix + gd * a.res_gs + cc * CBY) : kOob;
        dma16(r_res, base + (uint32_t)at + (64 * wave + i * NT) * 16, vo, (uint32_t)(id.cbk * (TN * B / 8)));
      }
  };
  int res_at = RING + CST;
  if constexpr (MODE == 1 && !LATE) fetch_res(res_at);

  // this thread's weight pieces and pixels
  uint32_t woff[C::WL];
#pragma unroll
  for (int i = 0; i < C::WL; ++i) {
    const int c = tid + i * NT, sub = c / (C::W1 / 16), r = c % (C::W1 / 16);
    woff[i] = (uint32_t)((((g * a.coutp + id.cbk * TN) / 32 + r / (T::SLAB / 16)) * a.kb + sub) * T::SLAB +
                         r % (T::SLAB / 16) * 16);
  }
  constexpr int NP = T::PPX * KPS;
  static_assert(PAIR || T::PPX == 1, "a piece per K-block");
  PixelGeo px[C::XL];
#pragma unroll
  for (int i = 0; i < C::XL; ++i) {
    int pixel = (tid + i * NT) % TM, chunk = 0;
    if constexpr (PAIR) {
      pixel = (tid + i * NT) / NP;
      chunk = (((tid + i * NT) % NP) ^ piece_swizzle<NP>(pixel)) * (T::XB / T::PPX);
    }
    px[i] = pixel_geo<MODE == 2>(a, m0 + pixel);
    px[i].off0 += g * a.in_gs + chunk;
    if constexpr (MODE == 2) px[i].poff += (uint32_t)(gd * a.proj_gs + chunk);
  }
  const int row_adj = (a.w - a.kw) * a.in_pix;
  const int KB = a.kb, NS = (KB + KPS - 1) / KPS;
  const uint32_t wdst = base + (uint32_t)(wave * 1024);
  // Stage s into slot `slot`.
  auto fetch = [&](int s, int slot) __attribute__((always_inline)) {
    const uint32_t so = (uint32_t)(slot * C::SST);
#pragma unroll
    for (int i = 0; i < C::WL; ++i)
      if ((i + 1) * NT <= C::WP || 64 * wave + i * NT < C::WP)
        dma16(r_w, wdst + so + i * NT * 16, woff[i], (uint32_t)(s * KPS * T::SLAB));
#pragma unroll
    for (int i = 0; i < C::XL; ++i)
      if ((i + 1) * NT <= C::XP || 64 * wave + i * NT < C::XP) {
        const int sub = KPS == 1 || PAIR ? 0 : (64 * wave + i * NT) / (C::XP / KPS);
        const int kb = s * KPS + sub;
        const uint32_t dst = wdst + so + C::WST + i * NT * 16;
        if (MODE == 2 && kb >= a.km) {
          dma16(rsrc4(a.proj, a.proj_bytes), dst, px[i].poff, (uint32_t)((kb - a.km) * T::XB));
        } else {
          const int tap = (int)a.d_cpb.div((uint32_t)kb), ky = (int)a.d_kw.div((uint32_t)tap);
          const int tapoff = tap * a.in_pix + ky * row_adj;
          // sign-extended bit `tap` of the mask: all ones outside the image
          const uint32_t o = (uint32_t)__builtin_amdgcn_sbfe((int)px[i].out_mask, (uint32_t)tap, 1u);
          dma16(r_in, dst, (uint32_t)(px[i].off0 + tapoff) | (o & kOob), (uint32_t)((kb - tap * a.cpb) * T::XB));
        }
      }
  };
#pragma unroll
  for (int s = 0; s < (S == 1 ? 1 : S - 1); ++s)
    if (s < NS) fetch(s, s);

  // operands of K-block `sub` of the slot at byte so
  constexpr int J = T::J;
  const int xl = C::WST + (wm * PB * 32 + l32) * 16 * (PAIR ? NP : 1) + (B == 2 ? half * 8 : 0);
  // piece PPX sub + j' of the lane's pixel: B = 3, 4, j' = half; B = 8, j' = 2 half + j
  const int xsw = PAIR ? 16 * (piece_swizzle<NP>(l32) ^ (B == 2 ? 0 : B == 8 ? 2 * half : half)) : 0;
  const int al = wn * CB * T::SLAB + lane * 16, bl = wn * CB * T::SLAB + 1024 + lane * 8;
  struct Ops { v4i x[PB][J], a0[CB][J]; v2i a1[CB]; };
  auto read = [&](Ops &o, int so, int sub) __attribute__((always_inline)) {
    const uint8_t *p = lds + so;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
      for (int j = 0; j < J; ++j) o.a0[cb][j] = *(const v4i *)(p + al + sub * C::W1 + cb * T::SLAB + j * 1024);
      if constexpr (B == 3 || B == 4) o.a1[cb] = *(const v2i *)(p + bl + sub * C::W1 + cb * T::SLAB);
    }
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const uint8_t *q = PAIR ? p + xl + ((16 * (T::PPX * sub + j)) ^ xsw) + pb * 512 * NP
                                : p + xl + sub * C::X1 + pb * 512;
        if constexpr (B == 2) {
          const v2i v = *(const v2i *)q;
          o.x[pb][j] = v4i{v[0], v[1], 0, 0};
        } else {
          o.x[pb][j] = *(const v4i *)q;
        }
      }
  };
  typename T::Acc acc[CB][PB];
  auto mfmas = [&](const Ops &o) __attribute__((always_inline)) {
    if constexpr (B == 8) {
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const v4i X = flip_i8(o.x[pb][j]);
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
            acc[cb][pb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(o.a0[cb][j], X, acc[cb][pb], 0, 0, 0);
        }
    } else {
      v8i A[CB];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) A[cb] = wt_fp<B>(o.a0[cb][0], o.a1[cb]);
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        const v8i X = act_fp<B>(o.x[pb][0]);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[cb][pb] = mfma_fp<B>(A[cb], X, acc[cb][pb]);
      }
    }
  };

  const bool more = C::LMAX != C::LMIN && wave < C::full();
  int so = 0, slot_f = S - 1;  // byte offset of the stage's slot; slot of the next fetch
  const float *cst = (const float *)(lds + RING) + wn * 256;
  const double *csd = (const double *)cst;                // B = 8 and kWide
  const int32_t *csi = (const int32_t *)cst;
  for (int s = 0; s < NS; ++s) {
    // stage s has landed; up to S - 2 younger ones may be in flight
    if (S > 1 && s + S - 2 < NS) {
      if (C::LMAX != C::LMIN && !more) wait_barrier<(S > 1 ? S - 2 : 0) * C::LMIN>();
      else wait_barrier<(S > 1 ? S - 2 : 0) * C::LMAX>();
    } else {
      wait_barrier<0>();
    }
    // two K-blocks' reads in flight before the next fetch, then one ahead
    Ops o[KPS];
#pragma unroll
    for (int i = 0; i < KPS; ++i) read(o[i], so, i);
    if (S > 1 && s + S - 1 < NS) {
      fetch(s + S - 1, slot_f);
    } else if constexpr (LATE) {
      res_at = slot_f * C::SST;
      fetch_res(res_at);
    }
    if (s == 0) {
      // element r of block cb is channel 32 cb + 8 (r / 4) + 4 half + r % 4
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int qi = 0; qi < 4; ++qi) {
          const int c0 = cb * 32 + 8 * qi + 4 * half;
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
              if constexpr (B == 8) acc[cb][pb][4 * qi + e] = csi[128 + c0 + e];
              else if constexpr (EP == kWide) acc[cb][pb][4 * qi + e] = 0.0f;
              else acc[cb][pb][4 * qi + e] = cst[64 + c0 + e];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < KPS; ++i) {
      if (i > 0 && s * KPS + i >= KB) break;  // uniform; an odd last K-block
      mfmas(o[i]);
    }
    so = so + C::SST == S * C::SST ? 0 : so + C::SST;
    slot_f = slot_f + 1 == S ? 0 : slot_f + 1;
  }

  // ---- epilogue
  if constexpr (LATE) wait_barrier<0>();
  const int ch0 = id.cbk * TN + wn * 64;
  const int mw = m0 + wm * PB * 32;
  if constexpr (DUMP) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int c = cb * 32 + 8 * (r >> 2) + 4 * half + (r & 3), m = mw + pb * 32 + l32;
          if (m < a.M && ch0 + c < a.cout)
            if constexpr (B == 8)  // without bias and 128 sum(w), exact modulo 2^32
              a.dump[((int64_t)m * a.G + gd) * a.cout + ch0 + c] =
                  acc[cb][pb][r] - csi[128 + c] + a.wsum[g * a.cout + ch0 + c];
            else
              a.dump[((int64_t)m * a.G + gd) * a.cout + ch0 + c] = (int)(acc[cb][pb][r] * (float)(1 << T::L));
        }
  }
  constexpr uint32_t qmax = (1u << B) - 1u;
  uint32_t w2[CB][PB];
  if constexpr (EP != kFp4) {
    set_round_down();
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) asm volatile("" : "+v"(acc[cb][pb]));
  }
  if constexpr (B == 8) {
    const uint32_t q8 = (1u << a.out_bits) - 1u;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      uint32_t qv[PB][4];
#pragma unroll
      for (int qi = 0; qi < 4; ++qi) {
        __builtin_amdgcn_sched_barrier(0);
        const int c0 = cb * 32 + 8 * qi + 4 * half;
        double sc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[e] = csd[c0 + e];
        v4i rm = {0, 0, 0, 0};
        if constexpr (MODE == 1) rm = *(const v4i *)(csi + 192 + c0);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
          uint32_t rc = 0, w = 0;
          if constexpr (MODE == 1)
            rc = *(const uint32_t *)(lds + res_at +
                                     ((wn * 4 + cb * 2 + (qi >> 1)) * TM + wm * PB * 32 + pb * 32 + l32) * 16 +
                                     8 * (qi & 1) + 4 * half);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int32_t v = acc[cb][pb][4 * qi + e], code = (int32_t)((rc >> (8 * e)) & 255u);
            double u;
            if constexpr (MODE == 1 && EP == kWide) u = __builtin_fma((double)rm[e], (double)code, (double)v);
            else u = (double)(MODE == 1 ? v + rm[e] * code : v);
            w |= requant_f64(u, sc[e], q8) << (8 * e);
          }
          qv[pb][qi] = w;
        }
      }
      const int wq = (ch0 + cb * 32) / 4 + 4 * half;  // the lane's 16 channels: their first word of the row
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        const auto p0 = __builtin_amdgcn_permlane32_swap(qv[pb][0], qv[pb][2], false, false);  // as below
        const auto p1 = __builtin_amdgcn_permlane32_swap(qv[pb][1], qv[pb][3], false, false);
        const int m = mw + pb * 32 + l32;
        if (m >= a.M) continue;
        uint32_t *cw = (uint32_t *)(a.out + (int64_t)m * a.out_pix + (int64_t)gd * a.out_gs) + wq;
        const uint32_t v[4] = {p0[0], p0[1], p1[0], p1[1]};
        if (wq + 4 <= a.out_words) {
          *(uint4 *)cw = make_uint4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (wq + e < a.out_words) cw[e] = v[e];
        }
      }
    }
  } else if constexpr (EP == kFp4) {
    // 2-bit codes, 2.1 VALU instructions a value instead of 4.3 (and 2 instead
    // of 3 for a shortcut): both ways between codes and floats by the FP4
    // conversions, even and odd codes in nibbles of their own
    const float o = 0x1p-24f;
    const uint32_t sel = half ? 0x07030602u : 0x05010400u;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      uint32_t E[PB], O[PB], re[PB][2], ro[PB][2];
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        E[pb] = O[pb] = 0;
        if constexpr (MODE == 1) {
          const v2i v = *(const v2i *)(lds + res_at + (wn * TM + wm * PB * 32 + pb * 32 + l32) * 16 + 8 * cb);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const uint32_t x = (uint32_t)v[j] >> (8 * half);
            re[pb][j] = x & 0x33333333u;
            ro[pb][j] = (x >> 2) & 0x33333333u;
          }
        }
      }
#define PALQ_QUAD(QI)                                                                                             \
  {                                                                                                               \
    __builtin_amdgcn_sched_barrier(0);                                                                            \
    const int c0 = cb * 32 + 8 * QI + 4 * half;                                                                   \
    const v4f sc = *(const v4f *)(cst + c0) * 0.25f;                                                              \
    v4f rm = {0.0f, 0.0f, 0.0f, 0.0f};                                                                            \
    if constexpr (MODE == 1) rm = *(const v4f *)(cst + 128 + c0);                                                 \
    _Pragma("unroll") for (int pb = 0; pb < PB; ++pb) {                                                           \
      float u[4];                                                                                                 \
      _Pragma("unroll") for (int e = 0; e < 4; ++e) u[e] = acc[cb][pb][4 * QI + e];                               \
      if constexpr (MODE == 1) {                                                                                  \
        const v2f c02 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(re[pb][QI >> 1], 2.0f, 2 * (QI & 1));            \
        const v2f c13 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(ro[pb][QI >> 1], 2.0f, 2 * (QI & 1));            \
        u[0] = __builtin_fmaf(rm[0], c02[0], u[0]);                                                               \
        u[2] = __builtin_fmaf(rm[2], c02[1], u[2]);                                                               \
        u[1] = __builtin_fmaf(rm[1], c13[0], u[1]);                                                               \
        u[3] = __builtin_fmaf(rm[3], c13[1], u[3]);                                                               \
      }                                                                                                           \
      float z[4];                                                                                                 \
      _Pragma("unroll") for (int e = 0; e < 4; ++e) z[e] = requant_z(u[e], sc[e], o);                             \
      E[pb] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(E[pb], z[0], z[2], 0.5f, QI);                              \
      O[pb] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(O[pb], z[1], z[3], 0.5f, QI);                              \
    }                                                                                                             \
  }
      PALQ_QUAD(0)
      PALQ_QUAD(1)
      PALQ_QUAD(2)
      PALQ_QUAD(3)
#undef PALQ_QUAD
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        // byte qi: the lane's quad qi; both lane halves' words meet in every
        // lane, and each lane takes the bytes of its 16 channels in order
        const uint32_t t = fp4_codes(E[pb]) | (fp4_codes(O[pb]) << 2);
        const auto r = __builtin_amdgcn_permlane32_swap(t, t, false, false);
        w2[cb][pb] = __builtin_amdgcn_perm(r[1], r[0], sel);
      }
    }
  } else {
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    uint32_t qv[PB][4], hv[PB][4], rc[PB][4];
    if constexpr (MODE == 1)
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        const int p = wm * PB * 32 + pb * 32 + l32;
        if constexpr (B == 2) {
          const v2i v = *(const v2i *)(lds + res_at + (wn * TM + p) * 16 + 8 * cb);
          rc[pb][0] = (uint32_t)v[0];
          rc[pb][1] = (uint32_t)v[1];
        } else {
          const v4i v = *(const v4i *)(lds + res_at + ((wn * 2 + cb) * TM + p) * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) rc[pb][e] = (uint32_t)v[e];
        }
      }
#pragma unroll
    for (int qi = 0; qi < 4; ++qi) {
      // one quad at a time: keeps the constants of the others out of registers
      __builtin_amdgcn_sched_barrier(0);
      const int c0 = cb * 32 + 8 * qi + 4 * half;
      v4f sc, rm = {0.0f, 0.0f, 0.0f, 0.0f};
      double sd[4];
      v4i bw, rw = {0, 0, 0, 0};
      if constexpr (EP == kWide) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sd[e] = csd[c0 + e];
        bw = *(const v4i *)(csi + 128 + c0);
        if constexpr (MODE == 1) rw = *(const v4i *)(csi + 192 + c0);
      } else {
        sc = *(const v4f *)(cst + c0);
        if constexpr (MODE == 1) rm = *(const v4f *)(cst + 128 + c0);
      }
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        typename std::conditional<EP == kWide, int32_t, float>::type rcode[4];
        if constexpr (MODE == 1) quad_codes<B>(rc[pb], qi, half, rcode);
        uint32_t w = 0, h = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float u = acc[cb][pb][4 * qi + e];
          uint32_t q;
          if constexpr (EP == kWide) {
            int32_t v = (int32_t)(u * (float)(1 << T::L)) + bw[e];
            if constexpr (MODE == 1) v += __mul24(rw[e], rcode[e]);  // |res_mult| < 2^15
            q = requant_f64((double)v, sd[e], qmax);
          } else {
            if constexpr (MODE == 1) u = __builtin_fmaf(rm[e], rcode[e], u);  // exact
            q = requant_rd(u, sc[e], qmax);
          }
          if constexpr (B == 3) {
            w |= (q & 3u) << (2 * e);
            h |= (q >> 2) << (2 * e);
          } else {
            w |= q << (B * e);
          }
        }
        qv[pb][qi] = w;
        hv[pb][qi] = h;
      }
    }
    const int wd = (ch0 + cb * 32) / 32 * B;  // the block's first word of the row
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      // v_permlane32_swap exchanges the upper lane half of its first operand
      // with the lower lane half of its second; afterwards every lane holds
      // quads 0..3 of its 16 channels in order
      const auto p0 = __builtin_amdgcn_permlane32_swap(qv[pb][0], qv[pb][2], false, false);
      const auto p1 = __builtin_amdgcn_permlane32_swap(qv[pb][1], qv[pb][3], false, false);
      const int m = mw + pb * 32 + l32;
      uint8_t *row = a.out + (int64_t)m * a.out_pix + (int64_t)gd * a.out_gs;
      if constexpr (B == 2) {
        w2[cb][pb] = p0[0] | (p0[1] << 8) | (p1[0] << 16) | (p1[1] << 24);
      } else if constexpr (B == 3) {
        uint32_t hp = 0;
#pragma unroll
        for (int qi = 0; qi < 4; ++qi) hp |= hv[pb][qi] << (16 * (qi & 1) + 8 * half + (qi >> 1));
        const auto hs = __builtin_amdgcn_permlane32_swap(hp, hp, false, false);
        if (m < a.M && wd < a.out_words) {
          uint32_t *cw = (uint32_t *)row + wd;
          cw[half] = p0[0] | (p0[1] << 8) | (p1[0] << 16) | (p1[1] << 24);
          if (half == 0) cw[2] = hs[0] | hs[1];
        }
      } else {
        const int wq = wd + 2 * half;
        uint32_t *cw = (uint32_t *)row + wq;
        const uint32_t v0 = p0[0] | (p0[1] << 16), v1 = p1[0] | (p1[1] << 16);
        if (m < a.M) {
          if (wq + 2 <= a.out_words) *(uint2 *)cw = make_uint2(v0, v1);
          else if (wq < a.out_words) cw[0] = v0;
        }
      }
    }
  }
  }
  if constexpr (B == 2) {
    // pixel blocks 2 i and 2 i + 1: lanes of half 0 take block 2 i, lanes of
    // half 1 block 2 i + 1 and gather its 64 channels, stored at once
    const int wd = ch0 / 32 * 2;
#pragma unroll
    for (int i = 0; i < PB / 2; ++i) {
      const auto s0 = __builtin_amdgcn_permlane32_swap(w2[0][2 * i], w2[0][2 * i + 1], false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(w2[1][2 * i], w2[1][2 * i + 1], false, false);
      const int m = mw + (2 * i + half) * 32 + l32;
      if (m >= a.M) continue;
      uint32_t *dst = (uint32_t *)(a.out + (int64_t)m * a.out_pix + (int64_t)gd * a.out_gs) + wd;
      const uint32_t v[4] = {s0[0], s0[1], s1[0], s1[1]};
      if (wd + 4 <= a.out_words) {
        *(uint4 *)dst = make_uint4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (wd + e < a.out_words) dst[e] = v[e];
      }
    }
  }
}

// ------------------------------------------------------------ split kernel
// Layers with few tiles (one image, the deep stages at small batches): what
// bounds those is one workgroup's serial K loop on an idle chip, so a tile is
// small (32 channels x 32 PB pixels) and its K-blocks are dealt to the NW waves
// of a workgroup.  A wave loads its operands straight into registers, U
// K-blocks at once, with no barrier; the accumulators meet in LDS, each wave
// adds and requantises its share of the quads and the codes are packed there.
template <int B, int PB, int NW, int MODE, bool DUMP, int EP>
__device__ __forceinline__ void conv_fp_split(const FpArgs &a) {
  static_assert(EP != kFp4 && (!DUMP || EP == kWide), "fp32 or any parameters; the dump with the latter");
  using T = FpT<B>;
  constexpr int U = B == 8 ? 2 : 4, Q = PB * 4;
  using V4 = typename std::conditional<B == 8, v4i, v4f>::type;
  static_assert(Q % NW == 0 || NW % Q == 0, "whole quads per wave");
  __shared__ V4 red[NW * Q * 64];
  __shared__ uint32_t cw[32 * PB * 9];  // packed quads of a pixel's 32 channels (9: no bank conflicts)
  if (a.gated && (a.bad[0] != 0) != (EP == kWide)) return;
  TileId id;
  if (!tile_of(a, id)) return;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int g = id.g, gd = g + a.shuffle < a.G ? g + a.shuffle : g + a.shuffle - a.G;
  const int m0 = id.pt * 32 * PB, KB = a.kb;
  const auto r_w = __builtin_amdgcn_make_buffer_rsrc((void *)a.wp, (short)0, (int)a.w_bytes, 0x00020000);
  const auto r_in = __builtin_amdgcn_make_buffer_rsrc((void *)a.in, (short)0, (int)a.in_bytes, 0x00020000);
  PixelGeo px[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    px[pb] = pixel_geo<MODE == 2>(a, m0 + 32 * pb + l32);
    px[pb].off0 += g * a.in_gs + half * T::CHS;
    if constexpr (MODE == 2) px[pb].poff += (uint32_t)(gd * a.proj_gs + half * T::CHS);
  }
  const int row_adj = (a.w - a.kw) * a.in_pix;
  const int slab0 = (g * (a.coutp / 32) + id.cbk) * KB;
  constexpr int J = T::J;
  auto load_x = [&](auto rs, uint32_t vo, int so) __attribute__((always_inline)) {
    v4i x = {0, 0, 0, 0};
    if constexpr (B == 2) {
      const v2i v = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)vo, so, 0));
      x[0] = v[0];
      x[1] = v[1];
    } else if constexpr (B == 3) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b96(rs, (int)vo, so, 0);
      x[0] = (int)v[0];
      x[1] = (int)v[1];
      x[2] = (int)v[2];
    } else {
      x = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)vo, so, 0));
    }
    return x;
  };
  typename T::Acc acc[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[pb][r] = 0;
  for (int k0 = wave; k0 < KB; k0 += NW * U) {
    v4i x[U][PB][J], w0[U][J];
    v2i w1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kb = k0 + u * NW;
      if (kb >= KB) break;  // uniform
      const int so = (slab0 + kb) * T::SLAB;
#pragma unroll
      for (int j = 0; j < J; ++j)
        w0[u][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r_w, lane * 16 + j * 1024, so, 0));
      if constexpr (B == 3 || B == 4)
        w1[u] = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(r_w, 1024 + lane * 8, so, 0));
      if (MODE == 2 && kb >= a.km) {
        const auto r_pj = __builtin_amdgcn_make_buffer_rsrc((void *)a.proj, (short)0, (int)a.proj_bytes, 0x00020000);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
          for (int j = 0; j < J; ++j) x[u][pb][j] = load_x(r_pj, px[pb].poff + 16 * j, (kb - a.km) * T::XB);
      } else {
        const int tap = (int)a.d_cpb.div((uint32_t)kb), ky = (int)a.d_kw.div((uint32_t)tap);
        const int tapoff = tap * a.in_pix + ky * row_adj;
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
          const uint32_t o = (uint32_t)__builtin_amdgcn_sbfe((int)px[pb].out_mask, (uint32_t)tap, 1u);
#pragma unroll
          for (int j = 0; j < J; ++j)
            x[u][pb][j] = load_x(r_in, (uint32_t)(px[pb].off0 + tapoff + 16 * j) | (o & kOob), (kb - tap * a.cpb) * T::XB);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u * NW >= KB) break;
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
#pragma unroll
        for (int j = 0; j < J; ++j) {
          if constexpr (B == 8)
            acc[pb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w0[u][j], flip_i8(x[u][pb][j]), acc[pb], 0, 0, 0);
          else
            acc[pb] = mfma_fp<B>(wt_fp<B>(w0[u][j], w1[u]), act_fp<B>(x[u][pb][j]), acc[pb]);
        }
    }
  }
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const auto &v = acc[j >> 2];
    red[(wave * Q + j) * 64 + lane] = V4{v[4 * (j & 3)], v[4 * (j & 3) + 1], v[4 * (j & 3) + 2], v[4 * (j & 3) + 3]};
  }
  __syncthreads();
  const int k32 = id.cbk * 32;  // the tile's first channel of the group
  set_round_down();             // the sums below are exact; only the requant rounds
#pragma unroll
  for (int j0 = 0; j0 < Q; j0 += NW) {
    const int j = j0 + wave;  // quad j: pixel block j / 4, channels 8 (j % 4) + 4 half .. + 3
    if (j >= Q) break;
    V4 v = red[j * 64 + lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[(w * Q + j) * 64 + lane];
    if constexpr (B == 8) asm volatile("" : "+v"(v));  // after set_round_down
    const int qi = j & 3, pixel = 32 * (j >> 2) + l32, m = m0 + pixel;
    const int c0 = 8 * qi + 4 * half;
    const float *blk = a.cst + (int64_t)((g * a.coutp + k32) >> 6) * (kCstBlock / 4);
    if constexpr (B == 8) {
      const double *sc = (const double *)blk + (k32 & 32) + c0;
      const int32_t *ci = (const int32_t *)blk + 128 + (k32 & 32) + c0;
      const uint32_t q8 = (1u << a.out_bits) - 1u;
      uint32_t rc = 0, w = 0;
      if constexpr (MODE == 1) {
        const auto r_res = __builtin_amdgcn_make_buffer_rsrc((void *)a.res, (short)0, (int)a.res_bytes, 0x00020000);
        const uint32_t vo = m < a.M ? (uint32_t)(m * a.res_pix + gd * a.res_gs + c0) : kOob;
        rc = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r_res, (int)vo, k32, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int32_t t = v[e] + ci[e];
        if constexpr (DUMP)
          if (m < a.M && k32 + c0 + e < a.cout)
            a.dump[((int64_t)m * a.G + gd) * a.cout + k32 + c0 + e] = v[e] + a.wsum[g * a.cout + k32 + c0 + e];
        const int32_t code = (int32_t)((rc >> (8 * e)) & 255u);
        double u;
        if constexpr (MODE == 1 && EP == kWide) u = __builtin_fma((double)ci[64 + e], (double)code, (double)t);
        else u = (double)(MODE == 1 ? t + ci[64 + e] * code : t);
        w |= requant_f64(u, sc[e], q8) << (8 * e);
      }
      cw[pixel * 9 + 2 * qi + half] = w;
      continue;
    } else {
    const float *cst = blk + (k32 & 32) + c0;
    const double *csd = (const double *)blk + (k32 & 32) + c0;  // kWide
    const int32_t *csi = (const int32_t *)blk + 128 + (k32 & 32) + c0;
    v4f sc, b, rm = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (EP != kWide) {
      sc = *(const v4f *)cst;
      b = *(const v4f *)(cst + 64);
      if constexpr (MODE == 1) rm = *(const v4f *)(cst + 128);
    }
    typename std::conditional<EP == kWide, int32_t, float>::type rcode[4] = {0, 0, 0, 0};
    if constexpr (MODE == 1) {
      const auto r_res = __builtin_amdgcn_make_buffer_rsrc((void *)a.res, (short)0, (int)a.res_bytes, 0x00020000);
      const uint32_t vo = m < a.M ? (uint32_t)(m * a.res_pix + gd * a.res_gs) : kOob;
      uint32_t rc[4];
#pragma unroll
      for (int e = 0; e < B; ++e)
        rc[e] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r_res, (int)vo, id.cbk * 4 * B + 4 * e, 0);
      quad_codes<B>(rc, qi, half, rcode);
    }
    if constexpr (DUMP)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (m < a.M && k32 + c0 + e < a.cout)
          a.dump[((int64_t)m * a.G + gd) * a.cout + k32 + c0 + e] = (int)(v[e] * (float)(1 << T::L));
    uint32_t w = 0, h = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t q;
      if constexpr (EP == kWide) {
        int32_t t = (int32_t)(v[e] * (float)(1 << T::L)) + csi[e];
        if constexpr (MODE == 1) t += __mul24(csi[64 + e], rcode[e]);
        asm volatile("" : "+v"(t));  // after set_round_down
        q = requant_f64((double)t, csd[e], (1u << B) - 1u);
      } else {
        float u = v[e] + b[e];
        if constexpr (MODE == 1) u = __builtin_fmaf(rm[e], rcode[e], u);
        asm volatile("" : "+v"(u));  // after set_round_down
        q = requant_rd(u, sc[e], (1u << B) - 1u);
      }
      if constexpr (B == 3) {
        w |= (q & 3u) << (2 * e);
        h |= (q >> 2) << (2 * e);
      } else {
        w |= q << (B * e);
      }
    }
    cw[pixel * 9 + 2 * qi + half] = w | (h << 16);
    }
  }
  __syncthreads();
  for (int i = tid; i < 32 * PB * B; i += NW * 64) {
    const int pixel = i / B, wi = i - pixel * B, m = m0 + pixel, wd = id.cbk * B + wi;
    if (m >= a.M || wd >= a.out_words) continue;
    const uint32_t *q = cw + pixel * 9;
    uint32_t v;
    if constexpr (B == 8) {
      v = q[wi];
    } else if constexpr (B == 4) {
      v = q[2 * wi] | (q[2 * wi + 1] << 16);
    } else if (B == 3 && wi == 2) {
      v = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) v |= (q[k] >> 16) << (8 * (k & 3) + (k >> 2));
    } else {
      v = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) v |= (q[4 * wi + k] & 0xffu) << (8 * k);
    }
    *(uint32_t *)(a.out + (int64_t)m * a.out_pix + (int64_t)gd * a.out_gs + 4 * wd) = v;
  }
}

// Entry points by matrix-core format.
#define PALQ_FP_TILE(NAME)                                                                            \
  template <int B, int PB, int WN, int WM, int MODE, bool DUMP, int KPS, int S, int EP, bool PAIR>     \
  __global__ __launch_bounds__(WN *WM * 64, B == 2 ? 4 : B == 8 ? 2 : 3) void NAME(FpArgs a) {        \
    conv_fp_tile<B, PB, WN, WM, MODE, DUMP, KPS, S, EP, PAIR>(a);                                     \
  }
#define PALQ_FP_SPLIT(NAME)                                                     \
  template <int B, int PB, int NW, int MODE, bool DUMP, int EP>                  \
  __global__ __launch_bounds__(NW * 64, 4) void NAME(FpArgs a) {                \
    conv_fp_split<B, PB, NW, MODE, DUMP, EP>(a);                                \
  }
PALQ_FP_TILE(conv_fp4_kernel)
PALQ_FP_TILE(conv_fp6_kernel)
PALQ_FP_TILE(conv_i8_kernel)
PALQ_FP_SPLIT(conv_fp4_split_kernel)
PALQ_FP_SPLIT(conv_fp6_split_kernel)
PALQ_FP_SPLIT(conv_i8_split_kernel)

// ------------------------------------------------------------ host side
int64_t code_max(int bits, int is_signed) {
  return is_signed ? ((int64_t)1 << (bits - 1)) : (((int64_t)1 << bits) - 1);
}
int64_t fp_acc_bound(const ConvArgs &a) {
  int64_t b = (int64_t)a.kh * a.kw * a.in.cpg * code_max(a.in.bits, 0) * code_max(a.w_bits, 1);
  if (a.proj.data) b += (int64_t)a.proj.cpg * code_max(a.proj.bits, 0) * code_max(a.w_bits, 1);
  return b;
}

int cpb_of(int cin) { return (cin + 63) / 64; }
int fp_km(const ConvArgs &a) { return a.kh * a.kw * cpb_of(a.in.cpg); }
int fp_kb(const ConvArgs &a) { return fp_km(a) + (a.proj.data ? cpb_of(a.proj.cpg) : 0); }
int fp_coutp(const ConvArgs &a) { return (a.cout + 63) / 64 * 64; }
int64_t fp_slab(int bits) { return bits == 2 ? 1024 : bits >= 6 ? 2048 : 1536; }

FpArgs fp_args(const ConvArgs &a, const uint8_t *wp, const int32_t *thr) {
  FpArgs f{};
  f.in = a.in.data; f.wp = wp; f.res = a.res.data; f.proj = a.proj.data; f.out = a.out.data;
  f.cst = (const float *)thr;
  f.bad = conv_fp_flag(a, thr);
  f.fast = a.fp_fast;
  f.dump = a.acc_dump;
  f.cout = a.cout;
  f.coutp = fp_coutp(a);
  f.G = a.in.groups;
  f.cpb = cpb_of(a.in.cpg);
  f.km = fp_km(a);
  f.kb = fp_kb(a);
  f.in_bytes = (uint32_t)a.in.bytes;
  f.w_bytes = (uint32_t)((int64_t)f.G * f.coutp / 32 * f.kb * fp_slab(a.in.bits));
  f.cst_bytes = (uint32_t)((int64_t)f.G * f.coutp * 16);
  f.in_pix = (int32_t)a.in.pixel; f.in_gs = (int32_t)a.in.gstride;
  f.out_pix = (int32_t)a.out.pixel; f.out_gs = (int32_t)a.out.gstride;
  f.out_words = (int32_t)(a.out.row / 4);
  if (a.res.data) { f.res_bytes = (uint32_t)a.res.bytes; f.res_pix = (int32_t)a.res.pixel; f.res_gs = (int32_t)a.res.gstride; }
  if (a.proj.data) {
    f.proj_bytes = (uint32_t)a.proj.bytes; f.proj_pix = (int32_t)a.proj.pixel; f.proj_gs = (int32_t)a.proj.gstride;
    f.ph = a.proj.h; f.pw = a.proj.w; f.pstride = a.proj_stride;
  }
  f.M = a.out.n * a.ho * a.wo;
  f.h = a.in.h; f.w = a.in.w; f.stride = a.stride; f.pad = a.pad; f.kh = a.kh; f.kw = a.kw;
  f.hw_out = a.ho * a.wo; f.wo = a.wo;
  f.shuffle = a.shuffle;
  f.out_bits = a.out.bits;
  for (int ky = 0; ky < a.kh; ++ky) f.rowpat |= 1u << (ky * a.kw);
  f.d_hw = FastDiv::of((uint32_t)f.hw_out);
  f.d_wo = FastDiv::of((uint32_t)f.wo);
  f.d_cpb = FastDiv::of((uint32_t)f.cpb);
  f.d_kw = FastDiv::of((uint32_t)f.kw);
  return f;
}

// Tiles of tn channels x tm pixels; 32 pixel chunks where the packed input
// outweighs the filter (every XCD then reads all of the filter: about 7 W
// extra against (G - 1) X saved), else one.  Returns the workgroups, a multiple
// of 8.
unsigned fp_tiles(FpArgs &f, int tn, int tm, int64_t in_bytes) {
  const int npt = (f.M + tm - 1) / tm;
  f.ncb = (f.cout + tn - 1) / tn;
  f.ncombo = f.ncb * f.G;
  f.tiles = npt * f.ncombo;
  const int want = 7 * (int64_t)f.w_bytes < (int64_t)(f.G - 1) * in_bytes ? std::min(32, npt) : 1;
  f.cl = (npt + want - 1) / want;
  f.nchunk = (npt + f.cl - 1) / f.cl;
  f.llen = npt - (f.nchunk - 1) * f.cl;
  f.d_chunk = FastDiv::of((uint32_t)(f.cl * f.ncombo));
  f.d_cl = FastDiv::of((uint32_t)f.cl);
  f.d_llen = FastDiv::of((uint32_t)f.llen);
  f.d_ncb = FastDiv::of((uint32_t)f.ncb);
  return (unsigned)((f.tiles + 7) / 8 * 8);
}

// Compute units of the current device (cached per device).
int cu_count() {
  static std::mutex mu;
  static int devs[16], vals[16], used = 0;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  std::lock_guard<std::mutex> lock(mu);
  for (int i = 0; i < used; ++i)
    if (devs[i] == dev) return vals[i];
  int cus = 256;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
  if (used < 16) {
    devs[used] = dev;
    vals[used] = cus;
    ++used;
  }
  return cus;
}

template <int B, int PB, int WN, int WM, int MODE, bool DUMP, int KPS, int S, bool PAIR, int EP>
hipError_t launch_tile_ep(const FpArgs &f, unsigned g, hipStream_t s) {
  const dim3 block(WN * WM * 64), grid(g);
  if constexpr (B == 8)
    hipLaunchKernelGGL((conv_i8_kernel<B, PB, WN, WM, MODE, DUMP, KPS, S, EP, PAIR>), grid, block, 0, s, f);
  else if constexpr (B != 2)
    hipLaunchKernelGGL((conv_fp6_kernel<B, PB, WN, WM, MODE, DUMP, KPS, S, EP, PAIR>), grid, block, 0, s, f);
  else
    hipLaunchKernelGGL((conv_fp4_kernel<B, PB, WN, WM, MODE, DUMP, KPS, S, EP, PAIR>), grid, block, 0, s, f);
  return hipGetLastError();
}
template <int B, int PB, int WN, int WM, int MODE, bool DUMP, int KPS, int S, bool PAIR, bool WIDE>
hipError_t launch_tile_mode(const FpArgs &f, unsigned grid, hipStream_t s) {
  if constexpr (WIDE) return launch_tile_ep<B, PB, WN, WM, MODE, DUMP, KPS, S, PAIR, kWide>(f, grid, s);
  else if constexpr (B == 2)
    if (f.fast) return launch_tile_ep<B, PB, WN, WM, MODE, DUMP, KPS, S, PAIR, kFp4>(f, grid, s);
  if constexpr (!WIDE) return launch_tile_ep<B, PB, WN, WM, MODE, DUMP, KPS, S, PAIR, kBase>(f, grid, s);
}
template <int B, int PB, int WN, int WM, int KPS, int S, bool PAIR, bool WIDE = false, bool DUMP = false>
hipError_t launch_tile(FpArgs f, int64_t in_bytes, hipStream_t s) {
  const unsigned grid = fp_tiles(f, 64 * WN, 32 * PB * WM, in_bytes);
  if (f.res) return launch_tile_mode<B, PB, WN, WM, 1, DUMP, KPS, S, PAIR, WIDE>(f, grid, s);
  if (f.proj) return launch_tile_mode<B, PB, WN, WM, 2, DUMP, KPS, S, PAIR, WIDE>(f, grid, s);
  return launch_tile_mode<B, PB, WN, WM, 0, DUMP, KPS, S, PAIR, WIDE>(f, grid, s);
}

template <int B, int PB, int NW, int MODE, bool DUMP, int EP>
hipError_t launch_split_ep(const FpArgs &f, unsigned g, hipStream_t s) {
  const dim3 block(NW * 64), grid(g);
  if constexpr (B == 8)
    hipLaunchKernelGGL((conv_i8_split_kernel<B, PB, NW, MODE, DUMP, EP>), grid, block, 0, s, f);
  else if constexpr (B != 2)
    hipLaunchKernelGGL((conv_fp6_split_kernel<B, PB, NW, MODE, DUMP, EP>), grid, block, 0, s, f);
  else
    hipLaunchKernelGGL((conv_fp4_split_kernel<B, PB, NW, MODE, DUMP, EP>), grid, block, 0, s, f);
  return hipGetLastError();
}
template <int B, int PB, int NW, bool DUMP, int EP>
hipError_t launch_split(FpArgs f, int64_t in_bytes, hipStream_t s) {
  const unsigned grid = fp_tiles(f, 32, 32 * PB, in_bytes);
  if (f.res) return launch_split_ep<B, PB, NW, 1, DUMP, EP>(f, grid, s);
  if (f.proj) return launch_split_ep<B, PB, NW, 2, DUMP, EP>(f, grid, s);
  return launch_split_ep<B, PB, NW, 0, DUMP, EP>(f, grid, s);
}

// Which build takes a layer (times for the 14x14, 256-channel layer unless
// stated; K-blocks of 64 codes):
//  * few 32 x 64 tiles: the split kernel up to two per CU (14x14, 512 channels
//    3x3, 2-bit, 304 and 496 tiles: 12.4 and 12.7 us against 14.0 and 14.2 on
//    128 x 128 tiles, at 688 and 992 tiles 17.6 and 22.3 against 14.4 and 14.5;
//    8-bit 20.9, 21.6, 30.0 and 42.9 against 26.2, 26.7, 26.9 and 27.3; 1024
//    channels, 992 tiles: 38.6 against 24.7), 3- and 4-bit layers of 64 K-blocks
//    and more three (4-bit 688 tiles 18.8 against 20.3, 848 23.4 against 20.3; 704
//    tiles of 1024 channels 33.7 against 36.3).  64 x 256 tiles leave more of the
//    chip idle: there it pays up to four per CU with 24 K-blocks and more, 8-bit
//    excepted (320 channels 3x3, 860 tiles: 2-bit 10.3 against 11.6, 4-bit 12.7
//    against 17.5; 20 K-blocks, 860 tiles: 8.4 against 7.6 and 11.0 against 9.0).
//    With one or two K-blocks (2-bit: four) most of its waves have none: one per
//    CU (128 -> 512 channels 1x1 with a shortcut, 448 tiles, 2-bit 5.4 against 4.2,
//    4-bit 6.1 against 4.6, but at 64 and 128 tiles 4.3-4.8 against 4.1-4.5);
//  * 128 x 128 tiles, else (channel blocks that are no multiple of 128) 64 x 256;
//  * 2-bit, four or more K-blocks per tap in fours: stages of four K-blocks,
//    whose pieces fill whole lines.  Two stages take a third of a CU's LDS and
//    the smaller stages a quarter, so with more than three and up to four tiles
//    per CU the fours need a second, nearly empty round and the others none
//    (14x14, 256 channels 3x3, G = 4: 704 tiles 17.9 -> 16.5 us, 776 20.5 -> 21.5,
//    1208 31.8 -> 27.2, 1536 35.4 -> 30.9; 1x1 with 8 K-blocks: 704 8.4 -> 7.5, 848
//    9.4 -> 10.0, 1400 13.6 -> 11.8); four K-blocks in all are one stage (14x14
//    256 -> 1024 with shortcut, 3136 tiles, 19.6 -> 18.9; for 64-channel tiles and
//    two K-blocks in all one stage measured the same as three of one);
//  * else from 12 K-blocks on, two stages of two K-blocks: half the barriers (batch 64,
//    2-bit, 18.2 us against 20.4 with three stages of one); below, three stages
//    of one, which leave LDS for more workgroups (56x56, 64 -> 256 channels 1x1
//    with a shortcut, batch 128, 43.5 us against 49.1).  3- and 4-bit stages of
//    two need an even number of K-blocks per tap (pieces by pixel: ResNet-18 G = 2
//    4-bit batch 32, stage 3, 16.2 -> 13.7 us; 14x14 3-bit batch 128 with shortcut
//    55.9 -> 51.5).
// The wide builds come without the stages of four (2-bit) and of two (3- and
// 4-bit), the accumulator dump in one build for every layer.
template <int B>
hipError_t launch_fp(const FpArgs &f, bool wide_ep, int64_t in_bytes, hipStream_t s) {
  const int64_t cus = cu_count();
  const int64_t few = (int64_t)((f.M + 63) / 64) * ((f.cout + 31) / 32) * f.G;
  const bool wide = f.coutp % 128 == 0;
  int per_cu = f.kb <= (B == 2 ? 4 : 2) ? 1 : 2;
  if (B != 8 && !wide && f.kb >= 24) per_cu = 4;
  else if ((B == 3 || B == 4) && f.kb >= 64) per_cu = 3;
  if (few <= per_cu * cus) {
    if (f.dump) return launch_split<B, 2, 8, true, kWide>(f, in_bytes, s);
    if (wide_ep) return launch_split<B, 2, 8, false, kWide>(f, in_bytes, s);
    return launch_split<B, 2, 8, false, kBase>(f, in_bytes, s);
  }
  constexpr int KW = B == 2 ? 2 : 1, SW = B == 2 ? 2 : 3;
  if (f.dump) return launch_tile<B, 2, 1, 4, KW, SW, B != 2, true, true>(f, in_bytes, s);
  if (wide_ep) {
    if constexpr (B == 2)
      if (f.kb < 12)
        return wide ? launch_tile<B, 2, 2, 2, 1, 3, false, true>(f, in_bytes, s)
                    : launch_tile<B, 2, 1, 4, 1, 3, false, true>(f, in_bytes, s);
    return wide ? launch_tile<B, 2, 2, 2, KW, SW, B != 2, true>(f, in_bytes, s)
                : launch_tile<B, 2, 1, 4, KW, SW, B != 2, true>(f, in_bytes, s);
  }
  if constexpr (B == 2) {
    if (wide && f.cpb % 4 == 0) {
      if (f.kb == 4) return launch_tile<B, 2, 2, 2, 4, 1, true>(f, in_bytes, s);
      const int64_t tiles = (int64_t)((f.M + 127) / 128) * (f.coutp / 128) * f.G;
      if (f.kb >= 8 && (tiles <= 3 * cus || tiles > 4 * cus))
        return launch_tile<B, 2, 2, 2, 4, 2, true>(f, in_bytes, s);
    }
    if (f.kb < 12)
      return wide ? launch_tile<B, 2, 2, 2, 1, 3, false>(f, in_bytes, s)
                  : launch_tile<B, 2, 1, 4, 1, 3, false>(f, in_bytes, s);
    return wide ? launch_tile<B, 2, 2, 2, 2, 2, false>(f, in_bytes, s)
                : launch_tile<B, 2, 1, 4, 2, 2, false>(f, in_bytes, s);
  } else {
    if constexpr (B != 8)
      if (f.kb >= 12 && f.cpb % 2 == 0)
        return wide ? launch_tile<B, 2, 2, 2, 2, 2, true>(f, in_bytes, s)
                    : launch_tile<B, 2, 1, 4, 2, 2, true>(f, in_bytes, s);
    return wide ? launch_tile<B, 2, 2, 2, 1, 3, true>(f, in_bytes, s)
                : launch_tile<B, 2, 1, 4, 1, 3, true>(f, in_bytes, s);
  }
}

}  // namespace

// Layers on the int8 form (6- and 8-bit codes): 128 sum(w) per channel follows the slabs.
static bool fp_is_i8(const ConvArgs &a) { return a.in.bits >= 6; }
static size_t fp_slab_bytes(const ConvArgs &a) {
  return (size_t)a.in.groups * fp_coutp(a) / 32 * fp_kb(a) * fp_slab(a.in.bits);
}

// 2-, 3- and 4-bit layers (unless the context keeps them on int8) and 6- and
// 8-bit ones, with filter, output and shortcut codes of the same
// width, whose accumulator bound leaves the fp32 accumulator room for bias and
// shortcut (each channel is checked on the device), tensors and slabs the
// buffer loads can address, and a tap mask of 32 bits.
bool conv_fp_applies(const ConvArgs &a) {
  const int b = a.in.bits;
  const bool i8 = b == 6 || b == 8;
  if (a.int8_only || a.in.is_signed || (!i8 && (!a.fp4 || (b != 2 && b != 3 && b != 4))) || a.w_bits != b || a.out.bits != b)
    return false;
  if (a.bitdecomp && b >= 4) return false;
  if (a.res.data && (a.res.bits != b || a.res.is_signed)) return false;
  if (a.proj.data && (a.proj.bits != b || a.proj.is_signed)) return false;
  if ((int64_t)a.kh * a.kw > 32 || fp_acc_bound(a) >= ((int64_t)1 << (i8 ? 30 : 23))) return false;
  const int64_t lim = (int64_t)1 << 30;
  auto bytes = [](const ActView &v) { return v.data ? v.bytes : 0; };
  if (bytes(a.in) >= lim || bytes(a.out) >= lim || bytes(a.res) >= lim || bytes(a.proj) >= lim) return false;
  if ((int64_t)a.out.n * a.ho * a.wo >= (1 << 24)) return false;
  const int64_t ch = (int64_t)a.in.groups * fp_coutp(a);
  if (ch / 32 * fp_kb(a) * fp_slab(b) >= lim || ch * 16 >= lim) return false;
  // tile indices in 31 bits (the smallest tile: 32 x 64)
  return ((int64_t)a.out.n * a.ho * a.wo + 63) / 64 * ((a.cout + 31) / 32) * a.in.groups < lim;
}

// Words of one set of constants (base or wide; B = 8 has one).
static int64_t fp_cst_words(const ConvArgs &a) { return (int64_t)a.in.groups * fp_coutp(a) * 4; }

ConvPlan conv_fp_plan(const ConvArgs &a) {
  return {fp_slab_bytes(a) + (fp_is_i8(a) ? (size_t)a.in.groups * a.cout * 4 : 0),
          (size_t)(fp_cst_words(a) * (fp_is_i8(a) ? 4 : 8) + 16)};
}

const int32_t *conv_fp_flag(const ConvArgs &a, const int32_t *thr) {
  return thr + fp_cst_words(a) * (fp_is_i8(a) ? 1 : 2);
}

bool conv_fp_fast(const ConvArgs &a, const int32_t *thr) {
  int32_t wide = 1;
  return conv_fp_applies(a) && hipMemcpy(&wide, conv_fp_flag(a, thr) + 1, sizeof(wide), hipMemcpyDeviceToHost) == hipSuccess &&
         wide == 0;
}

hipError_t launch_conv_fp_prepare(const ConvArgs &a, uint8_t *wp, int32_t *thr, hipStream_t s) {
  PrepArgs p{};
  p.w = a.w; p.pw = a.proj_w;
  p.mult = a.mult; p.shift = a.shift; p.bias = a.bias;
  p.res_mult = a.res.data ? a.res_mult : nullptr;
  p.G = a.in.groups; p.cout = a.cout; p.coutp = fp_coutp(a);
  p.taps = a.kh * a.kw; p.cin = a.in.cpg; p.pcin = a.proj.data ? a.proj.cpg : 0;
  p.cpb = cpb_of(a.in.cpg); p.km = fp_km(a); p.kb = fp_kb(a);
  p.shuffle = a.shuffle;
  p.res_max = a.res.data ? (int)code_max(a.res.bits, 0) : 0;
  p.row = row_bytes(a.in.cpg, a.w_bits);
  p.prow = a.proj.data ? row_bytes(a.proj.cpg, a.w_bits) : 0;
  p.acc_bound = fp_acc_bound(a);
  p.wp = wp;
  p.cst = (float *)thr;
  p.wide = (uint8_t *)(thr + (fp_is_i8(a) ? 0 : fp_cst_words(a)));
  p.bad = (int32_t *)conv_fp_flag(a, thr);
  p.w_bits = a.w_bits;
  if (fp_is_i8(a)) {
    p.wsum = (int32_t *)(wp + fp_slab_bytes(a));
    hipLaunchKernelGGL(wsum_i8_kernel, dim3((unsigned)((p.G * p.cout + 3) / 4)), dim3(256), 0, s, p);
  }
  const int64_t lanes = (int64_t)p.G * (p.coutp / 32) * p.kb * 64 * (fp_is_i8(a) ? 2 : 1);
  const dim3 grid((unsigned)(1 + (lanes + 511) / 512));
  if (a.in.bits == 2) hipLaunchKernelGGL(conv_fp_prep_kernel<2>, grid, dim3(512), 0, s, p);
  else if (a.in.bits == 3) hipLaunchKernelGGL(conv_fp_prep_kernel<3>, grid, dim3(512), 0, s, p);
  else if (a.in.bits == 4) hipLaunchKernelGGL(conv_fp_prep_kernel<4>, grid, dim3(512), 0, s, p);
  else hipLaunchKernelGGL(conv_fp_prep_kernel<8>, grid, dim3(512), 0, s, p);
  return hipGetLastError();
}

const char *conv_fp_label(const ConvArgs &a, int epi) {
  if (a.in.bits == 2) return epi == 1 ? "conv_fp4_kernel[wide]" : "conv_fp4_kernel";
  if (a.in.bits >= 6) return epi == 1 ? "conv_i8_kernel[wide]" : "conv_i8_kernel";
  return epi == 1 ? "conv_fp6_kernel[wide]" : "conv_fp6_kernel";
}

static hipError_t launch_fp_ep(const ConvArgs &a, FpArgs f, const int32_t *thr, bool wide, hipStream_t s) {
  if (wide && !fp_is_i8(a)) f.cst = (const float *)(thr + fp_cst_words(a));
  if (fp_is_i8(a)) return launch_fp<8>(f, wide, a.in.bytes, s);
  if (a.in.bits == 2) return launch_fp<2>(f, wide, a.in.bytes, s);
  if (a.in.bits == 3) return launch_fp<3>(f, wide, a.in.bytes, s);
  return launch_fp<4>(f, wide, a.in.bytes, s);
}

hipError_t launch_conv_fp(const ConvArgs &a, const uint8_t *wp, const int32_t *thr, int epi, hipStream_t s) {
  if ((int64_t)a.out.n * a.ho * a.wo == 0) return hipSuccess;
  FpArgs f = fp_args(a, wp, thr);
  if (fp_is_i8(a)) f.wsum = (const int32_t *)(wp + fp_slab_bytes(a));
  if (a.acc_dump) return launch_fp_ep(a, f, thr, true, s);
  if (epi >= 0) return launch_fp_ep(a, f, thr, epi == 1, s);
  f.fast = 0;
  // B = 8: within the interface's |bias| < 2^30 and |res_mult| < 2^15 only sums
  // next to their own bound can need the wide build
  const int64_t res = a.res.data ? code_max(a.res.bits, 0) << 15 : 0;
  if (fp_is_i8(a) && fp_acc_bound(a) + ((int64_t)1 << 30) + res <= (int64_t)1 << 31)
    return launch_fp_ep(a, f, thr, false, s);
  f.gated = 1;
  const hipError_t e = launch_fp_ep(a, f, thr, false, s);
  return e == hipSuccess ? launch_fp_ep(a, f, thr, true, s) : e;
}

}  // namespace palq
