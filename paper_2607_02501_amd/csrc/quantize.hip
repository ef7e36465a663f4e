// quantize.hip -- fp32 weights -> Q8_0 / Q4_0 / Q6_S planar layout, and
// conversion between the planar device layout and the canonical
// array-of-blocks bytes.
//
// The scale is fl32(amax / 127) or fl32(m / -8) (IEEE binary32 division),
// rounded to binary16 ties-to-even by the hardware conversion.  Each code is
// the one that the exact quotient w / d16 rounds to, decided without a
// division: an estimate by the reciprocal is off by at most one, and the
// rounding thresholds (q - 1/2) d16 are exact in binary32 (at most 9 + 11
// significant bits), so comparing w with one decides exactly.  Q6_S super-blocks: the sub-block scales s_j = fl32(m_j / -32), the
// binary16 super-scale from fl32(max |s_j| / 127), the int8 sub-scales decided
// in the same way on s_j / d16 and the 6-bit codes on x / (d16 sc_j) (divisor
// of at most 18 bits, thresholds up to 31.5 of them: 24 bits, exact).
// Block formats: paper section 4, Table 3 (8-, 6- and 4-bit configurations).
//
// Bound by memory: 4 bytes read per weight.  Lanes read 16 bytes each, side by
// side (a 32-weight block is 8 lanes, a Q6_S sub-block one), and find a block's
// extreme element by exchanges.  With a thread per block, 128 bytes (Q6_S 1 KiB)
// apart, and binary64 quotients, 11008 x 4096 weights took 54 us to Q4_0, 58 us
// to Q8_0 and 419 us to Q6_S; now 38, 38 and 35 us (5.4 TB/s).
#include <hip/hip_runtime.h>

#include "eb_internal.h"

namespace eb {
namespace {

__device__ inline uint16_t f32_to_f16_bits(float f) {
  _Float16 h = (_Float16)f;  // v_cvt_f16_f32, round to nearest even
  return __builtin_bit_cast(uint16_t, h);
}

__device__ inline float f16_bits_to_f32(uint16_t b) {
  return (float)__builtin_bit_cast(_Float16, b);
}

// floor(a / d + 1/2) of the exact quotient, plus z, for d > 0 and r = 1 / d to
// an ulp or two; c0 = z + 1/2.  The estimate is raised by 2^-14, more than its
// error where it matters (quotients up to 128 in size: at most 1.5 2^-16), so
// it is the result or one more, and the lower threshold of that, (q - 1/2) d,
// is exact in binary32 there.
__device__ inline float half_up(float a, float d, float r, float c0) {
  float q = floorf(__builtin_fmaf(a, r, c0 + 0x1p-14f));
  q -= a < (q - c0) * d ? 1.0f : 0.0f;
  return q;
}

// The same kept within [lo, hi]; a quotient that is not a number gives lo.
__device__ inline float round_half_up(float a, float d, float r, float c0, float lo, float hi) {
  return __builtin_amdgcn_fmed3f(half_up(a, d, r, c0), lo, hi);
}

// The exact quotient a / d rounded half away from zero, within [-lim, lim]
// (-lim if it is not a number).
__device__ inline int round_half_away(float a, float d, float r, float lim) {
  return (int)__builtin_amdgcn_fmed3f(copysignf(half_up(fabsf(a), d, r, 0.5f), a), -lim, lim);
}

// Zero the alignment gaps of the planar layout: [qs_end, d_off) and
// [d_end, round_up(d_end, 256)), so that equal weights give equal buffers.
__device__ inline void zero_gaps(uint8_t *out, int64_t qs_end, int64_t d_off, int64_t d_end) {
  const int64_t end = round_up(d_end, 256);
  for (int64_t i = qs_end + threadIdx.x; i < d_off; i += blockDim.x) out[i] = 0;
  for (int64_t i = d_end + threadIdx.x; i < end; i += blockDim.x) out[i] = 0;
}

// Zero [a, b) of the buffer (workgroup 0's threads).
__device__ inline void zero_range(uint8_t *out, int64_t a, int64_t b) {
  for (int64_t i = a + threadIdx.x; i < b; i += blockDim.x) out[i] = 0;
}

// The gaps of the Q6_S planar layout: after the code plane, after the
// sub-scale plane and after the scale plane, up to each next 256-byte start.
__device__ inline void zero_gaps_q6(uint8_t *out, int64_t n, const Layout &L) {
  zero_range(out, n * L.qs_row, L.sc_off);
  zero_range(out, L.sc_off + n * L.ss, L.d_off);
  zero_range(out, L.d_off + n * L.ds * 2, L.total);
}

constexpr int kAhead = 4;  // wave items whose weights are requested together

// A wave takes items of 8 blocks (one 16-byte row of the scale plane): lane
// 8 b + j holds weights 4 j .. 4 j + 3 of block b.
template <int QT>
__global__ void __launch_bounds__(256) quantize_kernel(const float *__restrict__ w, int64_t n,
                                                       int64_t k, uint8_t *__restrict__ out) {
  const int64_t nb = k / kQK, groups = round_up(nb, 8) / 8;  // of a row
  constexpr int qsb = (QT == EB_Q8_0) ? 32 : 16;
  const int64_t d_off = round_up(n * nb * qsb, 256);
  const int64_t items = n * groups;
  if (blockIdx.x == 0) zero_gaps(out, n * nb * qsb, d_off, d_off + items * 16);
  uint16_t *dplane = reinterpret_cast<uint16_t *>(out + d_off);
  const int lane = threadIdx.x & 63, j = lane & 7;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t waves = (int64_t)gridDim.x * 4, first = (int64_t)blockIdx.x * 4 + wave;
  for (int64_t it0 = first * kAhead; it0 < items; it0 += waves * kAhead) {
    float4 v[kAhead];
    int64_t blk[kAhead];  // its block of the code plane, or -1
    int64_t row = it0 / groups, g = it0 - row * groups;
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      const int64_t b = g * 8 + (lane >> 3);
      blk[a] = it0 + a < items && b < nb ? row * nb + b : -1;
      v[a] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (blk[a] >= 0) v[a] = *reinterpret_cast<const float4 *>(w + blk[a] * kQK + 4 * j);
      if (++g == groups) {
        g = 0;
        ++row;
      }
    }
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      const float e[4] = {v[a].x, v[a].y, v[a].z, v[a].w};
      float amax = fmaxf(fmaxf(fabsf(e[0]), fabsf(e[1])), fmaxf(fabsf(e[2]), fabsf(e[3])));
#pragma unroll
      for (int o = 4; o >= 1; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
      amax = fmaxf(amax, 0.0f);  // a block with no number in it counts as zeros
      float d32;
      if constexpr (QT == EB_Q8_0) {
        d32 = amax / 127.0f;
      } else {
        // the sign of the first element of that magnitude: the least of
        // 2 index + sign over the elements that have it
        int key = 64;
#pragma unroll
        for (int i = 3; i >= 0; --i)
          if (fabsf(e[i]) == amax) key = 2 * (4 * j + i) + (e[i] < 0.0f ? 1 : 0);
#pragma unroll
        for (int o = 4; o >= 1; o >>= 1) key = min(key, __shfl_xor(key, o));
        d32 = ((key & 1) ? -amax : amax) / -8.0f;
      }
      uint16_t d16 = f32_to_f16_bits(d32);
      // All-zero block: the scale is +0 / 127 = +0 (Q8_0) or +0 / -8 = -0 (Q4_0).
      // Written out because the compiler may fuse the product into a mixed-precision
      // FMA with a +0 addend, which loses the sign of an exact zero.
      if (amax == 0.0f) d16 = (QT == EB_Q8_0) ? 0x0000 : 0x8000;
      const float d = f16_bits_to_f32(d16), m = fabsf(d), r = __builtin_amdgcn_rcpf(m);
      const float sg = d < 0.0f ? -1.0f : 1.0f;
      uint32_t word = 0;
      if (m != 0.0f) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (QT == EB_Q8_0)
            word |= (uint32_t)(round_half_away(e[i], m, r, 127.0f) & 255) << (8 * i);
          else
            word = __builtin_amdgcn_cvt_pk_u8_f32(
                round_half_up(e[i] * sg, m, r, 8.5f, 0.0f, 15.0f), i, word);
        }
      } else if (QT == EB_Q4_0) {
        word = 0x08080808u;
      }
      // Q4_0: byte t holds weights t and t + 16, four lanes apart
      if constexpr (QT == EB_Q4_0) word |= (uint32_t)__shfl_xor((int)word, 4) << 4;
      if (blk[a] >= 0 && (QT == EB_Q8_0 || j < 4))
        *reinterpret_cast<uint32_t *>(out + blk[a] * qsb + 4 * j) = word;
      if (j == 0 && it0 + a < items) dplane[(it0 + a) * 8 + (lane >> 3)] = blk[a] >= 0 ? d16 : 0;
    }
  }
}

// planar -> canonical: one thread per block, byte stores (no alignment on dst).
template <int QT>
__global__ void __launch_bounds__(256) to_canonical_kernel(const uint8_t *__restrict__ planar,
                                                           int64_t n, int64_t k,
                                                           uint8_t *__restrict__ dst) {
  const int64_t nb = k / kQK;
  const int64_t ds = round_up(nb, 8);
  const int64_t qsb = (QT == EB_Q8_0) ? 32 : 16;
  const int64_t d_off = round_up(n * nb * qsb, 256);
  const uint16_t *dplane = reinterpret_cast<const uint16_t *>(planar + d_off);
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n * nb;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / nb, b = t % nb;
    uint8_t *o = dst + t * (2 + qsb);
    uint16_t d16 = dplane[r * ds + b];
    o[0] = (uint8_t)(d16 & 0xff);
    o[1] = (uint8_t)(d16 >> 8);
    const uint8_t *q = planar + t * qsb;
    for (int i = 0; i < qsb; ++i) o[2 + i] = q[i];
  }
}

// canonical -> planar (scale-plane padding written as zero).
template <int QT>
__global__ void __launch_bounds__(256) from_canonical_kernel(const uint8_t *__restrict__ src,
                                                             int64_t n, int64_t k,
                                                             uint8_t *__restrict__ out) {
  const int64_t nb = k / kQK;
  const int64_t ds = round_up(nb, 8);
  const int64_t qsb = (QT == EB_Q8_0) ? 32 : 16;
  const int64_t d_off = round_up(n * nb * qsb, 256);
  uint16_t *dplane = reinterpret_cast<uint16_t *>(out + d_off);
  if (blockIdx.x == 0) zero_gaps(out, n * nb * qsb, d_off, d_off + n * ds * 2);
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n * ds;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / ds, b = t % ds;
    if (b >= nb) {
      dplane[t] = 0;
      continue;
    }
    const uint8_t *c = src + (r * nb + b) * (2 + qsb);
    dplane[t] = (uint16_t)(c[0] | (c[1] << 8));
    uint8_t *q = out + (r * nb + b) * qsb;
    for (int i = 0; i < qsb; ++i) q[i] = c[2 + i];
  }
}

// ---- Q6_S ----

// One 256-weight super-block per 16 lanes at a time: lane 16 g + j of a wave
// holds sub-block j of super-block g (16 weights, four 16-byte loads).
__global__ void __launch_bounds__(256) quantize_q6_kernel(const float *__restrict__ w, int64_t n,
                                                          int64_t k, uint8_t *__restrict__ out) {
  const Layout L = layout_of(EB_Q6_S, n, k);
  const int64_t nsb = k / kQK6;
  if (blockIdx.x == 0) zero_gaps_q6(out, n, L);
  uint16_t *dplane = reinterpret_cast<uint16_t *>(out + L.d_off);
  const int lane = threadIdx.x & 63, j = lane & 15;
  const int64_t total = n * L.ds;  // one item per scale-plane slot (incl. padding)
  const int64_t step = (int64_t)gridDim.x * 16;
  for (int64_t t0 = (int64_t)blockIdx.x * 16; t0 < total; t0 += step) {
    const int64_t t = t0 + (threadIdx.x >> 4);
    const int64_t row = t / L.ds, sb = t - row * L.ds;
    const bool ok = t < total && sb < nsb;
    float v[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
      if (ok) q = *reinterpret_cast<const float4 *>(w + row * k + sb * kQK6 + 16 * j + 4 * i);
      v[4 * i] = q.x;
      v[4 * i + 1] = q.y;
      v[4 * i + 2] = q.z;
      v[4 * i + 3] = q.w;
    }
    // the sub-block's scale: its signed element of largest magnitude (first index) / -32
    float mag = 0.0f, m = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (fabsf(v[i]) > mag) {
        mag = fabsf(v[i]);
        m = v[i];
      }
    const float s = m / -32.0f;
    float amax = fabsf(s);
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
    uint16_t d16 = f32_to_f16_bits(amax / 127.0f);
    if (amax == 0.0f) d16 = 0x0000;  // +0 / 127
    const float d = f16_bits_to_f32(d16);
    const int sc = d != 0.0f ? round_half_away(s, d, __builtin_amdgcn_rcpf(d), 127.0f) : 0;
    const float e = d * (float)sc, ea = fabsf(e), r = __builtin_amdgcn_rcpf(ea);  // exact
    int u[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
      u[i] = ea != 0.0f ? (int)round_half_up(e < 0.0f ? -v[i] : v[i], ea, r, 32.5f, 0.0f, 63.0f) : 32;
    // a chunk's two sub-blocks are in lanes 2 c, 2 c + 1: byte i of the low
    // nibbles holds u_i and u_{i+16}, the top-bit byte t the top two bits of
    // u_t, u_{t+8}, u_{t+16}, u_{t+24}
    uint32_t lo[4], hi[2] = {0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) lo[i] |= (uint32_t)(u[4 * i + b] & 15) << (8 * b);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        hi[i] |= ((uint32_t)(u[4 * i + b] >> 4) | (uint32_t)(u[4 * i + b + 8] >> 4) << 2) << (8 * b);
#pragma unroll
    for (int i = 0; i < 4; ++i) lo[i] |= (uint32_t)__shfl_xor((int)lo[i], 1) << 4;
#pragma unroll
    for (int i = 0; i < 2; ++i) hi[i] |= (uint32_t)__shfl_xor((int)hi[i], 1) << 4;
    if (ok) {
      out[L.sc_off + row * L.ss + sb * 16 + j] = (uint8_t)(int8_t)sc;
      if (!(j & 1)) {  // chunks are 8-byte aligned
        uint2 *dst = reinterpret_cast<uint2 *>(out + (row * L.nb + sb * 8 + (j >> 1)) * 24);
        dst[0] = make_uint2(lo[0], lo[1]);
        dst[1] = make_uint2(lo[2], lo[3]);
        dst[2] = make_uint2(hi[0], hi[1]);
      }
    }
    if (j == 0 && t < total) dplane[t] = ok ? d16 : 0;
  }
}

// planar <-> canonical.  A workgroup takes kConv super-blocks.  They pass
// through LDS in their canonical form, so that the planes and (where their
// pointer allows it) the canonical bytes are read and written in 16-byte
// words; a thread per super-block, 210 bytes apart, took 1.8 times as long
// (11008 x 4096: 25 -> 14 us each way).
constexpr int kConv = 64, kConvBytes = 2 + 16 + 192;
static_assert(kConv * kConvBytes % 16 == 0, "whole words");

// `bytes` canonical bytes between LDS and memory.
template <bool STORE>
__device__ inline void conv_bytes(uint8_t *lds, uint8_t *mem, int bytes) {
  if ((reinterpret_cast<uintptr_t>(mem) & 15) == 0) {
    const int words = bytes / 16;
    for (int i = threadIdx.x; i < words; i += 256) {
      if (STORE)
        reinterpret_cast<uint4 *>(mem)[i] = reinterpret_cast<const uint4 *>(lds)[i];
      else
        reinterpret_cast<uint4 *>(lds)[i] = reinterpret_cast<const uint4 *>(mem)[i];
    }
    for (int i = words * 16 + threadIdx.x; i < bytes; i += 256) {
      if (STORE) mem[i] = lds[i]; else lds[i] = mem[i];
    }
  } else {
    for (int i = threadIdx.x; i < bytes; i += 256) {
      if (STORE) mem[i] = lds[i]; else lds[i] = mem[i];
    }
  }
}

// 16-byte pieces of a plane with B bytes per super-block <-> their place in the
// canonical super-blocks (2-byte aligned, at OFF).
template <int B, int OFF, bool STORE>
__device__ inline void conv_plane(uint8_t *lds, uint8_t *plane, int cnt) {
  for (int i = threadIdx.x; i < cnt * (B / 16); i += 256) {
    uint16_t *l = reinterpret_cast<uint16_t *>(lds + (i / (B / 16)) * kConvBytes + OFF + (i % (B / 16)) * 16);
    uint32_t w[4];
    if (STORE) {
#pragma unroll
      for (int q = 0; q < 4; ++q) w[q] = (uint32_t)l[2 * q] | (uint32_t)l[2 * q + 1] << 16;
      reinterpret_cast<uint4 *>(plane)[i] = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
      const uint4 v = reinterpret_cast<const uint4 *>(plane)[i];
      w[0] = v.x;
      w[1] = v.y;
      w[2] = v.z;
      w[3] = v.w;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        l[2 * q] = (uint16_t)w[q];
        l[2 * q + 1] = (uint16_t)(w[q] >> 16);
      }
    }
  }
}

__global__ void __launch_bounds__(256) to_canonical_q6_kernel(const uint8_t *__restrict__ planar,
                                                              int64_t n, int64_t k,
                                                              uint8_t *__restrict__ dst) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kConv * kConvBytes];
  const Layout L = layout_of(EB_Q6_S, n, k);
  const int64_t nsb = k / kQK6, total = n * nsb;
  uint8_t *const p = const_cast<uint8_t *>(planar);
  const uint16_t *dplane = reinterpret_cast<const uint16_t *>(planar + L.d_off);
  for (int64_t t0 = (int64_t)blockIdx.x * kConv; t0 < total; t0 += (int64_t)gridDim.x * kConv) {
    const int cnt = (int)(total - t0 < kConv ? total - t0 : kConv);
    conv_plane<192, 18, false>(lds, p + t0 * 192, cnt);
    conv_plane<16, 2, false>(lds, p + L.sc_off + t0 * 16, cnt);
    if ((int)threadIdx.x < cnt) {
      const int64_t t = t0 + threadIdx.x, r = t / nsb;
      *reinterpret_cast<uint16_t *>(lds + threadIdx.x * kConvBytes) = dplane[r * L.ds + (t - r * nsb)];
    }
    __syncthreads();
    conv_bytes<true>(lds, dst + t0 * kConvBytes, cnt * kConvBytes);
    __syncthreads();
  }
}

// (padding and gaps written as zero)
__global__ void __launch_bounds__(256) from_canonical_q6_kernel(const uint8_t *__restrict__ src,
                                                                int64_t n, int64_t k,
                                                                uint8_t *__restrict__ out) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kConv * kConvBytes];
  const Layout L = layout_of(EB_Q6_S, n, k);
  const int64_t nsb = k / kQK6, total = n * nsb;
  uint16_t *dplane = reinterpret_cast<uint16_t *>(out + L.d_off);
  if (blockIdx.x == 0) zero_gaps_q6(out, n, L);
  for (int64_t t0 = (int64_t)blockIdx.x * kConv; t0 < total; t0 += (int64_t)gridDim.x * kConv) {
    const int cnt = (int)(total - t0 < kConv ? total - t0 : kConv);
    conv_bytes<false>(lds, const_cast<uint8_t *>(src) + t0 * kConvBytes, cnt * kConvBytes);
    __syncthreads();
    conv_plane<192, 18, true>(lds, out + t0 * 192, cnt);
    conv_plane<16, 2, true>(lds, out + L.sc_off + t0 * 16, cnt);
    if ((int)threadIdx.x < cnt) {
      const int64_t t = t0 + threadIdx.x, r = t / nsb, b = t - r * nsb;
      dplane[r * L.ds + b] = *reinterpret_cast<const uint16_t *>(lds + threadIdx.x * kConvBytes);
      if (b == nsb - 1)  // the row's padding entries (at most 7)
        for (int64_t q = nsb; q < L.ds; ++q) dplane[r * L.ds + q] = 0;
    }
    __syncthreads();
  }
}

inline unsigned grid_for(int64_t threads) {
  int64_t g = (threads + 255) / 256;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (unsigned)g;
}

}  // namespace

hipError_t launch_quantize(int32_t type, const float *w, int64_t n, int64_t k, void *out,
                           hipStream_t s) {
  uint8_t *o = static_cast<uint8_t *>(out);
  if (type == EB_Q6_S) {
    const int64_t items = n * round_up(k / kQK6, 8);
    if (items == 0) return hipSuccess;
    quantize_q6_kernel<<<grid_for(items * 16), 256, 0, s>>>(w, n, k, o);
    return hipGetLastError();
  }
  const int64_t items = n * (round_up(k / kQK, 8) / 8);  // of 8 blocks, one per wave at a time
  if (items == 0) return hipSuccess;
  const unsigned grid = grid_for((items + kAhead - 1) / kAhead * 64);
  if (type == EB_Q8_0)
    quantize_kernel<EB_Q8_0><<<grid, 256, 0, s>>>(w, n, k, o);
  else
    quantize_kernel<EB_Q4_0><<<grid, 256, 0, s>>>(w, n, k, o);
  return hipGetLastError();
}

hipError_t launch_to_canonical(int32_t type, const void *planar, int64_t n, int64_t k, void *dst,
                               hipStream_t s) {
  if (type == EB_Q6_S) {
    const int64_t groups = (n * (k / kQK6) + kConv - 1) / kConv;
    if (groups == 0) return hipSuccess;
    to_canonical_q6_kernel<<<grid_for(groups * 256), 256, 0, s>>>((const uint8_t *)planar, n, k,
                                                             (uint8_t *)dst);
    return hipGetLastError();
  }
  const int64_t threads = n * (k / kQK);
  if (threads == 0) return hipSuccess;
  if (type == EB_Q8_0)
    to_canonical_kernel<EB_Q8_0>
        <<<grid_for(threads), 256, 0, s>>>((const uint8_t *)planar, n, k, (uint8_t *)dst);
  else
    to_canonical_kernel<EB_Q4_0>
        <<<grid_for(threads), 256, 0, s>>>((const uint8_t *)planar, n, k, (uint8_t *)dst);
  return hipGetLastError();
}

hipError_t launch_from_canonical(int32_t type, const void *src, int64_t n, int64_t k, void *out,
                                 hipStream_t s) {
  if (type == EB_Q6_S) {
    const int64_t groups = (n * (k / kQK6) + kConv - 1) / kConv;
    if (groups == 0) return hipSuccess;
    from_canonical_q6_kernel<<<grid_for(groups * 256), 256, 0, s>>>((const uint8_t *)src, n, k,
                                                               (uint8_t *)out);
    return hipGetLastError();
  }
  const int64_t threads = n * round_up(k / kQK, 8);
  if (threads == 0) return hipSuccess;
  if (type == EB_Q8_0)
    from_canonical_kernel<EB_Q8_0>
        <<<grid_for(threads), 256, 0, s>>>((const uint8_t *)src, n, k, (uint8_t *)out);
  else
    from_canonical_kernel<EB_Q4_0>
        <<<grid_for(threads), 256, 0, s>>>((const uint8_t *)src, n, k, (uint8_t *)out);
  return hipGetLastError();
}

}  // namespace eb
