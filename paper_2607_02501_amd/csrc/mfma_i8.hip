// mfma_i8.hip -- the low-precision prefill variant (paper section 3.2,
// backend-specific dispatch) on the integer matrix cores: activations
// quantized per 32-element block along k to int8 with a binary32 scale,
// Q8_0 / Q4_0 weight codes fed to v_mfma_i32_32x32x32_i8 as they are, one
// MFMA k-step per block, and each block's exact int32 tile scaled by
// s_ib * d_nb into fp32 accumulators.
//
// Activation step:
//   s = fl32(max |x| / 127) (0 for an all-zero block),
//   xq = clamp(round_half_away(x / s), -127, 127), as the exact quotient rounds.  Codes go to xq[m][k] (int8, row
// major), scales to xs[k/32][ms] (block major, ms = m rounded up to 4), both
// in the caller's workspace.
//
// Product kernel: a workgroup of 4 waves owns a 128 (rows of x) x 128 (weight
// rows) output tile, or 64 x 64; wave (wm, wn) owns a quarter of it as 2 x 2
// (or one) MFMA tiles of 32 x 32.  k runs in steps of 4 blocks, whose codes
// and scales are copied to LDS in whole row segments one step ahead.  Per block
// a lane holds, for each of its x sub-tiles, the 16 codes k = 32 b + 16 (lane /
// 32) .. + 15 of row lane % 32 (A operand), and for each weight sub-tile the
// same 16 weight codes of row lane % 32 (B operand; Q4_0 nibbles are unpacked
// to int8 c - 8 in registers).  The int32 result (lane: weight row lane % 32, x
// rows 8 (e / 4) + 4 (lane / 32) + e % 4) is converted to fp32 and added with
// weight s_ib d_nb: fma(float(P), s_ib d_nb, acc) -- three vector ALU
// operations per output element and block, which bound this kernel: 192 cycles
// per 32 x 32 x 32 product, about 770 TOP/s at the clock it runs at.
// Measured, a whole call with its activation step (Q8_0, 816 bf16 rows and
// outputs): 2048 -> 32768 289 -> 222 us (493 TOP/s; the product alone 213 us),
// 16384 -> 2048 378 -> 137 us, with operands read from memory by each wave
// before, 32 rows a power of two apart per load, and 128 x 128 tiles only.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "eb_internal.h"
#include "epilogue.h"
#include "mfma_common.h"

namespace eb {
namespace {

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// ---- activation quantization ----

// v / s of the exact quotient, rounded half away from zero, within [-127, 127];
// -127 where it is not a number.
// The estimate by the reciprocal is raised by 2^-14, more than its error, so it
// is the result or one more; the lower threshold (q - 1/2) s has at most 33
// significant bits, exact in binary64, and decides.  A scale so small that its
// reciprocal may overflow takes the binary64 quotient.
__device__ inline float code_x8(float v, float s, float r) {
  const float a = fabsf(v);
  float q;
  if (s >= 0x1p-100f) {
    q = floorf(__builtin_fmaf(a, r, 0.5f + 0x1p-14f));
    q -= (double)a < ((double)q - 0.5) * (double)s ? 1.0f : 0.0f;
  } else {
    q = (float)round((double)a / (double)s);
  }
  return __builtin_amdgcn_fmed3f(copysignf(q, v), -127.0f, 127.0f);
}

// Four lanes per row and block, 16 blocks of a row per wave: a wave reads 1 KiB
// and writes 512 bytes of codes, side by side (a thread per block, 64 bytes
// apart, and binary64 quotients took 19 us for 816 x 16384, now 12.5).
template <int XT>
__global__ void __launch_bounds__(256)
    quantize_x8_kernel(const uint16_t *__restrict__ x, int64_t m, int64_t k, int64_t ms,
                       int8_t *__restrict__ xq, float *__restrict__ xs) {
  const int64_t nb = k / kQK, groups = (nb + 15) / 16, items = ms * groups;
  const int lane = threadIdx.x & 63, j = lane & 3;
  for (int64_t it = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); it < items; it += (int64_t)gridDim.x * 4) {
    const int64_t i = it / groups, b = (it - i * groups) * 16 + (lane >> 2);
    uint4 w = make_uint4(0, 0, 0, 0);
    if (i < m && b < nb) w = *reinterpret_cast<const uint4 *>(x + i * k + b * kQK + 8 * j);
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
    float v[8], a = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint16_t lo = (uint16_t)(ws[e] & 0xffffu), hi = (uint16_t)(ws[e] >> 16);
      v[2 * e] = XT == EB_F16 ? (float)__builtin_bit_cast(_Float16, lo) : __uint_as_float((uint32_t)lo << 16);
      v[2 * e + 1] = XT == EB_F16 ? (float)__builtin_bit_cast(_Float16, hi) : __uint_as_float((uint32_t)hi << 16);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf(v[e]));
    a = fmaxf(a, __shfl_xor(a, 1));
    a = fmaxf(a, __shfl_xor(a, 2));
    const float s = a / 127.0f, r = __builtin_amdgcn_rcpf(s);
    if (b >= nb) continue;  // (whole groups of four lanes)
    if (j == 0) xs[b * ms + i] = s;
    if (i >= m) continue;
    uint32_t words[2] = {0, 0};
    if (s != 0.f) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        words[e / 4] |= (uint32_t)(uint8_t)(int8_t)(int)code_x8(v[e], s, r) << (8 * (e % 4));
    }
    *reinterpret_cast<uint2 *>(xq + i * k + b * kQK + 8 * j) = make_uint2(words[0], words[1]);
  }
}

// ---- product ----

constexpr int kBMi = 128, kBNi = 128;  // the larger tile

// 16 Q4_0 nibbles (half h of a block's 16 bytes) -> int8 codes c - 8
__device__ inline v4i_t q4_codes(const uint4 raw, int h) {
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
  v4i_t o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t v = (w[e] >> (4 * h)) & 0x0f0f0f0fu;
    // per byte (v | 0x80) - 8 stays in 120..135 (no borrow across bytes), and
    // the xor maps it to v - 8 modulo 256
    o[e] = (int)(((v | 0x80808080u) - 0x08080808u) ^ 0x80808080u);
  }
  return o;
}

// One stage of LDS: kSB blocks of k of the tile's x codes, weight codes and
// scales of both.
constexpr int kSB = 4;
template <int QT, int F>
struct I8Stage {
  static constexpr int QSB = (QT == EB_Q8_0) ? 32 : 16;  // code bytes per block
  static constexpr int kXcpr = 2 * kSB, kWcpr = QSB / 16 * kSB;  // 16-byte chunks per row
  static constexpr int T = 64 * F;                               // tile rows of x and of the weights
  static constexpr int kX = T * kXcpr * 16, kW = T * kWcpr * 16;
  static constexpr int kS = kSB * T * 4, kD = T * 16;  // x scales block by block; 16 bytes of d16 per row
  static constexpr int kBytes = kX + kW + kS + kD;
  static constexpr int kXper = kX / 4096, kWper = kW / 4096;  // 1 KiB copies per wave
  static constexpr int kJobs = kXper + kWper + 1;
  static_assert(kS == 1024 * F && kD == 1024 * F, "F copies of each kind of scale");
};

// F: 32 x 32 tiles per wave in either direction
template <int QT, int F>
__global__ void __launch_bounds__(256, 4 / F)
    mm_i8_kernel(const uint8_t *__restrict__ wdata, int64_t n, int64_t k, int64_t d_off, int64_t ds,
                 const int8_t *__restrict__ xq, const float *__restrict__ xs, int64_t ms, int64_t m,
                 void *__restrict__ y, int yt, Fuse f) {
  using ST = I8Stage<QT, F>;
  constexpr int QSB = ST::QSB, R = 2, T = ST::T, TW = 32 * F;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[R * ST::kBytes];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int r = lane & 31, h = lane >> 5;
  // tiles of x rows fastest in groups of 8 weight tiles: an XCD's workgroups
  // share weight rows in its L2
  const int tiles_m = (int)((m + T - 1) / T);
  int nt, mt;
  {
    const int g = (int)blockIdx.x / (kXcds * tiles_m), q = (int)blockIdx.x % (kXcds * tiles_m);
    nt = g * kXcds + q % kXcds;
    mt = q / kXcds;
  }
  const int64_t n0 = (int64_t)nt * T, m0 = (int64_t)mt * T;
  if (n0 >= n) return;
  const int rows_n = (int)min((int64_t)T, n - n0), rows_m = (int)min((int64_t)T, m - m0);
  const int nb = (int)(k / kQK), steps = (nb + kSB - 1) / kSB;

  // descriptors over the tile's rows (rows past the end read zeros), advanced
  // step by step
  const uint32_t qrow = (uint32_t)nb * QSB, drow = (uint32_t)ds * 2, xrow = (uint32_t)k;
  i32x4_t xr = rsrc4(xq + m0 * k, (uint32_t)rows_m * xrow);
  i32x4_t qr = rsrc4(wdata + n0 * qrow, (uint32_t)rows_n * qrow);
  i32x4_t sr = wave < F ? rsrc4(xs + m0, (uint32_t)(nb * ms - m0) * 4u)
                        : rsrc4(wdata + d_off + n0 * drow, (uint32_t)rows_n * drow);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
  uint32_t xo[ST::kXper], qo[ST::kWper], so;
#pragma unroll
  for (int i = 0; i < ST::kXper; ++i) {
    const uint32_t row = (i * 4 + wave) * (64 / ST::kXcpr) + lane / ST::kXcpr;
    xo[i] = row * xrow + (((lane % ST::kXcpr) ^ chunk_swz<ST::kXcpr>(row)) << 4);
  }
#pragma unroll
  for (int i = 0; i < ST::kWper; ++i) {
    const uint32_t row = (i * 4 + wave) * (64 / ST::kWcpr) + lane / ST::kWcpr;
    qo[i] = row * qrow + (((lane % ST::kWcpr) ^ chunk_swz<ST::kWcpr>(row)) << 4);
  }
  // waves 0 .. F - 1: the x scales of 4 / F blocks, T rows of 4 bytes each; the
  // others: d16 of 64 weight rows (F = 1: three waves copy the same bytes)
  const int sj = wave < F ? wave : (F == 2 ? wave - F : 0);
  if (wave < F)
    so = (uint32_t)(sj * (kSB / F) + lane / (16 * F)) * (uint32_t)ms * 4u + (lane % (16 * F)) * 16u;
  else
    so = (uint32_t)(sj * 64 + lane) * drow;
  const uint32_t slds = lds0 + ST::kX + ST::kW + (wave < F ? 0 : ST::kS) + sj * 1024;
  const uint32_t sstep = wave < F ? (uint32_t)(kSB * ms * 4) : 2u * kSB;
  auto issue = [&](uint32_t st) __attribute__((always_inline)) {
    const uint32_t base = lds0 + st + wave * 1024;
#pragma unroll
    for (int i = 0; i < ST::kXper; ++i) copy_lds(xr, xo[i], base + i * 4096);
#pragma unroll
    for (int i = 0; i < ST::kWper; ++i) copy_lds(qr, qo[i], base + ST::kX + i * 4096);
    copy_lds(sr, so, slds + st);
    advance(xr, kSB * 32);
    advance(qr, kSB * QSB);
    advance(sr, sstep);
  };

  // LDS addresses of this lane's operands in block 0; block b is at chunk
  // index 2 b + h of x (Q8_0 weights too) or b of Q4_0 weights
  uint32_t xa[F], wa[F], xsw[F], wsw[F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    const uint32_t row = TW * wm + 32 * i + r, col = TW * wn + 32 * i + r;
    xa[i] = row * (ST::kXcpr * 16);
    xsw[i] = chunk_swz<ST::kXcpr>(row);
    wa[i] = ST::kX + col * (ST::kWcpr * 16);
    wsw[i] = chunk_swz<ST::kWcpr>(col);
  }

  f32x16_t acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  auto block = [&](const uint8_t *L, int b) __attribute__((always_inline)) {
    v4i_t a[F], w[F];
    float dv[F];
#pragma unroll
    for (int i = 0; i < F; ++i) {
      a[i] = *reinterpret_cast<const v4i_t *>(L + xa[i] + (((2u * b + h) ^ xsw[i]) << 4));
      if constexpr (QT == EB_Q8_0)
        w[i] = *reinterpret_cast<const v4i_t *>(L + wa[i] + (((2u * b + h) ^ wsw[i]) << 4));
      else
        w[i] = q4_codes(*reinterpret_cast<const uint4 *>(L + wa[i] + (((uint32_t)b ^ wsw[i]) << 4)), h);
      dv[i] = (float)*reinterpret_cast<const _Float16 *>(L + ST::kX + ST::kW + ST::kS + (TW * wn + 32 * i + r) * 16 + 2 * b);
    }
    f32x4_t sv[F][4];
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        sv[i][g] = *reinterpret_cast<const f32x4_t *>(L + ST::kX + ST::kW + (b * T + TW * wm + 32 * i + 8 * g + 4 * h) * 4);
    v16i_t p[F][F];
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) {
        const v16i_t zero = {};
        p[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], w[j], zero, 0, 0, 0);
      }
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          acc[i][j][e] = __builtin_fmaf((float)p[i][j][e], sv[i][e >> 2][e & 3] * dv[j], acc[i][j][e]);
  };

  issue(0);
  for (int s = 0; s < steps; ++s) {
    const uint32_t st = (s & 1) ? ST::kBytes : 0;
    wait_vm_barrier<0>();  // step s is in LDS, and every wave is done with step s - 1
    if (s + 1 < steps) issue(ST::kBytes - st);
    const uint8_t *L = smem + st;
    if (nb - s * kSB >= kSB) {
#pragma unroll
      for (int b = 0; b < kSB; ++b) block(L, b);
    } else {
      for (int b = 0; b < nb - s * kSB; ++b) block(L, b);
    }
  }

  // epilogue: lane holds weight row (column of y) 64 wn + 32 j + r and x rows
  // 64 wm + 32 i + 8 (e / 4) + 4 h + e % 4
#pragma unroll
  for (int j = 0; j < F; ++j) {
    const int cl = TW * wn + 32 * j + r;
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int rl = TW * wm + 32 * i + 8 * (e >> 2) + 4 * h + (e & 3);
        float v = acc[i][j][e];
        if (f.epi == EB_EPI_GLU) {  // rows 2c, 2c + 1 of the weights sit in lanes r, r ^ 1
          const float up = __shfl_xor(v, 1);
          if ((r & 1) == 0 && rl < rows_m && cl < rows_n)
            store_y(y, (m0 + rl) * (n / 2) + (n0 + cl) / 2, silu_mul(v, up), yt);
          continue;
        }
        if (rl < rows_m && cl < rows_n) put_y(y, (m0 + rl) * n + n0 + cl, v, yt, f);
      }
  }
}

inline unsigned grid1(int64_t threads) {
  int64_t g = (threads + 255) / 256;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, 65536));
}

}  // namespace

size_t i8_workspace_bytes(int64_t m, int64_t k) {
  const int64_t ms = (m + 3) / 4 * 4;
  return (size_t)round_up(m * k, 256) + (size_t)round_up(k / kQK * ms * 4, 256);
}

bool i8_fits(int64_t m, int64_t n, int64_t k) {
  const int64_t ms = (m + 3) / 4 * 4;
  return m >= 1 && (int64_t)kBMi * k < 0x7fff0000LL && (int64_t)kBNi * (k / kQK) * 32 < 0x7fff0000LL &&
         (k / kQK) * ms * 4 < 0x7fff0000LL && (n + kBNi - 1) / kBNi <= 0x7fffffffLL &&
         (m + kBMi - 1) / kBMi <= 65535;
}

hipError_t launch_mfma_i8(int32_t type, const void *wdata, int64_t n, int64_t k, const void *x,
                          int32_t xt, int64_t m, void *y, int32_t yt, const Fuse &f, void *ws,
                          hipStream_t s) {
  if (!i8_fits(m, n, k)) return hipErrorInvalidValue;
  const int64_t ms = (m + 3) / 4 * 4, nb = k / kQK;
  int8_t *xq = static_cast<int8_t *>(ws);
  float *xsc = reinterpret_cast<float *>(static_cast<uint8_t *>(ws) + round_up(m * k, 256));
  const auto *xp = static_cast<const uint16_t *>(x);
  if (xt == EB_F16)
    quantize_x8_kernel<EB_F16><<<grid1(ms * ((nb + 15) / 16) * 64), 256, 0, s>>>(xp, m, k, ms, xq, xsc);
  else
    quantize_x8_kernel<EB_BF16><<<grid1(ms * ((nb + 15) / 16) * 64), 256, 0, s>>>(xp, m, k, ms, xq, xsc);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const Layout L = layout_of(type, n, k);
  const auto *wp = static_cast<const uint8_t *>(wdata);
  // 128 x 128 tiles where they give every CU its two workgroups, else 64 x 64
  // (measured, a whole call, Q8_0, 816 rows: 16384 -> 2048, 112 large tiles,
  // 306 us against 137; 2048 -> 2560, 140 of them, 50 us against 30)
  auto launch = [&](auto fc) {
    constexpr int F = decltype(fc)::value;
    const int64_t tiles = round_up((n + 64 * F - 1) / (64 * F), kXcds) * ((m + 64 * F - 1) / (64 * F));
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    if (type == EB_Q8_0)
      mm_i8_kernel<EB_Q8_0, F><<<(unsigned)tiles, 256, 0, s>>>(wp, n, k, L.d_off, L.ds, xq, xsc, ms, m, y, yt, f);
    else
      mm_i8_kernel<EB_Q4_0, F><<<(unsigned)tiles, 256, 0, s>>>(wp, n, k, L.d_off, L.ds, xq, xsc, ms, m, y, yt, f);
    return hipGetLastError();
  };
  const int64_t large = ((n + kBNi - 1) / kBNi) * ((m + kBMi - 1) / kBMi);
  if (large >= 2 * (int64_t)device_cu_count()) return launch(std::integral_constant<int, 2>{});
  return launch(std::integral_constant<int, 1>{});
}

}  // namespace eb
