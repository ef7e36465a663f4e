// mfma_rows.h -- small projections (m <= 128, or more rows of small matrices;
// action-chunk denoising, several robots or speculated tokens) on the matrix cores, Q8_0 and Q4_0:
// the kernel of lone projections and the one of fused runs of independent
// ones (paper section 3.2: latency-first batch-1 execution, operator fusion;
// the action-expert projections of section 2.1 / Table 1).  Included only by
// mfma_rows_<format>.hip; mfma_rows.hip holds the choice of tiles and splits.
//
// A workgroup of W waves computes 16 NT weight rows x 16 MB rows of x.  k runs
// in steps of W blocks of 32; wave w multiplies block w of every step for the
// whole tile, so that each staged byte of x and of the codes is read from LDS
// once, and the waves' partial tiles are added through LDS at the end.
//
// Weights enter the matrix cores as their integer codes, exact in bfloat16
// and binary16 (|code| <= 128), one v_mfma_f32_16x16x32 per block and 16 x 16
// outputs with a zero accumulator; its result is scaled by the block's d16 as
// it is added in fp32.  Against rounding w_hat to hi/lo bfloat16 pairs this
// halves the MFMAs, takes 12 instead of about 45 VALU instructions per 8
// weights, and every product is exact.
//
// What bounds it: lone launches (2-9 MB of weights) the latency of the copies
// and the launch itself; long fused runs the VALU (4 multiply-adds per MFMA,
// 3 per 2 codes) and the copies, both near half busy.  x, codes and scales are copied to
// LDS in 1 KiB pieces of whole 128- to 512-byte row segments (R - 1 steps
// ahead): read by each wave in operand order instead, 16 rows a power of two
// apart per load, the same loads took 2-3 times as long.  Measured against the
// kernels that did so, graph of launches on distinct weights, Q8_0, bfloat16 x,
// 50 rows: 1024 -> 2048 8.5 -> 4.7 us, 1024 -> 8192 gated 14.6 -> 6.6, 4096 ->
// 1024 split 12.0 -> 8.8 with its reduction; 77 rows 1504 -> 3008 19.4 -> 6.8;
// 128 rows 4096 -> 8192 35 -> 25; 128 fused projections of 32 action-expert
// layers 281 -> 180 us.
#ifndef EB_MFMA_ROWS_H
#define EB_MFMA_ROWS_H

#include <hip/hip_runtime.h>

#include <type_traits>

#include "eb_internal.h"
#include "epilogue.h"
#include "mfma_common.h"

namespace eb {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int XT>
__device__ inline f32x4_t mfma16(const uint4 a, const uint4 b, f32x4_t c) {
  if (XT == EB_BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a),
                                                __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

// The four codes in the bytes of v, as two pairs of 16-bit floats (exact:
// |code| <= 128).  Bytes hold code + Z, Z = 128 (Q8_0, after the xor) or 8.
template <int XT, int Z>
__device__ inline uint2 codes4(uint32_t v) {
  if constexpr (XT == EB_F16) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    const h2 z = {(_Float16)(1024 + Z), (_Float16)(1024 + Z)};
    const h2 a = __builtin_bit_cast(h2, under_1024(v, 0x04010400u)) - z;
    const h2 b = __builtin_bit_cast(h2, under_1024(v, 0x04030402u)) - z;
    return make_uint2(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b));
  } else {
    float f[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (Z == 128)
        f[i] = (float)(int8_t)((v ^ 0x80808080u) >> (8 * i));
      else
        f[i] = (float)((v >> (8 * i)) & 255u) - (float)Z;
    }
    // the high halves hold the whole value (at most 8 significant bits)
    return make_uint2(__builtin_amdgcn_perm(__float_as_uint(f[1]), __float_as_uint(f[0]), 0x07060302u),
                      __builtin_amdgcn_perm(__float_as_uint(f[3]), __float_as_uint(f[2]), 0x07060302u));
  }
}

// 8 codes of one block (Q8_0: 8 int8 bytes; Q4_0: the nibble `hi` of 8 bytes)
template <int QT, int XT>
__device__ inline uint4 codes8(uint2 q, bool hi) {
  uint2 a, b;
  if constexpr (QT == EB_Q8_0) {
    a = codes4<XT, 128>(q.x ^ 0x80808080u);
    b = codes4<XT, 128>(q.y ^ 0x80808080u);
  } else {
    const int sh = hi ? 4 : 0;
    a = codes4<XT, 8>((q.x >> sh) & 0x0f0f0f0fu);
    b = codes4<XT, 8>((q.y >> sh) & 0x0f0f0f0fu);
  }
  return make_uint4(a.x, a.y, b.x, b.y);
}

// Blocks [b0, b1) of one output as sums of x * w_hat (exact products).  The
// matrix cores add 32 products with the integer codes before the block's scale
// comes in, which bfloat16 activations above 3.4e38 / (32 * 128) = 8e34 can take
// past the range of fp32 although the output is within it (or the scale is
// zero); such sums are not finite, and their outputs are computed again here.
// Ends with the first block after which the sum cannot become finite again, so
// that rows of NaNs (unused ones, say) cost little.
template <int QT>
__device__ inline float plain_output(const MMOp &o, int64_t row, int64_t col, int b0, int b1) {
  constexpr int C = QT == EB_Q8_0 ? 4 : 2;  // 8-byte pieces of codes per block
  const uint4 *x = reinterpret_cast<const uint4 *>(o.x + row * o.k);
  const uint2 *q = reinterpret_cast<const uint2 *>(o.w) + col * (o.k / kQK) * C;
  const _Float16 *d = reinterpret_cast<const _Float16 *>(o.w + o.d_off) + col * o.ds;
  float acc = 0.f;
#pragma unroll 1
  for (int p = 4 * b0; p < 4 * b1 && __builtin_isfinite(acc); ++p) {  // 8 weights
    const float dv = (float)d[p / 4];
    const uint4 xv = x[p];
    uint2 qv = q[p / 4 * C + p % C];
    if (QT == EB_Q4_0) {
      const int sh = p & 2 ? 4 : 0;
      qv = make_uint2(qv.x >> sh & 0x0f0f0f0fu, qv.y >> sh & 0x0f0f0f0fu);
    }
    const uint32_t xs[4] = {xv.x, xv.y, xv.z, xv.w}, qs[2] = {qv.x, qv.y};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int8_t c = (int8_t)(qs[j / 4] >> (8 * (j % 4)));
      const float w = (float)(QT == EB_Q8_0 ? c : c - 8) * dv;
      acc = __builtin_fmaf(__uint_as_float(j % 2 ? xs[j / 2] & 0xffff0000u : xs[j / 2] << 16), w, acc);
    }
  }
  return acc;
}

template <int QT, int NT, int MB, int W, int R>
struct RowsTile {
  static constexpr int kXcpr = 4 * W;                               // 16-byte chunks per staged row of x
  static constexpr int kWcpr = (QT == EB_Q8_0 ? 2 : 1) * W;         // of weight codes
  static constexpr int kXbytes = MB * 16 * kXcpr * 16;
  static constexpr int kWbytes = (NT * 16 * kWcpr * 16 + 1023) / 1024 * 1024;
  static constexpr int kDbytes = 1024;                              // 16 bytes of scales per weight row
  static constexpr int kStage = kXbytes + kWbytes + kDbytes;
  static constexpr int kXjobs = kXbytes / 1024, kWjobs = kWbytes / 1024;
  static constexpr int kXper = kXjobs / W, kWper = kWjobs / W;      // copies of every wave
  static constexpr int kJobs = kXper + kWper + 1;                   // and one more (see rows_unit)
  static constexpr int kSlot = NT * MB * 1024;                      // a wave's partial tile
  static constexpr int kLds = R * kStage > W * kSlot ? R * kStage : W * kSlot;
  static_assert(kXjobs % W == 0 && kWjobs % W < W, "");
  static_assert(kLds <= 160 * 1024, "fits the LDS");
};

template <int QT, int XT, int NT, int MB, int W, int R>
__device__ inline void rows_unit(const MMOp &o, int nt, int mt, int sp, int splits,
                                 float *__restrict__ ws, int64_t ws_stride, uint8_t *smem) {
  using TL = RowsTile<QT, NT, MB, W, R>;
  constexpr int BN = 16 * NT, BM = 16 * MB;
  constexpr int ELEMS = NT * MB * 64;                 // float4 outputs of the tile
  constexpr int EPT = (ELEMS + W * 64 - 1) / (W * 64);
  constexpr int QSB = (QT == EB_Q8_0) ? 32 : 16;      // code bytes per block
  constexpr uint32_t kNoElem = 0x3fffffffu;           // an element past every output tile
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r16 = lane & 15, g4 = lane >> 4;
  const int n = o.n, k = o.k, yt = o.yt, epi = o.f.epi;
  const int64_t n0 = (int64_t)nt * BN, m0 = (int64_t)mt * BM;
  const int rows_n = (int)min((int64_t)BN, n - n0), rows_m = (int)min((int64_t)BM, o.m - m0);

  const int nb = k / kQK, nsteps = (nb + W - 1) / W;
  const int s0 = (int)((int64_t)nsteps * sp / splits), s1 = (int)((int64_t)nsteps * (sp + 1) / splits);

  const uint32_t qrow = (uint32_t)nb * QSB, drow = (uint32_t)o.ds * 2, xrow = (uint32_t)k * 2;
  // descriptors from this split's first step on; each step advances them, so
  // that the range checks always end with the tile's rows
  const uint8_t *const xb = reinterpret_cast<const uint8_t *>(o.x) + m0 * xrow + s0 * (64 * W);
  const uint8_t *const qb = o.w + n0 * qrow + s0 * (QSB * W);
  const uint8_t *const db = o.w + o.d_off + n0 * drow + s0 * (2 * W);
  i32x4_t xr = rsrc4(xb, (uint32_t)rows_m * xrow - s0 * (64 * W));
  i32x4_t qr = rsrc4(qb, (uint32_t)rows_n * qrow - s0 * (QSB * W));
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;

  // copies of this wave, 1 KiB each: kXper of x rows, kWper of weight rows,
  // and one of the remaining weight rows or (the other waves, all the same
  // bytes) of the scales
  uint32_t xo[TL::kXper], qo[TL::kWper + 1];
#pragma unroll
  for (int i = 0; i < TL::kXper; ++i) {
    const uint32_t j = i * W + wave;
    const uint32_t r = j * (64 / TL::kXcpr) + lane / TL::kXcpr, c = (lane % TL::kXcpr) ^ chunk_swz<TL::kXcpr>(r);
    xo[i] = r * xrow + c * 16;
  }
  const bool last_w = TL::kWper * W + wave < TL::kWjobs;
#pragma unroll
  for (int i = 0; i <= TL::kWper; ++i) {
    const uint32_t j = i * W + wave;
    const uint32_t r = j * (64 / TL::kWcpr) + lane / TL::kWcpr, c = (lane % TL::kWcpr) ^ chunk_swz<TL::kWcpr>(r);
    qo[i] = r * qrow + c * 16;
  }
  if (!last_w) qo[TL::kWper] = (uint32_t)lane * drow;
  i32x4_t lr = last_w ? qr : rsrc4(db, (uint32_t)rows_n * drow - s0 * (2 * W));
  const uint32_t lstep = last_w ? QSB * W : 2 * W;
  const uint32_t llds = lds0 + (TL::kXjobs + (last_w ? TL::kWper * W + wave : TL::kWjobs)) * 1024;
  const uint32_t wlds = lds0 + wave * 1024;
  auto issue = [&](uint32_t st) __attribute__((always_inline)) {  // the next step, to byte st of the stages
#pragma unroll
    for (int i = 0; i < TL::kXper; ++i) copy_lds(xr, xo[i], wlds + st + i * W * 1024);
#pragma unroll
    for (int i = 0; i < TL::kWper; ++i) copy_lds(qr, qo[i], wlds + st + TL::kXbytes + i * W * 1024);
    copy_lds(lr, qo[TL::kWper], llds + st);
    advance(xr, 64 * W);
    advance(qr, QSB * W);
    advance(lr, lstep);
  };

  f32x4_t acc[NT][MB];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // this thread's outputs: float4 e = t + 64 W u of the tile is column cl,
  // rows rl .. rl + 3; their elements from the tile's first, or past the end
  const bool glu = epi == EB_EPI_GLU && !ws, add = epi == EB_EPI_ADD && !ws;
  const uint32_t nout = glu ? (uint32_t)n / 2 : (uint32_t)n;
  uint32_t el[EPT][4];
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int e = t + u * W * 64, l = e & 63, tile = e >> 6;
    const int cl = 16 * (tile / MB) + (l & 15), rl = 16 * (tile % MB) + 4 * (l >> 4);
    const bool ok = e < ELEMS && cl < rows_n && !(glu && (cl & 1));
    const uint32_t first = (uint32_t)rl * nout + (glu ? cl / 2 : cl);
#pragma unroll
    for (int i = 0; i < 4; ++i) el[u][i] = ok && rl + i < rows_m ? first + i * nout : kNoElem;
  }
  const int64_t out0 = m0 * nout + (glu ? n0 / 2 : n0);
  const uint32_t out_n = (uint32_t)rows_m * nout - (uint32_t)(glu ? n0 / 2 : n0);  // elements from out0
  float res[EPT][4];
  if (add) {  // the residuals, requested ahead of the product
    if (yt == EB_F32) {
      const auto rr = rsrc(static_cast<const float *>(o.f.r) + out0, out_n * 4);
#pragma unroll
      for (int u = 0; u < EPT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          res[u][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rr, (int)(el[u][i] * 4), 0, 0));
    } else {
      const auto rr = rsrc(static_cast<const uint16_t *>(o.f.r) + out0, out_n * 2);
#pragma unroll
      for (int u = 0; u < EPT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          res[u][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b16(rr, (int)(el[u][i] * 2), 0, 0));
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // LDS addresses of this lane's operands: wave w takes block w of a step
  uint32_t xa[MB], wa[NT];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const uint32_t r = 16 * i + r16;
    xa[i] = r * (TL::kXcpr * 16) + (((4u * wave + g4) ^ chunk_swz<TL::kXcpr>(r)) << 4);
  }
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const uint32_t r = 16 * i + r16;
    const uint32_t c = QT == EB_Q8_0 ? 2u * wave + (g4 >> 1) : (uint32_t)wave;
    wa[i] = TL::kXbytes + r * (TL::kWcpr * 16) + ((c ^ chunk_swz<TL::kWcpr>(r)) << 4) + 8u * (g4 & 1);
  }
  const uint32_t da = TL::kXbytes + TL::kWbytes + r16 * 16 + 2 * wave;
  const bool nib_hi = (g4 >> 1) != 0;

  auto compute = [&](const uint8_t *L) __attribute__((always_inline)) {
    uint4 x[MB];
    uint2 q[NT];
    float d[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      q[i] = *reinterpret_cast<const uint2 *>(L + wa[i]);
      d[i] = (float)*reinterpret_cast<const _Float16 *>(L + da + 256 * i);
    }
#pragma unroll
    for (int b = 0; b < MB; ++b) x[b] = *reinterpret_cast<const uint4 *>(L + xa[b]);
    uint4 w = codes8<QT, XT>(q[0], nib_hi);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      f32x4_t p[MB];
#pragma unroll
      for (int b = 0; b < MB; ++b) p[b] = mfma16<XT>(x[b], w, f32x4_t{0.f, 0.f, 0.f, 0.f});
      if (i + 1 < NT) w = codes8<QT, XT>(q[i + 1], nib_hi);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][b][e] = __builtin_fmaf(p[b][e], d[i], acc[i][b][e]);
    }
  };
  const int ns = s1 - s0;
  constexpr uint32_t kEnd = R * TL::kStage;
#pragma unroll
  for (int a = 0; a < R - 1; ++a)
    if (a < ns) issue(a * TL::kStage);
  uint32_t st = 0, sn = (R - 1) * TL::kStage;  // stage of step s, stage that step s + R - 1 goes to
  for (int s = 0; s < ns; ++s) {
    // step s is in LDS (later ones may be in flight), and every wave is done
    // with step s - 1
    if (R > 3 && s + 2 < ns)
      wait_vm_barrier<(R > 3 ? 2 : 0) * TL::kJobs>();
    else if (R > 2 && s + 1 < ns)
      wait_vm_barrier<(R > 2 ? 1 : 0) * TL::kJobs>();
    else
      wait_vm_barrier<0>();
    if (s + R - 1 < ns) issue(sn);
    if ((s0 + s) * W + wave < nb) compute(smem + st);
    st = st + TL::kStage == kEnd ? 0 : st + TL::kStage;
    sn = sn + TL::kStage == kEnd ? 0 : sn + TL::kStage;
  }
  wait_vm_barrier<0>();

  // partial tiles of the waves, added in wave order
  auto slot = [&](int w) __attribute__((always_inline)) {
    return reinterpret_cast<f32x4_t *>(smem + w * TL::kSlot);
  };
  {
    f32x4_t *const mine = slot(wave);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int b = 0; b < MB; ++b) mine[(i * MB + b) * 64 + lane] = acc[i][b];
  }
  __syncthreads();
  f32x4_t v[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int e = t + u * W * 64;
    v[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (ELEMS % (W * 64) != 0 && e >= ELEMS) continue;
    v[u] = slot(0)[e];
#pragma unroll
    for (int w = 1; w < W; ++w) {
      const f32x4_t a = slot(w)[e];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[u][i] += a[i];
    }
  }
  if constexpr (XT == EB_BF16) {
    // sums that are not finite (0 times one is no number), all at once: a branch
    // per float4 would have every LDS read above wait for the one before
    float z = 0.f;
#pragma unroll
    for (int u = 0; u < EPT; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) z = __builtin_fmaf(v[u][i], 0.f, z);
    if (__builtin_expect(z != 0.f, 0)) {
      uint32_t lost = 0;
#pragma unroll
      for (int u = 0; u < EPT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) lost |= __builtin_isfinite(v[u][i]) ? 0u : 1u << (4 * u + i);
#pragma unroll 1
      for (; lost; lost &= lost - 1) {
        const int j = __builtin_ctz(lost), e = t + (j >> 2) * W * 64, l = e & 63, tile = e >> 6;
        const int cl = 16 * (tile / MB) + (l & 15), rl = 16 * (tile % MB) + 4 * (l >> 4) + (j & 3);
        if (rl >= rows_m || cl >= rows_n) continue;
        const float r = plain_output<QT>(o, m0 + rl, n0 + cl, s0 * W, min(nb, s1 * W));
#pragma unroll
        for (int u = 0; u < EPT; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (4 * u + i == j) v[u][i] = r;
      }
    }
  }
  if (ws) {  // a split of k: the raw partial sums, for the ordered reduction
    const auto wr = rsrc(ws + (int64_t)sp * ws_stride + out0, out_n * 4);
#pragma unroll
    for (int u = 0; u < EPT; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[u][i]), wr, (int)(el[u][i] * 4), 0, 0);
    return;
  }
  auto put = [&](auto ytc) __attribute__((always_inline)) {
    constexpr int YT = decltype(ytc)::value;
    constexpr uint32_t es = YT == EB_F32 ? 4 : 2;
    const auto yr = rsrc(static_cast<const uint8_t *>(o.y) + out0 * es, out_n * es);
    auto store = [&](float v, uint32_t e) __attribute__((always_inline)) {
      if constexpr (YT == EB_F32)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), yr, (int)(e * es), 0, 0);
      else
        __builtin_amdgcn_raw_buffer_store_b16(to_y16(v, YT), yr, (int)(e * es), 0, 0);
    };
    if (glu) {  // the gate/up pair of columns 2c, 2c + 1 sits in lanes l, l ^ 1
#pragma unroll
      for (int u = 0; u < EPT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float g = v[u][i];
          const float up = __builtin_bit_cast(
              float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, g), 0xB1, 0xF, 0xF, true));
          store(silu_mul(g, up), el[u][i]);
        }
    } else if (add) {
#pragma unroll
      for (int u = 0; u < EPT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          store(v[u][i] + (YT == EB_F32 ? res[u][i] : from_y16((uint16_t)__float_as_uint(res[u][i]), YT)), el[u][i]);
    } else {
#pragma unroll
      for (int u = 0; u < EPT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) store(v[u][i], el[u][i]);
    }
  };
  if (yt == EB_F32)
    put(std::integral_constant<int, EB_F32>{});
  else if (yt == EB_F16)
    put(std::integral_constant<int, EB_F16>{});
  else
    put(std::integral_constant<int, EB_BF16>{});
}

// Unit u of an op's tiles -> (n tile, m tile).  Units of one residue modulo 8
// run on one XCD: it takes a stretch of the tiles in n-major order, so that its
// L2 serves the weights of an n tile again, and the stretches differ by at most
// one tile (whole columns per XCD left some idle: Q4_0, 925 rows of 10592 -> 237
// took 36.8 us, the tile kernel 27.1, this order 21.5 with the tiles chosen for it).
__device__ inline void unit_tile(uint32_t u, uint32_t tiles, uint32_t tiles_m, int &nt, int &mt) {
  const uint32_t x = u % kXcds, t = x * (tiles / kXcds) + min(x, tiles % kXcds) + u / kXcds;
  nt = (int)(t / tiles_m);
  mt = (int)(t - (uint32_t)nt * tiles_m);
}

template <int QT, int XT, int NT, int MB, int W, int R>
__global__ void __launch_bounds__(W * 64)
    mm_rows_kernel(MMOp o, int tiles_m, int splits, float *__restrict__ ws, int64_t ws_stride) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem[RowsTile<QT, NT, MB, W, R>::kLds];
  int nt, mt;
  unit_tile(blockIdx.x, gridDim.x, tiles_m, nt, mt);
  rows_unit<QT, XT, NT, MB, W, R>(o, nt, mt, (int)blockIdx.y, splits, ws, ws_stride, smem);
}

template <int QT, int XT, int NT, int MB, int W, int R>
__global__ void __launch_bounds__(W * 64)
    mm_rows_multi_kernel(const MMOp *__restrict__ ops, int nops) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem[RowsTile<QT, NT, MB, W, R>::kLds];
  const int64_t u = blockIdx.x;
  int lo = 0, hi = nops - 1;
  while (lo < hi) {
    const int mid = (lo + hi) / 2;
    if (ops[mid].unit_end <= u) lo = mid + 1; else hi = mid;
  }
  const MMOp &o = ops[lo];
  const int64_t first = lo ? ops[lo - 1].unit_end : 0;
  const int tiles_m = (o.m + 16 * MB - 1) / (16 * MB);
  int nt, mt;
  unit_tile((uint32_t)(u - first), (uint32_t)(o.unit_end - first), tiles_m, nt, mt);
  rows_unit<QT, XT, NT, MB, W, R>(o, nt, mt, 0, 1, nullptr, 0, smem);
}

// one launch of the tile (NT, MB); splits of k write partial sums to sp.ws
template <int QT, int XT, int NT, int MB, int W = 8>
hipError_t launch_lone(const MMOp &op, int splits, float *ws, int64_t ws_stride, hipStream_t s) {
  constexpr int R = 3;
  const int64_t tiles_n = (op.n + 16 * NT - 1) / (16 * NT), tiles_m = (op.m + 16 * MB - 1) / (16 * MB);
  const dim3 grid((unsigned)(tiles_n * tiles_m), (unsigned)splits);
  mm_rows_kernel<QT, XT, NT, MB, W, R><<<grid, W * 64, 0, s>>>(op, (int)tiles_m, splits, ws, ws_stride);
  return hipGetLastError();
}

template <int QT, int XT, int NT, int MB>
hipError_t launch_lone4(const MMOp &op, int splits, float *ws, int64_t ws_stride, hipStream_t s) {
  return launch_lone<QT, XT, NT, MB, 4>(op, splits, ws, ws_stride, s);
}

template <int QT, int XT, int NT, int MB>
hipError_t launch_multi(const MMOp *ops, int nops, int64_t units, hipStream_t s) {
  // NT = 4 runs are long: four waves per workgroup, so that two workgroups
  // share a CU and one's copies pass under the other's arithmetic
  constexpr int W = NT == 4 ? 4 : 8, R = 3;
  mm_rows_multi_kernel<QT, XT, NT, MB, W, R><<<(unsigned)units, W * 64, 0, s>>>(ops, nops);
  return hipGetLastError();
}

#define EB_ROWS_MB(F, NT, MB, ...)                                                 \
  (MB == 1   ? F<QT, XT, NT, 1>(__VA_ARGS__)                                       \
   : MB == 2 ? F<QT, XT, NT, 2>(__VA_ARGS__)                                       \
   : MB == 3 ? F<QT, XT, NT, 3>(__VA_ARGS__)                                       \
             : F<QT, XT, NT, 4>(__VA_ARGS__))

template <int QT, int XT>
hipError_t rows_lone_x(const RowsTiles &t, const MMOp &o, int splits, float *ws, int64_t stride,
                       hipStream_t s) {
  if (t.nt == 1) return EB_ROWS_MB(launch_lone, 1, t.mb, o, splits, ws, stride, s);
  if (t.nt == 2) return EB_ROWS_MB(launch_lone, 2, t.mb, o, splits, ws, stride, s);
  if (t.w == 4) return EB_ROWS_MB(launch_lone4, 4, t.mb, o, splits, ws, stride, s);
  return EB_ROWS_MB(launch_lone, 4, t.mb, o, splits, ws, stride, s);
}

template <int QT, int XT>
hipError_t rows_multi_x(const RowsTiles &t, const MMOp *ops, int nops, int64_t units, hipStream_t s) {
  if (t.nt == 1) return EB_ROWS_MB(launch_multi, 1, t.mb, ops, nops, units, s);
  if (t.nt == 2) return EB_ROWS_MB(launch_multi, 2, t.mb, ops, nops, units, s);
  return EB_ROWS_MB(launch_multi, 4, t.mb, ops, nops, units, s);
}
#undef EB_ROWS_MB

}  // namespace

template <int QT>
hipError_t rows_lone(int32_t xt, const RowsTiles &t, const MMOp &o, int splits, float *ws,
                     int64_t ws_stride, hipStream_t s) {
  if (xt == EB_F16) return rows_lone_x<QT, EB_F16>(t, o, splits, ws, ws_stride, s);
  return rows_lone_x<QT, EB_BF16>(t, o, splits, ws, ws_stride, s);
}

template <int QT>
hipError_t rows_multi(int32_t xt, const RowsTiles &t, const MMOp *ops, int nops, int64_t units,
                      hipStream_t s) {
  if (xt == EB_F16) return rows_multi_x<QT, EB_F16>(t, ops, nops, units, s);
  return rows_multi_x<QT, EB_BF16>(t, ops, nops, units, s);
}

}  // namespace eb

#endif  // EB_MFMA_ROWS_H
