// Batched variant of the column-sparse projection for gfx950: B tokens with independent per-token
// index sets.  The union of the tokens' kept rows is what has to be read; at the sparsities of
// interest it is nearly every row once B >= 4 (1 - p^B of them), so the weight is streamed once
// over all rows and each token's dropped channels simply carry a zero coefficient:
//     y[b,:] = sum_j C[b,j] * W[j,:],   C[b,j] = h[b,j] if j in idx_b else 0.
// The same kernels serve the batched rotation / adapter / dense baseline (C = x).
//
//   * the product is a skinny dense contraction (all rows x B tokens), so it runs on the matrix
//     cores (f16/bf16, fp32 accumulate): M = 16 output columns, N = 16 tokens, K = 16 rows, token blocks padded to 16.
//     Measured on MI355X this is the fastest for every B >= 2 (the fp32-FMA kernel needed 205 us per LLaMA3-8B layer at
//     B = 4 where the first matrix-core kernel needed 160 us), because the product is HBM-bound and the FMA variant spends
//     its issue slots on B x 8 multiply-adds and coefficient reads per 16 bytes loaded.  Two kernels, which add a token's
//     products in the same order (its bits do not depend on the size of its batch):
//     up to 16 tokens (skinny16) a lane loads 8 consecutive columns of 4 rows (16 lanes x 16 bytes = 256 contiguous bytes
//     per row), and a byte permute regroups those registers into the K-runs the instruction wants; the weight never
//     passes through LDS.  More tokens (skinny32, groups of 32; small weights stay with groups of 16) keep the matrix
//     cores busy longer per row, so the loads go straight to LDS, ahead of the products and without registers of their
//     own, and transposing LDS reads make the K-runs (LLaMA2-7B layer, 32 tokens: 161 -> 152 us);
//   * an fp32-FMA kernel (2 or 4 tokens per workgroup) remains for the one case the 16-bit B
//     operand cannot express: a per-channel coefficient scale applied in fp32 (learned pre-norm
//     scale in front of an explicit rotation).
// Work split (one strip per workgroup, equal runs of rows), cross-workgroup hand-off (16-byte coherent
// stores and loads, arrival counter, the last arrival finishes) and epilogue follow the single-token
// kernel (gemv_core.hpp), with one arrival per workgroup for all its tokens.
#include "gemv_core.hpp"
#include "lds_load.hpp"

namespace larosa {

namespace {

constexpr int kBRW = 8;                 // row-waves of the FMA kernel
constexpr int kBThreads = 512;

// ------------------------------------------------------------------------------------------------
// masked coefficient matrix from (h, idx): C[b,:] = 0, then C[b, idx[b,t]] = h[b, idx[b,t]]
// ------------------------------------------------------------------------------------------------
// A workgroup fills a slice of one token's channels: it reads the token's whole index list (it need not be sorted),
// marks the kept channels of its slice in LDS and writes the slice once.  Latency-bound (under 1 MB moved): with one
// workgroup per token, its scattered stores and the barrier between them, 5 tokens of 14336 channels took 6.9 us, so
// slices of several workgroups per token and 16 index loads in flight per lane; now 3.9 us (5.2 with 8 in flight and 256
// lanes).  Every slice reads the list again, so from 64 slices of 4096 on the slices grow instead of their number (16
// tokens of 2^22 channels, whole call: 0.70 ms; 5.9 ms in slices of 4096, 3.6 with one workgroup per token).
constexpr int kPrepThreads = 512, kPrepPass = kPrepThreads * 8;   // channels per pass of the workgroup over its slice
constexpr int kPrepSlices = 64, kPrepSliceMax = 1 << 17;
template <bool ONE_PASS>   // slices of kPrepPass channels, 0.06 us a call faster than with the loops and LDS sized at the launch
__global__ __launch_bounds__(kPrepThreads) void batch_prep_kernel(const uint16_t* __restrict__ h, const int32_t* __restrict__ idx,
                                                                  uint16_t* __restrict__ C, int d_in, int K, int any_slice) {
  extern __shared__ __attribute__((aligned(16))) unsigned char any_kept[];
  __shared__ __attribute__((aligned(16))) unsigned char pass_kept[ONE_PASS ? kPrepPass : 16];
  unsigned char* const kept = ONE_PASS ? pass_kept : any_kept;   // [slice]
  const int slice = ONE_PASS ? kPrepPass : any_slice;
  const int b = blockIdx.y;
  const int c0 = blockIdx.x * slice, n = min(slice, d_in - c0);   // the slice's channels
  const size_t at = static_cast<size_t>(b) * d_in + c0;
  const int i0 = threadIdx.x * 8;                // the lane's 8 channels of the first pass (d_in % 8 == 0: all inside or none)
  uint4 first = make_uint4(0u, 0u, 0u, 0u);
  if (i0 < n) first = *reinterpret_cast<const uint4*>(h + at + i0);
  if (ONE_PASS) *reinterpret_cast<uint2*>(kept + i0) = make_uint2(0u, 0u);
  else
    for (int i = i0; i < n; i += kPrepPass) *reinterpret_cast<uint2*>(kept + i) = make_uint2(0u, 0u);
  __syncthreads();
  const int32_t* ib = idx + static_cast<size_t>(b) * K;
  constexpr int kAhead = 16;
  for (int t0 = 0; t0 < K; t0 += kPrepThreads * kAhead) {
    int j[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) j[q] = ib[min(t0 + q * kPrepThreads + static_cast<int>(threadIdx.x), K - 1)];   // the last one again: no matter
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const unsigned e = static_cast<unsigned>(j[q] - c0);
      if (e < static_cast<unsigned>(slice)) kept[e] = 1;
    }
  }
  __syncthreads();
  for (int i = i0; i < n; i += kPrepPass) {
    uint4 v = i == i0 ? first : *reinterpret_cast<const uint4*>(h + at + i);
    const uint2 k = *reinterpret_cast<const uint2*>(kept + i);
    // bytes 0 / 1 of a channel pair to the two halves of its dword
    const auto mask2 = [](uint32_t bytes, int sh) { return ((bytes >> sh) & 1u) * 0xFFFFu | ((bytes >> (sh + 8)) & 1u) * 0xFFFF0000u; };
    v.x &= mask2(k.x, 0);
    v.y &= mask2(k.x, 16);
    v.z &= mask2(k.y, 0);
    v.w &= mask2(k.y, 16);
    *reinterpret_cast<uint4*>(C + at + i) = v;
  }
}

struct Geometry {
  int s, t0, t1;          // strip and row range of a segment
  int g_first, g_last;    // workgroups that contribute to the strip
};

// Workgroup g works on strip g / wps only, rows [(g % wps) * chunk, + chunk) of it (plan_batched: every
// workgroup of a strip has rows, all but the last one `chunk` of them).
__device__ __forceinline__ Geometry strip_geometry(int g, int wps, int K, int chunk) {
  const int s = g / wps;
  const int t0 = (g - s * wps) * chunk;
  Geometry q{s, t0, min(K, t0 + chunk), s * wps, s * wps + wps - 1};
  return q;
}

// per-token pre-norm factor 1/sqrt(mean(x^2)+eps): wave w handles tokens w, w+NW, ...
template <typename T, int NW>
__device__ __forceinline__ void token_scales(const BatchArgs& a, int b0, int ntok, float* scale_s, int lane, int wave) {
  for (int bb = wave; bb < ntok; bb += NW) {
    float sc = 1.f;
    const int tok = b0 + bb;
    if (a.rms_src && tok < a.B) {
      const uint16_t* xs = a.rms_src + static_cast<size_t>(tok) * a.d_in;
      float ss = 0.f;
      for (int i = lane * 8; i < a.d_in; i += 64 * 8) {
        float w[8];
        unpack8<T>(*reinterpret_cast<const uint4*>(xs + i), w);
#pragma unroll
        for (int k = 0; k < 8; ++k) ss = fmaf(w[k], w[k], ss);
      }
      ss = wave_sum(ss);
      sc = 1.0f / sqrtf(ss / static_cast<float>(a.d_in) + a.rms_eps);
    }
    if (lane == 0) scale_s[bb] = sc;
  }
}

// epilogue for 8 consecutive columns of one token
template <typename T>
__device__ __forceinline__ void store_out8(const BatchArgs& a, int tok, int col, float (&v)[8], float scale) {
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] *= scale;
  const size_t off = static_cast<size_t>(tok) * a.d_out + col;
  if (a.residual) {
    if (a.y_pre) *reinterpret_cast<uint4*>(a.y_pre + off) = pack8<T>(v);
    float r[8];
    unpack8<T>(*reinterpret_cast<const uint4*>(a.residual + off), r);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = r[k] + round_store<T>(v[k]);
  }
  *reinterpret_cast<uint4*>(a.y + off) = pack8<T>(v);
}

// the same for 4 consecutive columns (d_out % 4 == 0: all four are inside)
template <typename T>
__device__ __forceinline__ void store_out4(const BatchArgs& a, int tok, int col, const float __attribute__((ext_vector_type(4))) & sum,
                                           float scale) {
  const size_t off = static_cast<size_t>(tok) * a.d_out + col;
  float v[4] = {sum.x * scale, sum.y * scale, sum.z * scale, sum.w * scale};
  if (a.residual) {
    if (a.y_pre) *reinterpret_cast<uint2*>(a.y_pre + off) = pack4<T>(v);
    const uint2 r = *reinterpret_cast<const uint2*>(a.residual + off);
    float f[4];
    T::unpack2(r.x, f[0], f[1]);
    T::unpack2(r.y, f[2], f[3]);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = f[k] + round_store<T>(v[k]);
  }
  *reinterpret_cast<uint2*>(a.y + off) = pack4<T>(v);
}

// ------------------------------------------------------------------------------------------------
// FMA kernel, NB <= 4 tokens per workgroup
// ------------------------------------------------------------------------------------------------
// Geometry: a workgroup is 8 waves on ONE strip of 128 columns.  Lane (kgrp, m) = (lane / 16,
// lane % 16) owns columns 8m..8m+7 of the strip; one load instruction of a wave covers 4 rows (one
// per kgrp), 256 contiguous bytes each, and 8 such loads are in flight.  The four row groups of a
// wave are summed by two lane exchanges, the 8 waves through LDS, workgroups through the workspace.
// Narrow strips keep the number of workgroups per strip, and so the partial-sum traffic, small.
constexpr int kFStrip = 128;

template <typename T, int NB>
__global__ __launch_bounds__(kBThreads) void skinny_fma_kernel(BatchArgs a) {
  __shared__ float coef[NB][kBatchChunkMax];
  __shared__ float red[kBRW - 1][NB][8][16];
  __shared__ float scale_s[NB];
  __shared__ int s_last;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int rw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kgrp = lane >> 4;
  const int m = lane & 15;
  const int g = blockIdx.x;
  const int grp = blockIdx.y;
  const int b0 = grp * NB;
  const int K = a.d_in;
  const int chunk = a.chunk;

  {
    const Geometry ge = strip_geometry(g, a.wps, K, chunk);
    const int s = ge.s, t0 = ge.t0, t1 = ge.t1;
    const int n = t1 - t0;
    const int col = s * kFStrip + m * 8;
    const bool colv = col < a.d_out;

    // this segment's coefficients, as floats, for the NB tokens
    for (int e = tid; e < NB * n; e += kBThreads) {
      const int bb = e / n;
      const int t = e - bb * n;
      const int tok = b0 + bb;
      float c = 0.f;
      if (tok < a.B) {
        c = T::to_f32(a.C[static_cast<size_t>(tok) * K + t0 + t]);
        if (a.coef_scale) c *= T::to_f32(a.coef_scale[t0 + t]);
      }
      coef[bb][t] = c;
    }
    __syncthreads();

    float acc[NB][8];
#pragma unroll
    for (int bb = 0; bb < NB; ++bb)
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[bb][k] = 0.f;
    const int per = (n + kBRW - 1) / kBRW;
    const int ra = t0 + rw * per;
    const int re = min(t1, ra + per);
    if (colv) {
      const uint16_t* wcol = a.W + col;
      for (int t = ra; t < re; t += 4 * kUnroll) {
        uint4 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
          v[u] = load_stream16(wcol + static_cast<size_t>(min(t + 4 * u + kgrp, re - 1)) * a.d_out);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
          float w[8];
          unpack8<T>(v[u], w);
          const int r = t + 4 * u + kgrp;
          const bool ok = r < re;
          const int ti = min(r, re - 1) - t0;
#pragma unroll
          for (int bb = 0; bb < NB; ++bb) {
            const float c = ok ? coef[bb][ti] : 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[bb][k] = fmaf(c, w[k], acc[bb][k]);
          }
        }
      }
    }
    // the four row groups of the wave (fixed order), then the 8 waves through LDS
#pragma unroll
    for (int bb = 0; bb < NB; ++bb)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        acc[bb][k] += __shfl_xor(acc[bb][k], 16, kWave);
        acc[bb][k] += __shfl_xor(acc[bb][k], 32, kWave);
      }
    if (rw > 0 && kgrp == 0) {
#pragma unroll
      for (int bb = 0; bb < NB; ++bb)
#pragma unroll
        for (int k = 0; k < 8; ++k) red[rw - 1][bb][k][m] = acc[bb][k];
    }
    __syncthreads();
    if (rw == 0 && kgrp == 0) {
      for (int r = 0; r < kBRW - 1; ++r)
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
#pragma unroll
          for (int k = 0; k < 8; ++k) acc[bb][k] += red[r][bb][k][m];
    }
    __syncthreads();

    const int n_s = ge.g_last - ge.g_first + 1;
    bool last = (n_s == 1);
    if (n_s > 1) {
      // slot: [NB][4][16] float pairs; lane m of the first wave holds columns 8m..8m+7
      const size_t slot_floats = static_cast<size_t>(NB) * kFStrip;
      unsigned long long* slot = reinterpret_cast<unsigned long long*>(
          a.partial + (static_cast<size_t>(grp) * a.G + g) * slot_floats);
      unsigned* ctr = a.counters + (static_cast<size_t>(grp) * a.nstrips + s) * kCounterStride;
      if (rw == 0 && kgrp == 0) {
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const unsigned long long v = static_cast<unsigned long long>(__float_as_uint(acc[bb][2 * k])) |
                                         (static_cast<unsigned long long>(__float_as_uint(acc[bb][2 * k + 1])) << 32);
            __hip_atomic_store(slot + bb * 64 + k * 16 + m, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0) {
        const unsigned old = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = (old == static_cast<unsigned>(n_s - 1)) ? 1 : 0;
      }
      __syncthreads();
      last = (s_last != 0);
      if (last) {
        if (tid == 0) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // lane group kgrp of wave rw adds partials g_first + 4*rw + kgrp, + 32, ...: 32 partials per pass
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
#pragma unroll
          for (int k = 0; k < 8; ++k) acc[bb][k] = 0.f;
        for (int gg = ge.g_first + 4 * rw + kgrp; gg <= ge.g_last; gg += 4 * kBRW) {
          const unsigned long long* p = reinterpret_cast<const unsigned long long*>(
              a.partial + (static_cast<size_t>(grp) * a.G + gg) * slot_floats);
          unsigned long long v[NB][4];
#pragma unroll
          for (int bb = 0; bb < NB; ++bb)
#pragma unroll
            for (int k = 0; k < 4; ++k)
              v[bb][k] = __hip_atomic_load(p + bb * 64 + k * 16 + m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int bb = 0; bb < NB; ++bb)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              acc[bb][2 * k] += __uint_as_float(static_cast<unsigned>(v[bb][k] & 0xFFFFFFFFull));
              acc[bb][2 * k + 1] += __uint_as_float(static_cast<unsigned>(v[bb][k] >> 32));
            }
        }
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            acc[bb][k] += __shfl_xor(acc[bb][k], 16, kWave);
            acc[bb][k] += __shfl_xor(acc[bb][k], 32, kWave);
          }
        if (rw > 0 && kgrp == 0) {
#pragma unroll
          for (int bb = 0; bb < NB; ++bb)
#pragma unroll
            for (int k = 0; k < 8; ++k) red[rw - 1][bb][k][m] = acc[bb][k];
        }
        __syncthreads();
        if (rw == 0 && kgrp == 0) {
          for (int r = 0; r < kBRW - 1; ++r)
#pragma unroll
            for (int bb = 0; bb < NB; ++bb)
#pragma unroll
              for (int k = 0; k < 8; ++k) acc[bb][k] += red[r][bb][k][m];
        }
        __syncthreads();
      }
    }
    if (last) {   // uniform over the workgroup
      token_scales<T, kBRW>(a, b0, NB, scale_s, lane, rw);
      __syncthreads();
      if (rw == 0 && kgrp == 0 && colv) {
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
          if (b0 + bb < a.B) store_out8<T>(a, b0 + bb, col, acc[bb], scale_s[bb]);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// matrix-core kernels: up to 16 tokens (skinny16), groups of 32 tokens (skinny32)
// ------------------------------------------------------------------------------------------------
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float float4_t __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ float4_t mfma16(uint2 a, uint2 b, float4_t c);
template <>
__device__ __forceinline__ float4_t mfma16<F16>(uint2 a, uint2 b, float4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4_t, a), __builtin_bit_cast(half4_t, b), c, 0, 0, 0);
}
template <>
__device__ __forceinline__ float4_t mfma16<BF16>(uint2 a, uint2 b, float4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4_t, a), __builtin_bit_cast(short4_t, b), c, 0,
                                                   0, 0);
}

constexpr int k16Strip = 128;        // output columns per workgroup of the kernel for up to 16 tokens
constexpr int k16Waves = 8;             // its row-waves
constexpr int k16Pitch = 130;   // floats per token row of an LDS tile (8-byte aligned, spreads tokens over banks)

// Up to 16 tokens per group.  Geometry: a workgroup is 8 waves on ONE strip of 128 columns (256 contiguous bytes per row), each
// wave taking its own run of 16-row tiles, two tiles (8 row loads of 16 bytes per lane) in flight.
// Narrow strips keep the number of workgroups that share a strip -- and with it the partial-sum
// traffic, which grows with the token count -- small.
template <typename T>
__device__ __forceinline__ void skinny16_body(const BatchArgs& a, int g, int grp) {
  __shared__ float tile[4][16][k16Pitch];
  // blocks of 16 tokens.  The three loops over it stay: written straight, the compiler lays this kernel's tail out
  // differently and its launches take 0.3 - 0.4 % longer (8B-shaped halves of 13 tokens 129.5 -> 129.9 us)
  constexpr int NTB = 1;
  __shared__ float scale_s[16];
  __shared__ int s_last;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int rw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kgrp = lane >> 4;    // K-run of 4 rows inside a 16-row tile
  const int m = lane & 15;       // column group (A operand) / token (B operand)
  const int b0 = grp * 16;
  const int K = a.d_in;
  const int chunk = a.chunk;

  LAROSA_STAMP(0);
  {
    const Geometry ge = strip_geometry(g, a.wps, K, chunk);
    const int s = ge.s, t0 = ge.t0, t1 = ge.t1;
    const int n = t1 - t0;
    const int colbase = s * k16Strip + 8 * m;   // this lane's 8 columns (A operand)
    const bool colv = colbase < a.d_out;

    float4_t acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = float4_t{0.f, 0.f, 0.f, 0.f};

    const int ntiles = (n + 15) / 16;
    const int per = (ntiles + k16Waves - 1) / k16Waves;
    const int tl0 = rw * per;
    const int tl1 = min(ntiles, tl0 + per);
    for (int tl = tl0; tl < tl1; tl += 2) {
      uint4 v[2][4];
      uint2 bf[2];
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        // first of this lane's 4 rows; t0 % 8 == 0, so j0 % 4 == 0.  A tile past this wave's run
        // starts at t1: its rows clamp to a valid address and its B operand is zero.
        const int j0 = (tl + h2 < tl1) ? t0 + (tl + h2) * 16 + 4 * kgrp : t1;
        // Every load is unconditional, from an address clamped into the operand (columns past d_out
        // read the strip's first column, tokens past B the last token, rows past t1 a valid row), and
        // what must not count is zeroed afterwards: a load under a lane condition sits in a branch of
        // its own, and the compiler then waits for the earlier loads half-way through issuing them.
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = min(j0 + q, t1 - 1);
          v[h2][q] = load_stream16(a.W + static_cast<size_t>(r) * a.d_out + (colv ? colbase : s * k16Strip));
        }
        // B operand: 4 consecutive rows of token b0 + m; rows at or past t1 belong to another workgroup
        // (or do not exist) and must contribute nothing
        const int tok = b0 + m;
        // j0 % 4 == 0 and K % 8 == 0, so min(j0, K - 4) keeps the four rows inside the token's vector
        uint2 c = *reinterpret_cast<const uint2*>(a.C + static_cast<size_t>(min(tok, a.B - 1)) * K + min(j0, K - 4));
        if (j0 + 1 >= t1) c.x &= 0x0000FFFFu;
        if (j0 + 2 >= t1) c.y = 0u;
        if (j0 + 3 >= t1) c.y &= 0x0000FFFFu;
        if (j0 >= t1 || tok >= a.B) c.x = 0u;
        if (tok >= a.B) c.y = 0u;
        bf[h2] = c;
      }
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        // A operand for column offset i: element i of each of the 4 row registers
        const uint32_t* vw0 = reinterpret_cast<const uint32_t*>(&v[h2][0]);
        const uint32_t* vw1 = reinterpret_cast<const uint32_t*>(&v[h2][1]);
        const uint32_t* vw2 = reinterpret_cast<const uint32_t*>(&v[h2][2]);
        const uint32_t* vw3 = reinterpret_cast<const uint32_t*>(&v[h2][3]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;
          uint2 af;
          af.x = __builtin_amdgcn_perm(vw1[i >> 1], vw0[i >> 1], sel);
          af.y = __builtin_amdgcn_perm(vw3[i >> 1], vw2[i >> 1], sel);
          acc[i] = mfma16<T>(af, bf[h2], acc[i]);
        }
      }
    }

    LAROSA_STAMP(1);
    const int n_s = ge.g_last - ge.g_first + 1;
    const size_t slot_floats = 16 * k16Strip;
    unsigned* ctr = a.counters + (static_cast<size_t>(grp) * a.nstrips + s) * kCounterStride;
    // every partial of this token group as one buffer (slot of workgroup w at byte w * slot bytes; a thread's 16 bytes at tid * 16 within it);
    // 16-byte accesses with the sc1 cache policy are coherent across the chip, see gemv_core.hpp
    const int slot_bytes = 8192;
    const __amdgpu_buffer_rsrc_t slots = __builtin_amdgcn_make_buffer_rsrc(
        a.partial + static_cast<size_t>(grp) * a.G * slot_floats, 0, a.G * slot_bytes, 0x00027000);
    constexpr int kCoherent = 16;
    const int my_slot = g * slot_bytes;

    // Sum the 8 row-waves: waves 0-3 write their tiles, waves 4-7 add theirs on
    // top, then every thread adds the four tiles for its two float pairs (pair q: token q / 64,
    // columns 2*(q % 64), +1).  D element e of MFMA i in lane (kgrp, m) is column 32*kgrp + 8*e + i
    // of token m.  The order of the additions is fixed.
    auto reduce = [&](float2 (&sm)[2]) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if ((rw >> 2) == r) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float* p = &tile[rw & 3][m][32 * kgrp + 8 * e + i];
              *p = (r == 0) ? acc[i][e] : *p + acc[i][e];
            }
        }
        __syncthreads();
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int q = tid + k * kBThreads;
        float2 t = *reinterpret_cast<const float2*>(&tile[0][q >> 6][(q & 63) * 2]);
#pragma unroll
        for (int w = 1; w < 4; ++w) {
          const float2 u = *reinterpret_cast<const float2*>(&tile[w][q >> 6][(q & 63) * 2]);
          t.x += u.x;
          t.y += u.y;
        }
        sm[k] = t;
      }
      __syncthreads();
    };
    // epilogue: the 16 x 128 sums (pairs held as in reduce) go through tile[0]
    auto tile_out = [&](const float2 (&sm)[2]) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int q = tid + k * kBThreads;
        *reinterpret_cast<float2*>(&tile[0][q >> 6][(q & 63) * 2]) = sm[k];
      }
      __syncthreads();
      if (tid < 256) {
        const int tok = b0 + (tid >> 4);
        const int col = s * k16Strip + (tid & 15) * 8;
        if (tok < a.B && col < a.d_out) {
          float v[8];
          const float* p = &tile[0][tid >> 4][(tid & 15) * 8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = p[e];
          store_out8<T>(a, tok, col, v, scale_s[tid >> 4]);
        }
      }
      __syncthreads();
    };

    if (n_s == 1) {
      token_scales<T, k16Waves>(a, b0, 16, scale_s, lane, rw);
      __syncthreads();
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) {
        float2 sm[2];
        reduce(sm);
        tile_out(sm);
      }
    } else {
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) {
        float2 sm[2];
        reduce(sm);
        // the thread's two float pairs of the block as one 16-byte chip-coherent store
        const u32x4 v = {__float_as_uint(sm[0].x), __float_as_uint(sm[0].y), __float_as_uint(sm[1].x), __float_as_uint(sm[1].y)};
        __builtin_amdgcn_raw_buffer_store_b128(v, slots, my_slot + tb * 8192 + tid * 16, 0, kCoherent);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      LAROSA_STAMP(2);
      if (tid == 0) {
        const unsigned old = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = (old == static_cast<unsigned>(n_s - 1)) ? 1 : 0;
      }
      __syncthreads();
      LAROSA_STAMP(3);
      if (s_last != 0) {   // uniform over the workgroup
        if (tid == 0) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        token_scales<T, k16Waves>(a, b0, 16, scale_s, lane, rw);
        for (int tb = 0; tb < NTB; ++tb) {
          // each thread owns 2 float pairs of the block and adds the partials in workgroup order
          float2 sum[2];
          sum[0] = sum[1] = make_float2(0.f, 0.f);
          for (int gg = ge.g_first; gg <= ge.g_last; gg += 8) {
            u32x4 v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              if (gg + q <= ge.g_last) {          // uniform over the workgroup: no partial is read twice
                v[q] = __builtin_amdgcn_raw_buffer_load_b128(slots, (gg + q) * slot_bytes + tid * 16, 0, kCoherent);
              }
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              if (gg + q <= ge.g_last) {
                sum[0].x += __uint_as_float(v[q].x);
                sum[0].y += __uint_as_float(v[q].y);
                sum[1].x += __uint_as_float(v[q].z);
                sum[1].y += __uint_as_float(v[q].w);
              }
            }
          }
          tile_out(sum);
        }
      }
    }
  }
  LAROSA_STAMP(5);
}

// More than 16 tokens, in groups of 32.  What bounded the kernel above here: with two blocks of tokens a wave spends twice
// as long between its batches of loads, so fewer are in flight (4096 x 22016, 32 tokens: 47.5 us on 172 workgroups; this
// one 43.1).  For 16 tokens the two are level, and the one above keeps its smaller hand-off.
// The sums are formed in that kernel's order, so a token's result does not depend on the size of its batch: eight runs of
// 16-row tiles per workgroup, one 16-deep product after the other along a run, the runs added as (0 + 4) + (1 + 5) + ...
constexpr int kMRuns = 8;           // runs of rows per workgroup
constexpr int kMTokens = 32;
constexpr int kMLds = 160 * 1024;   // a compute unit's LDS: the rings of all waves

// Sizes of the kernel for strips of SC columns, NW waves and tiles of R rows.
template <int SC, int NW, int R>
struct SkinnyShape {
  static constexpr int kTileBytes = R * SC * 2;
  static constexpr int kStage = kTileBytes + kMTokens * R * 2;   // a tile and the tokens' coefficients of its rows
  static constexpr int kStages = kMLds / NW / kStage;           // tiles in a wave's ring
  static constexpr int kRing = kStages * kStage;
  static constexpr int kPitch = SC + 4;                          // floats per token row of a wave's sums in LDS
  static_assert(sizeof(float) * (4 * kMTokens * kPitch + kMTokens + 1) <= NW * kRing, "sums, scales and flag reuse the rings");
};

// Position of row k's 32-byte granules in a tile with G of them per row: granule q sits at q ^ granule_swap(k), so that
// the eight rows that half a wave's transposing read touches lie in different banks.
template <int G>
__device__ __forceinline__ int granule_swap(int k) { return k & (G - 1); }

// Geometry: a workgroup is NW waves on ONE strip of SC columns (2 SC contiguous bytes per row).  Each wave streams its own
// runs of rows (one, or with four waves two) through a ring of its own in LDS: the loads go straight to LDS and run ahead
// of the products by what the ring holds (at least 16 KiB a wave), and no wave waits for another until the sums meet.
//   W tile    [R rows][SC columns] as in memory, granules exchanged as above.  16 lanes of a transposing read point at
//             4 rows x 16 columns and receive 4 consecutive rows of one column each: the A operand (M = 16 columns,
//             K = 16 rows).
//   C tile    R = 32: two blocks of [16 tokens][32 rows], 16-byte piece p of token m at position p ^ (m / 4 % 4);
//             R = 16: [32 tokens][16 rows].  The B operand.
// Rows past the run arrive as zeros (beyond the end of the buffer the tile's loads go through), and so do columns past
// d_out, tokens past B and the coefficients of rows past the run.
template <typename T, int SC, int NW, int R>
__device__ __forceinline__ void skinny32_body(const BatchArgs& a, int g, int grp) {
  typedef SkinnyShape<SC, NW, R> Sh;
  constexpr int NTB = kMTokens / 16;             // blocks of 16 tokens
  constexpr int kTokens = kMTokens, kStage = Sh::kStage, kRing = Sh::kRing, kPitch = Sh::kPitch;
  constexpr int kThreads = NW * 64;
  constexpr int kGroups = SC / 16;               // 16-column groups of the strip
  constexpr int kLoadsW = Sh::kTileBytes / 1024; // wave-loads per tile
  constexpr int kLoadsC = R / 16;
  constexpr int kLoads = kLoadsW + kLoadsC;
  constexpr int kRowLanes = SC / 8;              // lanes that load one row
  constexpr int kLoadRows = 64 / kRowLanes;
  constexpr int kCLanes = R / 8;                 // lanes that load one token's coefficients
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int rw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b0 = grp * kTokens;
  const int K = a.d_in, d_out = a.d_out;

  LAROSA_STAMP(0);
  Geometry ge = strip_geometry(g, a.wps, K, a.chunk);
  ge.t0 = __builtin_amdgcn_readfirstlane(ge.t0);   // uniform, but the division leaves it in vector registers
  ge.t1 = __builtin_amdgcn_readfirstlane(ge.t1);
  const int s = ge.s;

  // runs of whole 16-row tiles, the last one possibly short; run rw and (four waves) run rw + 4
  const int per = ((ge.t1 - ge.t0 + 15) / 16 + kMRuns - 1) / kMRuns * 16;   // rows of a run
  auto run_begin = [&](int run) __attribute__((always_inline)) { return min(ge.t1, ge.t0 + run * per); };
  int r0 = run_begin(rw);                        // first row not yet asked for
  int left = run_begin(rw + 1) - r0;             // rows of the run not yet asked for

  // ---- loads.  Wave-load q covers kLoadRows rows of the tile; a lane's place in the row is lane % kRowLanes pieces.
  uint32_t offW[kLoadsW];
#pragma unroll
  for (int q = 0; q < kLoadsW; ++q) {
    const int row = q * kLoadRows + lane / kRowLanes, pos = lane % kRowLanes;
    const int col = (((pos >> 1) ^ granule_swap<kGroups>(row)) << 4) + (pos & 1) * 8;
    offW[q] = s * SC + col < d_out ? (static_cast<uint32_t>(row) * d_out + s * SC + col) * 2u : kOutside;
  }
  uint32_t offC[kLoadsC];
  // first row of the lane's piece: token lane / kCLanes (of its block), position lane % kCLanes
  const int kC = R == 32 ? 8 * ((lane & 3) ^ ((lane >> 4) & 3)) : 8 * (lane & 1);
#pragma unroll
  for (int q = 0; q < kLoadsC; ++q) {
    const int tok = q * 16 + lane / kCLanes;
    offC[q] = b0 + tok < a.B ? (static_cast<uint32_t>(tok) * K + kC) * 2u : kOutside;
  }
  const uint32_t ring = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_char*)lds)) + rw * kRing;
  const char* nextW = reinterpret_cast<const char*>(a.W) + static_cast<size_t>(r0) * d_out * 2;
  const char* nextC = reinterpret_cast<const char*>(a.C) + (static_cast<size_t>(b0) * K + r0) * 2;
  const int steps0 = (left + R - 1) / R;         // tiles of the wave's first run, of its second
  const int second = NW < kMRuns ? run_begin(rw + NW) : 0;
  int left2 = NW < kMRuns ? run_begin(rw + NW + 1) - second : 0;
  const int steps1 = (left2 + R - 1) / R;
  uint32_t in_stage = 0;
  const uint32_t bytesC = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(min(kTokens, a.B - b0)) * K * 2u);
  auto fetch = [&]() __attribute__((always_inline)) {
    const int rows = __builtin_amdgcn_readfirstlane(max(0, min(R, left)));   // (the clamp is a vector instruction)
    const u32x4 bufW = raw_buffer(nextW, static_cast<uint32_t>(rows) * d_out * 2u);
    const u32x4 bufC = raw_buffer(nextC, bytesC);
#pragma unroll
    for (int q = 0; q < kLoadsC; ++q)
      load_to_lds(bufC, ring + in_stage + Sh::kTileBytes + q * 1024, kC < rows ? offC[q] : kOutside);
#pragma unroll
    for (int q = 0; q < kLoadsW; ++q) load_to_lds_stream(bufW, ring + in_stage + q * 1024, offW[q]);
    left -= R;
    nextW += static_cast<size_t>(R) * d_out * 2;
    nextC += R * 2;
    if (NW < kMRuns && left <= 0 && left2 > 0) { // on to the second run (once)
      left = left2;
      left2 = 0;
      nextW = reinterpret_cast<const char*>(a.W) + static_cast<size_t>(second) * d_out * 2;
      nextC = reinterpret_cast<const char*>(a.C) + (static_cast<size_t>(b0) * K + second) * 2;
    }
    in_stage = in_stage == (Sh::kStages - 1) * kStage ? 0 : in_stage + kStage;
  };

  // ---- operand reads
  const int grp16 = lane >> 4, j = lane & 15;
  const int rowk = 4 * grp16 + (j >> 2);
  const int sw = granule_swap<kGroups>(rowk);    // (and of row rowk + 16)
  const uint32_t rdW = ring + rowk * (SC * 2) + 8 * (j & 3);
  const uint32_t rdC = ring + Sh::kTileBytes + (R == 32 ? j * 64 + (((grp16 >> 1) ^ ((j >> 2) & 3)) * 16) + (grp16 & 1) * 8 : j * 32 + grp16 * 8);
  float4_t acc[NTB][kGroups], run_sum[NTB][kGroups];   // of the run at hand; of the runs before it
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
    for (int i = 0; i < kGroups; ++i) acc[tb][i] = run_sum[tb][i] = float4_t{0.f, 0.f, 0.f, 0.f};

  for (int i = 0; i < Sh::kStages; ++i) fetch();
  uint32_t stage = 0;
#pragma nounroll
  for (int run = 0; run < kMRuns / NW; ++run) {
    const int steps = run == 0 ? steps0 : steps1;
    for (int t = 0; t < steps; ++t) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((Sh::kStages - 1) * kLoads) : "memory");   // this tile has landed
      uint2 av[R / 16][kGroups], bv[R / 16][NTB];
#pragma unroll
      for (int h = 0; h < R / 16; ++h)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
          bv[h][tb] = __builtin_bit_cast(uint2, *reinterpret_cast<const __attribute__((address_space(3))) u32x2*>(
              R == 32 ? (rdC ^ (32 * h)) + stage + tb * 1024 : rdC + stage + tb * 512));
#pragma unroll
      for (int h = 0; h < R / 16; ++h)
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
          const uint32_t p = rdW + stage + ((i ^ sw) * 32) + h * (16 * SC * 2);
          av[h][i] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<__attribute__((address_space(3))) short4_t*>(p)));
        }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // it is in registers: its stage takes the next loads
      fetch();
#pragma unroll
      for (int h = 0; h < R / 16; ++h)
#pragma unroll
        for (int i = 0; i < kGroups; ++i)
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) acc[tb][i] = mfma16<T>(av[h][i], bv[h][tb], acc[tb][i]);
      stage = stage == (Sh::kStages - 1) * kStage ? 0 : stage + kStage;
    }
    if constexpr (NW < kMRuns) {
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
          run_sum[tb][i] += acc[tb][i];
          acc[tb][i] = float4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
  }
  // every load has landed and every wave has left its ring: the LDS is free for the sums
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  LAROSA_STAMP(1);

  float* sums = reinterpret_cast<float*>(lds);                         // [run % 4][token][kPitch]
  float* scale_s = sums + 4 * kTokens * kPitch;                        // [token]
  int* s_last = reinterpret_cast<int*>(scale_s + kTokens);
  // D element e of product i in lane (grp16, j) is column 16 i + 4 grp16 + e of token j
#pragma unroll
  for (int half = 0; half < NW / 4; ++half) {
    if ((rw >> 2) == half) {
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
          float4_t* q = reinterpret_cast<float4_t*>(sums + ((rw & 3) * kTokens + tb * 16 + j) * kPitch + 16 * i + 4 * grp16);
          const float4_t v = NW < kMRuns ? run_sum[tb][i] : acc[tb][i];
          *q = half == 0 ? v : *q + v;
        }
    }
    if (half + 1 < NW / 4) __syncthreads();
  }
  const int n_s = SC == kBatchStrip ? ge.g_last - ge.g_first + 1 : 1;   // workgroups of the strip; wide strips have one (plan_batched)
  if (n_s == 1) token_scales<T, NW>(a, b0, kTokens, scale_s, lane, rw);
  __syncthreads();
  // a thread owns pieces tid + kThreads p: columns 4 (piece % (SC / 4)) .. + 3 of token piece / (SC / 4)
  constexpr int kPieces = kTokens * (SC / 4) / kThreads;
  constexpr int kPass = kPieces < 8 ? kPieces : 8;                     // pieces a finisher holds at a time
  auto wave_sum_of = [&](int piece) __attribute__((always_inline)) {   // the four pairs of runs, in order
    const float* q = sums + piece / (SC / 4) * kPitch + piece % (SC / 4) * 4;
    float4_t v = *reinterpret_cast<const float4_t*>(q);
#pragma unroll
    for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const float4_t*>(q + w * kTokens * kPitch);
    return v;
  };
  auto store_piece = [&](int piece, const float4_t& v) __attribute__((always_inline)) {
    const int tok = piece / (SC / 4), col = s * SC + piece % (SC / 4) * 4;
    if (b0 + tok < a.B && col < d_out) store_out4<T>(a, b0 + tok, col, v, scale_s[tok]);
  };
  if (n_s == 1) {
#pragma unroll
    for (int p = 0; p < kPieces; ++p) store_piece(tid + p * kThreads, wave_sum_of(tid + p * kThreads));
    LAROSA_STAMP(5);
    return;
  }

  // every partial of this strip as one buffer: slot of workgroup w at byte w * slot bytes, piece i of it at 16 i; 16-byte
  // accesses with the sc1 cache policy are coherent across the chip, see gemv_core.hpp
  constexpr int kSlotBytes = kTokens * SC * 4;
  constexpr int kCoherent = 16;
  unsigned* ctr = a.counters + (static_cast<size_t>(grp) * a.nstrips + s) * kCounterStride;
  const __amdgpu_buffer_rsrc_t slots = __builtin_amdgcn_make_buffer_rsrc(
      a.partial + (static_cast<size_t>(grp) * a.G + ge.g_first) * (kTokens * SC), 0, n_s * kSlotBytes, 0x00027000);
  const int mine = (g - ge.g_first) * kSlotBytes;
#pragma unroll
  for (int p = 0; p < kPieces; ++p)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, wave_sum_of(tid + p * kThreads)), slots,
                                           mine + (tid + p * kThreads) * 16, 0, kCoherent);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  LAROSA_STAMP(2);
  if (tid == 0) {
    const unsigned old = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_last = (old == static_cast<unsigned>(n_s - 1)) ? 1 : 0;
  }
  __syncthreads();
  LAROSA_STAMP(3);
  if (*s_last == 0) {                            // uniform over the workgroup
    LAROSA_STAMP(5);
    return;
  }
  if (tid == 0) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  token_scales<T, NW>(a, b0, kTokens, scale_s, lane, rw);
  __syncthreads();
  // the thread's pieces of every partial, added in workgroup order
  constexpr int kAhead = 16 / kPass;             // partials in flight
  for (int p0 = 0; p0 < kPieces; p0 += kPass) {
    float4_t sm[kPass];
#pragma unroll
    for (int p = 0; p < kPass; ++p) sm[p] = float4_t{0.f, 0.f, 0.f, 0.f};
    for (int w = 0; w < n_s; w += kAhead) {
      u32x4 v[kAhead][kPass];
#pragma unroll
      for (int q = 0; q < kAhead; ++q)
        if (w + q < n_s) {                       // uniform over the workgroup: no partial is read twice
#pragma unroll
          for (int p = 0; p < kPass; ++p)
            v[q][p] = __builtin_amdgcn_raw_buffer_load_b128(slots, (w + q) * kSlotBytes + (tid + (p0 + p) * kThreads) * 16, 0, kCoherent);
        }
#pragma unroll
      for (int q = 0; q < kAhead; ++q)
        if (w + q < n_s) {
#pragma unroll
          for (int p = 0; p < kPass; ++p) sm[p] += __builtin_bit_cast(float4_t, v[q][p]);
        }
    }
#pragma unroll
    for (int p = 0; p < kPass; ++p) store_piece(tid + (p0 + p) * kThreads, sm[p]);
  }
  LAROSA_STAMP(5);
}


// One launch, up to two independent products: workgroups [0, side_G) of the grid run the side product
// (a residual adapter on a block's shortcut, which needs only the block's input), the others the main
// one.  Both use the same token grouping (blockIdx.y).
template <typename T>
__global__ __launch_bounds__(k16Waves * 64) void skinny16_kernel(BatchPair p) {
  const int g = blockIdx.x;
  const bool side = g < p.side_G;                       // uniform over the workgroup
  skinny16_body<T>(side ? p.side : p.main, side ? g : g - p.side_G, blockIdx.y);
}

// NW = 4 waves of tiles of 32 rows, or 8 of 16 rows (launch_batched_t).  The four waves' two sets of sums take more than
// the 256 registers that a second wave per SIMD would leave; the LDS holds one workgroup per compute unit anyway.
template <typename T, int NW>
__global__ __launch_bounds__(NW * 64, NW == 4 ? 1 : 2) void skinny32_kernel(BatchPair p) {
  constexpr int R = NW == 4 ? 32 : 16;
  const int g = blockIdx.x;
  const bool side = g < p.side_G;
  const BatchArgs& a = side ? p.side : p.main;
  const int own = side ? g : g - p.side_G;
  if (a.strip_cols == 256) skinny32_body<T, 256, NW, R>(a, own, blockIdx.y);
  else skinny32_body<T, 128, NW, R>(a, own, blockIdx.y);
}

}  // namespace
bool batched_uses_mfma(int B, bool coef_scale);
namespace {

template <typename T>
hipError_t launch_batched_t(const BatchPair& p, hipStream_t st) {
  const BatchArgs& a = p.main;
  const dim3 block(kBThreads);
  if (!batched_uses_mfma(a.B, a.coef_scale != nullptr)) {
    if (p.side_G > 0) return hipErrorInvalidValue;   // the FMA kernel carries no side product
    // (a per-channel coefficient scale is applied in fp32, which only the FMA kernel does)
    if (a.B <= 2) {
      hipLaunchKernelGGL((skinny_fma_kernel<T, 2>), dim3(a.G, (a.B + 1) / 2), block, 0, st, a);
    } else {
      hipLaunchKernelGGL((skinny_fma_kernel<T, 4>), dim3(a.G, (a.B + 3) / 4), block, 0, st, a);
    }
  } else if (a.group_tokens <= 16) {
    hipLaunchKernelGGL((skinny16_kernel<T>), dim3(a.G + p.side_G, (a.B + 15) / 16), dim3(k16Waves * 64), 0, st, p);
  } else {
    const dim3 grid(a.G + p.side_G, (a.B + kMTokens - 1) / kMTokens);
    // rows of a workgroup at which four waves, with twice the tile, overtake eight, whose runs stay even when there are few
    // tiles (32 tokens, eight / four waves: 4096 x 4096 (512 rows each) 14.0 / 14.7 us, 4096 x 8192 (1024) 18.9 / 19.0,
    // 11008 x 4096 (1376) 24.0 / 23.9, 14336 x 4096 (1792) 28.6 / 27.7, 4096 x 12288 (2048) 29.4 / 26.7, 4096 x 22016
    // (4096) 47.3 / 42.7; in strips of 256: 600 x 48720 19.1 / 20.2, 8192 x 57344 168 / 149)
    if (a.chunk <= 1024) hipLaunchKernelGGL((skinny32_kernel<T, 8>), grid, dim3(512), kMLds, st, p);
    else hipLaunchKernelGGL((skinny32_kernel<T, 4>), grid, dim3(256), kMLds, st, p);
  }
  return hipGetLastError();
}

}  // namespace

bool batched_uses_mfma(int B, bool coef_scale) { return B >= 2 && !coef_scale; }

int batched_g_total() { return tuning().g_target > 0 ? tuning().g_target : 256; }

int batched_tokens_per_group(int B, bool coef_scale, int d_in, int d_out) {
  if (!batched_uses_mfma(B, coef_scale)) return B <= 2 ? 2 : 4;
  // 17 .. 32 tokens on a small weight: reading it twice, out of the caches, costs less than the larger hand-off of a group
  // of 32.  Measured from 0.5 to 15 M values, tall and flat (two groups of 16 / one of 32, 32 tokens): 1024 x 1024 11.8 /
  // 14.6 us, 8192 x 512 15.1 / 20.1, 512 x 8192 8.6 / 9.4, 2560 x 2560 11.0 / 12.4, 2048 x 4096 11.5 / 12.5, 8192 x 1024
  // 14.3 / 16.5, 1024 x 8192 10.7 / 10.9 (512 x 16384, the flattest, 10.5 / 10.2); level at 9.4 M (3072 x 3072 13.3 / 13.0);
  // then 2560 x 4096 13.7 / 13.1, 2048 x 5632 14.8 / 12.0, 1024 x 11008 14.7 / 11.6.  A side product shares the
  // main one's launch and with it the size of its groups.
  const bool small = B <= 32 && d_out <= 32768 && static_cast<long>(d_in) * d_out <= 8L << 20;
  // groups of 32 address their coefficients with 32-bit byte offsets: below 2 GiB a group
  return B <= 16 || small || d_in >= 1 << 25 ? 16 : 32;
}

GemvPlan plan_batched(int d_in, int d_out, bool mfma, int g_hint, bool many) {
  GemvPlan p;
  p.strip_cols = kBatchStrip;
  p.nstrips = (d_out + p.strip_cols - 1) / p.strip_cols;
  // one workgroup per compute unit: each strip gets the same number of workgroups, each of those an equal run
  // of whole 16-row tiles (keeps row starts 8-aligned), so a workgroup never works on two strips
  long G = g_hint > 0 ? g_hint : batched_g_total();
  long wps = G / p.nstrips;
  if (wps < 1) wps = 1;
  long chunk = (d_in + wps - 1) / wps;
  chunk = (chunk + 15) / 16 * 16;
  if (!mfma && chunk > kBatchChunkMax) chunk = kBatchChunkMax;   // LDS staging of the coefficients
  wps = (d_in + chunk - 1) / chunk;
  p.chunk = static_cast<int>(chunk);
  p.wps = static_cast<int>(wps);
  p.G = static_cast<int>(p.nstrips * wps);
  p.partial_floats = static_cast<size_t>(p.G) * p.strip_cols;  // per token
  // 512 contiguous bytes per row instead of 256 stream faster (8192 x 57344, 32 tokens: 149 against 168 us), but where the
  // narrow strips fill the chip once, wide ones need a hand-off that those do not (512 x 22016: 13.5 against 10 us): wide
  // from more than one narrow strip per compute unit on, one workgroup each, so without a hand-off (and without the
  // counters and partial sums that the narrow plan provides)
  if (mfma && many && wps == 1 && p.nstrips > 256) {
    p.strip_cols = 256;
    p.nstrips = (d_out + 255) / 256;
    p.G = p.nstrips;
  }
  return p;
}

hipError_t launch_batch_prep(const uint16_t* h, const int32_t* idx, uint16_t* C, int B, int d_in, int K, hipStream_t s) {
  const long passes = (static_cast<long>(d_in) + kPrepPass - 1) / kPrepPass;
  const long even = (passes + kPrepSlices - 1) / kPrepSlices * kPrepPass;
  const int slice = even < kPrepSliceMax ? static_cast<int>(even) : kPrepSliceMax;
  const unsigned slices = static_cast<unsigned>((static_cast<long>(d_in) + slice - 1) / slice);
  if (slice == kPrepPass) hipLaunchKernelGGL(batch_prep_kernel<true>, dim3(slices, B), dim3(kPrepThreads), 0, s, h, idx, C, d_in, K, slice);
  else hipLaunchKernelGGL(batch_prep_kernel<false>, dim3(slices, B), dim3(kPrepThreads), slice, s, h, idx, C, d_in, K, slice);
  return hipGetLastError();
}

hipError_t launch_batched(const BatchArgs& a, bool bf16, hipStream_t s) {
  BatchPair p{};
  p.main = a;
  return bf16 ? launch_batched_t<BF16>(p, s) : launch_batched_t<F16>(p, s);
}

hipError_t launch_batched_pair(const BatchPair& p, bool bf16, hipStream_t s) {
  return bf16 ? launch_batched_t<BF16>(p, s) : launch_batched_t<F16>(p, s);
}

}  // namespace larosa
