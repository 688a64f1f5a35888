// Stand-alone Top-K sparsifier kernel (Sec. 4.3, Eq. 8): one workgroup of 2, 8 or 16 waves per token;
// the selection itself is in topk_core.hpp.
#include <type_traits>

#include "kernels.hpp"
#include "topk_core.hpp"

namespace larosa {

namespace {

constexpr int kTopkThreads = 1024;        // (threshold kernel)
constexpr int kTopkWaves = kTopkThreads / 64;

// Copies of pass 1's histogram: 32 where the workgroup can sum them by itself (topk_core.hpp), else 8.
template <int NW> constexpr int kTopkKernelCopies = NW % 4 == 0 ? kTopkCopiesWide : kTopkCopies;

// One workgroup of NW waves per token, E elements per lane (a multiple of 4).
// Where the selected vector comes from (batched decoder layer): the plain vector, the context-length-1
// attention output read straight from q|k|v (value head of the query head's group), or
// R(SiLU(gate) * up) computed from gate|up.  The vector itself can be written out as well.
// VALS: the kept values are written beside the index list.
// RUN: the sum of squares of kSrcNorm is formed from the squares of runs of RUN elements, 64 runs by halves, the sums of
// 64 runs one after the other -- whatever NW is, so that the choice of NW changes no bit.
template <typename T, int NW, int E, int RUN, bool VALS>
__global__ __launch_bounds__(NW * 64) void topk_kernel(const uint16_t* __restrict__ h, int d, int K,
                                                       int32_t* __restrict__ idx,
                                                       uint16_t* __restrict__ vals,
                                                       uint16_t* __restrict__ masked, TopkSource sc) {
  __shared__ TopkShared<NW, kTopkKernelCopies<NW>> sm;
  const int b = blockIdx.x;
  const uint16_t* hb = h + static_cast<size_t>(b) * d;
  const int base = threadIdx.x * E;

  LAROSA_STAMP(0);
  topk_clear<NW>(sm);                     // made visible by the first barrier below
  // All of the lane's loads are issued first, unconditionally and from addresses clamped into the
  // vector (d % 4 == 0: a group of four is all valid or all past the end; groups past the end re-read
  // the last group and are ignored).  Loads under a lane or mode condition sit in branches of their
  // own, and each is then waited for before the next is issued: one memory round trip per group.
  uint2 ld0[E / 4], ld1[E / 4];
  if (sc.mode == kSrcGqa) {
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      const int i = min(base + q * 4, d - 4);
      const int head = quotient_by(i, sc.head_magic);
      const int src = quotient_by(head, sc.group_magic) * sc.head_dim + (i - head * sc.head_dim);
      ld0[q] = *reinterpret_cast<const uint2*>(sc.src + static_cast<size_t>(b) * (sc.d_q + 2 * sc.d_kv) + sc.d_q +
                                               sc.d_kv + src);
      ld1[q] = make_uint2(0u, 0u);
    }
  } else if (sc.mode == kSrcSilu) {
    const uint16_t* gb = sc.src + static_cast<size_t>(b) * 2 * d;
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      const int i = min(base + q * 4, d - 4);
      ld0[q] = *reinterpret_cast<const uint2*>(gb + i);
      ld1[q] = *reinterpret_cast<const uint2*>(gb + d + i);
    }
  } else {
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      ld0[q] = *reinterpret_cast<const uint2*>(hb + min(base + q * 4, d - 4));
      ld1[q] = make_uint2(0u, 0u);
    }
  }
  uint32_t raw[E / 2];                    // the lane's elements as stored, two to a register (zeros past the end)
#pragma unroll
  for (int q = 0; q < E / 4; ++q) {
    const int i = base + q * 4;
    uint2 v = ld0[q];
    if (sc.mode == kSrcSilu) {
      float g[4], u[4], o[4];
      T::unpack2(ld0[q].x, g[0], g[1]);
      T::unpack2(ld0[q].y, g[2], g[3]);
      T::unpack2(ld1[q].x, u[0], u[1]);
      T::unpack2(ld1[q].y, u[2], u[3]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        o[k] = silu_f32(g[k]) * u[k];
        // rounded to fp32 before the storage rounding; left to itself the compiler does both in one for some sizes and not
        // for others, and a batched layer's bits would change with the width (above 16384 it always has done both in one)
        if constexpr (RUN <= 16) asm("" : "+v"(o[k]));
      }
      v = pack4<T>(o);
    }
    if (i >= d) v = make_uint2(0u, 0u);
    if (i < d && sc.h_out && sc.mode != kSrcNorm) *reinterpret_cast<uint2*>(sc.h_out + static_cast<size_t>(b) * d + i) = v;
    raw[2 * q] = v.x;
    raw[2 * q + 1] = v.y;
  }
  if (sc.mode == kSrcNorm) {
    // h = R(x * rsqrt(mean(x^2) + eps) * scale): the pre-norm of a block whose rotation is absorbed
    // the lane's slice of the learned scale, fetched up front (loads at each use would each wait for memory)
    uint2 sc2[E / 4];
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      const int i = base + q * 4;
      sc2[q] = (sc.norm_scale && i < d) ? *reinterpret_cast<const uint2*>(sc.norm_scale + i) : make_uint2(0u, 0u);
    }
    constexpr int kRuns = E / RUN;        // runs per lane; 64 / kRuns lanes hold 64 of them
    static_assert(E % RUN == 0 && (kRuns == 1 || kRuns == 2 || kRuns == 4), "lane exchanges of kRuns runs");
    __shared__ float tot_w[NW * kRuns];
    float ss[kRuns];
#pragma unroll
    for (int k = 0; k < kRuns; ++k) {
      ss[k] = 0.f;
#pragma unroll
      for (int q = k * (RUN / 2); q < (k + 1) * (RUN / 2); ++q) {
        float x0, x1;
        T::unpack2(raw[q], x0, x1);
        ss[k] = fmaf(x0, x0, ss[k]);
        ss[k] = fmaf(x1, x1, ss[k]);
      }
      ss[k] = lanes_sum<64 / kRuns>(ss[k]);
    }
#pragma unroll
    for (int o = kRuns / 2; o > 0; o >>= 1)
#pragma unroll
      for (int k = 0; k < o; ++k) ss[k] += ss[k + o];
    if ((threadIdx.x & (64 / kRuns - 1)) == 0) tot_w[threadIdx.x / (64 / kRuns)] = ss[0];
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < NW * kRuns; ++w2) tot += tot_w[w2];
    const float rinv = 1.0f / sqrtf(tot / static_cast<float>(d) + sc.norm_eps);
#pragma unroll
    for (int q = 0; q < E / 2; ++q) {
      float x0, x1;
      T::unpack2(raw[q], x0, x1);
      x0 *= rinv;
      x1 *= rinv;
      if (sc.norm_scale) {
        float s0, s1;
        T::unpack2((q & 1) ? sc2[q >> 1].y : sc2[q >> 1].x, s0, s1);
        x0 *= s0;
        x1 *= s1;
      }
      raw[q] = base + 2 * q < d ? T::from_f32(x0) | (static_cast<uint32_t>(T::from_f32(x1)) << 16) : 0u;   // past the end: zeros
    }
    if (sc.h_out) {
#pragma unroll
      for (int q = 0; q < E / 4; ++q) {
        const int i = base + q * 4;
        if (i < d) *reinterpret_cast<uint2*>(sc.h_out + static_cast<size_t>(b) * d + i) = make_uint2(raw[2 * q], raw[2 * q + 1]);
      }
    }
  }
  if (sc.mode != kSrcNorm) __syncthreads();
  LAROSA_STAMP(1);
  uint32_t key[E / 2];
#pragma unroll
  for (int q = 0; q < E / 2; ++q) key[q] = raw[q] & kPairKeys;
  const auto st = block_select<NW, E>(key, K, sm);
  LAROSA_STAMP(2);

  // The index list goes through LDS, so that memory sees whole lines: written from the lanes that hold the elements, a wave's
  // stores touch a line per lane or two (14336 wide, 8601 kept: whole kernel 8.4 -> 7.0 us, 28672: 16.2 -> 11.3).  Values (VALS) are stored
  // from the lanes in the same loop, ahead of the barrier, and a kernel without them holds no code for them (in a loop of their own
  // after the list they cost 4104 wide 5.1 -> 5.4 us, now 4.95; 28672 21.9 -> 17.0, now 14.3).
  if (idx) {
    __shared__ uint16_t list[NW * 64 * E];
    uint16_t* valb = VALS ? vals + static_cast<size_t>(b) * K : nullptr;
    unsigned pos = st.first;
#pragma unroll
    for (int q = 0; q < E; ++q) {
      if (kept_bit(st, q)) {
        if constexpr (VALS) valb[pos] = static_cast<uint16_t>(raw[q >> 1] >> (16 * (q & 1)));
        list[pos++] = static_cast<uint16_t>(base + q);
      }
    }
    __syncthreads();
    int32_t* idxb = idx + static_cast<size_t>(b) * K;
    for (int i = threadIdx.x; i < K; i += NW * 64) idxb[i] = list[i];
  }
  LAROSA_STAMP(3);
  if (masked) {
    uint16_t* mb = masked + static_cast<size_t>(b) * d;
    // bits 15 and 31 spread over their halves
    auto mask = [](uint32_t signs) __attribute__((always_inline)) { return ((signs >> 15) & 1u) * 0xFFFFu | (signs >> 31) * 0xFFFF0000u; };
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      const int i = base + q * 4;
      if (i < d)
        *reinterpret_cast<uint2*>(mb + i) = make_uint2(raw[2 * q] & mask(st.kept[2 * q]), raw[2 * q + 1] & mask(st.kept[2 * q + 1]));
    }
  }
  LAROSA_STAMP(4);
}

// Magnitude-threshold sparsifier (Eq. 4-5), the comparison method with a data-dependent kept count:
// lane t owns elements [tE, (t+1)E); kept positions come from a block prefix sum of the lanes' counts.
template <typename T, int E>
__global__ __launch_bounds__(kTopkThreads) void threshold_kernel(const uint16_t* __restrict__ h, int d, float eps,
                                                                 int32_t* __restrict__ idx,
                                                                 int32_t* __restrict__ count) {
  __shared__ unsigned wave_total[kTopkWaves];
  const int b = blockIdx.x;
  const uint16_t* hb = h + static_cast<size_t>(b) * d;
  const int base = threadIdx.x * E;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  unsigned keep = 0;     // bit q: element base + q is kept
  unsigned n = 0;
#pragma unroll
  for (int q = 0; q < E / 4; ++q) {
    const int i = base + q * 4;
    if (i < d) {
      const uint2 v = *reinterpret_cast<const uint2*>(hb + i);
      const uint16_t r[4] = {static_cast<uint16_t>(v.x & 0xFFFFu), static_cast<uint16_t>(v.x >> 16),
                             static_cast<uint16_t>(v.y & 0xFFFFu), static_cast<uint16_t>(v.y >> 16)};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (T::to_f32(r[k] & 0x7FFFu) > eps) {
          keep |= 1u << (q * 4 + k);
          n += 1;
        }
      }
    }
  }
  const unsigned incl = wave_scan_inclusive(n, lane);
  if (lane == 63) wave_total[wv] = incl;
  __syncthreads();
  unsigned before = incl - n, total = 0;
#pragma unroll
  for (int w2 = 0; w2 < kTopkWaves; ++w2) {
    const unsigned tw = wave_total[w2];
    if (w2 < wv) before += tw;
    total += tw;
  }
  int32_t* idxb = idx + static_cast<size_t>(b) * d;
#pragma unroll
  for (int q = 0; q < E; ++q) {
    if (keep & (1u << q)) idxb[before++] = base + q;
  }
  if (threadIdx.x == 0) count[b] = static_cast<int32_t>(total);
}

template <typename T>
hipError_t launch_threshold_t(const uint16_t* h, int B, int d, float eps, int32_t* idx, int32_t* count, hipStream_t s) {
  dim3 grid(B), block(kTopkThreads);
  const int e = (d + kTopkThreads - 1) / kTopkThreads;
  if (e <= 4)
    hipLaunchKernelGGL((threshold_kernel<T, 4>), grid, block, 0, s, h, d, eps, idx, count);
  else if (e <= 8)
    hipLaunchKernelGGL((threshold_kernel<T, 8>), grid, block, 0, s, h, d, eps, idx, count);
  else if (e <= 16)
    hipLaunchKernelGGL((threshold_kernel<T, 16>), grid, block, 0, s, h, d, eps, idx, count);
  else if (e <= 32)
    hipLaunchKernelGGL((threshold_kernel<T, 32>), grid, block, 0, s, h, d, eps, idx, count);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_threshold_select(const uint16_t* h, int B, int d, float eps, int32_t* idx, int32_t* count, bool bf16,
                                   hipStream_t s) {
  return bf16 ? launch_threshold_t<BF16>(h, B, d, eps, idx, count, s) : launch_threshold_t<F16>(h, B, d, eps, idx, count, s);
}

// Waves and elements per lane by width: what a wave executes is mostly fixed, and two waves or more share a SIMD, so narrow vectors
// take few waves; but element by element a wave is slower than two.  Whole kernel, us, one token, f16 (with index list):
// 512 wide 2 waves 2.8, 1 wave 3.1 (16: 4.1); 1024: 2 waves 3.2, 4 waves 3.3; 2048: 8 waves 3.4, 4 waves 3.6; 4096: 8 waves
// 4.0, 4 waves 4.6, 16 waves 4.3; 8192: 16 waves 5.2, 8 waves 5.9 (before the index list went through LDS);
// 14336: 16 waves 7.1, 8 waves 9.6 (likewise).  With 16 waves at every width and the index list written directly:
// 4.1 (512) 4.5 (4096) 5.5 (8192) 8.7 (14336) 16.4 (28672, now 11.5).
template <typename T>
hipError_t launch_topk_t(const uint16_t* h, int B, int d, int K, int32_t* idx, uint16_t* vals, uint16_t* masked,
                         TopkSource sc, hipStream_t s) {
  sc.head_magic = quotient_magic(sc.head_dim);
  sc.group_magic = quotient_magic(sc.group);
  auto launch = [&](auto nw, auto e, auto run) {
    constexpr int NW = decltype(nw)::value, E = decltype(e)::value, RUN = decltype(run)::value;
    if constexpr (std::is_same_v<T, F16>) {      // (values are asked for through launch_topk alone, with the index list)
      if (vals) {
        hipLaunchKernelGGL((topk_kernel<T, NW, E, RUN, true>), dim3(B), dim3(64 * NW), 0, s, h, d, K, idx, vals, masked, sc);
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((topk_kernel<T, NW, E, RUN, false>), dim3(B), dim3(64 * NW), 0, s, h, d, K, idx, nullptr, masked, sc);
    return hipGetLastError();
  };
#define LAROSA_TOPK(NW, E, RUN) launch(std::integral_constant<int, NW>{}, std::integral_constant<int, E>{}, std::integral_constant<int, RUN>{})
  if (d <= 512) return LAROSA_TOPK(2, 4, 4);
  if (d <= 1024) return LAROSA_TOPK(2, 8, 4);
  if (d <= 2048) return LAROSA_TOPK(8, 4, 4);
  if (d <= 4096) return LAROSA_TOPK(8, 8, 4);
  if (d <= 8192) return LAROSA_TOPK(16, 8, 8);
  if (d <= 16384) return LAROSA_TOPK(16, 16, 16);
  if (d <= 24576) return LAROSA_TOPK(16, 24, 24);
  if (d <= 32768) return LAROSA_TOPK(16, 32, 32);
#undef LAROSA_TOPK
  return hipErrorInvalidValue;
}

hipError_t launch_topk(const uint16_t* h, int B, int d, int K, int32_t* idx, uint16_t* vals, uint16_t* masked,
                       hipStream_t s) {
  TopkSource sc{};
  sc.mode = kSrcPlain;
  return launch_topk_t<F16>(h, B, d, K, idx, vals, masked, sc, s);   // the type matters for kSrcSilu only
}

hipError_t launch_topk_from(const TopkSource& sc, int B, int d, int K, int32_t* idx, uint16_t* masked, bool bf16,
                            hipStream_t s) {
  return bf16 ? launch_topk_t<BF16>(sc.src, B, d, K, idx, nullptr, masked, sc, s)
              : launch_topk_t<F16>(sc.src, B, d, K, idx, nullptr, masked, sc, s);
}

}  // namespace larosa
