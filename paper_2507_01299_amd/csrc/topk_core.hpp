// Workgroup-level radix select for the Top-K sparsifier S_k (Sec. 4.3, Eq. 8), shared by the
// stand-alone Top-K kernel and the Top-K prologue of the fused projection kernel.
//
// The ordering key is the stored 16-bit pattern with the sign cleared (15 bits, unsigned), so
// the selection is pure integer work and identical for binary16 and bfloat16.  Lane t owns the
// contiguous elements [t*E, (t+1)*E) and keeps them in registers through all phases:
//   1. 256-bin histogram of the top 8 key bits.  Activations crowd into a few of these bins (for
//      bfloat16 the 8 bits are the exponent alone), and lanes of one wave that add to the same LDS
//      word are served one per clock; so there are kTopkCopies histograms (in different banks for one
//      bin) and a lane adds to copy (lane mod kTopkCopies): at most 64 / kTopkCopies lanes meet in a
//      word whatever the data.  After a barrier wave 0 sums the copies and walks the bins from the top
//      (suffix sums on the data-parallel path); a second barrier publishes the bin holding the K-th largest key;
//   2. 128-bin histogram of the low 7 bits inside that bin, one copy PER WAVE.  After one more barrier
//      every wave reads all copies: their sum gives the threshold key T and r = K - #{key > T}, the
//      number of threshold ties to keep, and the copies of the waves before it give the number of
//      kept elements of that bin in front of the wave -- the block prefix needs no barrier of its own.
//      (The counts of elements in higher bins travel as one total per wave with the same barrier.)
//   3. a wave-level prefix sum of the ">T" and "==T" counts then gives every lane the number of kept
//      elements before its own, so an index-ordered compaction keeps every key > T and the first
//      r keys == T: ascending indices and the lower-index tie rule with no sort.
// Three barriers in all, four with kTopkCopiesWide (after the one that makes the cleared histograms and the vector visible).
//
// What bounds it: the instructions each wave executes one after the other (about 3 ns each with two waves per SIMD, whatever
// they are), not LDS or memory.  So the keys are worked on in pairs, two to a register (packed 16-bit subtractions; the keys
// have 15 bits, so a difference's sign is the comparison), counts come from bit counts of the signs, and nothing per element
// is branched on: what does not count goes to a word that nobody reads.  (Select and row list of a batch-1 projection, 4096
// wide, 512 lanes: 3.4 -> 2.8 us in the phase clocks; LLaMA2-7B layer 75.3 -> 74.5 us, with the batch kernels 152.3 -> 147.8
// for 32 tokens.)
#pragma once
#include <cstddef>

#include "kernels.hpp"
#include "numeric.hpp"

namespace larosa {

constexpr int kTopkCopies = 8;
// Pass 1's 256 bins times kTopkCopies are 8 KiB to read: one wave walks them and hands the bin on through
// LDS (one more barrier); every wave doing it by itself measured slower with two workgroups per compute unit.
constexpr int kTopkCopyStride = 260;   // words between copies: 16-byte aligned, and the copies of one bin fall in different LDS banks
constexpr int kTopkCopyStride2 = 132;  // the same for the 128-bin pass (one copy per wave)

// A workgroup that selects for a wide vector, or for bfloat16 (whose top 8 key bits are the exponent alone,
// so nearly every lane of a wave adds to the same few bins), is bound by those same-word additions: with
// kTopkCopiesWide copies (lane mod 32 picks the copy; stride 1 mod 32, so the 32 copies of one bin lie
// in 32 different banks) at most two lanes of a wave ever meet in a word.  The copies are then summed by
// the whole workgroup (one more barrier) before wave 0 walks the bins.
constexpr int kTopkCopiesWide = 32;
constexpr int kTopkCopyStrideWide = 257;
// words of the pass-1 histograms, padded to a multiple of 4 (they are cleared in 16-byte pieces)
template <int C> struct TopkHist1 { static constexpr int words = kTopkCopyStride * C; static constexpr int stride = kTopkCopyStride; };
template <> struct TopkHist1<kTopkCopiesWide> {
  static constexpr int words = (kTopkCopyStrideWide * kTopkCopiesWide + 3) / 4 * 4;
  static constexpr int stride = kTopkCopyStrideWide;
};

template <int NW, int C = kTopkCopies>
struct TopkShared {
  alignas(16) unsigned hist[TopkHist1<C>::words];             // pass 1: word copy * stride + bin
  unsigned hist2[kTopkCopyStride2 * NW];                      // pass 2: word wave * kTopkCopyStride2 + bin (adjacent: cleared in one step)
  alignas(16) unsigned part[C == kTopkCopiesWide ? 256 * (NW / 4) : 4];   // wide copies: sums over NW/4 groups of copies
  unsigned unread[64];                                        // pass 2's additions of elements outside the bin
  unsigned wave_tot[NW];                                      // per wave: elements in bins above the threshold bin
  int bin;                                                    // pass-1 bin holding the K-th largest key, and the
  unsigned above;                                             // count strictly above it (written by wave 0)
};

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kPairSigns = 0x80008000u;   // the sign bits of a pair
constexpr uint32_t kPairKeys = 0x7FFF7FFFu;

__device__ __forceinline__ unsigned popcount32(uint32_t v) { return static_cast<unsigned>(__popc(v)); }
__device__ __forceinline__ uint32_t pair_of(unsigned key) { return key | (key << 16); }
// per half: bit 15 set if the half of b (15 bits) is the larger one; zero if they are equal
__device__ __forceinline__ uint32_t pair_sub(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, static_cast<u16x2>(__builtin_bit_cast(u16x2, a) - __builtin_bit_cast(u16x2, b)));
}
// per half: 1 unless it is zero
__device__ __forceinline__ uint32_t pair_nonzero(uint32_t a) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), u16x2{1, 1}));
}

// Selection state of one lane after block_select.
template <int E>
struct TopkLane {
  unsigned first;          // rank of the lane's first kept element in the ascending kept list
  unsigned n;              // its kept elements
  uint32_t kept[E / 2];    // pair q: bit 15 (element 2 q) and bit 31 (element 2 q + 1) set if it is kept
};

// Zero both histograms; every lane of the workgroup calls it.  No barrier: the caller's next barrier
// (it usually has one of its own while it builds the vector) makes the zeros visible.
template <int NW, int C>
__device__ __forceinline__ void topk_clear(TopkShared<NW, C>& sm) {
  constexpr int kWords = TopkHist1<C>::words + kTopkCopyStride2 * NW;   // hist and hist2 are adjacent
  typedef TopkShared<NW, C> Sh;
  static_assert(offsetof(Sh, hist2) == sizeof(unsigned) * TopkHist1<C>::words, "histograms must be adjacent");
  static_assert(offsetof(Sh, hist) % 16 == 0 && kWords % 4 == 0, "cleared and read in 16-byte pieces");
  uint4* flat = reinterpret_cast<uint4*>(sm.hist);
  for (int i = threadIdx.x; i < kWords / 4; i += NW * 64) flat[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Sum over the 64 lanes, the same value in every lane (and known to be uniform).
__device__ __forceinline__ unsigned wave_total(unsigned v, int lane) {
  return static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(wave_scan_inclusive(v, lane)), 63));
}

// key[q]: this lane's elements 2 q (low half) and 2 q + 1 with their signs cleared; positions past the end of the vector
// MUST hold zero.
// Such padding is counted like a zero at an index above every real element: it is never above the
// threshold, and among threshold ties the lower-index rule takes the real elements first (K is at most
// their number), so it is never kept -- and the passes over the elements need no per-element predicate.
// Every lane of the NW-wave workgroup must call this, after topk_clear and a workgroup barrier.
// 1 <= K <= total number of valid elements <= 32768.
template <int NW, int E, int C>
__device__ __forceinline__ TopkLane<E> block_select(const uint32_t (&key)[E / 2], int K, TopkShared<NW, C>& sm) {
  constexpr bool kWide = C == kTopkCopiesWide;
  static_assert(!kWide || (NW % 4 == 0 && 32 % (NW / 4) == 0), "the copies are summed by NW/4 groups of 256 lanes");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- pass 1: top 8 key bits
  unsigned* mine = sm.hist + (static_cast<unsigned>(lane) & (C - 1)) * TopkHist1<C>::stride;
#pragma unroll
  for (int q = 0; q < E / 2; ++q) {
    atomicAdd(&mine[(key[q] >> 7) & 255u], 1u);
    atomicAdd(&mine[key[q] >> 23], 1u);
  }
  __syncthreads();
  if constexpr (kWide) {
    // lane group g = tid / 256 sums its 32 / (NW/4) copies of bin tid % 256 (consecutive lanes, consecutive banks)
    constexpr int kGroups = NW / 4, kPer = kTopkCopiesWide / kGroups;
    const int bin = tid & 255, grp = tid >> 8;
    unsigned sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) sum += sm.hist[(grp * kPer + k) * kTopkCopyStrideWide + bin];
    sm.part[grp * 256 + bin] = sum;
    __syncthreads();
  }
  if (wave == 0) {
    // lane covers 4 bins counted from the top: position p = 4*lane + q is bin 255 - p; its four
    // counts of one copy are one aligned 16-byte read
    unsigned c[4] = {0u, 0u, 0u, 0u};
    if constexpr (kWide) {
#pragma unroll
      for (int k = 0; k < NW / 4; ++k) {
        const uint4 v = *reinterpret_cast<const uint4*>(sm.part + k * 256 + 252 - 4 * lane);
        c[0] += v.w; c[1] += v.z; c[2] += v.y; c[3] += v.x;
      }
    } else {
#pragma unroll
      for (int k = 0; k < C; ++k) {
        const uint4 v = *reinterpret_cast<const uint4*>(sm.hist + k * kTopkCopyStride + 252 - 4 * lane);
        c[0] += v.w; c[1] += v.z; c[2] += v.y; c[3] += v.x;
      }
    }
    const unsigned local = (c[0] + c[1]) + (c[2] + c[3]);
    const unsigned need = static_cast<unsigned>(K);
    unsigned run = wave_scan_inclusive(local, lane) - local;
    int cand = -1;
    unsigned cand_above = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned before = run;
      run += c[q];
      if (before < need && run >= need) {
        cand = 255 - (lane * 4 + q);
        cand_above = before;
      }
    }
    // exactly one lane holds the bin (1 <= K <= number of counted elements)
    if (cand >= 0) {
      sm.bin = cand;
      sm.above = cand_above;
    }
  }
  __syncthreads();
  const unsigned bin1 = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(sm.bin));
  const unsigned above1 = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(sm.above)));

  // ---- pass 2: low 7 bits inside bin1 (this wave's copy), and the wave's count of elements in higher bins
  unsigned* mine2 = sm.hist2 + wave * kTopkCopyStride2;
  unsigned n_hi = 0;
  const uint32_t flip = pair_of(bin1 << 7), bin_end = pair_of((bin1 << 7) | 127u);
#pragma unroll
  for (int q = 0; q < E / 2; ++q) {
    n_hi += popcount32(pair_sub(bin_end, key[q]) & kPairSigns);
    const uint32_t x = key[q] ^ flip;            // below 128 in the bin: its low 7 bits
    const unsigned x0 = x & 0xFFFFu, x1 = x >> 16;
    atomicAdd(x0 < 128u ? mine2 + x0 : sm.unread + lane, 1u);
    atomicAdd(x1 < 128u ? mine2 + x1 : sm.unread + lane, 1u);
  }
  {
    const unsigned tot_hi = wave_total(n_hi, lane);
    if (lane == 0) sm.wave_tot[wave] = tot_hi;
  }
  __syncthreads();
  unsigned T, r;               // threshold key; threshold ties to keep (>= 1)
  unsigned base;               // kept-by-magnitude elements | threshold ties << 16 in the waves before this one
  {
    // lane covers bins 127 - 2*lane (c[0]) and 126 - 2*lane (c[1]): one 8-byte read per wave copy;
    // p[] = the same two bins summed over the waves before this one
    unsigned c[2] = {0u, 0u}, p[2] = {0u, 0u};
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const uint2 v = *reinterpret_cast<const uint2*>(sm.hist2 + k * kTopkCopyStride2 + 126 - 2 * lane);
      if (k == wave) { p[0] = c[0]; p[1] = c[1]; }   // uniform condition
      c[0] += v.y; c[1] += v.x;
    }
    const unsigned local = c[0] + c[1];
    const unsigned need = static_cast<unsigned>(K) - above1;
    unsigned run = wave_scan_inclusive(local, lane) - local;
    int cand = -1;
    unsigned cand_above = 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const unsigned before = run;
      run += c[q];
      if (before < need && run >= need) {
        cand = 127 - (lane * 2 + q);
        cand_above = before;
      }
    }
    const unsigned long long found = __builtin_amdgcn_ballot_w64(cand >= 0);
    const int src = found ? __builtin_ctzll(found) : 0;
    const int bin2 = __builtin_amdgcn_readlane(cand, src);
    const unsigned above2 = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(cand_above), src));
    T = (bin1 << 7) | static_cast<unsigned>(bin2);
    r = static_cast<unsigned>(K) - (above1 + above2);
    // elements of the threshold bin above / at T in earlier waves, plus earlier waves' higher-bin totals
    // (lane k < wave adds wave_tot[k]); packed as gt | eq << 16: of at most 32768 elements, so neither half overflows
    const int b0 = 127 - 2 * lane, b1 = 126 - 2 * lane;
    unsigned gt = (b0 > bin2 ? p[0] : 0u) + (b1 > bin2 ? p[1] : 0u);
    const unsigned eq = (b0 == bin2 ? p[0] : 0u) + (b1 == bin2 ? p[1] : 0u);
    if (lane < wave) gt += sm.wave_tot[lane];      // wave <= NW <= 16 < 64
    base = wave_total(gt | (eq << 16), lane);
  }

  // the lane's elements above and at T
  TopkLane<E> out;
  uint32_t ties[E / 2];        // bits 15, 31: at T
  const uint32_t TT = pair_of(T);
  unsigned n_gt = 0, n_eq = 0;
#pragma unroll
  for (int q = 0; q < E / 2; ++q) {
    const uint32_t x = pair_sub(TT, key[q]);
    out.kept[q] = x & kPairSigns;
    ties[q] = (pair_nonzero(x) << 15) ^ kPairSigns;
    n_gt += popcount32(out.kept[q]);
    n_eq += popcount32(ties[q]);
  }
  // within the wave: one wave holds at most 64 * E <= 4096 elements, so both counts fit 16-bit halves
  const unsigned packed = n_gt | (n_eq << 16);
  const unsigned before = base + (wave_scan_inclusive(packed, lane) - packed);
  const unsigned gt_before = before & 0xFFFFu, eq_before = before >> 16;
  out.first = gt_before + min(eq_before, r);
  // the lane's ties that are kept: its first `keep` ones
  const unsigned keep = min(n_eq, r - min(eq_before, r));
  out.n = n_gt + keep;
  if (keep == n_eq) {
#pragma unroll
    for (int q = 0; q < E / 2; ++q) out.kept[q] |= ties[q];
  } else if (keep > 0) {       // rare: the tie quota ends inside this lane
    unsigned left = keep;
#pragma unroll
    for (int q = 0; q < E / 2; ++q) {
      const uint32_t lo = ties[q] & 0x8000u, hi = ties[q] & 0x80000000u;
      if (lo && left > 0) { out.kept[q] |= lo; --left; }
      if (hi && left > 0) { out.kept[q] |= hi; --left; }
    }
  }
  return out;
}

// ---- selection from histograms that the producer of the vector has already built ------------------
//
// A vector that one of the library's own kernels writes (the MLP intermediate vector, a rotated block
// input) can arrive with the two histograms of its keys in device memory: hist[0 .. 256) counts the top
// 8 key bits, hist[256 + key] every 15-bit key (the workgroups that store the vector's strips add their
// elements with device atomics).  The threshold then costs two small dependent reads by one wave instead
// of two histogram passes over the vector in every workgroup.

// Threshold key T and tie quota r = K - #{key > T} from such histograms, in two steps so that the caller
// can issue the loads where it wants them (the second read depends on the first step's result); all 64
// lanes of one wave take part, results in every lane.  1 <= K <= number of counted elements.
// Lane's words: coarse bins 255 - 4 lane - q (q = 0..3) are hist[252 - 4 lane + (3 - q)], one 16-byte read.
__device__ __forceinline__ const uint4* hist_coarse_ptr(const unsigned* hist, int lane) {
  return reinterpret_cast<const uint4*>(hist + 252 - 4 * lane);
}
// fine bins 127 - 2 lane, 126 - 2 lane of coarse bin `bin1`: one 8-byte read
__device__ __forceinline__ const uint2* hist_fine_ptr(const unsigned* hist, int bin1, int lane) {
  return reinterpret_cast<const uint2*>(hist + kHistCoarse + bin1 * 128 + 126 - 2 * lane);
}
// step 1: the coarse bin that holds the K-th largest key, and the count above it
__device__ __forceinline__ void hist_coarse_step(const uint4& v, int K, int lane, int& bin1, unsigned& above1) {
  const unsigned c[4] = {v.w, v.z, v.y, v.x};
  const unsigned local = (c[0] + c[1]) + (c[2] + c[3]);
  const unsigned need = static_cast<unsigned>(K);
  unsigned run = wave_scan_inclusive(local, lane) - local;
  int cand = -1;
  unsigned cand_above = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const unsigned before = run;
    run += c[q];
    if (before < need && run >= need) {
      cand = 255 - (lane * 4 + q);
      cand_above = before;
    }
  }
  const unsigned long long found = __builtin_amdgcn_ballot_w64(cand >= 0);
  const int src = found ? __builtin_ctzll(found) : 0;
  bin1 = max(0, __builtin_amdgcn_readlane(cand, src));
  above1 = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(cand_above), src));
}
// step 2: the threshold key and the tie quota
__device__ __forceinline__ void hist_fine_step(const uint2& f, int K, int bin1, unsigned above1, int lane, unsigned& T,
                                               unsigned& r) {
  const unsigned c2[2] = {f.y, f.x};
  const unsigned need = static_cast<unsigned>(K) - above1;
  unsigned run = wave_scan_inclusive(c2[0] + c2[1], lane) - (c2[0] + c2[1]);
  int cand = -1;
  unsigned cand_above = 0;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const unsigned before = run;
    run += c2[q];
    if (before < need && run >= need) {
      cand = 127 - (lane * 2 + q);
      cand_above = before;
    }
  }
  const unsigned long long found = __builtin_amdgcn_ballot_w64(cand >= 0);
  const int src = found ? __builtin_ctzll(found) : 0;
  const int bin2 = max(0, __builtin_amdgcn_readlane(cand, src));
  const unsigned above2 = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(cand_above), src));
  T = (static_cast<unsigned>(bin1) << 7) | static_cast<unsigned>(bin2);
  r = static_cast<unsigned>(K) - (above1 + above2);
}

// Producer side: the eight stored 16-bit values of each lane of ONE wave (valid lanes only) are added to
// the histograms, each counting `weight` times.  The coarse counts are summed in `scratch` (256 words of
// LDS owned by this wave) first, so a bin that many strips fill costs one device atomic per strip and
// not one per element.  All 64 lanes must call it.
__device__ __forceinline__ void histograms_add_wave(const uint16_t (&bits)[8], bool valid, unsigned weight,
                                                    unsigned* __restrict__ hist, unsigned* scratch, int lane) {
  // Lanes of the wave exchange counts through `scratch`: every access to it is an atomic, and the three
  // steps are separated by wavefront-scope fences (no instructions on this hardware, where a wave's LDS
  // operations complete in order; they keep the compiler from forwarding a lane's own zeros to its read).
#pragma unroll
  for (int k = 0; k < 4; ++k)
    __hip_atomic_store(scratch + 4 * lane + k, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (valid) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const unsigned key = bits[k] & 0x7FFFu;
      __hip_atomic_fetch_add(scratch + (key >> 7), weight, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
      atomicAdd(&hist[kHistCoarse + key], weight);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const unsigned c = __hip_atomic_load(scratch + 4 * lane + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    if (c) atomicAdd(&hist[4 * lane + k], c);
  }
}

// Element q of the lane (0 or 1): whether it is kept.
template <int E>
__device__ __forceinline__ unsigned kept_bit(const TopkLane<E>& st, int q) {
  return (q & 1) ? st.kept[q >> 1] >> 31 : (st.kept[q >> 1] >> 15) & 1u;
}

}  // namespace larosa
