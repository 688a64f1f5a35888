// Offline part of the method on the matrix cores (Sec. 4.2): the uncentred second moment X^T X of the
// calibration tokens, the folded weights Q^T W and W Q, and the residual adapters Q_l^T Q_{l+1}.
// All four are dense contractions  C[m,n] = sum_k A(k,m) B(k,n)  and share one kernel.
//
//  * v_mfma_f32_32x32x16 (f16 / bf16 inputs, fp32 accumulate).  A workgroup of 4 waves (one per SIMD) owns a
//    256 x 256 tile of C, each wave a 128 x 128 quarter (4 x 4 instruction tiles, 256 accumulator registers): eight
//    operand reads from LDS feed sixteen instructions, two thirds of the LDS traffic per flop of the 128 x 64 quarters that
//    eight waves would own.
//  * Global loads go straight into LDS (16 bytes per lane, no staging registers) and run three 32-deep k-tiles ahead of
//    the products: four stages of 32 KiB (the smallest tile: eight of 8 KiB, seven ahead; both terms of an f16 fold together: three of
//    48 KiB, two ahead; three bf16 terms: five of 32 KiB, four ahead), one barrier per k-tile, and the
//    loads, the LDS reads and the products of a k-tile are issued in one fixed interleaved order.
//  * Operands are stored k-major ([k][m], the layout of X, Q and W), the instruction wants 8 values along k per lane.
//    The LDS tile keeps the memory's layout and the transposing LDS read does the rest: 16 lanes point at 4 rows x 16
//    columns and receive 4 k-values of one column each.  A row's 64-byte granules are exchanged by its number
//    (granule_swizzle; the permutation sits in the addresses of the global loads), so the rows of one read lie in
//    different banks.  The k-contiguous operand of W Q is read as it is, with its 16-byte pieces exchanged likewise.
//  * A rotation comes from an eigen-solver in fp32 or better; rounding it to 16 bits before the
//    product would cost more than the 16-bit rounding of the folded weight itself.  It is therefore
//    split into 2 (f16) or 3 (bf16) 16-bit terms whose sum carries the fp32 value, and the kernel
//    adds the products of the listed term pairs into the same accumulators.
//  * The terms of a fold go through k together (TERMS): the weight's tile is loaded, and read from LDS, once for all of them.
//    Two f16 terms: three operands a k-tile instead of four; 4096 x 22016 1315 -> 1233 us, 11008 x 4096 (W Q) 698 -> 646, 1024 x
//    16384 76 -> 72.  Three bf16 terms: four operands instead of six, k-tiles of 16 in five stages of 32 KiB, a barrier per 48
//    products instead of 32; whole calls 4096 x 28672 2229 -> 2000 us, 14336 x 4096 (W Q) 1239 -> 1145 (with the split of the rotation).
//  * X^T X is symmetric: only tiles on and above the diagonal are computed; a tile above it is stored twice.
//  * Whole rounds of 256 tiles (one per compute unit) run in 256 x 256 tiles; what is left over runs as 128 x 128 or 64 x 64
//    parts in a second launch when that is shorter than another round (launch_shape).
// What bounds it: the matrix cores at the clock that the card's power allows.  A loop of nothing but these instructions on
// random operands reaches 1.63 PFLOP/s here (2.37 on zeros).  Issued in whole rounds (kernel trace): 4096 x
// 28672 x 4096 bf16, 3 terms, 1.43 PFLOP/s (2016 us; 1.29 with a pass per term); f16 folds of a 4096-wide layer 1.21 - 1.29, its adapter 1.22;
// second moment of 5000 x 8192 bf16, whose two rounds also store 268 MB: 311 us in the first traced passes, 350 - 399 once the card is warm, and
// 26 - 35 for the 16 tiles left over (36 - 38 before the waves shared k-tiles); untraced the whole call takes 327 (736 before the
// large tile; C stored in 16-byte pieces through LDS instead of from registers saved 45).  The matrix cores are busy 81 % of the cycles with three
// bf16 terms together, 69 - 79 % in f16 folds, 73 % in its adapter's passes, 59 % in the two rounds of that second moment, 20 % in parts of 64 that share
// the k-tiles (a chain's latency); LDS bank conflicts are under 1 % of the large tile's active cycles.  The design before (8 waves of 128 x 64,
// staging registers, two LDS stages) kept them busy 34 % and gave the XCDs of a symmetric product uneven shares.
#include <type_traits>

#include "kernels.hpp"
#include "lds_load.hpp"
#include "numeric.hpp"

namespace larosa {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bfloat8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));

constexpr int kKTile = 32;         // k rows per LDS stage
// LDS stages: loads run kStages - 1 k-tiles ahead of the products (a k-tile of the smallest workgroup tile is multiplied
// in a fraction of a memory round trip, so it looks further ahead)
template <int MI> constexpr int kStagesOf = MI == 1 ? 8 : 4;
constexpr int kBand = 4;           // tile rows of a band (see tile_of)

template <typename T> struct Mfma;
template <> struct Mfma<F16> {
  static __device__ __forceinline__ float16v run(u32x4 a, u32x4 b, float16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
  }
};
template <> struct Mfma<BF16> {
  static __device__ __forceinline__ float16v run(u32x4 a, u32x4 b, float16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bfloat8, a), __builtin_bit_cast(bfloat8, b), c, 0, 0,
                                                   0);
  }
};

// Operand loads go through buffer resources that span the whole (multi-term) operand: rows past Kd and columns outside
// the matrix only need the offset kOutside.
__device__ __forceinline__ u32x4 operand_buffer(const uint16_t* p, long elements) {
  return raw_buffer(p, static_cast<uint32_t>(elements * 2));
}

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>)
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// One 64-byte granule (32 columns) of a k-major LDS tile is moved by its row: granule q of row k sits at
// position q ^ granule_swizzle(k), so that the eight rows a transposing read touches lie in different banks.
template <int GR>   // granules per row (a power of two)
__device__ __forceinline__ int granule_swizzle(int k) { return ((k & 3) | (((k >> 3) & 1) << 2)) & (GR - 1); }

// Workgroup barrier once all but the wave's N youngest loads have landed in LDS and its own LDS reads are done.
template <int N>
__device__ __forceinline__ void tile_landed() {
  static_assert(N < 64, "vmcnt is a 6-bit field");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// LDS writes of a wave before it are seen by its reads after it (the hardware keeps a wave's LDS accesses in order; this
// keeps the compiler from moving a lane's read in front of another lane's write).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A tile of the product, as (row, column) of the grid of tiles.  Tiles are numbered band by band (kBand tile rows),
// column by column inside a band; workgroup b takes number (b % 8) * ceil(tiles / 8) + b / 8, so an XCD
// (workgroups b % 8) works on consecutive tiles: its 32 compute units on a patch of 4 x 8, sharing the panels of both
// operands in their L2.  Symmetric products number the tiles on and above the diagonal only.
struct TileAt { int m, n; };
__host__ __device__ __forceinline__ TileAt tile_of(int number, int tiles_m, int tiles_n, bool symmetric) {
  int band = 0;
  for (;;) {
    const int left = tiles_m - band * kBand, rows = left < kBand ? left : kBand;
    const int first = symmetric ? band * kBand : 0;          // first column of the band
    const int head = symmetric ? rows * (rows - 1) / 2 : 0;  // tiles in the columns that meet the diagonal above its last row
    const int cols = tiles_n - first - (symmetric ? rows - 1 : 0);
    const int count = head + cols * rows;
    if (number < count || (band + 1) * kBand >= tiles_m) {
      if (number < head) {       // column c of the corner holds c + 1 tiles
        int c = 0;
        while (number > c) { number -= c + 1; ++c; }
        return {band * kBand + number, first + c};
      }
      number -= head;
      return {band * kBand + number % rows, first + (symmetric ? rows - 1 : 0) + number / rows};
    }
    number -= count;
    ++band;
  }
}

constexpr int kBigTile = 256;      // tiles are numbered in this size; smaller workgroup tiles are parts of them

// A workgroup of 4 waves (2 x 2) owns a (64 MI) x (64 MI) tile of C, a wave (32 MI) x (32 MI) of it.
// TERMS > 1: all term pairs of a fold in one pass over k.  The operand that has terms (A if it is k-major, else B: the
// rotation) brings those of a k-tile together, the weight comes once for all: three operands are loaded and read from LDS where
// two passes take four, four where three passes take six (three terms: k-tiles of 16, so that five stages fit).
template <typename T, bool A_KMAJOR, int MI, int TERMS>
__global__ __launch_bounds__(256, MI == 4 ? 1 : 2) void contraction_kernel(ContractionArgs a) {
  constexpr int TC = 64 * MI;                    // tile side
  constexpr int KT = TERMS == 3 ? 16 : kKTile;   // k rows of a k-tile
  constexpr int kOperandBytes = TC * KT * 2;     // one operand of one stage
  constexpr int kStageBytes = (TERMS + 1) * kOperandBytes;     // A, B, further terms
  constexpr int CPR = TC / 8;                    // 16-byte pieces per row of a k-major tile
  constexpr int RPI = 64 / CPR;                  // rows that one wave-load covers
  constexpr int GR = 2 * MI;                     // granules per row
  constexpr int kStages = TERMS == 1 ? kStagesOf<MI> : TERMS == 2 ? 3 : 5;
  static_assert(TERMS == 1 || MI == 4, "several terms at once: the large tile only");
  constexpr int LQ = kOperandBytes / 4096;       // loads of a wave per operand and k-tile
  constexpr int kLoads = kStageBytes / 4096;     // of a wave per stage
  constexpr int kParts = 4 / MI;                 // a 256 x 256 tile is kParts x kParts tiles of this kernel
  __shared__ __attribute__((aligned(1024))) char lds[kStages * kStageBytes];

  const int per_xcd = (a.tiles + 7) >> 3;
  const int local = static_cast<int>(blockIdx.x & 7) * per_xcd + static_cast<int>(blockIdx.x >> 3);
  if (local >= a.tiles) return;
  const TileAt at = tile_of(a.tile0 + local / (kParts * kParts), a.tiles_m, a.tiles_n, a.symmetric != 0);
  const int part = local % (kParts * kParts);
  const int m0 = at.m * kBigTile + part / kParts * TC, n0 = at.n * kBigTile + part % kParts * TC;
  if (m0 >= a.M || n0 >= a.N) return;            // a part of an edge tile that holds nothing (uniform)

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int wm = w >> 1, wn = w & 1;

  const int ktiles = (a.Kd + KT - 1) / KT;
  const int iters = TERMS > 1 ? ktiles : ktiles * a.npairs;

  // ---- loads, straight into LDS: wave-load q of wave w fills pieces 64 (4 q + w) .. + 63 of the operand's tile
  const u32x4 bufA = operand_buffer(a.A, a.a_elements);
  const u32x4 bufB = operand_buffer(a.B, a.b_elements);
  uint32_t offA[LQ], offB[LQ];
  int kA[LQ], kB[LQ];                            // k inside the tile of the lane's piece (its first k value)
#pragma unroll
  for (int q = 0; q < LQ; ++q) {
    const int row = (4 * q + w) * RPI + lane / CPR, piece = lane % CPR;
    const int src = piece ^ (4 * granule_swizzle<GR>(row));
    kB[q] = row;
    offB[q] = n0 + 8 * src < a.N ? static_cast<uint32_t>((row * a.N + n0 + 8 * src) * 2) : kOutside;
    if (A_KMAJOR) {
      kA[q] = row;
      offA[q] = m0 + 8 * src < a.M ? static_cast<uint32_t>((row * a.M + m0 + 8 * src) * 2) : kOutside;
    } else {
      // [row m][KT k values]: piece p of the four (two) of 16 bytes of row m holds k values 8 (p ^ (m / 4 % 4)) .. (8 (p ^ (m / 8 % 2)) ..)
      const int m = KT == 32 ? (4 * q + w) * 16 + (lane >> 2) : (4 * q + w) * 32 + (lane >> 1);
      kA[q] = KT == 32 ? 8 * ((lane & 3) ^ ((m >> 2) & 3)) : 8 * ((lane & 1) ^ ((m >> 3) & 1));
      offA[q] = m0 + m < a.M ? static_cast<uint32_t>(((m0 + m) * a.Kd + kA[q]) * 2) : kOutside;
    }
  }
  const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_char*)lds));
  // The next k-tile to load: its first k, the stage it goes to and the byte offsets of its first element in the
  // operands.  Past the last tile f_k is 0: zeros are loaded, so that every step waits for the same count.
  const uint32_t stepA = static_cast<uint32_t>((A_KMAJOR ? KT * a.M : KT) * 2), stepB = static_cast<uint32_t>(KT * a.N * 2);
  int f_pair = 0, f_k = a.Kd, f_stage = 0;
  uint32_t ta = static_cast<uint32_t>(a.pa[0] * a.a_term_stride * 2), tb = static_cast<uint32_t>(a.pb[0] * a.b_term_stride * 2);
  uint32_t f_lds = lds_base + w * 1024;
  const uint32_t term2 = static_cast<uint32_t>((A_KMAJOR ? a.a_term_stride : a.b_term_stride) * 2);
  auto fetch_piece = [&](int q) {                // operand q / LQ: A, B, the further terms of one of them
    const int op = q / LQ, i = q % LQ;
    const uint32_t to = f_lds + op * kOperandBytes + i * 4096;
    const uint32_t term = op < 2 ? 0u : (op - 1) * term2;
    if (op == 0 || (op > 1 && A_KMAJOR)) load_to_lds(bufA, to, (kA[i] < f_k ? offA[i] : kOutside) + (ta + term));
    else load_to_lds(bufB, to, (kB[i] < f_k ? offB[i] : kOutside) + (tb + term));
  };
  auto fetch_next = [&]() {
    f_k -= KT;
    ta += stepA;
    tb += stepB;
    if (f_k <= 0) {                              // the next term pair (uniform, once per pass over k)
      ++f_pair;
      if (TERMS == 1 && f_pair < a.npairs) {
        f_k = a.Kd;
        ta = static_cast<uint32_t>(a.pa[f_pair] * a.a_term_stride * 2);
        tb = static_cast<uint32_t>(a.pb[f_pair] * a.b_term_stride * 2);
      } else {
        f_k = 0;
        ta = tb = 0;
      }
    }
    f_stage = TERMS > 1 ? (f_stage == kStages - 1 ? 0 : f_stage + 1) : (f_stage + 1) & (kStages - 1);
    f_lds = lds_base + f_stage * kStageBytes + w * 1024;
  };
  auto fetch = [&]() {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) fetch_piece(q);
    fetch_next();
  };

  // ---- operand reads.  k-major tiles: lane (g, j) = (lane / 16, lane % 16) of a transposing read points at four
  // columns of row 8 (g / 2) + j / 4 and receives column 16 (g % 2) + j of four rows.
  const int g = lane >> 4, j = lane & 15;
  const int rowk = 8 * (g >> 1) + (j >> 2);
  const int inrow = 32 * (g & 1) + 8 * (j & 3);
  const int sw = granule_swizzle<GR>(rowk);
  int adrA[MI], adrB[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    adrA[i] = A_KMAJOR ? rowk * (TC * 2) + ((wm * MI + i) ^ sw) * 64 + inrow
                       : (wm * MI * 32 + i * 32 + (lane & 31)) * (2 * KT) +
                             (((lane >> 5) ^ (KT == 32 ? (lane >> 2) & 3 : (lane >> 3) & 1)) * 16);
    adrB[i] = kOperandBytes + rowk * (TC * 2) + ((wn * MI + i) ^ sw) * 64 + inrow;
  }
  auto read_k = [&](int stage, int adr, int s) -> u32x4 {
    const lds_char* p = (const lds_char*)lds + stage + adr + s * (16 * TC * 2);
    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)p));
    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p + 4 * TC * 2)));
    return u32x4{lo.x, lo.y, hi.x, hi.y};
  };
  // piece r < 2 MI of a 16-deep slice s: the operand of tile row / column r / 2, alternating A and B
  auto read_piece = [&](int st, int s, int r, u32x4 (&av)[MI], u32x4 (&bv)[MI]) {
    const int i = r >> 1;
    if (r & 1) {
      bv[i] = read_k(st, adrB[i], s);
    } else if (A_KMAJOR) {
      av[i] = read_k(st, adrA[i], s);
    } else {
      av[i] = *(const __attribute__((address_space(3))) u32x4*)((const lds_char*)lds + st + (adrA[i] ^ (32 * s)));
    }
  };

  float16v acc[MI][MI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int jj = 0; jj < MI; ++jj)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][jj][r] = 0.0f;
  // The products of one slice, in a fixed order of instructions: between them the operand reads of the next slice
  // (stage st, slice s) and, with LOADS, the loads of a later k-tile.
  auto products = [&](const u32x4 (&av)[MI], const u32x4 (&bv)[MI], int st, int s, u32x4 (&an)[MI], u32x4 (&bn)[MI], auto loads) {
    static_for<MI * MI>([&](auto ij) {
      constexpr int x = decltype(ij)::value;
      constexpr int kEvery = MI * MI / (2 * MI);     // products per operand read and per load
      if constexpr (kEvery > 0) {
        if constexpr (x % kEvery == 0) read_piece(st, s, x / kEvery, an, bn);
        if constexpr (decltype(loads)::value && x % kEvery == kEvery - 1) fetch_piece(x / kEvery);
      } else {
        read_piece(st, s, 0, an, bn);
        read_piece(st, s, 1, an, bn);
        if constexpr (decltype(loads)::value) { fetch_piece(0); fetch_piece(1); }
      }
      acc[x / MI][x % MI] = Mfma<T>::run(av[x / MI], bv[x % MI], acc[x / MI][x % MI]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // ---- pipeline.  A stage's loads are issued kStages - 1 k-tiles before its products; the second half of tile it is read
  // while its first half is multiplied, then one barrier, then the first half of tile it + 1 while the second half is
  // multiplied.  The barrier follows a wait for this wave's own loads of tile it + 1 (the kStages - 2 tiles of 2 MI loads
  // after it may be outstanding) and for its LDS reads of tile it, whose stage the loads issued next overwrite.
  if constexpr (TERMS == 1) {
    u32x4 a0[MI], b0[MI], a1[MI], b1[MI];
    for (int i = 0; i < kStages - 1; ++i) fetch();
    tile_landed<(kStages - 2) * 2 * MI>();
    fetch();
    int stage = 0;
#pragma unroll
    for (int r = 0; r < 2 * MI; ++r) read_piece(stage, 0, r, a0, b0);
    for (int it = 0; it < iters; ++it) {
      products(a0, b0, stage, 1, a1, b1, std::false_type{});
      tile_landed<(kStages - 2) * 2 * MI>();
      stage = (stage + kStageBytes) & (kStages * kStageBytes - 1);
      products(a1, b1, stage, 0, a0, b0, std::true_type{});
      fetch_next();
    }
  } else {
    // The same with a group of products per term (two terms: of the tile's first half, then of its second).  The barrier stands
    // before the last group, which reads the next tile's first operands; a tile's loads are issued half in that group, half in
    // the one after.
    u32x4 p0[MI], p1[MI], s0[MI], s1[MI];        // terms; the shared operand of each half (of each tile)
    auto read_term = [&](int st, int s, int term, int i) -> u32x4 {
      return A_KMAJOR ? read_k(st + (term ? term + 1 : 0) * kOperandBytes, adrA[i], s) : read_k(st + term * kOperandBytes, adrB[i], s);
    };
    auto read_shared = [&](int st, int s, int i) -> u32x4 {
      if constexpr (A_KMAJOR) return read_k(st, adrB[i], s);
      else return *(const __attribute__((address_space(3))) u32x4*)((const lds_char*)lds + st + (adrA[i] ^ (32 * s)));
    };
    auto group = [&](const u32x4 (&p)[MI], const u32x4 (&sh)[MI], auto between) {
      static_for<MI * MI>([&](auto ij) {
        constexpr int x = decltype(ij)::value;
        between(x);
        acc[x / MI][x % MI] = A_KMAJOR ? Mfma<T>::run(p[x / MI], sh[x % MI], acc[x / MI][x % MI])
                                       : Mfma<T>::run(sh[x / MI], p[x % MI], acc[x / MI][x % MI]);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    for (int i = 0; i < kStages - 1; ++i) fetch();
    tile_landed<(kStages - 2) * kLoads>();
#pragma unroll
    for (int q = 0; q < kLoads / 2; ++q) fetch_piece(q);
    int stage = 0;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      p0[i] = read_term(stage, 0, 0, i);
      s0[i] = read_shared(stage, 0, i);
    }
    if constexpr (TERMS == 2) {
      for (int it = 0; it < iters; ++it) {
        group(p0, s0, [&](int x) __attribute__((always_inline)) {
          if (x % 4 == 0) p1[x / 4] = read_term(stage, 0, 1, x / 4);
          if (x % 2 == 1 && x / 2 < kLoads / 2) fetch_piece(kLoads / 2 + x / 2);
        });
        fetch_next();
        group(p1, s0, [&](int x) __attribute__((always_inline)) {
          if (x % 4 == 0) p0[x / 4] = read_term(stage, 1, 0, x / 4);
          if (x % 4 == 2) s1[x / 4] = read_shared(stage, 1, x / 4);
        });
        group(p0, s1, [&](int x) __attribute__((always_inline)) {
          if (x % 4 == 0) p1[x / 4] = read_term(stage, 1, 1, x / 4);
        });
        tile_landed<(kStages - 2) * kLoads>();     // of the tiles under way, all but the next may be outstanding
        stage = stage == (kStages - 1) * kStageBytes ? 0 : stage + kStageBytes;
        group(p1, s1, [&](int x) __attribute__((always_inline)) {
          if (x % 4 == 0) p0[x / 4] = read_term(stage, 0, 0, x / 4);
          if (x % 4 == 2) s0[x / 4] = read_shared(stage, 0, x / 4);
          if (x % 2 == 1 && x / 2 < kLoads / 2) fetch_piece(x / 2);
        });
      }
    } else {
      // terms 0 and 2 of a tile sit in `p`, term 1 and the next tile's term 0 in `q`
      auto tile = [&](u32x4 (&p)[MI], u32x4 (&q)[MI], u32x4 (&sh)[MI], u32x4 (&sh_next)[MI]) __attribute__((always_inline)) {
        group(p, sh, [&](int x) __attribute__((always_inline)) {
          if (x % 4 == 0) q[x / 4] = read_term(stage, 0, 1, x / 4);
          if (x % 4 == 1) fetch_piece(kLoads / 2 + x / 4);
        });
        fetch_next();
        group(q, sh, [&](int x) __attribute__((always_inline)) {
          if (x % 4 == 0) p[x / 4] = read_term(stage, 0, 2, x / 4);
        });
        tile_landed<(kStages - 2) * kLoads>();
        stage = stage == (kStages - 1) * kStageBytes ? 0 : stage + kStageBytes;
        group(p, sh, [&](int x) __attribute__((always_inline)) {
          if (x % 4 == 0) q[x / 4] = read_term(stage, 0, 0, x / 4);
          if (x % 4 == 2) sh_next[x / 4] = read_shared(stage, 0, x / 4);
          if (x % 4 == 1) fetch_piece(x / 4);
        });
      };
      static_assert(TERMS != 3 || kLoads == 8, "four loads in a group");
      for (int it = 0; it < iters; it += 2) {    // (an odd count: the last tile is zeros)
        tile(p0, p1, s0, s1);
        tile(p1, p0, s1, s0);
      }
    }
  }
  // ---- store.  Accumulator register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of its 32 x 32
  // block.  A strip of 32 rows at a time goes through the wave's own part of the LDS (every load into it has landed and
  // every wave has left the operands behind), so that memory sees runs of MI * 128 bytes.  The block indices are
  // compile-time constants (static_for): a run-time index would move the accumulators to scratch memory.
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  constexpr int W = 32 * MI;                     // side of the wave's block
  constexpr int kPitch32 = W + 4;                // floats per row: 16-byte rows whose pieces fall into different banks
  constexpr int kPitch16 = W + 8;                // 16-bit values per row
  static_assert(32 * kPitch32 * 4 * 4 <= kStages * kStageBytes, "the strips of four waves fit the LDS");
  float* strip = reinterpret_cast<float*>(lds + w * (32 * kPitch32 * 4));
  const int mw = m0 + wm * W, nw = n0 + wn * W;  // first row and column of the wave's block
  const int rq = 4 * (lane >> 5), cl = lane & 31;
  const int M = a.M, N = a.N;
  uint16_t* const C16 = a.C16;
  float* const C32 = a.C32;
  const float post_scale = a.post_scale;
  const bool mirror = a.symmetric != 0 && at.m != at.n;
  const bool add = a.accumulate != 0 && C32 != nullptr;
  // register r of block (i, jj) as it will be stored
  auto value = [&](float v, int i, int jj, int r) __attribute__((always_inline)) {
    v *= post_scale;
    if (add) {
      const int m = mw + i * 32 + 8 * (r >> 2) + rq + (r & 3), n = nw + jj * 32 + cl;
      if (m < M && n < N) v = C32[static_cast<long>(m) * N + n] + v;
    }
    return v;
  };
  // rows r0 .. r0 + 31 of the strip to rows of C, 16 bytes per lane
  auto store_strip = [&](int row0, int col0) __attribute__((always_inline)) {
    wave_lds_order();
    if (C16) {
      constexpr int kLanes = W / 8;              // lanes per row
#pragma unroll
      for (int p = 0; p < 32 * kLanes / 64; ++p) {
        const int r = p * (64 / kLanes) + lane / kLanes, c = lane % kLanes * 8;
        const uint4 v = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(strip) + r * kPitch16 + c);
        if (row0 + r < M && col0 + c < N) *reinterpret_cast<uint4*>(C16 + static_cast<long>(row0 + r) * N + col0 + c) = v;
      }
    } else {
      constexpr int kLanes = W / 4;
#pragma unroll
      for (int p = 0; p < 32 * kLanes / 64; ++p) {
        const int r = p * (64 / kLanes) + lane / kLanes, c = lane % kLanes * 4;
        const float4 v = *reinterpret_cast<const float4*>(strip + r * kPitch32 + c);
        if (row0 + r < M && col0 + c < N) *reinterpret_cast<float4*>(C32 + static_cast<long>(row0 + r) * N + col0 + c) = v;
      }
    }
    wave_lds_order();
  };
  // a symmetric product's elements below the diagonal: the transposed block (tiles on the diagonal hold both halves).
  // First, while the elements that are added to still hold their old values.
  if (mirror) {
    static_for<MI>([&](auto jc) {                // block columns of the wave
      constexpr int jj = decltype(jc)::value;
      static_for<MI>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *reinterpret_cast<float4*>(strip + cl * kPitch32 + i * 32 + 8 * r4 + rq) =
              make_float4(value(acc[i][jj][4 * r4], i, jj, 4 * r4), value(acc[i][jj][4 * r4 + 1], i, jj, 4 * r4 + 1),
                          value(acc[i][jj][4 * r4 + 2], i, jj, 4 * r4 + 2), value(acc[i][jj][4 * r4 + 3], i, jj, 4 * r4 + 3));
      });
      store_strip(nw + jj * 32, mw);
    });
  }
  static_for<MI>([&](auto ic) {                  // block rows of the wave
    constexpr int i = decltype(ic)::value;
    static_for<MI>([&](auto jc) {
      constexpr int jj = decltype(jc)::value;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + rq + (r & 3), col = jj * 32 + cl;
        if (C16) reinterpret_cast<uint16_t*>(strip)[row * kPitch16 + col] = T::from_f32(value(acc[i][jj][r], i, jj, r));
        else strip[row * kPitch32 + col] = value(acc[i][jj][r], i, jj, r);
      }
    });
    store_strip(mw + i * 32, nw);
  });
}

// Few tiles: a workgroup owns a 64 x 64 tile, and its four waves share the k-tiles instead of the tile.  What bounds such
// products is not the matrix cores but each wave's chain over k, so a wave takes every fourth k-tile through a ring of its own
// in LDS, with no barrier until the four sums meet, and multiplies the whole 64 x 64 (with a 32 x 32 quarter per wave and a
// barrier per k-tile, 16 tiles of 256 x 256 left over from a second moment of 5000 x 8192 took 36 us, 0.23 us a k-tile; now 26 - 32).
// Whole calls, us, quarters / shared k-tiles: second moment 5000 x 1024 f16 29.0 / 22.6, 2048 x 1024 (64 k-tiles) 14.4 / 12.0, fold
// 2048 x 512 f16 30.8 / 25.8, adapter 1024 bf16 46.8 / 38.4.  shares_chain says which products take it.
// The line at 64 k-tiles is not one of speed: sharing is level at 16 k-tiles and faster from 24 on (second moment 512 wide, 512 / 768 / 1024 /
// 2016 tokens: 6.90 / 8.03 / 9.08 / 13.7 in quarters, 7.01 / 7.77 / 8.47 / 11.4 shared).  Sums on the matrix cores are not symmetric under
// negation, and sums in four parts are two to five times less so (entries of Q^T W that round the other way for -Q, quarters / shared:
// f16 256 x 704 4 / 11, 1024 x 1024 92 / 191, bf16 2048 x 256 11 / 60): at 16 or 24 the flipped eigenvectors of a 256-wide layer reach its output's last
// bits at batch 1, where they did not before.
constexpr int kSharedChain = 64;   // k-tiles of all term pairs from which the four waves share them
constexpr int kSmallSide = 64;
constexpr int kSmallStages = 4;    // k-tiles in a wave's ring
constexpr int kSmallOperand = kSmallSide * kKTile * 2, kSmallStage = 2 * kSmallOperand, kSmallRing = kSmallStages * kSmallStage;
constexpr int kSmallPitch = kSmallSide + 4;    // floats per row of a wave's sums

template <typename T, bool A_KMAJOR>
__global__ __launch_bounds__(256, 1) void small_contraction_kernel(ContractionArgs a) {
  constexpr int kParts = kBigTile / kSmallSide;
  constexpr int kLoads = kSmallStage / 1024;     // of a wave per k-tile
  __shared__ __attribute__((aligned(1024))) char lds[4 * kSmallRing];
  static_assert(4 * kSmallSide * kSmallPitch * 4 <= static_cast<int>(sizeof(lds)), "the sums reuse the rings");

  const int per_xcd = (a.tiles + 7) >> 3;
  const int local = static_cast<int>(blockIdx.x & 7) * per_xcd + static_cast<int>(blockIdx.x >> 3);
  if (local >= a.tiles) return;
  const TileAt at = tile_of(a.tile0 + local / (kParts * kParts), a.tiles_m, a.tiles_n, a.symmetric != 0);
  const int part = local % (kParts * kParts);
  const int m0 = at.m * kBigTile + part / kParts * kSmallSide, n0 = at.n * kBigTile + part % kParts * kSmallSide;
  const int M = a.M, N = a.N, Kd = a.Kd;
  if (m0 >= M || n0 >= N) return;                // a part of an edge tile that holds nothing (uniform)

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- loads: wave-load q fills pieces 64 q .. + 63 of the operand's tile.  A k-major row is 128 bytes, two granules, which
  // every second pair of rows exchanges: the four rows that half a wave's transposing read touches lie in different banks.
  const u32x4 bufA = operand_buffer(a.A, a.a_elements);
  const u32x4 bufB = operand_buffer(a.B, a.b_elements);
  auto swap_of = [](int k) __attribute__((always_inline)) { return (k >> 1) & 1; };
  uint32_t offA[4], offB[4];
  int kA[4], kB[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = 8 * q + lane / 8, col = 8 * ((lane % 8) ^ (4 * swap_of(row)));
    kB[q] = row;
    offB[q] = n0 + col < N ? static_cast<uint32_t>((row * N + n0 + col) * 2) : kOutside;
    if (A_KMAJOR) {
      kA[q] = row;
      offA[q] = m0 + col < M ? static_cast<uint32_t>((row * M + m0 + col) * 2) : kOutside;
    } else {
      // [row m][32 k values], pieces exchanged as in the large tiles
      const int m = q * 16 + (lane >> 2);
      kA[q] = 8 * ((lane & 3) ^ ((m >> 2) & 3));
      offA[q] = m0 + m < M ? static_cast<uint32_t>(((m0 + m) * Kd + kA[q]) * 2) : kOutside;
    }
  }
  const uint32_t ring = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_char*)lds)) + w * kSmallRing;
  const uint32_t stepA = static_cast<uint32_t>((A_KMAJOR ? kKTile * M : kKTile) * 2), stepB = static_cast<uint32_t>(kKTile * N * 2);
  const int ktiles = (Kd + kKTile - 1) / kKTile;
  const int iters = ktiles * a.npairs;           // k-tiles of all term pairs, one pass after the other
  int f_pair = 0, f_tile = w, f_stage = 0;       // the k-tile to load next, the stage it goes to
  auto fetch = [&]() __attribute__((always_inline)) {
    while (f_tile >= ktiles && f_pair < a.npairs) { f_tile -= ktiles; ++f_pair; }   // (uniform)
    const bool any = f_pair < a.npairs;          // past the last: zeros, so that every step waits for the same count
    const int left = any ? Kd - f_tile * kKTile : 0;
    const uint32_t ta = any ? static_cast<uint32_t>(a.pa[f_pair] * a.a_term_stride * 2) + f_tile * stepA : 0u;
    const uint32_t tb = any ? static_cast<uint32_t>(a.pb[f_pair] * a.b_term_stride * 2) + f_tile * stepB : 0u;
    const uint32_t to = ring + f_stage * kSmallStage;
#pragma unroll
    for (int q = 0; q < 4; ++q) load_to_lds(bufA, to + q * 1024, (kA[q] < left ? offA[q] : kOutside) + ta);
#pragma unroll
    for (int q = 0; q < 4; ++q) load_to_lds(bufB, to + kSmallOperand + q * 1024, (kB[q] < left ? offB[q] : kOutside) + tb);
    f_tile += 4;
    f_stage = (f_stage + 1) & (kSmallStages - 1);
  };

  // ---- operand reads, as in the large tiles with two granules per row
  const int g = lane >> 4, j = lane & 15;
  const int rowk = 8 * (g >> 1) + (j >> 2);
  const int inrow = rowk * (kSmallSide * 2) + 32 * (g & 1) + 8 * (j & 3), swap = 64 * swap_of(rowk);
  const lds_char* const mine = (const lds_char*)lds + w * kSmallRing;
  auto read_k = [&](const lds_char* p) __attribute__((always_inline)) {
    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)p));
    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p + 4 * kSmallSide * 2)));
    return u32x4{lo.x, lo.y, hi.x, hi.y};
  };
  struct Operands { u32x4 a[2][2], b[2][2]; };   // [16-deep slice][32 rows or columns]
  auto read = [&](Operands& o, int stage) __attribute__((always_inline)) {
    const lds_char* p = mine + stage * kSmallStage;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int at16 = inrow + ((i * 64) ^ swap) + s * (16 * kSmallSide * 2);
        o.b[s][i] = read_k(p + kSmallOperand + at16);
        if constexpr (A_KMAJOR) o.a[s][i] = read_k(p + at16);
        else o.a[s][i] = *(const __attribute__((address_space(3))) u32x4*)(p + (((i * 32 + (lane & 31)) * 64 + (((lane >> 5) ^ ((lane >> 2) & 3)) * 16)) ^ (32 * s)));
      }
  };
  float16v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][jj][r] = 0.0f;
  auto multiply = [&](const Operands& o) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) acc[i][jj] = Mfma<T>::run(o.a[s][i], o.b[s][jj], acc[i][jj]);
  };

  // ---- the operands of the wave's next k-tile are read while one is multiplied
  Operands o0, o1;
  for (int i = 0; i < kSmallStages; ++i) fetch();
  int stage = 0;
  auto step = [&](Operands& now, Operands& next) __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // `now` is in registers: its stage takes the next loads
    fetch();
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kSmallStages - 1) * kLoads) : "memory");   // the next k-tile has landed
    stage = (stage + 1) & (kSmallStages - 1);
    read(next, stage);
    __builtin_amdgcn_sched_barrier(0);
    multiply(now);
    __builtin_amdgcn_sched_barrier(0);
  };
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kSmallStages - 1) * kLoads) : "memory");
  read(o0, 0);
  for (int t = w; t < iters; t += 8) {           // two of the wave's k-tiles at a time (past the last: zeros)
    step(o0, o1);
    step(o1, o0);
  }
  // every load has landed and every wave has left its ring: the LDS is free for the sums
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

  // ---- the four waves' sums, in wave order.  Accumulator register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column
  // l % 32 of its 32 x 32 block.
  float* const sums = reinterpret_cast<float*>(lds);
  constexpr int kCopy = kSmallSide * kSmallPitch;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        sums[w * kCopy + (i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * kSmallPitch + jj * 32 + (lane & 31)] = acc[i][jj][r];
  __syncthreads();
  const bool mirror = a.symmetric != 0 && at.m != at.n;
  const int tr = tid >> 4, tc = tid & 15;        // the thread's pieces: rows tr + 16 p, columns 4 tc .. + 3
  auto store4 = [&](int row, int col, const float (&v)[4]) __attribute__((always_inline)) {
    const long at4 = static_cast<long>(row) * N + col;
    if (a.C16) *reinterpret_cast<uint2*>(a.C16 + at4) = pack4<T>(v);
    else *reinterpret_cast<float4*>(a.C32 + at4) = make_float4(v[0], v[1], v[2], v[3]);
  };
  float v[4][4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = tr + 16 * p, row = m0 + r, col = n0 + 4 * tc;
    float* const q = sums + r * kSmallPitch + 4 * tc;
    float4 c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = *reinterpret_cast<const float4*>(q + k * kCopy);
    const bool in = row < M && col < N;          // (N % 4 == 0: the four are inside together)
    float4 old = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a.accumulate != 0 && a.C32 && in) old = *reinterpret_cast<const float4*>(a.C32 + static_cast<long>(row) * N + col);
    v[p][0] = old.x + (c[0].x + c[1].x + c[2].x + c[3].x) * a.post_scale;
    v[p][1] = old.y + (c[0].y + c[1].y + c[2].y + c[3].y) * a.post_scale;
    v[p][2] = old.z + (c[0].z + c[1].z + c[2].z + c[3].z) * a.post_scale;
    v[p][3] = old.w + (c[0].w + c[1].w + c[2].w + c[3].w) * a.post_scale;
    if (mirror) *reinterpret_cast<float4*>(q) = make_float4(v[p][0], v[p][1], v[p][2], v[p][3]);
    if (in) store4(row, col, v[p]);
  }
  if (mirror) {                                  // uniform; below the diagonal: the transposed tile
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int c = tr + 16 * p;                 // column of the tile, row of the transposed one
      float t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = sums[(4 * tc + e) * kSmallPitch + c];
      if (n0 + c < N && m0 + 4 * tc < M) store4(n0 + c, m0 + 4 * tc, t);
    }
  }
}

// Bits of a 16-bit rounding as T::from_f32 gives them, for bf16 as a choice between two values: the branch around a NaN there is one more
// serial step per rounding in a lane that has twelve of them.
__device__ __forceinline__ uint32_t term_bits(F16, float f) { return F16::from_f32(f); }
__device__ __forceinline__ uint32_t term_bits(BF16, float f) {
  const uint32_t u = __float_as_uint(f), rounded = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16, nan = (u >> 16) | 0x40u;
  return (u & 0x7FFFFFFFu) > 0x7F800000u ? nan : rounded;
}

// fp32 -> NT 16-bit terms with x * pre_scale = t0 + t1 (+ t2) up to the last term's rounding.  HBM-bound for wide rotations, 4 bytes in
// and 2 NT out per entry (4096 x 4096 in three terms: 49.8 us with one entry a lane, 28.8 with eight, 27.7 with four), latency-bound for narrow ones, where
// a lane's chain counts: bf16 fold 512 x 512 / adapter 256, whole calls, us: one entry 14.4 / 15.5, eight 15.0 / 16.7.  Four entries (16 bytes
// in, n is a multiple of 64) are as fast as the better of the two: 14.4 / 15.6, adapter 4096 bf16 660 (eight: 659, one: 702).
// DEALT: pieces of 256 entries, a wave's, go round the eight XCDs one by one (workgroup b runs on XCD b % 8), not four at a time: of a
// rotation 1024 wide each XCD then writes one column panel of 256 and can find it in its own L2.  Whole calls, us, four at a time / dealt: f16 W Q 2048 x
// 1024 24.9 / 23.0, Q^T W 1024 x 512 16.4 / 14.9, W Q 264 x 2048 27.1 / 23.8 (one entry a lane, which dealt them too: 23.6, 17.6, 31.5); elsewhere between
// 3 % faster and 1.5 % slower (Q^T W 1536 x 512 22.1 / 22.5).
template <typename T, int NT, int WAVES, bool DEALT>
__global__ __launch_bounds__(WAVES * 64) void split_terms_kernel(const float* __restrict__ src, uint16_t* __restrict__ dst, long n,
                                                          float pre_scale) {
  const long b = blockIdx.x, wave = threadIdx.x >> 6;
  const long piece = DEALT ? (b >> 3) * (8 * WAVES) + wave * 8 + (b & 7) : b * WAVES + wave;
  const long i = piece * 256 + (threadIdx.x & 63) * 4;
  if (i >= n) return;
  const float4 v = *reinterpret_cast<const float4*>(src + i);
  float r[4] = {v.x * pre_scale, v.y * pre_scale, v.z * pre_scale, v.w * pre_scale};
#pragma unroll
  for (int s = 0; s < NT; ++s) {
    uint32_t b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      b[k] = term_bits(T{}, r[k]);
      r[k] -= T::to_f32(static_cast<uint16_t>(b[k]));
    }
    *reinterpret_cast<uint2*>(dst + s * n + i) = make_uint2(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
  }
}

}  // namespace

int contraction_terms(bool bf16) { return bf16 ? 3 : 2; }

namespace {

template <typename T, int NT, int WAVES, bool DEALT>
void launch_split(const float* src, uint16_t* dst, long n, float pre_scale, hipStream_t s) {
  constexpr long kRound = 256L * WAVES * (DEALT ? 8 : 1);        // entries of the workgroups that share out a run of pieces
  const unsigned grid = static_cast<unsigned>((n + kRound - 1) / kRound * (DEALT ? 8 : 1));
  hipLaunchKernelGGL((split_terms_kernel<T, NT, WAVES, DEALT>), dim3(grid), dim3(64 * WAVES), 0, s, src, dst, n, pre_scale);
}

}  // namespace

hipError_t launch_split_terms(const float* src, uint16_t* dst, long n, float pre_scale, bool bf16, hipStream_t s) {
  // Up to 512 x 512 one wave a workgroup (f16 Q^T W 256 x 2048, four waves / one: 8.3 / 8.1 us a call, level at 512), above four, whose launch is
  // shorter (f16 adapter 976 26.7 / 27.3, W Q 992 x 600 17.0 / 17.4).  Dealt above 512 x 512, but for bf16 only up to 1448 x 1448: Q^T W
  // 1536 x 512 28.5 four at a time, 29.0 dealt, 3072 x 512 80.3 / 81.0 (f16 22.3 / 22.3, 54.7 / 54.7, W Q 2048 x 512 25.3 / 24.4), against means over 16
  // allocations of W Q 520 x 1288 38.6 / 38.2, 560 x 1288 40.6 / 38.3, 520 x 1352 46.4 / 45.9 and Q^T W 1280 x 512 26.1 / 26.3.
  // (A run-time size would cost 0.4 us a launch for the implicit arguments.)
  if (n <= 1L << 18) bf16 ? launch_split<BF16, 3, 1, false>(src, dst, n, pre_scale, s) : launch_split<F16, 2, 1, false>(src, dst, n, pre_scale, s);
  else if (!bf16) launch_split<F16, 2, 4, true>(src, dst, n, pre_scale, s);
  else if (n <= 1L << 21) launch_split<BF16, 3, 4, true>(src, dst, n, pre_scale, s);
  else launch_split<BF16, 3, 4, false>(src, dst, n, pre_scale, s);
  return hipGetLastError();
}

namespace {

// Whether 64 x 64 tiles of `count` (at most 32) tiles of 256 x 256 from number `first` run in the kernel whose waves share the
// k-tiles.  It takes 128 KiB of LDS, one workgroup per compute unit where the other fits two, so it is for launches of one round:
// no XCD's share of consecutive parts holds more than 32 (its compute units) that have anything to do.  Up to 16 tiles that is so;
// above, the edges decide.  Whole calls, us, quarters / shared: second moment 2048 x 1536 (21 tiles) 17.6 / 21.8, 4800 x 1792 (28)
// 33.8 / 38.9, fold f16 1024 x 2048 (32) 23.3 / 26.8, bf16 704 x 1400 (18 tiles, up to 36 parts an XCD) 23.4 / 28.8; W Q bf16 264 x 2504
// (20 tiles, up to 28 parts) 87.7 / 53.1.  Two rounds pay only for sums so long that the shorter chain outweighs them: second moment 1536
// wide of 16384 tokens (512 k-tiles) 117 / 108, of 32768 259 / 208, W Q bf16 256 x 8192 (768) 406 / 367; with more than 24 tiles of a
// second moment later (1792 wide: 16384 tokens 102 / 108, 32768 207 / 206, 65536 469 / 399).
// W Q of up to 16 tiles reads its weight along k, 64 bytes a row and k-tile.  Where rows are no whole number of those, pieces straddle cache lines, and
// sharing gains only if the XCDs' equal shares of the parts end with the tiles' columns (columns in fours).  Quarters / shared: bf16 1280 x 680
// 19.6 / 20.5, 768 x 1096 27.3 / 29.7, f16 768 x 1048 19.5 / 20.6, 200 x 2312 34.7 / 36.5; in fours 520 x 904 bf16 23.0 / 21.5, 520 x 1016 f16 18.1 /
// 17.2, 200 x 2008 31.0 / 26.6; whole pieces 1280 x 704 bf16 19.4 / 17.7, 200 x 1088 f16 19.2 / 17.3.  Q^T W of such sizes gains or is level.
template <bool A_KMAJOR>
bool shares_chain(const ContractionArgs& a, long first, long count) {
  const int chain = (a.Kd + kKTile - 1) / kKTile * a.npairs;
  if (chain < kSharedChain) return false;
  if (!A_KMAJOR && count <= 16 && a.Kd % kKTile != 0 && a.tiles_n % 4 != 0) return false;
  if (count <= 16 || chain >= (a.symmetric != 0 && count > 24 ? 1024 : 512)) return true;
  constexpr int kParts = kBigTile / kSmallSide, kTileParts = kParts * kParts;
  const int share = static_cast<int>(count) * kTileParts / 8;    // parts of an XCD, in the kernels' numbering
  TileAt at{};
  for (int part = 0, of_share = 0, busy = 0; part < share * 8; ++part, ++of_share) {
    if (of_share == share) of_share = busy = 0;
    // (once per tile: tile_of walks the bands before it, of which tall products have many)
    if (part % kTileParts == 0) at = tile_of(static_cast<int>(first) + part / kTileParts, a.tiles_m, a.tiles_n, a.symmetric != 0);
    const int m0 = at.m * kBigTile + part % kTileParts / kParts * kSmallSide, n0 = at.n * kBigTile + part % kParts * kSmallSide;
    if (m0 < a.M && n0 < a.N && ++busy > 32) return false;
  }
  return true;
}

// Tiles first .. first + count - 1 (numbered in 256 x 256 tiles) by workgroups of (64 MI) x (64 MI) tiles.
template <typename T, bool A_KMAJOR, int MI, int TERMS = 1>
hipError_t launch_tiles(ContractionArgs a, long first, long count, hipStream_t s) {
  const long parts = count * (4 / MI) * (4 / MI);
  const long grid = (parts + 7) / 8 * 8;
  if (grid > 0x7FFFFFFFL) return hipErrorInvalidValue;
  a.tile0 = static_cast<int>(first);
  a.tiles = static_cast<int>(parts);
  if (MI == 1 && shares_chain<A_KMAJOR>(a, first, count))
    hipLaunchKernelGGL((small_contraction_kernel<T, A_KMAJOR>), dim3(static_cast<unsigned>(grid)), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((contraction_kernel<T, A_KMAJOR, MI, TERMS>), dim3(static_cast<unsigned>(grid)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Time of `count` 256 x 256 tiles on the chip by workgroup tiles of 64 mi, in rounds (the time of one 256 x 256 tile per
// compute unit).  Whole calls by tiles of 64 / 128 / 256, us, Q^T W 2048 deep, f16: 16 tiles 26.9 / 44.5 / 88.1, 32 41.3 / 46.6 / 87.7, 40 59.4 /
// 46.7 / 86.8, 64 70.8 / 52.6 / 89.7, 128 128 / 81.2 / 98.2, 136 145 / 112 / 97.6, 256 244 / 151 / 127; the lines that follow, 32 and 128 tiles, are the same for
// bf16, W Q and adapters.  (Second moments of 129 to about 200 tiles would take less in tiles of 128: 136 tiles, 2048 tokens 58.6 / 67.3.)
double tile_rounds(long count, int mi) {
  if (mi == 4) return static_cast<double>((count + 255) / 256);
  if (mi == 2) return count <= 64 ? 0.5 : 0.7 * ((count + 127) / 128);   // one, two workgroups per compute unit
  return 0.1 + 0.16 * ((count + 15) / 16);
}

constexpr int kTogether = 112;     // k rows from which W Q takes three terms in one pass (launch_shape)

template <typename T, bool A_KMAJOR>
hipError_t launch_shape(ContractionArgs a, hipStream_t s) {
  a.tiles_m = (a.M + kBigTile - 1) / kBigTile;
  a.tiles_n = (a.N + kBigTile - 1) / kBigTile;
  // the operands are addressed with 32-bit byte offsets from their first term
  int ta = 0, tb = 0;
  for (int i = 0; i < a.npairs; ++i) {
    ta = a.pa[i] > ta ? a.pa[i] : ta;
    tb = a.pb[i] > tb ? a.pb[i] : tb;
  }
  a.a_elements = ta * a.a_term_stride + static_cast<long>(a.Kd) * a.M;
  a.b_elements = tb * a.b_term_stride + static_cast<long>(a.Kd) * a.N;
  if (a.a_elements * 2 >= 0x7FFFFFF0L || a.b_elements * 2 >= 0x7FFFFFF0L) return hipErrorInvalidValue;
  const long tiles = a.symmetric ? static_cast<long>(a.tiles_m) * (a.tiles_m + 1) / 2 : static_cast<long>(a.tiles_m) * a.tiles_n;
  // Whole rounds of 256 x 256 tiles (one per compute unit); what is left over by the tile size that takes least time,
  // so that a few last tiles do not keep the chip for a whole round.
  const int forced = tuning().contraction_tiles;   // 0: by size, 1: 128, 2: 256 (tests)
  long big = forced == 0 ? tiles / 256 * 256 : forced == 2 ? tiles : 0;
  const long rest = tiles - big;
  int mi = 2;
  if (forced == 0) {
    mi = 4;
    for (int m : {2, 1})
      if (tile_rounds(rest, m) < tile_rounds(rest, mi)) mi = m;
    if (mi == 4) big = tiles;
  }
  if (big > 0) {
    // A fold's term pairs: the rotation's terms, all of them, each with the weight.  Short sums of three terms keep a pass per term when
    // A is the weight: the longer start (four stages instead of three before the first product) is not won back.  W Q bf16, 65536 rows, us,
    // a pass per term / together: 8 wide 31.8 / 32.3, 96 wide 36.6 / 36.8, 120 wide 39.2 / 38.7, 256 wide 53.7 / 52.0 (Q^T W 8 wide 26.3 / 25.9).
    constexpr int kTerms = std::is_same_v<T, BF16> ? 3 : 2;
    bool fold = a.npairs == kTerms;
    for (int i = 0; fold && i < kTerms; ++i) fold = (A_KMAJOR ? a.pa[i] : a.pb[i]) == i && (A_KMAJOR ? a.pb[i] : a.pa[i]) == 0;
    hipError_t e;
    if constexpr (!A_KMAJOR && kTerms == 2) {    // only folds come here
      e = fold ? launch_tiles<T, A_KMAJOR, 4, kTerms>(a, 0, big, s) : hipErrorInvalidValue;
    } else {
      const bool together = fold && (A_KMAJOR || a.Kd >= kTogether);
      e = together ? launch_tiles<T, A_KMAJOR, 4, kTerms>(a, 0, big, s) : launch_tiles<T, A_KMAJOR, 4>(a, 0, big, s);
    }
    if (e != hipSuccess) return e;
  }
  if (big == tiles) return hipSuccess;
  return mi == 2 ? launch_tiles<T, A_KMAJOR, 2>(a, big, rest, s) : launch_tiles<T, A_KMAJOR, 1>(a, big, rest, s);
}

}  // namespace

hipError_t launch_contraction(ContractionArgs a, bool a_kmajor, bool bf16, hipStream_t s) {
  if (bf16) return a_kmajor ? launch_shape<BF16, true>(a, s) : launch_shape<BF16, false>(a, s);
  return a_kmajor ? launch_shape<F16, true>(a, s) : launch_shape<F16, false>(a, s);
}

}  // namespace larosa
