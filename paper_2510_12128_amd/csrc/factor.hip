// Block-Jacobi preconditioner (Section 3.2, eq. (cholesky factorization)): batched
// Cholesky K_ii = L_i L_i^T of every diagonal block, the explicit inverses L_i^-1 (the
// paper applies the factor as an explicit inverse followed by batched products, Table 2),
// log det of the preconditioner, and the right-hand sides B = [y | L Z].
//
// Products in blocks of 128 x 128, four waves of 64 x 64, on the bf16 matrix cores (an fp32 entry cut into three bf16 numbers without
// loss, see block_gemm); the diagonal blocks on the fp32 ones.
//   Cholesky: left-looking over block columns.  Step k: every block (m, k), m >= k, gets
//     A[m,k] - sum_{j<k} L[m,j] L[k,j]^T in one batched launch over clusters (most of
//     the sum one step ahead, see k_potrf_step); the workgroup that owns the diagonal
//     block factors and inverts it; a second launch multiplies the blocks
//     below by that inverse.
//   Inverse: the binary-tree identity
//     [L11 0; L21 L22]^-1 = [Y11 0; -Y22 L21 Y11, Y22]
//     applied bottom-up over tile ranges, two batched products per level
//     (T = L21 Y11, kept transposed in the still unused upper triangle; Y21 = -Y22 T).
//   The inverse is stored with its mirror image so that both halves of the
//   preconditioner apply, tril(G) r and triu(G) v, stream row-major strips.
// log det of the preconditioner is taken from the STORED inverse, -2 sum log Y_pp, so the
// split of eq. (logdet) holds exactly for the operator PCG really applies.
#include <algorithm>
#include <climits>
#include <cmath>

#include "nugpr_internal.h"

namespace nugpr {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// Blocked storage seen tile by tile: element (r, q) of the 64 x 64 tile (tr, tc) of a square block lies at
// tile_base(ld, tr, tc) + tile_offset(r, q) (= blocked_index(ld, 64 tr + r, 64 tc + q)).  The base is uniform over a
// workgroup and computed once; the offset is a few 32-bit shifts, and with the accumulator coordinates of
// for_each_acc most of it is a compile-time constant.
__device__ __forceinline__ uint64_t tile_base(uint32_t ld, int tr, int tc) {
  return (uint64_t)tr * TILE * ld + (uint64_t)tc * (2 * TILE * BLK_COLS);
}
__device__ __forceinline__ uint32_t tile_offset(int r, int q) {
  return (uint32_t)((q >> 5) * (TILE * BLK_COLS) + (((r >> 4) * 2 + ((q & 31) >> 4)) * FRAG) + (r & 15) * 16 + (q & 15));
}

// Workgroup -> (cluster, item) for a launch with a different number of items for every cluster.  The items of all clusters,
// the largest cluster first, form one list, and each of the 8 dies, to which workgroups go round-robin and which have an
// L2 of their own each, takes a contiguous piece of it: the tiles of a cluster all read the same panel, which then is
// fetched into one L2 (or two, where a piece ends) and not into eight.  The pieces are cut by work, so it makes no difference
// whether the clusters are alike.  (Before: one die per cluster for similar clusters, 14.9 -> 12.8 ms at 128 x 2048 points, and
// every cluster over all dies, workgroups past the end of a cluster leaving at once, for uneven ones, where the last level of
// the inverse of 64 uneven clusters of 4096 points ran at half the rate of the one before it: the valid rows of a block of
// tiles fell on the first dies.)
constexpr int NUM_DIES = 8;
struct Pieces {
  uint32_t from[NUM_DIES + 1];        // die d takes the items from[d] .. from[d + 1] - 1
  unsigned grid() const {
    uint32_t most = 0;
    for (int d = 0; d < NUM_DIES; ++d) most = std::max(most, from[d + 1] - from[d]);
    return most * NUM_DIES;
  }
};
// The clusters come in the order of ClusterInfo::by_size; the one of rank i has the items first[i] - i sub .. first[i + 1] -
// (i + 1) sub - 1 (n ranks with items).  rank, item (inside the cluster): uniform over the workgroup.
// An item may be shared by `parts` workgroups, which follow one another (part: which of them this one is).
__device__ __forceinline__ bool list_item(const Pieces& pieces, const uint32_t* __restrict__ first, uint32_t sub, int n, int id, int& rank, int& item,
                                          uint32_t parts, int& part) {
  const uint32_t die = (uint32_t)id % NUM_DIES;
  uint32_t g = pieces.from[die] + (uint32_t)id / NUM_DIES;
  if (g >= pieces.from[die + 1]) return false;
  part = (int)(g % parts);
  g /= parts;
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = n;                          // the rank lies in lo .. hi - 1: 64 places of it are looked at at a time
  while (hi - lo > 1) {
    const int stride = (hi - lo + 63) / 64, at = lo + lane * stride;
    const bool before = at < hi && first[at] - (uint32_t)at * sub <= g;
    lo += (__popcll(__ballot(before)) - 1) * stride;
    hi = min(hi, lo + stride);
  }
  rank = __builtin_amdgcn_readfirstlane(lo);
  item = (int)__builtin_amdgcn_readfirstlane(g - (first[rank] - (uint32_t)rank * sub));
  return true;
}

// ---------------------------------------------------------------------------
// Block products: a workgroup computes 128 x 128, each of its four waves one 64 x 64 tile
// ---------------------------------------------------------------------------
// acc += OpA[128 x K] OpB[128 x K]^T: wave w works on row tile w / 2 of OpA and w % 2 of OpB.
// The fp32 entries are multiplied on the bf16 matrix cores, whose rate is 16 times that of the fp32 ones: an entry is cut, without
// rounding, into three bf16 numbers h + m + l of 8 bits each (its 24 bits), and of the nine products of two entries the six that
// reach 2^-24 are taken; those left out (m l, l m, l l) are below half an ulp of the product.  The products are exact, the sums
// are kept in fp32.  These matrix cores do not round a sum but cut it, at the place of its largest term, so h h has
// accumulators of its own, whose terms are all alike, and the five small products another set, which is added at the end: rms
// error of a sum of K products in units of 2^-24 of its terms' magnitudes, fp32 instructions / this (probe on this card):
// K = 128 0.46 / 0.20, terms of one sign 2.9 / 1.3; K = 2048 0.47 / 0.17, one sign 11.8 / 4.2 (54 in one set of accumulators).
// A step is 32 columns: two fragments of 1 KiB of each of the sixteen row groups, eight a wave, are loaded a step ahead into
// registers, cut, and put into LDS as three fragments of bf16 each, once for the two waves that read them.  Lane (m, kg) has (row m,
// columns 4 kg .. + 3) of both fragments of a row group: its eight values are the operand of one contraction over 32 columns (of
// which lane takes which columns makes no difference as long as both operands agree).  A wave reads its four row groups of OpA
// and one of OpB after the other, 24 matrix instructions each.  The cutting (vector ALUs, which run beside the bf16 matrix cores,
// unlike beside the fp32 ones) hides behind the matrix instructions of the other workgroup on the compute unit.  The roles are
// swapped (OpB is the row operand of the instruction): lane l ends up with C[row l & 15][columns 4 (l >> 4) .. + 3] of each fragment,
// 16 bytes of a row.
// What bounds it: the bf16 matrix cores work 55 % of the last levels' cycles (clock 1.8 GHz under this load), the vector
// instructions (the cutting, mostly) take 46 % of the issue slots, partly beside them.  The two products of the tree, fp32 instructions / this: 128 x 2048 points 3.9 / 2.45 ms, 64 uneven
// clusters of 4096 points 23.7 / 13.3.  Not kept, whole factorisation of the latter (35.3 ms before RangeScale): every wave cuts what it reads, the fp32 fragments
// loaded straight into LDS, 36.7; cutting placed between the matrix instructions of the same wave, for the second half of a step 39.7
// (registers spill), for its last quarter 36.3; steps beyond a triangular tile multiplied as zeros and not passed over 35.8.
constexpr int stage_bytes(int F) { return 12 * F * 1024; }
// Powers of two for the operands of the products.  The parts of an entry are multiples of its last bit, 2^-149 at least, so every fp32
// number is cut without loss once it is multiplied by 2^23.  With a = alpha + sigma^2 the entries of L are sqrt(a) at most, those of the
// inverse factor Y 1 / sigma, those of the intermediate of the tree T = L Y sqrt(a) / sigma (below 2^12 where fp32 can factor): with sqrt(a)
// brought to 2^UP and 1 / sqrt(a) as well, products of any two and their sums stay below 2^127 for pivots down to 2^-70 a.
// Entries of L and Y between 2^-126 and 2^-100 (d = 20, lengthscale 0.45 of the spread, 142 .. 400 points): rms error of an entry
// without the powers 1.6e-4 to 5.8e-4, with them 1e-7 to 7e-7 as on the fp32 matrix cores; factorisation of 64 uneven clusters of 4096 points
// 35.0 / 35.7 ms.
struct RangeScale {
  static constexpr int UP = 24;
  static constexpr float UP_T = 0x1p24f;
  int l, a, y;                                   // exponents for L, for the block that a multiply starts from, for Y (for T: UP)
  float up_l, up_a, up_y;
};
struct Cut { v4u h, m, l; };                     // eight values each, two in a register
__device__ __forceinline__ Cut cut(const v4f& first, const v4f& second) {
  Cut c;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v2f x = i < 2 ? (v2f){first[2 * i], first[2 * i + 1]} : (v2f){second[2 * i - 4], second[2 * i - 3]};
    uint32_t part[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      part[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, v2bf));
      if (k < 2) {
        x[0] -= __builtin_bit_cast(float, part[k] << 16);
        x[1] -= __builtin_bit_cast(float, part[k] & 0xffff0000u);
      }
    }
    c.h[i] = part[0];
    c.m[i] = part[1];
    c.l[i] = part[2];
  }
  return c;
}
// up: a power of two that this wave's entries are multiplied by before they are cut, so that every fp32 entry is cut without loss (the
// matrix cores take what is below 2^-126 for zero, see RangeScale); the sums carry both operands' powers.
// F = 2: 64 x 64 per workgroup and 32 x 32 per wave (one row tile of either operand, whose fragments the waves load in pairs, F
// each), for launches that would not fill the chip otherwise: a step takes a quarter of the time.
// Columns 16 s0 .. 16 s1 - 1 (whole tiles).  mine: first element of the strip (64 rows of a square block) that this wave loads:
// row tile 0 / 1 of OpA, 0 / 1 of OpB for wave 0 .. 3 (F = 2: OpA, OpA, OpB, OpB).  TRI (of OpA): 0 none; 1 / 2: the tile of column tile diag is
// triangular for row tile 0 (column <= row / >= row is kept), the next one for row tile 1, and the tiles past it / before it count as zero
// whatever is stored there.
template <int TRI, bool SWAP = false, int F = 4>
__device__ __forceinline__ void block_gemm(v4f (&acc)[F][F], const float* mine, int s0, int s1, int diag, unsigned char* stage, float up) {
#if __HIP_DEVICE_COMPILE__
  typedef __attribute__((address_space(3))) v4u* lds_v4u;
  const int lane = threadIdx.x & 63, m = lane & 15, kg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t piece = (uint32_t)(m * 16 + 4 * kg) * 4u;      // (scalar base + 32-bit lane offset: one address register)
  const int n = (s1 - s0) / 2;
  if (n <= 0) return;
  v4f raw[F][2];
  auto load = [&](int q) {
    const float* at = mine + (uint64_t)(s0 / 2 + q) * (TILE * BLK_COLS);
    if (F == 2) at += (w & 1) * 4 * FRAG;
#pragma unroll
    for (int g = 0; g < F; ++g)
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) raw[g][sub] = *reinterpret_cast<const v4f*>(reinterpret_cast<const char*>(at + g * 2 * FRAG + sub * FRAG) + piece);
  };
  // the tile of a step, and whether it counts for row tile t of OpA
  auto tile_at = [&](int q) { return (s0 + 2 * q) >> 2; };
  const int my_diag = diag + (F == 4 ? w : 0);   // (waves 0 and 1 load OpA)
  v4f small[F][F];
#pragma unroll
  for (int g = 0; g < F; ++g)
#pragma unroll
    for (int j = 0; j < F; ++j) small[g][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  lds_v4u mine_lds = (lds_v4u)(stage + F * w * 3 * 1024 + lane * 16);
  const lds_v4u a_lds = (lds_v4u)(stage + F * (w >> 1) * 3 * 1024 + lane * 16), b_lds = (lds_v4u)(stage + (2 * F + F * (w & 1)) * 3 * 1024 + lane * 16);
  auto meet = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  load(0);
#pragma unroll 1
  for (int q = 0; q < n; ++q) {
    const int tile = tile_at(q);
    if (TRI != 0 && w < 2 && tile == my_diag) {
      const int row0 = F == 2 ? 32 * (w & 1) : 0;
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        const int k = 16 * ((s0 + 2 * q + sub) & 3) + 4 * kg;
#pragma unroll
        for (int g = 0; g < F; ++g)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const bool keep = TRI == 1 ? k + i <= row0 + 16 * g + m : k + i >= row0 + 16 * g + m;
            raw[g][sub][i] = keep ? raw[g][sub][i] : 0.f;
          }
      }
    }
#pragma unroll
    for (int g = 0; g < F; ++g)
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) raw[g][sub] *= up;
    Cut mc[F];
#pragma unroll
    for (int g = 0; g < F; ++g) mc[g] = cut(raw[g][0], raw[g][1]);
    if (q > 0) meet();                           // every wave has read step q - 1
#pragma unroll
    for (int g = 0; g < F; ++g) {
      mine_lds[(3 * g) * 64] = mc[g].h;
      mine_lds[(3 * g + 1) * 64] = mc[g].m;
      mine_lds[(3 * g + 2) * 64] = mc[g].l;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (q + 1 < n) load(q + 1);
    meet();
    const int counted = diag + (F == 4 ? w >> 1 : 0);
    if ((TRI == 1 && tile > counted) || (TRI == 2 && tile < counted)) continue;
    Cut a[F], b[2];
    auto get = [&](Cut& c, const lds_v4u from, int f) {
      c.h = from[(3 * f) * 64];
      c.m = from[(3 * f + 1) * 64];
      c.l = from[(3 * f + 2) * 64];
    };
    get(b[0], b_lds, 0);
#pragma unroll
    for (int g = 0; g < F; ++g) get(a[g], a_lds, g);
#pragma unroll
    for (int j = 0; j < F; ++j) {
      if (j + 1 < F) get(b[(j + 1) & 1], b_lds, j + 1);
      const Cut& y = b[j & 1];
      auto mult = [&](const v4u& x, const v4u& z, v4f& to) {
        to = SWAP ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, x), __builtin_bit_cast(v8bf, z), to, 0, 0, 0)
                  : __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, z), __builtin_bit_cast(v8bf, x), to, 0, 0, 0);
      };
#pragma unroll
      for (int g0 = 0; g0 < F; g0 += 2) {
#pragma unroll
        for (int g = g0; g < g0 + 2; ++g) mult(a[g].h, y.h, acc[g][j]);
#pragma unroll
        for (int g = g0; g < g0 + 2; ++g) mult(a[g].l, y.h, small[g][j]);
#pragma unroll
        for (int g = g0; g < g0 + 2; ++g) mult(a[g].h, y.l, small[g][j]);
#pragma unroll
        for (int g = g0; g < g0 + 2; ++g) mult(a[g].m, y.m, small[g][j]);
#pragma unroll
        for (int g = g0; g < g0 + 2; ++g) mult(a[g].m, y.h, small[g][j]);
#pragma unroll
        for (int g = g0; g < g0 + 2; ++g) mult(a[g].h, y.m, small[g][j]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int g = 0; g < F; ++g)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[g][j] += small[g][j];
#endif
}
template <int F>
__device__ __forceinline__ void zero_block(v4f (&acc)[F][F]) {
#pragma unroll
  for (int g = 0; g < F; ++g)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[g][j] = (v4f){0.f, 0.f, 0.f, 0.f};
}
// this lane's four values of fragment (g, j) of a 64 x 64 tile (a uniform pointer and a 32-bit lane offset)
__device__ __forceinline__ v4f* fragment(float* tile, int g, int j) {
  const uint32_t lane = threadIdx.x & 63, at = (lane & 15) * 64 + (lane >> 4) * 16;
  return reinterpret_cast<v4f*>(reinterpret_cast<char*>(tile + ((j >> 1) * (TILE * BLK_COLS) + (g * 2 + (j & 1)) * FRAG)) + at);
}
__device__ __forceinline__ const v4f* fragment(const float* tile, int g, int j) { return fragment(const_cast<float*>(tile), g, j); }
// keeps an address where it is used: per-lane addresses computed ahead of the products cost registers that these need
template <typename P> __device__ __forceinline__ P* here(P* p) {
#if __HIP_DEVICE_COMPILE__
  __attribute__((address_space(1))) P* g = (__attribute__((address_space(1))) P*)p;
  asm volatile("" : "+s"(g));
  p = (P*)g;
#endif
  return p;
}
// (four fragments at a time: with the whole tile's loads in flight at once the accumulators would not stay in registers)
__device__ __forceinline__ void add_tile(v4f (&acc)[4][4], const float* tile) {
  tile = here(tile);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[g][j] += *fragment(tile, g, j);
    __builtin_amdgcn_sched_barrier(0);
  }
}
__device__ __forceinline__ v4f times_power(const v4f& x, int e) {      // 2^e x
  return (v4f){ldexpf(x[0], e), ldexpf(x[1], e), ldexpf(x[2], e), ldexpf(x[3], e)};
}
__device__ __forceinline__ void put_difference(const float* from, const v4f (&acc)[4][4], int down, float* tile) {
  from = here(from);
  tile = here(tile);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int j = 0; j < 4; ++j) *fragment(tile, g, j) = *fragment(from, g, j) - times_power(acc[g][j], down);
    __builtin_amdgcn_sched_barrier(0);
  }
}
__device__ __forceinline__ void put_tile(const v4f (&acc)[4][4], float* tile) {
  tile = here(tile);
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int j = 0; j < 4; ++j) *fragment(tile, g, j) = acc[g][j];
}
// element offset of fragment (g, j)'s first value of this lane in the transposed tile
__device__ __forceinline__ uint32_t block_at_mirrored(int g, int j) {
  const int lane = threadIdx.x & 63;
  return tile_offset(16 * j + 4 * (lane >> 4), 16 * g + (lane & 15));
}

// ---------------------------------------------------------------------------
// Cholesky factor and inverse of one 64 x 64 tile in LDS (256 threads)
// ---------------------------------------------------------------------------
// This is the critical path of a step's launch (the next one needs its result), and it shares its compute unit with
// workgroups that keep the matrix cores busy, which slows every instruction it issues.  So the serial part is small: the
// tile is taken in four panels of 16 columns, a panel is factored by ONE wave in registers (lane = row; pivots and pivot
// rows reach the other lanes by v_readlane, no LDS and no barrier between the pivots), and everything else is 16 x 16 blocks
// on the matrix cores, a block per wave: the left-looking update of a panel's column of blocks, and the blocks of
// L^-1 = [Y11 0; -Y22 L21 Y11, Y22] over blocks, then pairs of blocks.
// Panel, elimination without square roots (A = Lu D Lu^T): pivot j: m_i = a_ij / d_j (i > j), a_ic -= m_i a_cj (c > j);
// then L = Lu D^1/2.  A pivot that is not positive and finite is replaced by 1 and reported.
// Before: 64 pivots of one LDS round trip and one barrier each, the inverse carried along: 37 us a tile on an idle chip, now 12.4.
constexpr int LT = TILE + 1;                    // row stride of a tile in LDS
constexpr int IP = 17;                          // and of an inverted diagonal block
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
// 2^-125 <= d < 2^125: the hardware's reciprocal neither takes nor gives subnormal numbers (a uniform test on the bits, which also
// holds off what is not positive or not finite)
__device__ __forceinline__ bool within_reciprocal(float d) {
  const uint32_t bits = __builtin_bit_cast(uint32_t, d), least = (127u - 125u) << 23, past = (127u + 125u) << 23;
  return bits - least < past - least;
}
// sT: the tile (lower triangle read), replaced by L; block (i, j), i > j, of L^-1 is left where block (j, i) of L would be.
// inv: four 16 x IP inverted diagonal blocks; rdiag: 64 values.  Returns whether a pivot was bad (true for wave 0's threads).
__device__ __forceinline__ bool factor_tile(float (*sT)[LT], float* inv, float* rdiag) {
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, kg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  bool bad = false;
  // inverse of diagonal block q by one wave, beside the next panel: lane m holds column m of it
  auto invert = [&](int q) {
    float l[16], y[16];
    const float r = rdiag[16 * q + m];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      l[u] = sT[16 * q + m][16 * q + u];
      y[u] = u == m ? 1.f : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      y[k] *= lane_value(r, k);
#pragma unroll
      for (int i = k + 1; i < 16; ++i) y[i] = fmaf(-lane_value(l[k], i), y[k], y[i]);
    }
    if (kg == 0) {
#pragma unroll
      for (int u = 0; u < 16; ++u) inv[(16 * q + u) * IP + m] = y[u];
    }
  };
#pragma unroll 1
  for (int p = 0; p < 4; ++p) {
    if (p > 0) {                                // block (w, p) -= sum over the panels before of L(w, q) L(p, q)^T
      if (w >= p) {
        v4f acc;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = sT[16 * w + 4 * kg + i][16 * p + m];
        for (int q = 0; q < p; ++q)
#pragma unroll
          for (int s = 0; s < 4; ++s)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-sT[16 * w + m][16 * q + 4 * s + kg], sT[16 * p + m][16 * q + 4 * s + kg], acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) sT[16 * w + 4 * kg + i][16 * p + m] = acc[i];
      }
      __syncthreads();
    }
    if (w == 0) {
      float a[16], d = 1.f;
#pragma unroll
      for (int u = 0; u < 16; ++u) a[u] = sT[lane][16 * p + u];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        float dj = lane_value(a[j], 16 * p + j), mi;
        if (within_reciprocal(dj)) {            // (one Newton step: 1 ulp, in place of a division's ten dependent instructions)
          float rd = __builtin_amdgcn_rcpf(dj);
          rd = fmaf(fmaf(-dj, rd, 1.f), rd, rd);
          mi = a[j] * rd;
        } else {
          if (!(dj > 0.f) || !(dj < INFINITY)) { bad = true; dj = 1.f; }
          mi = a[j] / dj;
        }
        d = lane == 16 * p + j ? dj : d;
        mi = lane > 16 * p + j ? mi : 0.f;
#pragma unroll
        for (int c = j + 1; c < 16; ++c) a[c] = fmaf(-mi, lane_value(a[j], 16 * p + c), a[c]);
      }
      const float sd = sqrtf(d), rs = 1.f / sd;
      if (lane >= 16 * p) {
#pragma unroll
        for (int u = 0; u < 16; ++u) sT[lane][16 * p + u] = lane == 16 * p + u ? sd : (lane > 16 * p + u ? a[u] * lane_value(rs, 16 * p + u) : 0.f);
        if (lane < 16 * p + 16) rdiag[lane] = rs;
      }
    } else if (w == 1 && p > 0) {
      invert(p - 1);
    }
    __syncthreads();
  }
  if (w == 1) invert(3);
  __syncthreads();
  // acc += X Y for blocks: X row-major at x, Y row-major at y; a product's result enters the next one as its right factor
  // as it stands (component i of lane (m, kg) is element (4 kg + i, m), contraction index 4 kg + i)
  auto mult = [&](const float* x, int ldx, const float* y, int ldy, v4f acc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[m * ldx + 4 * kg + i], y[(4 * kg + i) * ldy + m], acc, 0, 0, 0);
    return acc;
  };
  auto mult_reg = [&](const float* x, int ldx, const v4f& y, v4f acc) {      // acc -= X Y
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-x[m * ldx + 4 * kg + i], y[i], acc, 0, 0, 0);
    return acc;
  };
  const v4f zero = (v4f){0.f, 0.f, 0.f, 0.f};
  auto put = [&](int i, int j, const v4f& v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) sT[16 * j + 4 * kg + e][16 * i + m] = v[e];
  };
  if (w < 2) {                                  // blocks (1, 0) and (3, 2)
    const int j = 2 * w, i = j + 1;
    const v4f t = mult(&sT[16 * i][16 * j], LT, inv + 16 * j * IP, IP, zero);
    put(i, j, mult_reg(inv + 16 * i * IP, IP, t, zero));
  }
  __syncthreads();
  if (w < 2) {                                  // blocks (2, w) and (3, w)
    v4f t2 = mult(&sT[32][16 * w], LT, inv + 16 * w * IP, IP, zero), t3 = mult(&sT[48][16 * w], LT, inv + 16 * w * IP, IP, zero);
    if (w == 0) {
      t2 = mult(&sT[32][16], LT, &sT[0][16], LT, t2);
      t3 = mult(&sT[48][16], LT, &sT[0][16], LT, t3);
    }
    const v4f y2 = mult_reg(inv + 32 * IP, IP, t2, zero);
    const v4f y3 = mult_reg(&sT[32][48], LT, t2, mult_reg(inv + 48 * IP, IP, t3, zero));
    put(2, w, y2);
    put(3, w, y3);
  }
  __syncthreads();
  return bad;
}

// ---------------------------------------------------------------------------
// Cholesky, step k
// ---------------------------------------------------------------------------
// Left-looking over columns of blocks of 128 x 128 (two tiles by two; the last one of a cluster may be one tile), with the
// bulk of every block's update done one step ahead.  The launch of step k has two kinds of workgroups:
//   diagonal  block (k, k): subtract the contribution of block column k - 1 (the only one that was not final when the bulk of
//             this block was computed), then factor and invert the block
//   row m > k two blocks of the same block row, one after the other:
//             finish (m, k): subtract the contribution of block column k - 1, as above;
//             bulk (m, k + 1): L <- A - sum over the block columns < k, all final by now
//             Where there are too few blocks for the chip, the sum is shared by `parts` workgroups of k / parts columns each: the
//             first one as above, the others leave their sums in blocks of the inverse's row m that it does not need yet, in
//             turn even and odd columns, and the finish of the next step adds them up.
// The factorisation of the diagonal block is serial and keeps one workgroup per cluster busy for tens of
// microseconds; with the long products of the NEXT column in the same launch the rest of the chip has work
// meanwhile, where a launch that only finished column k would idle behind its diagonal blocks.
// Grid order = start order: the diagonal blocks of all clusters first, since the launch cannot end before they do.  Finish
// and bulk of a block row share a workgroup because, as workgroups of their own, the short finish ones either
// delay the start of the long ones or wait behind them for a free slot.
// A second launch multiplies the blocks below the diagonal by its inverse.
// What bounds it: the matrix cores and the cutting of their operands (block_gemm), and where a launch is one or two rounds of
// workgroups their number.  Steps and multiplies of 64 uneven clusters of 4096 points: 17.9 ms (fp32 matrix instructions 23.1, tiles of 64
// 33.2), of 128 x 2048 points 3.7 ms (5.1; 5.0).  A block column of 128 needs half as many steps as one of 64, reads the panel L[m, 0:k] half
// as often, and its diagonal workgroup (47 us on an idle chip) is still done before the rows are.
// (Rows past the end of a cluster: zero in the assembled blocks and therefore zero in L; identity in the diagonal tile.)
// the tile in LDS and its inverse (factor_tile) to memory: L lower, the inverse with its mirror image
__device__ __forceinline__ void store_factored(const float (*sT)[LT], const float* inv, float* l, float* y) {
  const int w = threadIdx.x >> 6, i = threadIdx.x & 63;
  const uint32_t at = tile_offset(i, 16 * w);     // one fragment row: 16 floats
#pragma unroll
  for (int u = 0; u < 16; u += 4) {
    float lo[4], yo[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int cc = 16 * w + u + v;
      lo[v] = cc <= i ? sT[i][cc] : 0.f;
      const int r = max(i, cc), q = min(i, cc);
      yo[v] = (r >> 4) == (q >> 4) ? inv[r * IP + (q & 15)] : sT[(q & ~15) + (r & 15)][(r & ~15) + (q & 15)];
    }
    *reinterpret_cast<float4*>(l + at + u) = make_float4(lo[0], lo[1], lo[2], lo[3]);
    *reinterpret_cast<float4*>(y + at + u) = make_float4(yo[0], yo[1], yo[2], yo[3]);
  }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_potrf_step(const ClusterInfo* __restrict__ cl, const float* Kd, float* Lf, float* G, int k, int n_diag, int grid_diag,
                  Pieces pieces, const uint32_t* __restrict__ first, int n_rows, int parts, int parts_before, RangeScale range, PcgState* __restrict__ st) {
  // the stage of the products and, once these are done, the tiles of the diagonal block share one piece of LDS
  __shared__ __attribute__((aligned(1024))) unsigned char stage[stage_bytes(4)];
  static_assert((2 * TILE * LT + 4 * 16 * IP + TILE) * sizeof(float) <= stage_bytes(4), "two tiles and the inverted blocks must fit");
  const int id = (int)blockIdx.x;
  const bool diag = id < grid_diag;
  int rank = id, item = 0, part = 0;
  if (diag) {
    if (id >= n_diag) return;
  } else {
    if (!list_item(pieces, first, (uint32_t)k + 1, n_rows, id - grid_diag, rank, item, (uint32_t)parts, part)) return;
  }
  const int ci = (int)cl[rank].by_size;
  const ClusterInfo c = cl[ci];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), ia = w >> 1, jb = w & 1;
  const int m = diag ? k : k + 1 + item;       // block row of this workgroup
  const int last = (int)c.nt - 1;
  const float* A = Kd + c.koff;
  float* L = Lf + c.koff;
  float* Y = G + c.koff;
  // where part p (1, 2, ..) of the sum for tile (ia, jb) of the block of row m and an even / odd column of blocks waits
  auto part_tile = [&](int column, int p) { return Y + tile_base(c.ld, 2 * m + ia, 2 * (2 * (p - 1) + (column & 1)) + jb); };
  auto strip = [&](int t) { return (const float*)(L + (uint64_t)min(t, last) * TILE * c.ld); };
  v4f acc[4][4];
  zero_block(acc);
#pragma unroll 1
  for (int ahead = part > 0 ? 1 : 0; k > 0; ahead = 1) {      // the block of column k, then (rows) that of column k + 1
    const int col = 2 * (k + ahead) + jb, row = 2 * m + ia;
    zero_block(acc);
    block_gemm<0>(acc, strip(w < 2 ? 2 * m + w : 2 * (k + ahead) + w - 2), ahead ? 8 * (k * part / parts) : 8 * (k - 1),
                  ahead ? 8 * (k * (part + 1) / parts) : 8 * k, 0, stage, range.up_l);
    if (!ahead && row <= last)
      for (int p = 1; p < parts_before; ++p) add_tile(acc, part_tile(k, p));
    if (diag) break;
    if (row <= last && col <= row) {           // (tiles above the diagonal are not part of the factor)
      const uint64_t tb = tile_base(c.ld, row, col);
      // what the products are subtracted from: the bulk result of the step before where there is one, or the assembled block
      if (part > 0) put_tile(acc, part_tile(k + 1, part));
      else put_difference((!ahead && k > 1 ? L : A) + tb, acc, -2 * range.l, L + tb);
    }
    if (ahead) return;
    __syncthreads();                           // the stage is written again
  }
  if (!diag) return;                           // (k = 0: k_potrf_solve reads the assembled block)
  // ---- diagonal block [A00 .; A10 A11]: L00, L00^-1 = Y00;  L10 = A10 Y00^T;  A11 -= L10 L10^T;  L11, Y11;  Y10 = -Y11 L10 Y00 ----
  float (*sT)[LT] = reinterpret_cast<float (*)[LT]>(stage);
  float (*sX)[LT] = sT + TILE;
  float *inv = &sX[TILE][0], *rdiag = inv + 4 * 16 * IP;
  const int lane = tid & 63, mm = lane & 15, kg = lane >> 4;
  const int b = (int)c.b;
  const bool two = 2 * k + 1 <= last;
  __syncthreads();                             // every wave is done with the stage
  const float* base = k > 1 ? L : A;
  if (jb <= ia && 2 * k + ia <= last) {        // wave 0: A00, wave 2: A10, wave 3: A11, which waits in memory
    const uint64_t tb = tile_base(c.ld, 2 * k + ia, 2 * k + jb);
    const int valid = w == 0 ? min(TILE, b - 2 * k * TILE) : TILE;       // (the rows of A10 past the end are zero)
    float (*s)[LT] = w == 0 ? sT : sX;
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const v4f x = *fragment(base + tb, g, j) - times_power(acc[g][j], -2 * range.l);
        if (w == 3) *fragment(L + tb, g, j) = x;
        else {
          const int r = 16 * g + mm, q = 16 * j + 4 * kg;
#pragma unroll
          for (int e = 0; e < 4; ++e) s[r][q + e] = r >= valid || q + e >= valid ? (r == q + e ? 1.f : 0.f) : x[e];
        }
        if (j == 3) __builtin_amdgcn_sched_barrier(0);
      }
  }
  __syncthreads();
  bool bad = factor_tile(sT, inv, rdiag);
  {
    const uint64_t tb = tile_base(c.ld, 2 * k, 2 * k);
    store_factored(sT, inv, L + tb, Y + tb);
  }
  if (two) {
    // blocks of 16 x 16: element (r, q) of block (i, j) of the inverse left by factor_tile
    auto yb = [&](int i, int j) { return i == j ? inv + 16 * i * IP : &sT[16 * j][16 * i]; };
    auto ldy = [&](int i, int j) { return i == j ? IP : LT; };
    v4f l10[4];                                // L10(w, j) = sum over q <= j of A10(w, q) Y00(j, q)^T
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      l10[j] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q <= j; ++q) {
        const float* y = yb(j, q);
        const int ld = ldy(j, q);
#pragma unroll
        for (int s = 0; s < 4; ++s)
          l10[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(sX[16 * w + mm][16 * q + 4 * s + kg], y[mm * ld + 4 * s + kg], l10[j], 0, 0, 0);
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) sX[16 * w + 4 * kg + e][16 * j + mm] = l10[j][e];
    __syncthreads();
    {
      float* lt = L + tile_base(c.ld, 2 * k + 1, 2 * k) + tile_offset(lane, 16 * w);
#pragma unroll
      for (int u = 0; u < 16; u += 4)
        *reinterpret_cast<float4*>(lt + u) = make_float4(sX[lane][16 * w + u], sX[lane][16 * w + u + 1], sX[lane][16 * w + u + 2], sX[lane][16 * w + u + 3]);
    }
    v4f t[4];                                  // column w of blocks of L10 Y00
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int q = w; q < 4; ++q) {
      const float* y = yb(q, w);
      const int ld = ldy(q, w);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          t[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(sX[16 * i + mm][16 * q + 4 * s + kg], y[(4 * s + kg) * ld + mm], t[i], 0, 0, 0);
    }
    __syncthreads();
    {                                          // A11; rows / columns past the cluster's end behave as identity
      const float* from = L + tile_base(c.ld, 2 * k + 1, 2 * k + 1) + tile_offset(lane, 16 * w);
      const int valid = min(TILE, b - (2 * k + 1) * TILE);
#pragma unroll
      for (int u = 0; u < 16; u += 4) {
        const v4f x = *reinterpret_cast<const v4f*>(from + u);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int q = 16 * w + u + e;
          sT[lane][q] = lane >= valid || q >= valid ? (lane == q ? 1.f : 0.f) : x[e];
        }
      }
    }
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j <= w; ++j) {             // row w of blocks of A11
      v4f x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = sT[16 * w + 4 * kg + e][16 * j + mm];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          x = __builtin_amdgcn_mfma_f32_16x16x4f32(-sX[16 * w + mm][16 * q + 4 * s + kg], sX[16 * j + mm][16 * q + 4 * s + kg], x, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) sT[16 * w + 4 * kg + e][16 * j + mm] = x[e];
    }
    __syncthreads();
    if (factor_tile(sT, inv, rdiag)) bad = true;
    {
      const uint64_t tb = tile_base(c.ld, 2 * k + 1, 2 * k + 1);
      store_factored(sT, inv, L + tb, Y + tb);
    }
    // column w of blocks of Y10 = -Y11 (L10 Y00), and its mirror image
    float *yl = Y + tile_base(c.ld, 2 * k + 1, 2 * k), *yu = Y + tile_base(c.ld, 2 * k, 2 * k + 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v4f x = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q <= i; ++q) {
        const float* y = yb(i, q);
        const int ld = ldy(i, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) x = __builtin_amdgcn_mfma_f32_16x16x4f32(-y[mm * ld + 4 * kg + e], t[q][e], x, 0, 0, 0);
      }
      *reinterpret_cast<v4f*>(yu + tile_offset(16 * w + mm, 16 * i + 4 * kg)) = x;
#pragma unroll
      for (int e = 0; e < 4; ++e) yl[tile_offset(16 * i + 4 * kg + e, 16 * w + mm)] = x[e];
    }
  }
  if (bad && tid == 0) atomicMin(&st->bad_cluster, ci);
}

// blocks below the diagonal: L[m,k] <- L[m,k] inv(L[k,k])^T
template <int F>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(F == 4 ? 2 : 4)))
void k_potrf_solve(const ClusterInfo* __restrict__ cl, const float* Kd, float* Lf, const float* G, int k, Pieces pieces,
                   const uint32_t* __restrict__ first, int n_rows, RangeScale range) {
  __shared__ __attribute__((aligned(1024))) unsigned char stage[stage_bytes(F)];
  int rank, item, part;
  if (!list_item(pieces, first, (uint32_t)k + 1, n_rows, (int)blockIdx.x, rank, item, F == 2 ? 2u : 1u, part)) return;
  const ClusterInfo c = cl[cl[rank].by_size];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ia = w >> 1, jb = w & 1, lane = threadIdx.x & 63;
  const int m = k + 1 + item, last = (int)c.nt - 1;
  float* L = Lf + c.koff;
  const float* from = k == 0 ? Kd + c.koff : L;
  // OpA = the inverse (columns of the result), OpB = the block's rows
  if (F == 2) {
    // a workgroup per row tile (its two column tiles read the same rows, in place: one after the other, the second first)
    const int row = 2 * m + part;
    if (row > last) return;
#pragma unroll 1
    for (int q = 1; q >= 0; --q) {
      v4f acc[F][F];
      zero_block(acc);
      block_gemm<1, true, F>(acc, w < 2 ? G + c.koff + (uint64_t)(2 * k + q) * TILE * c.ld : from + (uint64_t)row * TILE * c.ld, 8 * k, 8 * k + 4 * q + 4,
                             2 * k + q, stage, w < 2 ? range.up_y : range.up_a);
      __syncthreads();                         // the stage is written again
      float* lt = L + tile_base(c.ld, row, 2 * k + q);
#pragma unroll
      for (int g = 0; g < F; ++g)
#pragma unroll
        for (int j = 0; j < F; ++j)
          *reinterpret_cast<v4f*>(lt + tile_offset(32 * jb + 16 * j + (lane & 15), 32 * ia + 16 * g + 4 * (lane >> 4))) = times_power(acc[g][j], -(range.a + range.y));
    }
    return;
  }
  v4f acc[F][F];
  zero_block(acc);
  block_gemm<1, true, F>(acc, w < 2 ? G + c.koff + (uint64_t)(2 * k + w) * TILE * c.ld : from + (uint64_t)min(2 * m + w - 2, last) * TILE * c.ld,
                         8 * k, 8 * (k + 1), 2 * k, stage, w < 2 ? range.up_y : range.up_a);
  if (2 * m + jb > last) return;
  float* lt = L + tile_base(c.ld, 2 * m + jb, 2 * k + ia);
#pragma unroll
  for (int g = 0; g < F; ++g)
#pragma unroll
    for (int j = 0; j < F; ++j)
      *reinterpret_cast<v4f*>(lt + tile_offset(16 * j + (lane & 15), 16 * g + 4 * (lane >> 4))) = times_power(acc[g][j], -(range.a + range.y));
}

// ---------------------------------------------------------------------------
// triangular inverse, one tree level (half = tiles per child)
// ---------------------------------------------------------------------------
// T = L21 Y11 and Y21 = -Y22 T, T kept transposed in the upper triangle of L's storage, which nothing else uses, and Y21
// written with its mirror image: the next level reads Y11 transposed, and both operands of every product are then
// row-major strips.  Blocks of 128 x 128 (half is even, so a block's columns are whole; its second row tile may be missing).
// STAGE 1: T^T[n][m] over the columns tn ..; longest products (small tn) first.  STAGE 2: Y21[m][n] over the columns up to
// tm; longest (large tm) first.
// F = 2: four workgroups an item, each one 64 x 64 tile of the block.
template <int STAGE, int F>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(F == 4 ? 2 : 4)))
void k_trtri_block(const ClusterInfo* __restrict__ cl, float* Lf, float* G, int half, Pieces pieces,
                   const uint32_t* __restrict__ first, int n, RangeScale range) {
  __shared__ __attribute__((aligned(1024))) unsigned char stage[stage_bytes(F)];
  int rank, item, part;
  if (!list_item(pieces, first, 0u, n, (int)blockIdx.x, rank, item, F == 2 ? 4u : 1u, part)) return;
  const ClusterInfo c = cl[cl[rank].by_size];
  const int hb = half / 2, node = item / (hb * hb), within = item % (hb * hb), last = (int)c.nt - 1;
  const int start = node * 2 * half, mid = start + half;
  const int rows = min(hb, (last - mid) / 2 + 1);                 // block rows of this node
  int tm = mid + 2 * (STAGE == 1 ? within % rows : rows - 1 - within / hb), tn = start + 2 * (STAGE == 1 ? within / rows : within % hb);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ia = w >> 1, jb = w & 1;
  float* L = Lf + c.koff;
  float* Y = G + c.koff;
  auto strip = [&](const float* base, int t) { return base + (uint64_t)min(t, last) * TILE * c.ld; };
  v4f acc[F][F];
  zero_block(acc);
  if (F == 2) {
    tm += part >> 1;
    tn += part & 1;
    if (tm > last) return;
  }
  // the wave's tiles, and (F = 2) its fragments in them
  const int am = F == 2 ? 0 : STAGE == 1 ? jb : ia, an = F == 2 ? 0 : STAGE == 1 ? ia : jb, fa = F == 2 ? 2 * ia : 0, fb = F == 2 ? 2 * jb : 0;
  if (STAGE == 1) {
    block_gemm<2, false, F>(acc, w < 2 ? strip(Y, F == 2 ? tn : tn + w) : strip(L, F == 2 ? tm : tm + w - 2), 4 * tn, 4 * mid, tn, stage,
                            w < 2 ? range.up_y : range.up_l);
    if (tm + am > last) return;
    float* tt = here(L + tile_base(c.ld, tn + an, tm + am));
#pragma unroll
    for (int g = 0; g < F; ++g)
#pragma unroll
      for (int j = 0; j < F; ++j) *fragment(tt, fa + g, fb + j) = times_power(acc[g][j], -(range.y + range.l));
  } else {
    block_gemm<1, false, F>(acc, w < 2 ? strip(Y, F == 2 ? tm : tm + w) : strip(L, F == 2 ? tn : tn + w - 2), 4 * mid,
                            4 * (min(F == 2 ? tm : tm + 1, last) + 1), tm, stage, w < 2 ? range.up_y : RangeScale::UP_T);
    if (tm + am > last) return;
    float *yl = Y + tile_base(c.ld, tm + am, tn + an), *yu = Y + tile_base(c.ld, tn + an, tm + am);
#pragma unroll
    for (int g = 0; g < F; ++g)
#pragma unroll
      for (int j = 0; j < F; ++j) {
        const v4f y = times_power(-acc[g][j], -(range.y + RangeScale::UP));
        *fragment(yl, fa + g, fb + j) = y;
        float* to = yu + block_at_mirrored(fa + g, fb + j);
#pragma unroll
        for (int i = 0; i < 4; ++i) to[16 * i] = y[i];
      }
  }
}

// upper triangle <- transpose of the lower triangle (tile list of the assembly kernels)
__global__ __launch_bounds__(256) void k_mirror(const ClusterInfo* __restrict__ cl, const uint64_t* __restrict__ tiles,
                                                float* __restrict__ G) {
  __shared__ float sT[TILE][TILE + 1];
  const uint64_t t = tiles[blockIdx.x];
  const int ci = (int)(t >> 32), tr = (int)((t >> 16) & 0xffff), tc = (int)(t & 0xffff);
  const ClusterInfo c = cl[ci];
  float* Y = G + c.koff;
  const int tid = threadIdx.x;

  const float* ys = Y + tile_base(c.ld, tr, tc);
  float* yd = Y + tile_base(c.ld, tc, tr);
  for (int idx = tid; idx < TILE * TILE; idx += 256) {
    const int r = idx >> 6, q = idx & 63;
    sT[r][q] = ys[tile_offset(r, q)];
  }
  __syncthreads();
  for (int idx = tid; idx < TILE * TILE; idx += 256) {
    const int r = idx >> 6, q = idx & 63;      // element (r, q) of the destination tile
    if (tr != tc || q > r) yd[tile_offset(r, q)] = sT[q][r];
  }
}

// upper tiles of one square blocked matrix of nt x nt tiles <- transposes of the lower ones (1-D grid of nt * nt)
__global__ __launch_bounds__(256) void k_mirror_square(float* __restrict__ M, uint32_t ld, int nt) {
  __shared__ float sT[TILE][TILE + 1];
  const int tr = (int)(blockIdx.x / (unsigned)nt), tc = (int)(blockIdx.x % (unsigned)nt);
  if (tc >= tr) return;
  const int tid = threadIdx.x;
  const float* ms = M + tile_base(ld, tr, tc);
  float* md = M + tile_base(ld, tc, tr);
  for (int idx = tid; idx < TILE * TILE; idx += 256) {
    const int r = idx >> 6, q = idx & 63;
    sT[r][q] = ms[tile_offset(r, q)];
  }
  __syncthreads();
  for (int idx = tid; idx < TILE * TILE; idx += 256) {
    const int r = idx >> 6, q = idx & 63;
    md[tile_offset(r, q)] = sT[q][r];
  }
}

int ensure_c_upper(nugpr_ctx* c, hipStream_t s) {
  if (c->c_upper_valid || !c->built) return NUGPR_OK;
  const int nt = c->L.ldc / TILE;
  hipLaunchKernelGGL(k_mirror_square, dim3((unsigned)nt * (unsigned)nt), dim3(256), 0, s, c->C, (uint32_t)c->L.ldc, nt);
  NUGPR_HIP(hipGetLastError());
  c->c_upper_valid = true;
  return NUGPR_OK;
}

int ensure_kd_upper(nugpr_ctx* c, hipStream_t s) {
  if (c->kd_upper_valid || !c->built) return NUGPR_OK;
  hipLaunchKernelGGL(k_mirror, dim3((unsigned)c->L.n_diag_tiles), dim3(256), 0, s, c->d_cl, c->d_tiles, c->Kd);
  NUGPR_HIP(hipGetLastError());
  c->kd_upper_valid = true;
  return NUGPR_OK;
}

// log det of the preconditioner of one cluster from the stored inverse diagonal
__global__ __launch_bounds__(256) void k_logdet(const ClusterInfo* __restrict__ cl, const float* __restrict__ G,
                                                double* __restrict__ out) {
  __shared__ double red[256];
  const ClusterInfo c = cl[blockIdx.x];
  const float* Y = G + c.koff;
  double s = 0.0;
  for (uint32_t p = threadIdx.x; p < c.b; p += 256) s += log((double)Y[blocked_index(c.ld, p, p)]);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = -2.0 * red[0];
}

__global__ void k_reset_bad(PcgState* st) { st->bad_cluster = INT_MAX; }

// V = [0 | Z] (n x T) from the probes (n x t)
template <typename VT>
__global__ void k_probes_to_block(const float* __restrict__ Z, VT* __restrict__ V, int64_t n, int t) {
  const int T = t + 1;
  const int64_t total = n * T;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = idx / T;
    const int col = (int)(idx - p * T);
    V[idx] = col == 0 ? (VT)0 : (VT)Z[p * t + col - 1];
  }
}

template <typename VT>
__global__ void k_set_col0(VT* __restrict__ B, const float* __restrict__ y, int64_t n, int T) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x)
    B[p * T] = (VT)y[p];
}

// Diagonal blocks of the compensated matrix (eq. (kypp)) with the one-hot basis: tile (tr, tc), tc <= tr, of
// cluster ci gets  K_ii[p][q] + Cc[a(p)][a(q)],  a(p) = the row of the coupling matrix that point p belongs to and
// Cc = C - lambda_0 I as stored (same-cluster entries kept, float(alpha - lambda_0) on the diagonal).  Reads the
// lower triangle of Cc element-wise (row >= column), which every storage mode keeps.  One workgroup per tile of
// the assembly's tile list; writes the spare blocks, where the factorisation then runs in place.
__global__ __launch_bounds__(256) void k_compensated_blocks(const ClusterInfo* __restrict__ cl,
                                                            const uint64_t* __restrict__ tiles,
                                                            const float* __restrict__ Kd, float* __restrict__ out,
                                                            const float* __restrict__ Cc, uint32_t ldc,
                                                            const int32_t* __restrict__ assign) {
  __shared__ int32_t ar[TILE], ac[TILE];
  const uint64_t t = tiles[blockIdx.x];
  const int ci = (int)(t >> 32), tr = (int)((t >> 16) & 0xffff), tc = (int)(t & 0xffff);
  const ClusterInfo c = cl[ci];
  const int tid = threadIdx.x;
  if (tid < TILE) {
    const uint32_t p = (uint32_t)(tr * TILE + tid);
    ar[tid] = p < c.b ? assign[c.row0 + p] : -1;
  } else if (tid < 2 * TILE) {
    const uint32_t q = (uint32_t)(tc * TILE + tid - TILE);
    ac[tid - TILE] = q < c.b ? assign[c.row0 + q] : -1;
  }
  __syncthreads();
  const uint64_t tb = tile_base(c.ld, tr, tc);
  for (int idx = tid; idx < TILE * TILE; idx += 256) {
    const int r = idx >> 6, q = idx & 63;
    const uint32_t at = tile_offset(r, q);
    float v = Kd[c.koff + tb + at];
    const int a = ar[r], b = ac[q];
    if (a >= 0 && b >= 0) v += Cc[blocked_index(ldc, (uint32_t)max(a, b), (uint32_t)min(a, b))];
    out[c.koff + tb + at] = v;
  }
}

// Up to this many blocks of 128 x 128 in a launch leave half of the compute units idle: tiles of 64 x 64 then.
constexpr uint64_t FEW_BLOCKS = 128;

// How many workgroups share the bulk of a block (k_potrf_step's parts).  The chip holds 512 workgroups, two on a compute unit, which
// then share its matrix cores; what counts is how full the last round is.  A workgroup alone on its unit takes four fifths of the
// time that two take; the block of column k and both ends of a workgroup cost as much as 45 half steps (16 columns).  64 uneven clusters
// of 4096 points, whole factorisation: with sums never shared 40.6 ms, with the line of the fp32 instructions (768 workgroups, 14 half
// steps) 35.8, with 20 / 45 / 70 half steps 35.4 / 35.3 / 35.5.
static int bulk_parts(uint64_t items, int k) {
  int best = 1;
  double least = 0.0;
  for (int p = 1; p <= 8 && (p == 1 || 2 * p <= k); ++p) {
    const uint64_t n = items * (uint64_t)p, left = (n % 512 + 255) / 256;
    const double units = 2.0 * (double)(n / 512) + (left == 0 ? 0.0 : left == 1 ? 1.6 : 2.0);
    const double cost = units * (8.0 * k / p + 45.0);
    if (p == 1 || cost < least) { best = p; least = cost; }
  }
  return best;
}

static RangeScale range_scale(const nugpr_ctx* c) {
  const double a = c->theta_built[c->L.p - 2] + c->theta_built[c->L.p - 1];
  const int e = a > 0.0 && std::isfinite(a) ? std::max(-126, std::min(128, std::ilogb(a))) : 0;
  RangeScale r;
  r.l = RangeScale::UP - e / 2;
  r.a = std::min(RangeScale::UP - e, 120);
  r.y = RangeScale::UP + e / 2;
  r.up_l = std::ldexp(1.f, r.l);
  r.up_a = std::ldexp(1.f, r.a);
  r.up_y = std::ldexp(1.f, r.y);
  return r;
}

int launch_factor(nugpr_ctx* c, hipStream_t s) {
  const Layout& L = c->L;
  c->Lf = c->Kd2;                 // the factor goes into the spare blocks (see nugpr_ctx::lf_valid)
  c->lf_valid = true;
  // what is factored: the assembled K_ii, or (NUGPR_PRECOND_COMPENSATED) the diagonal blocks of K'' formed in the
  // spare blocks, where the factorisation then runs in place (every tile is read before it is written)
  const float* Afac = c->Kd;
  if (c->params.flags & NUGPR_PRECOND_COMPENSATED) {
    if (!c->onehot) { set_error("NUGPR_PRECOND_COMPENSATED needs the default one-hot basis"); return NUGPR_ERR_STATE; }
    hipLaunchKernelGGL(k_compensated_blocks, dim3((unsigned)L.n_diag_tiles), dim3(256), 0, s, c->d_cl, c->d_tiles, c->Kd,
                       c->Kd2, c->C, (uint32_t)L.ldc, c->assign);
    Afac = c->Kd2;
  }
  hipLaunchKernelGGL(k_reset_bad, dim3(1), dim3(1), 0, s, c->d_state);
  // (ranks are by size: the clusters with more than k block columns are the first ones)
  const int n_blocks = (L.ntmax + 1) / 2;
  auto with_blocks = [&](int least) {
    return (int)(std::partition_point(L.blocks_by_rank.begin(), L.blocks_by_rank.end(), [&](uint32_t nb) { return (int)nb >= least; }) - L.blocks_by_rank.begin());
  };
  int parts_before = 1;
  const RangeScale range = range_scale(c);
  for (int k = 0; k < n_blocks; ++k) {
    const int n_diag = with_blocks(k + 1), grid_diag = (n_diag + NUM_DIES - 1) / NUM_DIES * NUM_DIES, n_rows = with_blocks(k + 2);
    const uint64_t items = L.rows_before[n_rows] - (uint64_t)n_rows * (uint64_t)(k + 1);
    const int parts = items ? bulk_parts(items, k) : 1;
    Pieces pr, ps;
    for (int d = 0; d <= NUM_DIES; ++d) { pr.from[d] = (uint32_t)(items * parts * d / NUM_DIES); ps.from[d] = (uint32_t)(items * d / NUM_DIES); }
    hipLaunchKernelGGL(k_potrf_step, dim3((unsigned)grid_diag + (k > 0 ? pr.grid() : 0u)), dim3(256), 0, s, c->d_cl, Afac, c->Lf, c->G, k,
                       n_diag, grid_diag, pr, c->d_rows_before, n_rows, parts, parts_before, range, c->d_state);
    if (items > FEW_BLOCKS) hipLaunchKernelGGL((k_potrf_solve<4>), dim3(ps.grid()), dim3(256), 0, s, c->d_cl, Afac, c->Lf, c->G, k, ps, c->d_rows_before, n_rows, range);
    else if (items) {
      for (int d = 0; d <= NUM_DIES; ++d) ps.from[d] = (uint32_t)(2 * items * d / NUM_DIES);
      hipLaunchKernelGGL((k_potrf_solve<2>), dim3(ps.grid()), dim3(256), 0, s, c->d_cl, Afac, c->Lf, c->G, k, ps, c->d_rows_before, n_rows, range);
    }
    parts_before = parts;
  }
  for (const TreeLevel& t : L.tree) {
    const bool few = t.from1[NUM_DIES] <= FEW_BLOCKS;
    Pieces p1, p2;
    for (int d = 0; d <= NUM_DIES; ++d) { p1.from[d] = t.from1[d] * (few ? 4 : 1); p2.from[d] = t.from2[d] * (few ? 4 : 1); }
    const uint32_t* first = c->d_rows_before + t.at;
    if (few) {
      hipLaunchKernelGGL((k_trtri_block<1, 2>), dim3(p1.grid()), dim3(256), 0, s, c->d_cl, c->Lf, c->G, t.half, p1, first, t.ranks, range);
      hipLaunchKernelGGL((k_trtri_block<2, 2>), dim3(p2.grid()), dim3(256), 0, s, c->d_cl, c->Lf, c->G, t.half, p2, first, t.ranks, range);
    } else {
      hipLaunchKernelGGL((k_trtri_block<1, 4>), dim3(p1.grid()), dim3(256), 0, s, c->d_cl, c->Lf, c->G, t.half, p1, first, t.ranks, range);
      hipLaunchKernelGGL((k_trtri_block<2, 4>), dim3(p2.grid()), dim3(256), 0, s, c->d_cl, c->Lf, c->G, t.half, p2, first, t.ranks, range);
    }
  }
  hipLaunchKernelGGL(k_logdet, dim3(L.nc), dim3(256), 0, s, c->d_cl, c->G, c->d_logdet);
  NUGPR_HIP(hipGetLastError());
  // right-hand sides B = [y | L Z]
  if (L.t > 0) {
    if (c->acc64)
      hipLaunchKernelGGL((k_probes_to_block<double>), dim3(1024), dim3(256), 0, s, c->probes, (double*)c->Pv, (int64_t)L.n, L.t);
    else
      hipLaunchKernelGGL((k_probes_to_block<float>), dim3(1024), dim3(256), 0, s, c->probes, (float*)c->Pv, (int64_t)L.n, L.t);
    StripPort p0{};
    p0.A = c->Lf; p0.in = c->Pv; p0.out = c->Bv;
    int rc = launch_strip(c->tab_lowL, p0, p0, L.T, c->acc64, s);
    if (rc) return rc;
  }
  if (c->acc64) hipLaunchKernelGGL((k_set_col0<double>), dim3(1024), dim3(256), 0, s, (double*)c->Bv, c->y, (int64_t)L.n, L.T);
  else hipLaunchKernelGGL((k_set_col0<float>), dim3(1024), dim3(256), 0, s, (float*)c->Bv, c->y, (int64_t)L.n, L.T);
  NUGPR_HIP(hipGetLastError());
  // z_0 = M^-1 B of every later solve on these right-hand sides (x_0 = 0, so r_0 = B whatever theta is)
  c->z0_ready = false;
  int rc = run_precond(c, c->Bv, c->Z0v, L.T, s);
  if (rc) return rc;
  if ((rc = store_known_starts(c, s))) return rc;
  c->z0_ready = true;
  c->factor_gen = c->build_gen;
  c->stats.factorisations += 1;
  return NUGPR_OK;
}

}  // namespace nugpr
