// Strip GEMM: the product of a stored fp32 matrix strip (64 rows,
// any number of columns) with a tall-skinny vector block of T <= 33 columns.
//
// Every matrix of the hot path is applied through this one kernel:
//   K_ii D_i, C S (coupling), W_i^T D_i, W_i P_i        -- the block-low-rank product
//                                                          K' D of eq. (odsplit), Section 3.3
//   tril(L_i^-1) R_i, triu(L_i^-T) V_i                   -- the block-Jacobi preconditioner,
//                                                          applied as explicit inverses (Table 2)
//   tril(L_i) Z_i                                        -- probe right-hand sides
//
// One workgroup = one item (a strip of 64 rows and a column range), four waves.  The CONTRACTION is split among
// the waves: of every 64-column tile each wave takes 16 columns, for all 64 rows and all T columns, so a wave
// depends on no other one until the strip is done (no barrier in the loop; any number of tiles divides evenly
// among the waves) and a vector operand serves four 16-row groups.  The four partial sums meet in LDS at the end,
// in a fixed order, and the 64 x T result is written as one contiguous run.
// A step (16 columns): lane (m, kg) of a wave holds float4 A[row 16 g + m][4 kg ..] for the four row groups g; the
// four components feed four 16x16x4 MFMAs whose contraction index is the lane's kg.  Columns 1..T-1 go through the
// matrix cores in groups of 16; column 0 (y) rides on the vector ALUs from the same registers, so T = 17 costs one
// MFMA group, not two.
// Operands: the matrix goes from memory straight into registers, STAGES steps ahead (7 KiB a step and wave); the
// step's 16 vector rows arrive as contiguous 16-byte loads and take their operand order through a piece of LDS that
// belongs to the wave.  Loads past the last tile are issued out of range instead of being skipped: the number in
// flight is what the waits count.  Such a load still costs the address unit its 25 - 30 cycles, so the loop refills
// only while a whole turn of it remains, and a strip of few tiles wants few stages.
//
// What bounds it.  fp64: the matrix cores and the vector ALUs share one pipe (16 MFMAs x 64 cycles and 32 vector
// instructions a step: 550 ns at the sustained clock, measured without any memory access); 1 - 17 columns also the
// traffic behind the L2s.  Before (a loader wave feeding an LDS ring with one workgroup barrier per 32 columns, the
// strip's rows split among the waves) the barrier -> LDS -> MFMA chain left a fifth of the issue slots empty.
// 128 clusters of 2048 points, 128 representatives each, 17 columns: 556 -> 500 us, and the whole product 550 -> 534 us
// since the loop no longer refills past its last turn; 64 uneven clusters of 4096 points on average, 33 columns:
// 2297 -> 1870 us; preconditioner strips, 64 x 2048, 17 columns: 112 -> 108 us (4.9 TB/s of HBM); fp32 mode, 64 x 2048,
// 17 columns: whole squares -> lower tiles (see below).
// Tried and not kept: vector operands loaded in operand order from memory (the address unit takes 25 - 30 cycles
// for a load whatever its width: 640 us); workgroups that stay and take item after item (741 us), or whose start is
// staggered (580 us): both take the partner strips below out of step.
// Short triangular strips (clusters of up to about 1024 points) spend their time at the two ends, so what counts is how
// many workgroups a compute unit holds: two stages, the vector operands made ready when they are needed, and with two
// column groups two row groups a wave, which leaves four waves per SIMD in place of two.  With the long strips' two waves
// x four stages and streaming loads for every size, clusters this small were slower than under the loader wave.
// Preconditioner apply, fp64, 17 columns, loader wave / two waves x four stages / now: 2000 clusters of 64 points
// 48 / 60 / 46 us, 600 uneven ones of 100 35 / 48 / 38, 300 uneven ones of 200 41 / 53 / 42, 256 x 512 94 / 108 / 90,
// 32 x 1024 50 / 52 / 42; 33 columns 69 / 83 / 64, 50 / 63 / 52, 57 / 71 / 58, 146 / 154 / 126, 77 / 76 / 66.
//
// Two arithmetic modes, same data movement:
//   ACC64 = true   vector blocks are fp64; the fp32 matrix entries are widened in
//                  registers and contracted with v_mfma_f64_16x16x4_f64: products and
//                  sums carry no fp32 rounding at all.
//   ACC64 = false  vector blocks are fp32; v_mfma_f32_16x16x4_f32 in one chain of 16 columns
//                  per row and column group, folded into fp64 sums after every step.
// The CG coefficients and the SLQ estimate are Rayleigh quotients of these products
// scaled by n, so rounding in the running sums enters the loss at first order; the fp64
// mode removes it, the fp32 mode keeps it near sqrt(b) * 1e-7 per output entry.
//
// Strips of a symmetric matrix (StripItem::blocked bit 1).  The item's columns are the tiles of a square super-block
// whose rows are a group of `na` strips (0: the tile range of the item itself); the item is strip number jr of that
// group.  It visits its tiles in the rotating order p = (u - jr) mod the number of tiles.  A super-block on the
// diagonal of the matrix (kind 0: a cluster's K_ii, or a diagonal block of C) takes tile p from the strip's own rows
// when p <= jr and as the TRANSPOSE of the stored tile (p, strip) when p > jr; one below the diagonal (kind 1)
// always reads its own rows, one above it (kind 2) always the transposed tiles of its mirror image.  The partner
// strip visits the same stored tile at the same step, the two workgroups are dealt to the same die and start
// together, so the two requests for the same 16 KiB meet in that die's L2 and memory serves one: the lower triangle
// is streamed, the upper one is never read (and need not have been written).  A transposed tile passes the wave's
// LDS: each lane fetches the 16-byte piece (row 4 ((l / 4) % 4) + l / 16, columns 4 (l % 4) ..) of the stored
// fragment, which puts element (4 kg + i, m) at float 64 i + 16 kg + m, so both accesses have unit stride.
#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "nugpr_internal.h"

namespace nugpr {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));
typedef double v4d __attribute__((ext_vector_type(4)));

template <bool ACC64> struct VecT { typedef float type; };
template <> struct VecT<true> { typedef double type; };

// row of the 16x16 accumulator tile held in component i of lane `lane`:
// f32 16x16x4 keeps rows 4*(lane/16) + i, f64 16x16x4 keeps rows (lane/16) + 4*i
template <bool ACC64>
__device__ __forceinline__ int acc_row(int lane, int i) {
  return ACC64 ? (lane >> 4) + 4 * i : 4 * (lane >> 4) + i;
}

constexpr int NW = 4;                  // waves of a workgroup
// What the items of a table are.  STRIP_STREAMED (added to the first and the last): matrix loads with the streaming hint.
// STRIP_MANY (added to the symmetric ones): up to 16 tiles a strip, more workgroups than three on a compute unit.
// STRIP_QUARTERS (added to symmetric and short ones): four workgroups a strip, one for each of its 16-row groups, where the
// strips are too few for the chip: a wave's serial chain of matrix instructions is a quarter as long.
enum { STRIP_LONG = 0, STRIP_SYM = 1, STRIP_ROWMAJOR = 2, STRIP_SHORT = 3, STRIP_STREAMED = 4, STRIP_MANY = 8, STRIP_QUARTERS = 16 };
template <int NG, bool ACC64, int KIND> struct WaveCfg {
  typedef typename VecT<ACC64>::type VT;
  static constexpr int BASE = KIND & 3;
  static constexpr bool SHORT = (BASE == STRIP_SHORT && !(KIND & STRIP_QUARTERS)) || (KIND & STRIP_MANY) != 0;
  // Waves per SIMD and steps in flight, as the registers allow.  Symmetric strips in fp64 with one column group: 3
  // waves x 3 stages 500 us, 2 x 4 527 us (workload in the file's head); long strips without partners, which stream from
  // HBM: 2 x 4 108 us, 3 x 3 117 us.  Short strips: see the file's head.
  static constexpr bool QUARTERS = (KIND & STRIP_QUARTERS) != 0;
  static constexpr int WAVES_PER_EU = QUARTERS ? 2 : SHORT ? (NG == 1 && !ACC64 ? 3 : 4) : BASE == STRIP_SYM && ACC64 && NG == 1 ? 3 : 2;
  static constexpr int STAGES = QUARTERS ? 4 : SHORT || (NG == 2 && !ACC64) ? 2 : (WAVES_PER_EU == 3 || NG == 2 ? 3 : 4);
  // Row groups of a wave: all four with a quarter of a tile's columns, or two with half of them (short strips of two
  // column groups: half the accumulators, so that four waves fit; the vector rows are then read twice)
  static constexpr int ROW_GROUPS = QUARTERS ? 1 : BASE == STRIP_SHORT && NG == 2 ? 2 : 4;
  static constexpr int SHARES = ROW_GROUPS == 2 ? 2 : 4;         // waves that share a row's columns
  // the vector operands of the next step are made ready while the matrix cores work on the present one
  static constexpr bool AHEAD = !SHORT;
  static constexpr int NB = NG > 0 ? NG : 1;
  // 16-byte loads per lane that cover the vector rows of a step (16 rows of at most 16 NG + 1 columns; with one column the
  // lane's own four rows, which are contiguous)
  static constexpr int NV = NG > 0 ? (16 * (16 * NG + 1) * (int)sizeof(VT) + 1023) / 1024 : (int)sizeof(VT) / 4;
  static constexpr int TURN_LDS = BASE == STRIP_SYM ? 4096 : 0;  // a wave's LDS: a tile on its way to its transpose,
  static constexpr int WAVE_LDS = TURN_LDS + NV * 1024;          // vector rows
};

// Whether one of the tiles tb .. tb + nb - 1 of row j of the coupling matrix holds a value: those between clusters further apart than the
// kernel reaches hold none, and an item without any, whose vector rows are finite, only clears its slab.  Product of 17 columns, 128
// clusters of 2048 points in 20 dimensions with 128 representatives each, a third of whose tiles are the coupling's, 22 of 65536 with a
// value at a lengthscale of 1: 533 / 402 us.  Items of up to three tiles are not looked at (the words arrive no sooner than a tile does:
// 4 x 512 points 14.8 / 14.95 us), nor are those of more than 64.  Items of four tiles: 64 x 2048 points, 64 representatives each, 17 columns
// 213 / 204 us; but where most hold a value and there is little else, 2000 x 64, 2 each, 9 columns 48.9 / 49.5.
__device__ __forceinline__ bool any_live(const uint32_t* __restrict__ live, int j, int tb, int nb, int lane) {
  if (nb < 4 || nb > 64) return true;
  uint32_t word = 0;
  if (lane < nb) {
    const uint64_t hi = (uint64_t)max(j, tb + lane), lo = (uint64_t)min(j, tb + lane);
    word = live[hi * (hi + 1) / 2 + lo];
  }
  return __ballot(word != 0u) != 0;
}

template <int NG, bool ACC64, int KIND>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu((WaveCfg<NG, ACC64, KIND>::WAVES_PER_EU)))) void k_strip(const StripArgs a) {
  typedef WaveCfg<NG, ACC64, KIND> Cfg;
  typedef typename Cfg::VT VT;
  constexpr bool RM = Cfg::BASE == STRIP_ROWMAJOR, SYM = Cfg::BASE == STRIP_SYM, TRI = !RM && !SYM;
  constexpr int ST = Cfg::STAGES, NB = Cfg::NB, NV = Cfg::NV, RG = Cfg::ROW_GROUPS;
  constexpr int KP = Cfg::SHARES, SP = 4 / KP;               // waves that share a row's columns; steps of a wave in a tile
  constexpr int HINT = (KIND & STRIP_STREAMED) ? 2 : 0;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

  const int T = a.T;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, kg = lane >> 4;
  // which 16 SP columns of every 64-column tile are this wave's, and its first row group
  const int part = KP == NW ? wave : wave % KP, g0 = Cfg::QUARTERS ? (int)(blockIdx.x & 3u) : KP == NW ? 0 : wave / KP * RG;
  const uint32_t rowbytes = (uint32_t)T * (uint32_t)sizeof(VT);

  // What the loops need to know of an item.  Tile numbers p = 0 .. nb - 1 run from the item's first column on and are
  // visited in a rotating order (tile_of): a triangular item begins with its diagonal tile, which is masked.
  struct Strip {
    const char *A, *V;         // matrix (strip row 0, column 0) and the vector row of the item's first column
    uint32_t lda, vbytes;
    int c_begin, nrows, mode, cnt, jm, thr, tbj, j_abs;
  } S;
  auto setup = [&](const StripItem& it, const StripPort& pt) {
    const int c_begin = (int)it.c_begin, c_end = (int)it.c_end;
    const int nb = c_end > c_begin ? (c_end - c_begin + TILE - 1) >> 6 : 0;
    const uint32_t fl = it.blocked;
    const bool sym = SYM && (fl & 2u) != 0;
    const int kind = (int)((fl >> 2) & 3u);
    const int tb = c_begin >> 6;
    S.j_abs = (int)it.row_in_block >> 6;
    const int jr = ((fl >> 4) & 0x7ffu) ? (int)((fl >> 15) & 0x7ffu) : S.j_abs - tb;
    S.mode = (int)it.mode;
    S.cnt = nb;
    // (the diagonal tile is the last one of mode 1 and the first one of mode 2)
    S.jm = TRI ? (S.mode == 1 ? 1 : 0) : !sym || nb <= 0 ? 0 : (jr < nb ? jr : jr % nb);
    S.thr = !sym || kind == 1 ? 0x7fffffff : (kind == 2 ? -1 : jr);      // tiles past it are read transposed
    S.tbj = tb - S.j_abs;
    S.A = reinterpret_cast<const char*>(pt.A + it.a_off);
    S.V = reinterpret_cast<const char*>(pt.in) + (uint64_t)(it.in_row0 + (uint32_t)c_begin) * rowbytes;
    S.lda = it.lda;
    S.vbytes = (uint32_t)max(c_end - c_begin, 0) * rowbytes;
    S.c_begin = c_begin;
    S.nrows = (int)it.nrows;
  };
  auto tile_of = [&](const int u) { int p = min(u, S.cnt - 1) - S.jm; p += p < 0 ? S.cnt : 0; return p; };
  auto turned = [&](const int p) { return SYM && p > S.thr; };

  // Buffer loads: the address is a scalar base + a lane offset that never changes, so the loop computes no vector
  // addresses, and rows of the vector block past the item's last column read as zero (the padding of every stored
  // matrix is finite), so a tile that the last column cuts needs no masks.
  const uint32_t ooff = (uint32_t)((m * 16 + 4 * kg) * 4);
  const uint32_t toff = (uint32_t)(((((lane >> 2) & 3) * 4 + (lane >> 4)) * 16 + (lane & 3) * 4) * 4);
  // offsets of the vector operand in the wave's LDS: rows 4 kg + j of the step, column 0 and column 1 + 16 n + m
  // (clamped to the last one)
  uint32_t yoff[4], boff[NB][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    yoff[j] = (uint32_t)(4 * kg + j) * rowbytes;
#pragma unroll
    for (int n = 0; n < NB; ++n) boff[n][j] = yoff[j] + (uint32_t)min(1 + 16 * n + m, T - 1) * (uint32_t)sizeof(VT);
  }

  auto load_a = [&](v4f (&ra)[RG], const int p, const int sub, const bool valid) {
    const int c = S.c_begin + TILE * p;                      // first column of the tile
    // transposed: fragments (row group sub, columns 16 g ..) of the stored tile (column tile of p, tile row of the strip)
    const bool tr = turned(p);
    const int64_t own = RM ? (int64_t)(c + 16 * sub) : (int64_t)((c >> 5) + (sub >> 1)) * (TILE * BLK_COLS) + (sub & 1) * FRAG;
    const int64_t far = (int64_t)(S.tbj + p) * TILE * (int64_t)S.lda + (int64_t)(2 * S.j_abs) * (TILE * BLK_COLS) + sub * 2 * FRAG;
    const auto res = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(S.A + (tr ? far : own) * 4), 0, valid ? 0x7fffffff : 0, 0x00027000);
    const uint32_t off = tr ? toff : ooff;
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      const int so = RM || !valid ? 0 : (tr ? (((g0 + g) >> 1) * (TILE * BLK_COLS) + ((g0 + g) & 1) * FRAG) * 4 : (g0 + g) * 2 * FRAG * 4);
      const uint32_t ro = RM ? (uint32_t)min(16 * (g0 + g) + m, S.nrows - 1) * S.lda * 4u + 16u * (uint32_t)kg : off;
      ra[g] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(res, ro, so, HINT));
    }
  };
  struct VRegs { v4f q[NV]; };
  // (valid = false: past the wave's last tile; every load is out of range and touches no memory, so that the number of
  // loads in flight stays what the loop's waits count on)
  auto load = [&](v4f (&ra)[RG], VRegs& rv, const int u, const bool valid) {
    const int p = tile_of(SP == 1 ? u : u / SP), sub = SP == 1 ? part : part * SP + u % SP;
    load_a(ra, p, sub, valid);
    const auto vres = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(S.V), 0, (int)S.vbytes, 0x00027000);
    const int so = valid ? (int)min((uint32_t)(TILE * p + 16 * sub) * rowbytes, S.vbytes) : (int)S.vbytes;
    if constexpr (NG > 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
        // (a scalar offset past the range would not be out of range for the check: it is clamped)
        rv.q[i] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(vres, (uint32_t)lane * 16u,
                      1024u * i < 16u * rowbytes ? (int)min((uint32_t)(so + 1024 * i), S.vbytes) : (int)S.vbytes, 0));
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i)
        rv.q[i] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(vres, yoff[0] + 16u * i, so, 0));
    }
  };

  // Whether the project kernel met a value that is not finite among the item's vector rows (0 times it is NaN, so tiles of zeros
  // count then).  Looked for in the rows themselves, by each wave in its own: 402 -> 413 us in the workload of any_live.
  auto any_odd = [&](const StripItem& it, const StripPort& pt) {
    const uint8_t* __restrict__ at = static_cast<const uint8_t*>(pt.in) + (uint64_t)pt.odd_at * 256;
    if (pt.odd_rows == 0) return false;
    const uint32_t last = (it.c_end - 1) / pt.odd_rows;
    uint32_t some = 0;
    for (uint32_t i = it.c_begin / pt.odd_rows + lane; i <= last; i += 64) some |= at[i];
    return __any(some) != 0;
  };

  // accumulators: fp64 running sums; in the fp32 mode the matrix cores fill a fresh fp32 chain every 16 columns
  v4d acc[RG][NB];
  double accy[RG];
#pragma unroll
  for (int g = 0; g < RG; ++g) {
    accy[g] = 0.0;
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[g][n] = (v4d){0.0, 0.0, 0.0, 0.0};
  }
  float* tr_lds = reinterpret_cast<float*>(lds + wave * Cfg::WAVE_LDS);
  unsigned char* v_lds = lds + wave * Cfg::WAVE_LDS + Cfg::TURN_LDS;
  // vector rows of a step: through the wave's LDS into operand order
  auto spread = [&](const VRegs& rv, VT (&rb)[NB][4], VT (&ry)[4]) {
    if constexpr (NG > 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) reinterpret_cast<v4f*>(v_lds)[i * 64 + lane] = rv.q[i];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ry[j] = *reinterpret_cast<const VT*>(v_lds + yoff[j]);
#pragma unroll
        for (int n = 0; n < NB; ++n) rb[n][j] = *reinterpret_cast<const VT*>(v_lds + boff[n][j]);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (ACC64) ry[j] = __builtin_bit_cast(v2d, rv.q[j >> 1])[j & 1];
        else ry[j] = rv.q[0][j];
      }
    }
  };
  // the operand of a transposed tile passes the wave's own piece of LDS (a wave's LDS accesses are served in order)
  auto turn = [&](v4f (&ra)[RG]) {
#pragma unroll
    for (int g = 0; g < RG; ++g) reinterpret_cast<v4f*>(tr_lds)[g * 64 + lane] = ra[g];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) ra[g][i] = tr_lds[g * 256 + 64 * i + lane];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto compute = [&](const v4f (&ra)[RG], const VT (&rb)[NB][4], const VT (&ry)[4]) {
    if constexpr (ACC64) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        double ad[RG];
#pragma unroll
        for (int g = 0; g < RG; ++g) ad[g] = (double)ra[g][j];
        if (NG > 0) {
#pragma unroll
          for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int g = 0; g < RG; ++g) acc[g][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(ad[g], rb[n][j], acc[g][n], 0, 0, 0);
        }
#pragma unroll
        for (int g = 0; g < RG; ++g) accy[g] = fma(ad[g], ry[j], accy[g]);
      }
    } else {
      if (NG > 0) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          if (n > 0) __builtin_amdgcn_sched_barrier(0);     // one column group's chains at a time: registers
          v4f f[RG];
#pragma unroll
          for (int g = 0; g < RG; ++g) f[g] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int g = 0; g < RG; ++g) f[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(ra[g][j], rb[n][j], f[g], 0, 0, 0);
#pragma unroll
          for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[g][n][i] += (double)f[g][i];
        }
      }
#pragma unroll
      for (int g = 0; g < RG; ++g)
        accy[g] += (double)fmaf(ra[g][3], ry[3], fmaf(ra[g][2], ry[2], fmaf(ra[g][1], ry[1], ra[g][0] * ry[0])));
    }
    // pins the y sums to this place: the compiler otherwise moves them behind the loop's last use and keeps every
    // operand alive until then
#pragma unroll
    for (int g = 0; g < RG; ++g) asm volatile("" : "+v"(accy[g]));
  };

  v4f sa[ST][RG];
  VRegs sv[ST];
  VT cb[2][NB][4], cy[2][4];                                 // vector operands of the step at hand and of the next one
  auto ready = [&](auto s_c, const int u) {                  // operands of sequence number u, held by stage s
    constexpr int s = decltype(s_c)::value;
    if (turned(tile_of(u))) turn(sa[s % ST]);
    spread(sv[s % ST], cb[Cfg::AHEAD ? s & 1 : 0], cy[Cfg::AHEAD ? s & 1 : 0]);
  };
  const uint32_t id = Cfg::QUARTERS ? blockIdx.x >> 2 : blockIdx.x, die = id % NUM_XCD, row = id / NUM_XCD;
  const uint32_t at = a.from[die] + (row >> a.sys_log2), first_port = (row & ((1u << a.sys_log2) - 1)) * (uint32_t)a.sys_ports;
  if (at >= a.from[die + 1]) return;                         // (the other dies' lists are longer)
  const StripItem& it = a.items[at];
  const StripPort& pt = a.port[first_port + it.port];
  setup(it, pt);
  if (SYM && pt.live && !any_live(pt.live, S.j_abs, S.tbj + S.j_abs, S.cnt, lane) && !any_odd(it, pt)) S.cnt = 0;
  const int cnt = SP * S.cnt;                                // steps of a wave
  {
    if (cnt > 0) {
#pragma unroll
      for (int s = 0; s + 1 < ST; ++s) load(sa[s], sv[s], s, s < cnt);
      __builtin_amdgcn_sched_barrier(0);
      load(sa[ST - 1], sv[ST - 1], ST - 1, ST - 1 < cnt);
      if (TRI && S.mode != 0) {                              // the diagonal tile: the wave's first SP steps
#pragma unroll
        for (int s = 0; s < SP; ++s) {
          const int q0 = 16 * (part * SP + s) + 4 * kg;      // column of this lane's first element inside the tile
#pragma unroll
          for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int row = 16 * (g0 + g) + m;
              sa[s][g][i] = (S.mode == 1 ? q0 + i <= row : q0 + i >= row) ? sa[s][g][i] : 0.f;
            }
        }
      }
      int i = 0;
      if constexpr (Cfg::AHEAD) ready(std::integral_constant<int, 0>(), 0);
      constexpr int UN = ST % 2 == 0 ? ST : 2 * ST;          // the operand buffers alternate: an even number of steps
      auto step = [&](auto s_c, const bool refill) {
        constexpr int s = decltype(s_c)::value;
        if constexpr (Cfg::AHEAD) ready(std::integral_constant<int, s + 1>(), i + s + 1);
        else ready(s_c, i + s);
        compute(sa[s % ST], cb[Cfg::AHEAD ? s & 1 : 0], cy[Cfg::AHEAD ? s & 1 : 0]);
        __builtin_amdgcn_sched_barrier(0);
        if (refill) load(sa[s % ST], sv[s % ST], i + s + ST, i + s + ST < cnt);
        __builtin_amdgcn_sched_barrier(0);
      };
      for (; i + UN < cnt; i += UN) {
        step(std::integral_constant<int, 0>(), true);
        step(std::integral_constant<int, 1>(), true);
        if constexpr (UN > 2) { step(std::integral_constant<int, 2>(), true); step(std::integral_constant<int, 3>(), true); }
        if constexpr (UN > 4) { step(std::integral_constant<int, 4>(), true); step(std::integral_constant<int, 5>(), true); }
      }
      const int rem = cnt - i;                               // 1 .. UN; with UN = 2 ST the first steps still refill
      step(std::integral_constant<int, 0>(), UN > ST);
      if (rem > 1) step(std::integral_constant<int, 1>(), UN > ST);
      if constexpr (UN > 2) {
        if (rem > 2) step(std::integral_constant<int, 2>(), UN > ST);
        if (rem > 3) step(std::integral_constant<int, 3>(), false);
      }
      if constexpr (UN > 4) {
        if (rem > 4) step(std::integral_constant<int, 4>(), false);
        if (rem > 5) step(std::integral_constant<int, 5>(), false);
      }
    }

    VT* __restrict__ out = static_cast<VT*>(pt.out) + (uint64_t)it.out_part * pt.out_part_stride + (uint64_t)it.out_row0 * T;
    const VT* __restrict__ din = reinterpret_cast<const VT*>(pt.in) + (uint64_t)(it.in_row0 + it.row_in_block) * T;
    const double dadd = (double)it.diag_add * pt.diag_add, scale = pt.scale;
    const int per = TILE * T, total = (Cfg::QUARTERS ? min((int)it.nrows, 16 * g0 + 16) : (int)it.nrows) * T;
    const bool accumulate = pt.accumulate != 0;
    // ---- the waves' sums are added in a fixed order ----
    __syncthreads();                                         // every wave is done with its own piece of LDS
    double* red = reinterpret_cast<double*>(lds) + (size_t)part * per;
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      if (NG > 0) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const int col = 1 + 16 * n + m;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (col < T) red[(16 * (g0 + g) + acc_row<ACC64>(lane, i)) * T + col] = acc[g][n][i];
          acc[g][n] = (v4d){0.0, 0.0, 0.0, 0.0};
        }
      }
      double y = accy[g];
      y += __shfl_xor(y, 16);
      y += __shfl_xor(y, 32);
      if (kg == 0) red[(16 * (g0 + g) + m) * T] = y;
      accy[g] = 0.0;
    }
    __syncthreads();
    const double* all = reinterpret_cast<const double*>(lds);
    for (int e = tid + (Cfg::QUARTERS ? 16 * g0 * T : 0); e < total; e += 64 * NW) {
      double v = KP == 2 ? all[e] + all[per + e] : (all[e] + all[per + e]) + (all[2 * per + e] + all[3 * per + e]);
      v *= scale;
      if (dadd != 0.0) v = fma(dadd, (double)din[e], v);
      if (accumulate) v += (double)out[e];
      out[e] = (VT)v;
    }
  }
}

template <int NG, bool ACC64, int KIND>
static int launch_kind(int count, int T, hipStream_t s, const StripArgs& a) {
  typedef WaveCfg<NG, ACC64, KIND> Cfg;
  // LDS: the waves' own pieces in the loop, then the partial sums (one set for each wave that shares a row's columns)
  constexpr int wl = NW * Cfg::WAVE_LDS, per_col = Cfg::SHARES * TILE * (int)sizeof(double), rl = per_col * (16 * NG + 1);
  const size_t lds = std::max<size_t>(wl, (size_t)per_col * T);
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_strip<NG, ACC64, KIND>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, std::max(wl, rl));
  NUGPR_HIP(attr);
  hipLaunchKernelGGL((k_strip<NG, ACC64, KIND>), dim3(count), dim3(64 * NW), lds, s, a);
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}
template <bool ACC64, int KIND>
static int launch_width(int ng, int count, int T, hipStream_t s, const StripArgs& a) {
  if (ng == 0) return launch_kind<0, ACC64, KIND>(count, T, s, a);
  if (ng == 1) return launch_kind<1, ACC64, KIND>(count, T, s, a);
  return launch_kind<2, ACC64, KIND>(count, T, s, a);
}

// out[i] = sum over `parts` slabs of in[part * stride + i]  (fixed order: deterministic)
template <typename VT>
__global__ void k_sum_parts(const VT* __restrict__ in, VT* __restrict__ out, int64_t count, int parts,
                            uint64_t stride, uint64_t slot) {
  in = reinterpret_cast<const VT*>(reinterpret_cast<const char*>(in) + blockIdx.y * slot);
  out = reinterpret_cast<VT*>(reinterpret_cast<char*>(out) + blockIdx.y * slot);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
    VT s = in[i];
    for (int p = 1; p < parts; ++p) s += in[(uint64_t)p * stride + i];
    out[i] = s;
  }
}

int launch_sum_parts(const void* in, void* out, int64_t count, int parts, uint64_t stride, bool acc64,
                     hipStream_t s, int nsys, uint64_t slot) {
  const dim3 grid((unsigned)std::min<int64_t>((count + 255) / 256, 2048), (unsigned)nsys);
  if (acc64)
    hipLaunchKernelGGL((k_sum_parts<double>), grid, dim3(256), 0, s, (const double*)in, (double*)out, count,
                       parts, stride, slot);
  else
    hipLaunchKernelGGL((k_sum_parts<float>), grid, dim3(256), 0, s, (const float*)in, (float*)out, count,
                       parts, stride, slot);
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

uint64_t strip_tiles(const std::vector<StripItem>& items) {
  uint64_t tiles = 0;
  for (const StripItem& it : items) tiles += it.c_end > it.c_begin ? (it.c_end - it.c_begin + TILE - 1) / TILE : 0;
  return tiles;
}
bool short_strips(const std::vector<StripItem>& items) { return strip_tiles(items) <= 10 * items.size(); }

// Tables with strips of symmetric blocks take the instantiation that pairs their tiles, strips of a basis the caller
// supplied the row-major one, triangular strips the short or the long one by their mean number of tiles.
// Short: up to 10 tiles a strip on average.  Preconditioner apply, fp64, 17 columns, short against long: 256 clusters of
// 512 points (4.5 tiles) 91 / 109 us, 32 x 1024 (8.5) 46 / 48, 32 x 1280 (10.5) 61 / 61, 64 x 2048 (16.5) 258 / 264 but
// 3 x 4096 95 / 91; 33 columns: 131 / 165, 73 / 74, 100 / 93, 24 uneven clusters of 1536 on average 217 / 168.
// The streaming hint (each tile is used once).  A solver applies the K_ii and the factor, equally large, in turn, so it pays
// from the size on at which the two no longer fit the memory-side cache (256 MB) together.  Batched solve, 17 columns,
// without / with it: 64 x 512 points (64 MB each) 385 / 392 us, 96 x 512 (96 MB) 431 / 441, 128 x 512 (128 MB) 513 / 508,
// 48 x 1024 (192 MB) 550 / 530, 64 x 2048 (1 GB) 1614 / 1555; the apply by itself could do without up to 256 MB (48 x 1024:
// 60 / 66).  Row-major strips never gain: the basis is small beside the K_ii (96 x 2048 points, rank 256: 848 / 865 us).
int strip_kind(const std::vector<StripItem>& items, uint64_t matrix_bytes) {
  for (const StripItem& it : items)
    if (it.blocked & 2u) return strip_tiles(items) <= 16 * items.size() ? STRIP_SYM + STRIP_MANY : STRIP_SYM;
  if (!items.empty() && items[0].blocked == 0) return STRIP_ROWMAJOR;
  return (short_strips(items) ? STRIP_SHORT : STRIP_LONG) + (matrix_bytes >= (uint64_t)128 << 20 ? STRIP_STREAMED : 0);
}

// Up to 512 strips leave a compute unit two workgroups at most, so four waves per SIMD are no use to them; what two row
// groups a wave cost is then felt, and two column groups in fp64 run as long strips (three stages, four row groups).
// Preconditioner apply, 33 columns, short / long: 4 uneven clusters of 700 points on average 73 / 64 us, 24 x 1000 (384
// strips) 67 / 60, 64 x 300 (320) 33 / 35, 100 uneven ones of 300 (560) 53 / 54.  The other widths and the fp32 mode gain
// as much by the shorter start as they lose (17 columns: 4 of 700 40 / 39, 24 x 1000 38 / 40).
// Symmetric strips in fp64 with one column group, more of them than the 768 that three workgroups a compute unit make: with two
// stages a fourth workgroup fits, which pays while a strip has few tiles.  Product of 17 columns, three stages / two: 512 clusters
// of 128 points 52.0 / 48.7 us, 256 x 256 86.7 / 82.9, 128 x 512 64.2 / 63.2, 256 x 512 137.7 / 134.8, 128 x 1024 140.7 / 139.6, but
// 64 x 1536 126.2 / 130.5, 64 x 2048 198.0 / 208.6, and 2000 x 64, whose coupling strips are long, 212.9 / 219.7.
// Few strips: a strip's four row groups in workgroups of their own (STRIP_QUARTERS).  A wave then issues a quarter of the matrix
// instructions, of which it issued one after the other while most of the chip was idle; the vector rows are read four times.
// Symmetric up to 128 strips of three tiles or more; triangular ones, which are uneven, up to 256 of four (128 of two).  One
// column has no matrix instructions.  Whole strips / quarters, us, 17 columns fp64, 33 fp64, 17 fp32:
//   product  4 x 512 points (32 strips) 18.0 / 14.5, 23.3 / 15.6, 16.7 / 15.1; 2 x 2048 (64) 38.6 / 27.0, 57.9 / 38.1, 32.5 / 22.5;
//            8 x 1024 (128) 26.9 / 22.4, 36.4 / 28.6, 22.2 / 18.9; but 24 x 512 (192) 25.7 / 25.8, 32.9 / 36.4, 20.3 / 21.8, 2 x 128 13.5 / 14.8
//   apply    4 x 512 23.0 / 17.0, 34.0 / 19.2, 16.3 / 12.0; 2 x 4096 (128) 89 / 47.5, 161 / 76, 72 / 35.5; 16 x 1024 (256) 35.4 / 29.7, 56.6 / 48.6,
//            25.3 / 20.8; but 24 x 1024 (384) 37.1 / 40.2, 60.5 / 70.5, 26.4 / 29.2, 64 x 256 (256) 20.2 / 21.6, 28.7 / 31.5, 12.9 / 11.9
// Systems side by side (count = strips of all of them) take sums in the order of one alone.  All instantiations share a row's
// columns among four waves but whole short strips of two column groups, which share them between two: those are for
// several systems where they are for one, and where one takes quarters or long strips, several take quarters or long strips.
// (33 columns fp64, by the strips of all systems / by those of one: training step 24 x 1000 points 4.26 / 4.41 ms, 16 x 1024 2.56 / 2.59;
// prediction of 264 points 24 x 1000 2.60 / 2.71 ms, 40 x 300 1.12 / 1.18.)
static int kind_at(const StripTable& tab, int count, int T, bool acc64) {
  const bool sym = (tab.kind & 3) == STRIP_SYM;
  auto quarters = [&](int strips) {
    return T > 1 && (tab.kind & 3) != STRIP_ROWMAJOR && strips <= (sym ? 128 : 256) && tab.tiles >= tab.count * (sym ? 3 : strips > 128 ? 4 : 2);
  };
  if (quarters(count)) return (sym ? STRIP_SYM : STRIP_SHORT) + STRIP_QUARTERS;
  if (tab.kind & STRIP_MANY) return acc64 && T > 1 && T <= 17 && count > 768 ? tab.kind : tab.kind - STRIP_MANY;
  const bool as_long = (tab.kind & 3) == STRIP_SHORT && T > 17 && (quarters(tab.count) || (acc64 && tab.count <= 512));
  return as_long ? tab.kind - STRIP_SHORT + STRIP_LONG : tab.kind;
}

const char* strip_kernel_name(const StripTable& tab, int T, bool acc64) {
  static thread_local char name[32];
  std::snprintf(name, sizeof(name), "k_strip<%d, %s, %d>", (T - 1 + 15) / 16, acc64 ? "true" : "false", kind_at(tab, tab.count, T, acc64));
  return name;
}

template <bool ACC64>
static int launch_table(const StripTable& tab, int ng, int T, hipStream_t s, const StripArgs& a) {
  const int kind = kind_at(tab, tab.count << a.sys_log2, T, ACC64);
  uint32_t longest = 0;
  for (int d = 0; d < NUM_XCD; ++d) longest = std::max(longest, tab.from[d + 1] - tab.from[d]);
  const int count = (int)(NUM_XCD * longest) << a.sys_log2;      // workgroups (quarters of them)
  switch (kind) {
    case STRIP_SYM: return launch_width<ACC64, STRIP_SYM>(ng, count, T, s, a);
    case STRIP_SYM + STRIP_MANY:
      if constexpr (ACC64) return launch_kind<1, true, STRIP_SYM + STRIP_MANY>(count, T, s, a);
      break;
    case STRIP_LONG: return launch_width<ACC64, STRIP_LONG>(ng, count, T, s, a);
    case STRIP_SHORT: return launch_width<ACC64, STRIP_SHORT>(ng, count, T, s, a);
    case STRIP_SYM + STRIP_QUARTERS: return launch_width<ACC64, STRIP_SYM + STRIP_QUARTERS>(ng, 4 * count, T, s, a);
    case STRIP_SHORT + STRIP_QUARTERS: return launch_width<ACC64, STRIP_SHORT + STRIP_QUARTERS>(ng, 4 * count, T, s, a);
    case STRIP_ROWMAJOR: return launch_width<ACC64, STRIP_ROWMAJOR>(ng, count, T, s, a);
    case STRIP_LONG + STRIP_STREAMED: return launch_width<ACC64, STRIP_LONG + STRIP_STREAMED>(ng, count, T, s, a);
    case STRIP_SHORT + STRIP_STREAMED: return launch_width<ACC64, STRIP_SHORT + STRIP_STREAMED>(ng, count, T, s, a);
  }
  set_error("internal: strip table of an unknown kind");
  return NUGPR_ERR_INVALID;
}

int launch_strip(const StripTable& tab, const StripPort* ports, int nports, int T, bool acc64, hipStream_t s, int nsys) {
  if (tab.count == 0) return NUGPR_OK;
  if (nports < 1 || nports > 2 * MAX_SLOTS || (nsys != 1 && nsys != 2 && nsys != 4) || nports % nsys) { set_error("internal: number of strip ports"); return NUGPR_ERR_INVALID; }
  if (T < 1 || T > MAX_COLS) { set_error("vector block wider than 33 columns"); return NUGPR_ERR_INVALID; }
  StripArgs a{};
  for (int i = 0; i < nports; ++i) a.port[i] = ports[i];
  a.items = tab.dev;
  a.T = T;
  a.sys_log2 = nsys / 2;
  a.sys_ports = nports / nsys;
  std::copy(tab.from, tab.from + NUM_XCD + 1, a.from);
  const int ng = (T - 1 + 15) / 16;
  return acc64 ? launch_table<true>(tab, ng, T, s, a) : launch_table<false>(tab, ng, T, s, a);
}

}  // namespace nugpr
