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
// flight is what the waits count.
//
// What bounds it.  fp64: the matrix cores and the vector ALUs share one pipe (16 MFMAs x 64 cycles and 32 vector
// instructions a step: 550 ns at the sustained clock, measured without any memory access); 1 - 17 columns also the
// traffic behind the L2s.  Before (a loader wave feeding an LDS ring with one workgroup barrier per 32 columns, the
// strip's rows split among the waves) the barrier -> LDS -> MFMA chain left a fifth of the issue slots empty.
// 128 clusters of 2048 points, 128 representatives each, 17 columns: 556 -> 500 us; 64 uneven clusters of 4096
// points on average, 33 columns: 2297 -> 1870 us; preconditioner strips, 64 x 2048, 17 columns: 112 -> 108 us
// (4.9 TB/s of HBM); fp32 mode, 64 x 2048, 17 columns: whole squares -> lower tiles (see below).
// Tried and not kept: vector operands loaded in operand order from memory (the address unit takes 25 - 30 cycles
// for a load whatever its width: 640 us); workgroups that stay and take item after item (741 us), or whose start is
// staggered (580 us): both take the partner strips below out of step.
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
#include <type_traits>

#include "nugpr_internal.h"

namespace nugpr {

typedef float v4f __attribute__((ext_vector_type(4)));
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
enum { STRIP_PLAIN = 0, STRIP_SYM = 1, STRIP_ROWMAJOR = 2 };      // what the items of a table are
template <int NG, bool ACC64, int KIND> struct WaveCfg {
  typedef typename VecT<ACC64>::type VT;
  // Waves per SIMD and steps in flight, as the registers allow.  Symmetric strips in fp64 with one column group: 3
  // waves x 3 stages 500 us, 2 x 4 527 us (workload in the file's head); strips without partners, which stream from
  // HBM: 2 x 4 108 us, 3 x 3 117 us.
  static constexpr int WAVES_PER_EU = KIND == STRIP_SYM && ACC64 && NG == 1 ? 3 : 2;
  static constexpr int STAGES = NG == 2 && !ACC64 ? 2 : (WAVES_PER_EU == 3 || NG == 2 ? 3 : 4);
  static constexpr int NB = NG > 0 ? NG : 1;
  // 16-byte loads per lane that cover the vector rows of a step (16 rows of at most 16 NG + 1 columns)
  static constexpr int NV = NG > 0 ? (16 * (16 * NG + 1) * (int)sizeof(VT) + 1023) / 1024 : 1;
  static constexpr int WAVE_LDS = 4096 + NV * 1024;            // a wave's LDS: a tile on its way to its transpose, vector rows
};

template <int NG, bool ACC64, int KIND>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu((WaveCfg<NG, ACC64, KIND>::WAVES_PER_EU)))) void k_strip(const StripArgs a) {
  typedef WaveCfg<NG, ACC64, KIND> Cfg;
  typedef typename Cfg::VT VT;
  constexpr bool RM = KIND == STRIP_ROWMAJOR, SYM = KIND == STRIP_SYM;
  constexpr int ST = Cfg::STAGES, NB = Cfg::NB, NV = Cfg::NV;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

  const int T = a.T;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, kg = lane >> 4;
  const int sub = wave;                                      // which 16 columns of every 64-column tile are this wave's
  const uint32_t rowbytes = (uint32_t)T * (uint32_t)sizeof(VT);

  // What the loops need to know of an item.  Tile numbers p = 0 .. nb - 1 run from the item's first column on.  The
  // diagonal tile of a triangular item is masked and comes first, the others are taken in turn (tile_of).
  struct Strip {
    const char *A, *V;         // matrix (strip row 0, column 0) and the vector row of the item's first column
    uint32_t lda, vbytes;
    int c_begin, nrows, mode, p_lo, p_diag, cnt, jm, thr, tbj, j_abs;
  } S;
  auto setup = [&](const StripItem& it) {
    const StripPort& pt = a.port[it.port];
    const int c_begin = (int)it.c_begin, c_end = (int)it.c_end;
    const int nb = c_end > c_begin ? (c_end - c_begin + TILE - 1) >> 6 : 0;
    const uint32_t fl = it.blocked;
    const bool sym = SYM && (fl & 2u) != 0;
    const int kind = (int)((fl >> 2) & 3u);
    const int tb = c_begin >> 6;
    S.j_abs = (int)it.row_in_block >> 6;
    const int jr = ((fl >> 4) & 0x7ffu) ? (int)((fl >> 15) & 0x7ffu) : S.j_abs - tb;
    S.mode = (int)it.mode;
    int p_hi = nb;
    S.p_lo = 0; S.p_diag = -1;
    if (KIND == STRIP_PLAIN && nb > 0 && S.mode == 1) { p_hi -= 1; S.p_diag = p_hi; }
    if (KIND == STRIP_PLAIN && nb > 0 && S.mode == 2) { S.p_lo = 1; S.p_diag = 0; }
    S.cnt = p_hi - S.p_lo;
    S.jm = !sym || S.cnt <= 0 ? 0 : (jr < S.cnt ? jr : jr % S.cnt);
    S.thr = !sym || kind == 1 ? 0x7fffffff : (kind == 2 ? -1 : jr);      // tiles past it are read transposed
    S.tbj = tb - S.j_abs;
    S.A = reinterpret_cast<const char*>(pt.A + it.a_off);
    S.V = reinterpret_cast<const char*>(pt.in) + (uint64_t)(it.in_row0 + (uint32_t)c_begin) * rowbytes;
    S.lda = it.lda;
    S.vbytes = (uint32_t)max(c_end - c_begin, 0) * rowbytes;
    S.c_begin = c_begin;
    S.nrows = (int)it.nrows;
  };
  auto tile_of = [&](const int u) { int p = min(u, S.cnt - 1) - S.jm; p += p < 0 ? S.cnt : 0; return S.p_lo + p; };
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

  auto load_a = [&](v4f (&ra)[4], const int p, const bool valid) {
    const int c = S.c_begin + TILE * p;                      // first column of the tile
    // transposed: fragments (row group sub, columns 16 g ..) of the stored tile (column tile of p, tile row of the strip)
    const bool tr = turned(p);
    const int64_t own = RM ? (int64_t)(c + 16 * sub) : (int64_t)((c >> 5) + (sub >> 1)) * (TILE * BLK_COLS) + (sub & 1) * FRAG;
    const int64_t far = (int64_t)(S.tbj + p) * TILE * (int64_t)S.lda + (int64_t)(2 * S.j_abs) * (TILE * BLK_COLS) + sub * 2 * FRAG;
    const auto res = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(S.A + (tr ? far : own) * 4), 0, valid ? 0x7fffffff : 0, 0x00027000);
    const uint32_t off = tr ? toff : ooff;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int so = RM || !valid ? 0 : (tr ? ((g >> 1) * (TILE * BLK_COLS) + (g & 1) * FRAG) * 4 : g * 2 * FRAG * 4);
      const uint32_t ro = RM ? (uint32_t)min(16 * g + m, S.nrows - 1) * S.lda * 4u + 16u * (uint32_t)kg : off;
      ra[g] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(res, ro, so, SYM ? 0 : 2));
    }
  };
  struct VRegs { typename std::conditional<(NG > 0), v4f, VT>::type q[NG > 0 ? NV : 4]; };
  // (valid = false: past the wave's last tile; every load is out of range and touches no memory, so that the number of
  // loads in flight stays what the loop's waits count on)
  auto load = [&](v4f (&ra)[4], VRegs& rv, const int p, const bool valid) {
    load_a(ra, p, valid);
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
      for (int j = 0; j < 4; ++j) {
        if constexpr (ACC64) rv.q[j] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(vres, yoff[j], so, 0));
        else rv.q[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vres, yoff[j], so, 0));
      }
    }
  };

  // accumulators: fp64 running sums; in the fp32 mode the matrix cores fill a fresh fp32 chain every 16 columns
  v4d acc[4][NB];
  double accy[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    accy[g] = 0.0;
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[g][n] = (v4d){0.0, 0.0, 0.0, 0.0};
  }
  float* tr_lds = reinterpret_cast<float*>(lds + wave * Cfg::WAVE_LDS);
  unsigned char* v_lds = lds + wave * Cfg::WAVE_LDS + 4096;
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
      for (int j = 0; j < 4; ++j) ry[j] = rv.q[j];
    }
  };
  // the operand of a transposed tile passes the wave's own piece of LDS (a wave's LDS accesses are served in order)
  auto turn = [&](v4f (&ra)[4]) {
#pragma unroll
    for (int g = 0; g < 4; ++g) reinterpret_cast<v4f*>(tr_lds)[g * 64 + lane] = ra[g];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) ra[g][i] = tr_lds[g * 256 + 64 * i + lane];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto compute = [&](const v4f (&ra)[4], const VT (&rb)[NB][4], const VT (&ry)[4]) {
    if constexpr (ACC64) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        double ad[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) ad[g] = (double)ra[g][j];
        if (NG > 0) {
#pragma unroll
          for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int g = 0; g < 4; ++g) acc[g][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(ad[g], rb[n][j], acc[g][n], 0, 0, 0);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) accy[g] = fma(ad[g], ry[j], accy[g]);
      }
    } else {
      if (NG > 0) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          if (n > 0) __builtin_amdgcn_sched_barrier(0);     // one column group's chains at a time: registers
          v4f f[4];
#pragma unroll
          for (int g = 0; g < 4; ++g) f[g] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) f[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(ra[g][j], rb[n][j], f[g], 0, 0, 0);
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[g][n][i] += (double)f[g][i];
        }
      }
#pragma unroll
      for (int g = 0; g < 4; ++g)
        accy[g] += (double)fmaf(ra[g][3], ry[3], fmaf(ra[g][2], ry[2], fmaf(ra[g][1], ry[1], ra[g][0] * ry[0])));
    }
    // pins the y sums to this place: the compiler otherwise moves them behind the loop's last use and keeps every
    // operand alive until then
#pragma unroll
    for (int g = 0; g < 4; ++g) asm volatile("" : "+v"(accy[g]));
  };

  v4f sa[ST][4];
  VRegs sv[ST];
  VT cb[2][NB][4], cy[2][4];                                 // vector operands of the step at hand and of the next one
  auto ready = [&](auto s_c, const int u) {                  // operands of sequence number u, held by stage s
    constexpr int s = decltype(s_c)::value;
    if (turned(tile_of(u))) turn(sa[s % ST]);
    spread(sv[s % ST], cb[s & 1], cy[s & 1]);
  };
  // the diagonal tile passes through the last stage's registers before the loop needs them
  auto start = [&]() {
    if (S.p_diag >= 0) load(sa[ST - 1], sv[ST - 1], S.p_diag, true);
#pragma unroll
    for (int s = 0; s + 1 < ST; ++s) load(sa[s], sv[s], tile_of(s), s < S.cnt);
  };
  const StripItem& it = a.items[blockIdx.x];
  setup(it);
  start();
  {
    if (S.p_diag >= 0) {
      const int q0 = 16 * sub + 4 * kg;                      // column of this lane's first element inside the tile
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool keep = S.mode == 1 ? q0 + i <= 16 * g + m : q0 + i >= 16 * g + m;
          sa[ST - 1][g][i] = keep ? sa[ST - 1][g][i] : 0.f;
        }
      spread(sv[ST - 1], cb[1], cy[1]);
      compute(sa[ST - 1], cb[1], cy[1]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (S.cnt > 0) {
      load(sa[ST - 1], sv[ST - 1], tile_of(ST - 1), ST - 1 < S.cnt);
      int i = 0;
      ready(std::integral_constant<int, 0>(), 0);
      constexpr int UN = ST % 2 == 0 ? ST : 2 * ST;          // the operand buffers alternate: an even number of steps
      auto step = [&](auto s_c, const bool refill) {
        constexpr int s = decltype(s_c)::value;
        ready(std::integral_constant<int, s + 1>(), i + s + 1);
        compute(sa[s % ST], cb[s & 1], cy[s & 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (refill) load(sa[s % ST], sv[s % ST], tile_of(i + s + ST), i + s + ST < S.cnt);
        __builtin_amdgcn_sched_barrier(0);
      };
      for (; i + UN <= S.cnt; i += UN) {
        step(std::integral_constant<int, 0>(), true);
        step(std::integral_constant<int, 1>(), true);
        if constexpr (UN > 2) { step(std::integral_constant<int, 2>(), true); step(std::integral_constant<int, 3>(), true); }
        if constexpr (UN > 4) { step(std::integral_constant<int, 4>(), true); step(std::integral_constant<int, 5>(), true); }
      }
      const int rem = S.cnt - i;                             // < UN; with UN = 2 ST the first steps still refill
      if (rem > 0) step(std::integral_constant<int, 0>(), UN > ST);
      if constexpr (UN > 2) {
        if (rem > 1) step(std::integral_constant<int, 1>(), UN > ST);
        if (rem > 2) step(std::integral_constant<int, 2>(), false);
      }
      if constexpr (UN > 4) {
        if (rem > 3) step(std::integral_constant<int, 3>(), false);
        if (rem > 4) step(std::integral_constant<int, 4>(), false);
      }
    }

    const StripPort& pt = a.port[it.port];
    VT* __restrict__ out = static_cast<VT*>(pt.out) + (uint64_t)it.out_part * pt.out_part_stride + (uint64_t)it.out_row0 * T;
    const VT* __restrict__ din = reinterpret_cast<const VT*>(pt.in) + (uint64_t)(it.in_row0 + it.row_in_block) * T;
    const double dadd = (double)it.diag_add * pt.diag_add, scale = pt.scale;
    const int per = TILE * T, total = (int)it.nrows * T;
    const bool accumulate = pt.accumulate != 0;
    // ---- the waves' sums are added in a fixed order ----
    __syncthreads();                                         // every wave is done with its own piece of LDS
    double* red = reinterpret_cast<double*>(lds) + (size_t)wave * per;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (NG > 0) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const int col = 1 + 16 * n + m;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (col < T) red[(16 * g + acc_row<ACC64>(lane, i)) * T + col] = acc[g][n][i];
          acc[g][n] = (v4d){0.0, 0.0, 0.0, 0.0};
        }
      }
      double y = accy[g];
      y += __shfl_xor(y, 16);
      y += __shfl_xor(y, 32);
      if (kg == 0) red[(16 * g + m) * T] = y;
      accy[g] = 0.0;
    }
    __syncthreads();
    const double* all = reinterpret_cast<const double*>(lds);
    for (int e = tid; e < total; e += 64 * NW) {
      double v = (all[e] + all[per + e]) + (all[2 * per + e] + all[3 * per + e]);
      v *= scale;
      if (dadd != 0.0) v = fma(dadd, (double)din[e], v);
      if (accumulate) v += (double)out[e];
      out[e] = (VT)v;
    }
  }
}

template <int NG, bool ACC64, int KIND>
static int launch_kind(int count, int T, hipStream_t s, const StripArgs& a) {
  constexpr int wl = NW * WaveCfg<NG, ACC64, KIND>::WAVE_LDS, rl = NW * TILE * (16 * NG + 1) * (int)sizeof(double);
  const size_t lds = std::max<size_t>(wl, (size_t)NW * TILE * T * sizeof(double));
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
                            uint64_t stride) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
    VT s = in[i];
    for (int p = 1; p < parts; ++p) s += in[(uint64_t)p * stride + i];
    out[i] = s;
  }
}

int launch_sum_parts(const void* in, void* out, int64_t count, int parts, uint64_t stride, bool acc64,
                     hipStream_t s) {
  const int grid = (int)std::min<int64_t>((count + 255) / 256, 2048);
  if (acc64)
    hipLaunchKernelGGL((k_sum_parts<double>), dim3(grid), dim3(256), 0, s, (const double*)in, (double*)out, count,
                       parts, stride);
  else
    hipLaunchKernelGGL((k_sum_parts<float>), dim3(grid), dim3(256), 0, s, (const float*)in, (float*)out, count,
                       parts, stride);
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

// Tables with strips of symmetric blocks take the instantiation that pairs their tiles, strips of a basis the caller
// supplied the row-major one, triangular strips the plain one (streaming loads: each tile is used once).
static int strip_kind(const StripTable& tab) { return tab.rowmajor ? STRIP_ROWMAJOR : tab.sym ? STRIP_SYM : STRIP_PLAIN; }

const char* strip_kernel_name(const StripTable& tab, int T, bool acc64) {
  static const char* const names[3][2][3] = {
      {{"k_strip<0, false, 0>", "k_strip<0, false, 1>", "k_strip<0, false, 2>"}, {"k_strip<0, true, 0>", "k_strip<0, true, 1>", "k_strip<0, true, 2>"}},
      {{"k_strip<1, false, 0>", "k_strip<1, false, 1>", "k_strip<1, false, 2>"}, {"k_strip<1, true, 0>", "k_strip<1, true, 1>", "k_strip<1, true, 2>"}},
      {{"k_strip<2, false, 0>", "k_strip<2, false, 1>", "k_strip<2, false, 2>"}, {"k_strip<2, true, 0>", "k_strip<2, true, 1>", "k_strip<2, true, 2>"}}};
  return names[(T - 1 + 15) / 16][acc64 ? 1 : 0][strip_kind(tab)];
}

int launch_strip(const StripTable& tab, const StripPort& p0, const StripPort& p1, int T, bool acc64,
                 hipStream_t s) {
  if (tab.count == 0) return NUGPR_OK;
  if (T < 1 || T > MAX_COLS) { set_error("vector block wider than 33 columns"); return NUGPR_ERR_INVALID; }
  StripArgs a;
  a.port[0] = p0;
  a.port[1] = p1;
  a.items = tab.dev;
  a.T = T;
  const int ng = (T - 1 + 15) / 16;
  switch (strip_kind(tab)) {
    case STRIP_ROWMAJOR: return acc64 ? launch_width<true, STRIP_ROWMAJOR>(ng, tab.count, T, s, a) : launch_width<false, STRIP_ROWMAJOR>(ng, tab.count, T, s, a);
    case STRIP_SYM: return acc64 ? launch_width<true, STRIP_SYM>(ng, tab.count, T, s, a) : launch_width<false, STRIP_SYM>(ng, tab.count, T, s, a);
    default: return acc64 ? launch_width<true, STRIP_PLAIN>(ng, tab.count, T, s, a) : launch_width<false, STRIP_PLAIN>(ng, tab.count, T, s, a);
  }
}

}  // namespace nugpr
