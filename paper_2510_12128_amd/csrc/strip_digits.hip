// Strips on the integer matrix cores: products of k_strip's symmetric and triangular items with vector blocks of 18 to 33 columns
// which the caller holds in fp32 and wants in fp32 (nugpr_matvec, nugpr_precond_apply).  The solver keeps the fp64 instructions: with its
// directions in digits too, a solve on 256 clusters of 4096 points took 157 iterations in place of 152.
//
// A 16 x 16 x 64 product of 8-bit integers takes a quarter of the cycles of a 16 x 16 x 4 one in fp64 for sixteen times the
// terms, its sums are exact, and unlike the fp64 instructions it runs beside the vector ALUs.  So both factors are written
// in digits to base 256 (balanced, -128 .. 127):
//   matrix  64 entries of a row as whole numbers of up to 2^31 in units of 2^-31 of the power of two above their largest: four
//           digits.  An entry keeps the 24 bits it is stored with down to 2^-7 of the largest, and is off by half a unit below; the
//           diagonal of a symmetric matrix, which is larger than the rest, is left out and multiplied in fp64.
//   vector  64 rows of a column as whole numbers of up to 2^38 in units of 2^-38 of the power of two above their largest: five digits.
// Of the twenty products of digits the fourteen are taken whose place is at least 2^-32 of the first one's; their sums over
// 64 columns, by place in 32 bits, then form one fp64 number, which is scaled and added to the fp64 sums.  A value that is not
// finite makes its column's scale, and with it the column's results in the cluster, NaN.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "nugpr_internal.h"

namespace nugpr {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int MAT_DIGITS = 4, VEC_DIGITS = 5, G = 2;

// ---------------------------------------------------------------------------
// vector blocks in digits
// ---------------------------------------------------------------------------
// A block of 64 rows (DIGIT_BLOCK bytes): VEC_DIGITS fragments of 1 KiB for each of two groups of 16 columns (columns 1 + 16 g ..), the first digit first; a
// fragment with the digits of column 0, which has none of the groups to fill, in its first five columns; then the scales (fp64)
// of the groups' columns and of column 0 in a KiB of their own.  Lane (m, kg) of a fragment has column m, rows 16 f + 4 kg + c in byte
// 4 f + c: the operand of one matrix instruction, in the order in which a lane of k_strip_digits holds the rows' entries.
// One workgroup per block; columns past T are zero.
__device__ __forceinline__ long long whole_number(double x) {      // |x| <= 2^38
  const double hi = rint(x * 0x1p-16);
  return (long long)(int)hi * 65536 + (int)rint(fma(hi, -65536.0, x));
}
__global__ __launch_bounds__(256) void k_digits(const ClusterInfo* __restrict__ cl, int nc, uint32_t cluster_blocks, const double* __restrict__ D,
                                                const double* __restrict__ S, int ncr, int T, unsigned char* __restrict__ out) {
  constexpr int COLS = 16 * G + 1;
  __shared__ double rows[TILE * COLS], part[4][COLS], unit[COLS];
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t block = blockIdx.x;
  out += (uint64_t)block * DIGIT_BLOCK;
  const double* from;
  int valid;
  if (block < cluster_blocks) {
    int lo = 0, hi = nc;                             // the cluster lies in lo .. hi - 1: 64 places of it are looked at at a time
    while (hi - lo > 1) {
      const int stride = (hi - lo + 63) / 64, at = lo + lane * stride;
      const bool before = at < hi && cl[at].prow / TILE <= block;
      lo += (__popcll(__ballot(before)) - 1) * stride;
      hi = min(hi, lo + stride);
    }
    const ClusterInfo& c = cl[__builtin_amdgcn_readfirstlane(lo)];
    const uint32_t r = (block - c.prow / TILE) * TILE;
    from = D + (uint64_t)(c.row0 + r) * T;
    valid = min(TILE, (int)(c.b - r));
  } else {
    const uint32_t r = (block - cluster_blocks) * TILE;
    from = S + (uint64_t)r * T;
    valid = min(TILE, ncr - (int)r);
  }
  for (int e = tid; e < TILE * T; e += 256) rows[e] = e < valid * T ? from[e] : 0.0;
  __syncthreads();
  // the largest magnitude of a column; not finite if one of its values is not
  if (tid < 4 * COLS) {
    const int col = tid % COLS, q = tid / COLS;
    double most = 0.0, odd = 0.0;
    if (col < T)
      for (int r = q; r < TILE; r += 4) {
        const double x = fabs(rows[r * T + col]);
        most = fmax(most, x);
        odd += x - x;                                // (zero, or NaN)
      }
    part[q][col] = most + odd;
  }
  __syncthreads();
  if (tid < COLS) {
    const double most = fmax(fmax(part[0][tid], part[1][tid]), fmax(part[2][tid], part[3][tid]));
    const double odd = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
    const bool bad = !(odd == odd) || !(most < INFINITY);
    const int e = most > 0.0 && !bad ? max(ilogb(most) + 1, -900) : 0;      // 2^e > most
    unit[tid] = bad ? 0.0 : ldexp(1.0, 38 - e);
    reinterpret_cast<double*>(out + (G * VEC_DIGITS + 1) * 1024)[tid == 0 ? 16 * G : tid - 1] = bad ? (double)NAN : ldexp(1.0, e - 38);
  }
  __syncthreads();
  if (tid >= 64 * (G + 1)) return;
  const int cg = tid >> 6, m = lane & 15, kg = lane >> 4, col = cg == G ? 0 : 1 + 16 * cg + m;
  const double u = col < T ? unit[col] : 0.0;
  v4i digit[VEC_DIGITS];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    uint32_t word[VEC_DIGITS] = {};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double x = u > 0.0 ? rows[(16 * f + 4 * kg + c) * T + col] * u : 0.0;
      const long long q = whole_number(x) + 0x8080808080ll;
#pragma unroll
      for (int i = 0; i < VEC_DIGITS; ++i) word[VEC_DIGITS - 1 - i] |= (uint32_t)((q >> (8 * i)) & 0xff) << (8 * c);
    }
#pragma unroll
    for (int i = 0; i < VEC_DIGITS; ++i) digit[i][f] = (int)(word[i] ^ 0x80808080u);
  }
  if (cg < G) {
#pragma unroll
    for (int i = 0; i < VEC_DIGITS; ++i) *reinterpret_cast<v4i*>(out + (cg * VEC_DIGITS + i) * 1024 + lane * 16) = digit[i];
  } else {
    v4i mine = (v4i){0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < VEC_DIGITS; ++i)
      if (m == i) mine = digit[i];
    *reinterpret_cast<v4i*>(out + G * VEC_DIGITS * 1024 + lane * 16) = mine;
  }
}

int launch_digits(nugpr_ctx* c, const void* D, const void* S, int T, hipStream_t s) {
  const Layout& L = c->L;
  const uint32_t cb = (uint32_t)(L.rows_pad / TILE), blocks = cb + (S ? (uint32_t)(L.ldc / TILE) : 0u);
  hipLaunchKernelGGL(k_digits, dim3(blocks), dim3(256), 0, s, c->d_cl, L.nc, cb, static_cast<const double*>(D), static_cast<const double*>(S), L.ncr, T,
                     static_cast<unsigned char*>(c->digits));
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

// ---------------------------------------------------------------------------
// the strips
// ---------------------------------------------------------------------------
// One workgroup = one item of k_strip's tables; the tiles of a symmetric one in the same order (its partner strip reads the same stored
// tile at the same step).  Wave g takes the rows 16 g .. 16 g + 15 of the strip, so no sums have to meet.  A tile's digits of the
// vector come into one of two stages of LDS (straight from memory, each wave a quarter) for all four waves, the wave's 16 x 64
// entries into registers, both a tile ahead; one workgroup barrier a tile.  32 KiB of LDS and 128 registers a lane: four workgroups on a
// compute unit.
// What bounds it: what memory delivers.  64 uneven clusters of 4096 points, 33 columns: 1.07 ms (fp64 instructions 1.40), 5.5 GB at 5.2 TB/s, with
// the matrix cores at 43 % and the vector ALUs at 75 % of the cycles; partner strips of clusters this large are not on the chip
// together for long enough to meet in L2.  Not kept there: three stages and two workgroups on a compute unit 1.26 ms, streaming
// hint for the matrix 1.2, the tiles in rotating blocks of 4, 8 or 16 1.07.  16 x 64 entries with one scale in place of
// one a row: 0.7 % more error of the product for the same time.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_strip_digits(const StripArgs a) {
#if __HIP_DEVICE_COMPILE__
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  typedef __attribute__((address_space(3))) const v4i* lds_v4i;
  typedef __attribute__((address_space(3))) const double* lds_double;
  constexpr int STAGE = DIGIT_BLOCK, NVL = STAGE / 4096;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];       // two stages, then 2 KiB a wave
  const int T = a.T, tid = threadIdx.x, lane = tid & 63, m = lane & 15, kg = lane >> 4;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t die = blockIdx.x % NUM_XCD, row = blockIdx.x / NUM_XCD;
  const uint32_t at = a.from[die] + (row >> a.sys_log2);
  if (at >= a.from[die + 1]) return;                 // (the other dies' lists are longer)
  const StripItem& it = a.items[at];
  const StripPort& pt = a.port[(row & ((1u << a.sys_log2) - 1)) * (uint32_t)a.sys_ports + it.port];
  const int c_begin = (int)it.c_begin, c_end = (int)it.c_end;
  int nb = c_end > c_begin ? (c_end - c_begin + TILE - 1) >> 6 : 0;
  const uint32_t fl = it.blocked;
  const bool sym = (fl & 2u) != 0;
  const int kind = (int)((fl >> 2) & 3u), tb = c_begin >> 6, j_abs = (int)it.row_in_block >> 6;
  if (pt.live && !any_live(pt.live, j_abs, tb, nb, lane)) nb = 0;
  const int jr = ((fl >> 4) & 0x7ffu) ? (int)((fl >> 15) & 0x7ffu) : j_abs - tb;
  const int jm = !sym || nb <= 0 ? 0 : (jr < nb ? jr : jr % nb);
  // the tile that holds the strip's own diagonal, and what becomes of it: multiplied apart (symmetric) or masked (triangular)
  const int mode = (int)it.mode, own_tile = mode == 1 ? nb - 1 : mode == 2 ? 0 : kind == 0 ? j_abs - tb : -1;
  const int thr = !sym || kind == 1 ? 0x7fffffff : (kind == 2 ? -1 : jr);      // tiles past it are read transposed
  const char* A = reinterpret_cast<const char*>(pt.A + it.a_off);
  const char* V = reinterpret_cast<const char*>(pt.digits) + (uint64_t)(it.in_block + (uint32_t)tb) * STAGE;
  const uint32_t lda = it.lda;
  auto tile_of = [&](const int u) { int p = min(u, nb - 1) - jm; p += p < 0 ? nb : 0; return p; };

  const uint32_t ooff = (uint32_t)((m * 16 + 4 * kg) * 4);
  const uint32_t toff = (uint32_t)(((((lane >> 2) & 3) * 4 + (lane >> 4)) * 16 + (lane & 3) * 4) * 4);
  v4f raw[2][4];
  auto load = [&](auto s_c, const int u) {           // tile of sequence number u into stage s; past the end out of range
    constexpr int s = decltype(s_c)::value;
    const bool valid = u < nb;
    const int p = tile_of(u), c = c_begin + TILE * p;
    const auto vres = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(V + (uint64_t)p * STAGE), 0, valid ? STAGE : 0, 0x00027000);
#pragma unroll
    for (int i = 0; i < NVL; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vres, (lds_ptr)(lds + s * STAGE + (g * NVL + i) * 1024), 16, (uint32_t)lane * 16u, (g * NVL + i) * 1024, 0, 0);
    const bool tr = p > thr;
    const int64_t own = (int64_t)(c >> 5) * (TILE * BLK_COLS) + g * 2 * FRAG;
    const int64_t far = (int64_t)(tb - j_abs + p) * TILE * (int64_t)lda + (int64_t)(2 * j_abs) * (TILE * BLK_COLS) + (g >> 1) * (TILE * BLK_COLS) + (g & 1) * FRAG;
    const auto res = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(A + (tr ? far : own) * 4), 0, valid ? 0x7fffffff : 0, 0x00027000);
#pragma unroll
    for (int q = 0; q < 4; ++q) {                    // columns 16 q .. of the tile
      const int so = !valid ? 0 : (tr ? q * 2 * FRAG : (q >> 1) * (TILE * BLK_COLS) + (q & 1) * FRAG) * 4;
      raw[s][q] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(res, tr ? toff : ooff, so, 0));
    }
  };
  // column 0: lane (m, kg) adds up what digit m < 5 gives
  double acc[G][4], acc0[4] = {0.0, 0.0, 0.0, 0.0};
  const double place0 = m < VEC_DIGITS ? ldexp(1.0, 8 * (VEC_DIGITS - 1 - m)) : 0.0;
#pragma unroll
  for (int n = 0; n < G; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[n][i] = 0.0;
  float diagonal = 0.f;                              // of row m, in the lane whose columns hold it (kg = m / 4)
  float* turn = reinterpret_cast<float*>(lds + 2 * STAGE + g * 2048);
  auto tile = [&](auto s_c, const int u) {
    constexpr int s = decltype(s_c)::value;
    const int p = tile_of(u);
    if (p > thr) {                          // to its transpose, through the wave's own piece of LDS
#pragma unroll
      for (int h = 0; h < 4; h += 2) {
#pragma unroll
        for (int q = h; q < h + 2; ++q) reinterpret_cast<v4f*>(turn)[(q - h) * 64 + lane] = raw[s][q];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int q = h; q < h + 2; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) raw[s][q][i] = turn[(q - h) * 256 + 64 * i + lane];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
    if (p == own_tile) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 16 * g + m, c = 16 * q + 4 * kg + i;
          if (mode == 0) {
            diagonal = r == c ? raw[s][q][i] : diagonal;
            raw[s][q][i] = r == c ? 0.f : raw[s][q][i];
          } else {
            raw[s][q][i] = (mode == 1 ? c <= r : c >= r) ? raw[s][q][i] : 0.f;
          }
        }
    }
    // the largest entry of row m, and the power of two that takes it to at most 127.5 / 128 2^31: the largest in balanced digits
    float most = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      most = fmaxf(most, fmaxf(fabsf(raw[s][q][0]), fabsf(raw[s][q][1])));
      most = fmaxf(most, fmaxf(fabsf(raw[s][q][2]), fabsf(raw[s][q][3])));
    }
    {                                                // over the four lanes of the row
      const auto near = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, most), __builtin_bit_cast(uint32_t, most), false, false);
      most = fmaxf(__builtin_bit_cast(float, (uint32_t)near[0]), __builtin_bit_cast(float, (uint32_t)near[1]));
      const auto far = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, most), __builtin_bit_cast(uint32_t, most), false, false);
      most = fmaxf(__builtin_bit_cast(float, (uint32_t)far[0]), __builtin_bit_cast(float, (uint32_t)far[1]));
    }
    const int ex = (int)((__builtin_bit_cast(uint32_t, most) + 0x20000u) >> 23), up_ex = min(284 - ex, 254);
    const float up = __builtin_bit_cast(float, (uint32_t)up_ex << 23);
    // its inverse, as the upper half of a double (NaN for entries that are not finite), and that of the rows that this lane's sums belong to
    const int back = ex >= 255 ? 0x7ff80000 : (1023 + 127 - up_ex) << 20;
    double weight[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) weight[i] = __hiloint2double(__shfl(back, 4 * kg + i), 0);
    v4i digit[MAT_DIGITS];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        int whole;
        asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(whole) : "v"(raw[s][q][i] * up));      // to the nearest
        x[i] = (uint32_t)whole + 0x80808080u;
      }
      const uint32_t lo01 = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u), lo23 = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u);
      const uint32_t hi01 = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u), hi23 = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
      digit[3][q] = (int)(__builtin_amdgcn_perm(lo23, lo01, 0x05040100u) ^ 0x80808080u);
      digit[2][q] = (int)(__builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u);
      digit[1][q] = (int)(__builtin_amdgcn_perm(hi23, hi01, 0x05040100u) ^ 0x80808080u);
      digit[0][q] = (int)(__builtin_amdgcn_perm(hi23, hi01, 0x07060302u) ^ 0x80808080u);
    }
    const unsigned char* st = lds + s * STAGE;
#pragma unroll
    for (int n = 0; n < G; ++n) {
      v4i v[VEC_DIGITS], place[VEC_DIGITS];
#pragma unroll
      for (int i = 0; i < VEC_DIGITS; ++i) v[i] = *(lds_v4i)(st + (n * VEC_DIGITS + i) * 1024 + lane * 16);
      const double unit = 0x1p24 * *(lds_double)(st + (G * VEC_DIGITS + 1) * 1024 + (16 * n + m) * 8);
#pragma unroll
      for (int i = 0; i < VEC_DIGITS; ++i) place[i] = (v4i){0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < MAT_DIGITS; ++i)
#pragma unroll
        for (int j = 0; i + j < VEC_DIGITS; ++j) place[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(digit[i], v[j], place[i + j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {                  // |place[k]| <= (k + 1) 2^20: two at a time fit 32 bits
        const int t0 = (place[0][i] << 8) + place[1][i], t1 = (place[2][i] << 8) + place[3][i];
        const double sum = fma((double)t0, 0x1p24, fma((double)t1, 0x1p8, (double)place[4][i]));
        acc[n][i] = fma(sum, weight[i] * unit, acc[n][i]);
      }
    }
    {
      const v4i v = *(lds_v4i)(st + G * VEC_DIGITS * 1024 + lane * 16);
      const double unit = place0 * *(lds_double)(st + (G * VEC_DIGITS + 1) * 1024 + 16 * G * 8);
      v4i place[MAT_DIGITS];
#pragma unroll
      for (int i = 0; i < MAT_DIGITS; ++i) place[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(digit[i], v, (v4i){0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t0 = (place[0][i] << 8) + place[1][i], t1 = (place[2][i] << 8) + place[3][i];
        acc0[i] = fma(fma((double)t0, 0x1p16, (double)t1), weight[i] * unit, acc0[i]);
      }
    }
  };
  // Every wave has read tile u - 1 when tile u is there, and its stage takes tile u + 1.
  auto step = [&](auto s_c, const int u) {
    constexpr int s = decltype(s_c)::value;
    __builtin_amdgcn_s_waitcnt(0x0F70u);             // vmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    load(std::integral_constant<int, 1 - s>(), u + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (u < nb) tile(s_c, u);
    __builtin_amdgcn_sched_barrier(0);
  };
  load(std::integral_constant<int, 0>(), 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
  for (int u = 0; u < nb; u += 2) {
    step(std::integral_constant<int, 0>(), u);
    step(std::integral_constant<int, 1>(), u + 1);
  }
  // (what is still on its way to LDS is out of range and stores nothing that anyone reads, but must not outlive the workgroup)
  __builtin_amdgcn_s_waitcnt(0x0F70u);
  double* out = static_cast<double*>(pt.out) + (uint64_t)it.out_part * pt.out_part_stride + (uint64_t)it.out_row0 * T;
  const double* din = static_cast<const double*>(pt.in) + (uint64_t)(it.in_row0 + it.row_in_block) * T;
  const double dadd = (double)it.diag_add * pt.diag_add, scale = pt.scale;
  const int nrows = (int)it.nrows;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int x = 1; x < 8; x *= 2) acc0[i] += __shfl_xor(acc0[i], x);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 16 * g + 4 * kg + i;
    const double d = (double)__shfl(diagonal, 20 * kg + i);      // (row 4 kg + i of the wave's)
    auto put = [&](const int col, double v) {
      if (own_tile >= 0 && mode == 0) v = fma(d, din[r * T + col], v);
      v *= scale;
      if (dadd != 0.0) v = fma(dadd, din[r * T + col], v);
      if (pt.accumulate) v += out[r * T + col];
      out[r * T + col] = v;
    };
    if (r < nrows) {
#pragma unroll
      for (int n = 0; n < G; ++n)
        if (1 + 16 * n + m < T) put(1 + 16 * n + m, acc[n][i]);
      if (m == 0) put(0, acc0[i]);
    }
  }
#endif
}

// The triangular strips (run_precond): from 768 of 16 tiles or more on average.  Apply of 33 columns, fp64 instructions / this: 12 x 4096 285 / 259 us,
// 32 x 4096 625 / 546, 64 x 2048 349 / 328; but 64 x 1024 (8.5 tiles) 105 / 116, 8 x 4096 (512 strips) 173 / 190, 128 x 512 71 / 77.
// From 512 strips and 5000 tiles on, of more than 17 columns.  Product of 33 columns, fp64 instructions / this: 8 clusters of
// 2048 points (256 strips) 62.8 / 68.0 us, 16 (512) 96.1 / 87.4, 64 349 / 265, 32 x 1024 (512) 65.8 / 63.8, 128 x 512 106 / 85, 32 x 4096 605 / 466; of
// 25 columns 59.5 / 64.3, 94.4 / 85.6, 336 / 251, 64.1 / 62.0, 99 / 78, 592 / 453.  Up to 17 columns there is nothing to gain: the matrix alone
// takes that long to arrive (64 x 2048 200 / 203, 32 x 4096 377 / 366).  With few tiles a strip the
// digits' launch is what is felt: 64 x 512 (5120 tiles) 55.9 / 53.9.
bool takes_digits(const nugpr_ctx* c, const StripTable& tab, int T) {
  return c->acc64 && c->digits && T > 17 && tab.count >= 512 && tab.tiles >= 5000;
}

int launch_strip_digits(const StripArgs& a, int count, hipStream_t s) {
  constexpr int lds = 2 * DIGIT_BLOCK + 4 * 2048;
  hipLaunchKernelGGL(k_strip_digits, dim3(count), dim3(256), lds, s, a);
  NUGPR_HIP(hipGetLastError());
  return NUGPR_OK;
}

}  // namespace nugpr
