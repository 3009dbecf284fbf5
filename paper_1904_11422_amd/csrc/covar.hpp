// Covariance form of the accumulated image (N = 64, 3 x 3 Gaussian kernels).
//
// The image summed over T samples is the transform of the autocorrelation of
// the gridded E-field (paper Sec. 2.1: the multiplication-convolution theorem
// that makes Eq. (5) the image of Eq. (1)).  With F_P = sum_a g_a b_a e_a,
//   sum_t F_P conj(F_Q) (k) = sum_d R_PQ(d) exp(+2 pi i d.k / N),
//   R_PQ(d) = sum_b sum_u conj(w_b(u) g_b) M_b(u + d),
//   M_b(u)  = sum_a w_a(u) g_a V_ab,     V_ab = sum_t e_a conj(e_b),
// so the time sum moves in front of the transform: V is a sum of products of
// 4-bit integers (exact in int32, and a contraction the matrix cores run at
// their int8 rate), and the gridding and the transform run once per channel
// instead of once per sample.  All offsets d are taken modulo N: the image is
// sampled at N points, so the circular autocorrelation is all it can see.
//
//   cov_corr_kernel   V of a channel, 128 x 128 antennas per workgroup;
//   cov_sum_kernel    where its samples are split, the splits added;
//   cov_fold_kernel   R of a range of a channel's antennas b, in float64;
//   cov_image_kernel  the ranges' sums added, transformed and written, in float64.
#pragma once
#include <type_traits>
#include <utility>

#include "fused.hpp"

namespace epic {

constexpr int kCovTile = 128;       // antennas per side of a workgroup's tile of V
constexpr int kCovStage = 64;       // samples staged in LDS at a time
constexpr int kCovPitch = 80;       // bytes per staged antenna row: 64 samples + 16, so that
                                    // 16 consecutive rows' 16-byte reads fall on distinct banks
constexpr int kCovMaxSplit = 32768; // samples per partial sum: 256 * 128 * T < 2^31

using i32x4 = __attribute__((ext_vector_type(4))) int;
using i32x16 = __attribute__((ext_vector_type(16))) int;

// Place of antenna a in the stored covariance: the staging transposes four
// antennas' samples at once and writes antenna 4 g + q to LDS row 32 q + g
// (of its 128), which spreads the writes over the banks; V keeps that order.
__host__ __device__ constexpr int cov_slot(int a) { return (a & ~127) | ((a & 3) << 5) | ((a >> 2) & 31); }
__host__ __device__ constexpr int cov_ant(int s) { return (s & ~127) | ((s & 31) << 2) | ((s >> 5) & 3); }

template <int P> struct CovShape {
  static constexpr int NPROD = P == 2 ? 3 : 1;   // planes of V: XX, YY, XY or XX
};

struct CovCorrArgs {
  const uint8_t* efield;    // [T][C][P][A]
  int2* v;                  // [channel - c0][split][n_prod][b: ap][a: ap] (re, im), slots of cov_slot
  int64_t n_time;
  int64_t t_split;          // samples per split, a multiple of kCovStage
  int n_chan, n_ant, ap;    // ap: n_ant rounded up to kCovTile
  int c0, n_split;
  int n_prod;               // planes written: NPROD, or 4 with YX = conj(XY) transposed (the gradient)
  int total;                // workgroups: channels * n_split * tiles
};

// Tiles (I, J) of a-block I and b-block J: the upper triangle (I <= J) of XX
// and of YY, whose mirror images the same workgroup writes, and all of XY.
__host__ __device__ __forceinline__ int cov_tiles(int nb, int P) {
  const int tri = nb * (nb + 1) / 2;
  return P == 2 ? 2 * tri + nb * nb : tri;
}

// Bound: the matrix cores' int8 rate.  A wave holds 64 x 64 pairs, real and
// imaginary (128 accumulator VGPRs), so every 16-byte operand read from LDS
// feeds four 32x32x32 products; samples stay packed (one byte) in LDS and are
// split into 16 re and 16 im (the nibble in the byte's high half, already a
// signed int8) after the read, half the LDS bytes of staging them split.  The
// imaginary part needs -im, which int8 cannot hold for 16 * (-8); the bitwise
// complement of the nibble is -im - 1, exact, and the excess sum_t re_a is
// taken from one dot product per operand.  132 channels of 256 dual-pol antennas,
// T = 1000: 132 us (41 at T = 64: mostly the covariances' 208 MB written) =
// 1.05 POP/s of 8 operations per pair and sample; 8.9 vector instructions per
// matrix one, of which about 4 are free, so the two take turns (matrix pipes 25 %,
// vector ALU 31 % busy).
// Four antennas' samples are one load at any address (the hardware loads an
// unaligned word); WHOLE: A % 4 = 0, no group of four reaches past its row.
template <int P, bool WHOLE>
__global__ __launch_bounds__(256, 2) void cov_corr_kernel(CovCorrArgs a) {
  __shared__ __align__(16) uint8_t lds[2][2 * kCovTile * kCovPitch];
  const int logical = wg_range_index(blockIdx.x, a.total, 1);
  const int nb = a.ap / kCovTile, tri = nb * (nb + 1) / 2, tiles = cov_tiles(nb, P);
  const int cl = logical / (a.n_split * tiles), rem = logical % (a.n_split * tiles);
  const int split = rem / tiles;
  int tile = rem % tiles;
  int prod = 0;
  if (P == 2 && tile >= tri) {
    tile -= tri;
    prod = 1;
    if (tile >= tri) {
      tile -= tri;
      prod = 2;
    }
  }
  int I, J;
  if (prod == 2) {
    I = tile % nb;
    J = tile / nb;
  } else {
    J = 0;
    while ((J + 1) * (J + 2) / 2 <= tile) ++J;
    I = tile - J * (J + 1) / 2;
  }
  const bool mirror = prod != 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave & 1, wj = wave >> 1;
  const bool works = !(mirror && I == J && wi > wj);

  // staging: lane -> four antennas of a (lanes 0-31) or b (lanes 32-63), the
  // wave's 16 samples of the stage
  const int side = lane >> 5, g = lane & 31;
  const int ant = kCovTile * (side ? J : I) + 4 * g;
  const int pol = prod == 1 ? 1 : (prod == 2 ? side : 0);
  const int64_t tstride = (int64_t)a.n_chan * P * a.n_ant;
  const int64_t t_begin = split * a.t_split;
  const int64_t t_end = t_begin + a.t_split < a.n_time ? t_begin + a.t_split : a.n_time;
  // uniform row address plus a 32-bit lane offset; lanes past the antennas
  // read the row's first and are cleared
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  const int n_row = (int)(t_end - t_begin);
  const uint8_t* src = a.efield + t_begin * tstride + (int64_t)(a.c0 + cl) * P * a.n_ant;
  const int nvalid = a.n_ant - ant;    // antennas of the four that exist
  const uint32_t lmask = nvalid >= 4 ? ~0u : nvalid <= 0 ? 0u : (1u << (8 * nvalid)) - 1u;
  // the row's last group reads its last four bytes and shifts them down
  const int first = nvalid <= 0 ? 0 : WHOLE || nvalid >= 4 || a.n_ant < 4 ? ant : a.n_ant - 4;
  const uint32_t loff = (uint32_t)(pol * a.n_ant + first);
  const int lshift = nvalid > 0 ? 8 * (ant - first) : 0;
  const int n_stage = (int)((t_end - t_begin + kCovStage - 1) / kCovStage);
  auto load = [&](int k, uint32_t (&raw)[16]) {
    if (k >= n_stage) k = n_stage - 1;
    // past the end the last row again, cleared when it is staged
    const int last = n_row - 1 - (k * kCovStage + 16 * uwave);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint8_t* row = src + (k * kCovStage + 16 * uwave + (i < last ? i : last)) * tstride;
      if (WHOLE || a.n_ant >= 4) {
        __builtin_memcpy(&raw[i], row + loff, 4);
      } else {                         // one to three antennas
        raw[i] = 0;
#pragma unroll
        for (int q = 0; q < 3; ++q)
          if (q < nvalid) raw[i] |= (uint32_t)row[loff + q] << (8 * q);
      }
    }
  };

  i32x16 re[2][2], im[2][2];          // [b tile][a tile]
  int sa[2] = {0, 0};                 // 16 sum_t re_a over the lane's half of the samples
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int i = 0; i < 16; ++i) re[x][y][i] = im[x][y][i] = 0;

  auto stage = [&](int k, uint32_t (&raw)[16]) {
    uint8_t* buf = lds[k & 1];
    const int rows = n_row - (k * kCovStage + 16 * uwave);   // of the wave's 16
    {
      uint32_t u[4][4];                // [antenna][four groups of four samples]
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        uint32_t in[4], tr[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) in[i] = (WHOLE ? raw[4 * s + i] : raw[4 * s + i] >> lshift) & (4 * s + i < rows ? lmask : 0u);
        transpose4(in, tr);
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q][s] = tr[q];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint4*>(buf + (size_t)(kCovTile * side + 32 * q + g) * kCovPitch + 16 * wave) =
            make_uint4(u[q][0], u[q][1], u[q][2], u[q][3]);
    }
    __syncthreads();
    load(k + 2, raw);
    if (works) {
#pragma unroll
      for (int ks = 0; ks < kCovStage / 32; ++ks) {
        const int off = 32 * ks + 16 * (lane >> 5);
        i32x4 ra[2], ia[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const i32x4 r = *reinterpret_cast<const i32x4*>(buf + (size_t)(32 * (2 * wi + x) + (lane & 31)) * kCovPitch + off);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            ra[x][i] = r[i] & 0xF0F0F0F0;
            ia[x][i] = (r[i] << 4) & 0xF0F0F0F0;
            sa[x] = __builtin_amdgcn_sdot4(ra[x][i], 0x01010101, sa[x], false);
          }
        }
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const i32x4 r = *reinterpret_cast<const i32x4*>(
              buf + (size_t)(kCovTile + 32 * (2 * wj + y) + (lane & 31)) * kCovPitch + off);
          i32x4 rb, ib, nb4;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            rb[i] = r[i] & 0xF0F0F0F0;
            ib[i] = (r[i] << 4) & 0xF0F0F0F0;
            nb4[i] = ib[i] ^ 0xF0F0F0F0;
          }
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            re[y][x] = __builtin_amdgcn_mfma_i32_32x32x32_i8(rb, ra[x], re[y][x], 0, 0, 0);
            im[y][x] = __builtin_amdgcn_mfma_i32_32x32x32_i8(rb, ia[x], im[y][x], 0, 0, 0);
            re[y][x] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ib, ia[x], re[y][x], 0, 0, 0);
            im[y][x] = __builtin_amdgcn_mfma_i32_32x32x32_i8(nb4, ra[x], im[y][x], 0, 0, 0);
          }
        }
      }
    }
  };
  uint32_t raw0[16], raw1[16];         // two stages' loads in flight
  if (n_stage > 0) {
    load(0, raw0);
    load(1, raw1);
  }
  for (int k = 0; k < n_stage; k += 2) {
    stage(k, raw0);
    if (k + 1 < n_stage) stage(k + 1, raw1);
  }
  if (!works) return;

  int2* v = a.v + ((int64_t)(cl * a.n_split + split) * a.n_prod + prod) * a.ap * a.ap;
  const bool yx = P == 2 && prod == 2 && a.n_prod == 4;
  int2* vm = yx ? v + (int64_t)a.ap * a.ap : v;      // plane of the mirror image
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int s1 = (sa[x] + __shfl_xor(sa[x], 32)) >> 4;
    const int as = kCovTile * I + 32 * (2 * wi + x) + (lane & 31);
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int i = 0; i < 16; i += 4) {
        const int bs = kCovTile * J + 32 * (2 * wj + y) + 2 * i + 4 * (lane >> 5);
        int2 val[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          val[j] = make_int2(re[y][x][i + j] >> 8, (im[y][x][i + j] >> 8) + s1);
          v[(int64_t)(bs + j) * a.ap + as] = val[j];
        }
        if (yx || (mirror && (I != J || wi != wj))) {
          int4* m = reinterpret_cast<int4*>(vm + (int64_t)as * a.ap + bs);
          m[0] = make_int4(val[0].x, -val[0].y, val[1].x, -val[1].y);
          m[1] = make_int4(val[2].x, -val[2].y, val[3].x, -val[3].y);
        }
      }
  }
}

struct CovSumArgs {
  int2* v;                  // cov_corr_kernel's output
  int64_t n;                // values of a channel and split (n_prod ap^2)
  int n_split;
  int64_t total;            // pairs of values: channels * n / 2
};

// Antenna b of a channel, in the order the fold takes them (by column): its
// first tap's cell in the programs' (possibly transposed) aperture and its
// kernel as row and column factors.
struct __align__(16) CovAnt {
  int ant, row, col;
  int voff;                 // its column in a plane of V, cov_slot(ant) * ap
  double wr[3];             // weights of rows row .. row + 2
  double wc[3];             // weights of columns col .. col + 2
  int lane, pad0[3];        // the gradient's lane of this index takes the antenna at index `lane`
};

constexpr int kCovAntsPast = 16;    // entries past the table that the fold's look-ahead may read

// Gridding program of the fold, per channel and wave: a wave grids RPW whole
// consecutive rows, its cells dealt to "slots" of 64 (one per lane) by number of
// entries, so that the lanes of a slot end together and a step is a read and
// the products, with no test per lane.  `ends` marks the steps that end a slot
// and store its cells; cells of no antenna are never written and stay zero.
// Padding reads a zero slot of E'.  Per lane: the cells' byte offsets and the
// steps' E' byte offsets, 16 bits each, and the steps' weights, all of it in
// registers for the whole range (a step read from memory in the loop would wait
// behind the prefetch of V).  A weight is the float64 product of the factors
// that the fold multiplies by on b's side: R is Hermitian in d to float64
// rounding only if the two sides agree, and half of it is taken from the other.
struct CovProgHead {
  uint32_t row_lo, row_hi;          // aperture rows of the wave
  uint32_t steps, ends;
};
template <int STEPS, int SLOTS> struct CovProgLane {
  uint32_t cell[SLOTS > 2 ? 2 : 1];
  uint32_t e[STEPS / 2];
  double w[STEPS];
};

struct CovFoldArgs {
  const int2* v;            // cov_corr_kernel's output, the splits added
  const float2* gains;      // [C][P][A]
  const CovProgHead* head;  // [C][waves]
  const void* prog;         // CovProgLane [C][waves][64]
  const CovAnt* ants;       // [C][A], and kCovAntsPast more that may be read
  double2* r;               // [workgroup + channel group][CovFold::ROWS][64]
  int n_ant, ap;
  int c0, n_split;
  int W;                    // workgroups
  int64_t units;            // channels * groups * antennas
};

// The fold's units, (channel, group of sets, antenna b) in that order, are cut
// into W consecutive ranges of equal length, one per workgroup; what a workgroup
// adds to channel group cg goes to slot w + cg (a boundary of either kind moves
// on by one).  First workgroup of the group's and its slots:
__host__ __device__ __forceinline__ int cov_owner(int64_t unit, int64_t units, int W) {
  return (int)(((unit + 1) * W - 1) / units);
}

// Shape of the fold: one workgroup of 1024 threads per CU and NV aperture grids at
// a time, R rows and W columns each, lanes along the columns (LR lanes per row)
// and "units" of LR lanes along d's rows, two rows of d per unit: the sums take
// 24 registers of a thread's 128, the program 36.  The products come in sets:
// Half the grid (two grids, 64 rows of d):
//   set 0  half planes of d: at P = 2 XX and YY of one antenna b, at P = 1 XX of
//          two;
//   set 1  (P = 2) the whole plane of XY, of two antennas b one after the other.
// Wide block (one grid, whose row takes a wave; 32 rows of d): XX, YY, and the
// halves d = 0 .. 31 and -32 .. -1 of XY; sets 0 and 2, 1 and 3 make a group.
// A workgroup makes all sets of a group for its antennas, so that ranges of equal
// length take equal time whatever a set costs.
// XX and YY need half of the plane of d (R(-d) = conj R(d)): rows 0 .. 31 for XX
// and 0 .. -31 for YY, row 32 riding in row 0's imaginary part (both are
// Hermitian in d's column alone, which tells them apart).  Of M_b a half plane
// reads only the rows at or past b's first (d >= 0) or up to its last (d <= 0),
// so about half of the waves grid for it.
// KIND: kCovMany, more than 256 antennas; kCovCrowded, more steps than the
// registers of the others hold (some of the program spills to scratch memory).
enum { kCovPlain, kCovMany, kCovCrowded };
template <int P, bool WIDE, int KIND> struct CovFold {
  static constexpr int N = 64, NT = 1024, NW = NT / 64;
  static constexpr int MAXA = KIND == kCovPlain ? 256 : 512;
  static constexpr int STEPS = KIND == kCovCrowded ? 24 : 12;     // program steps of a wave at most
  static constexpr int SLOTS = WIDE ? 4 : 1;                 // slots of a wave at most
  static constexpr int NV = WIDE ? 1 : 2;
  static constexpr int SETS = P == 1 ? 1 : WIDE ? 4 : 2;
  static constexpr int GROUPS = P == 2 && WIDE ? 2 : 1;      // of sets
  static constexpr int SROWS = 32 * NV;                      // rows of r per set
  static constexpr int ROWS = SETS / GROUPS * SROWS;         // ... and slot
  static constexpr int R = WIDE ? FusedShape<64>::HW : 32;   // rows of a grid
  static constexpr int W = WIDE ? 48 : 32;                   // columns of a grid
  static constexpr int RS = WIDE ? W + 1 : W + 4;            // row stride; column W stays zero
  static constexpr int RU = 2;                               // rows of d per unit
  static constexpr int PADR = RU + 1;                        // zero rows around each grid
  static constexpr int VS = (R + PADR) * RS;                 // grid stride
  static constexpr int MSIZE = PADR * RS + NV * VS;
  static constexpr int ES = MAXA + 16;                       // E' of one grid, with 16 zero slots
  static constexpr int LR = WIDE ? 64 : 32;
  static constexpr int HU = 32 / RU;                         // units of 32 rows of d
  static_assert(NT / LR * RU == SROWS, "a unit per two rows");
};

// f(0), f(1), .. f(N - 1) with compile-time indices, until one returns false.
template <typename F, int... I>
__device__ __forceinline__ void static_while_impl(F&& f, std::integer_sequence<int, I...>) {
  (void)(f(std::integral_constant<int, I>{}) && ...);
}
template <int N, typename F> __device__ __forceinline__ void static_while(F&& f) {
  static_while_impl(f, std::make_integer_sequence<int, N>{});
}

// The value of the lane before (DPP wave shift right by one, 0x138, or rotation,
// 0x13C: the first lane keeps its own, or takes the last one's).
template <int CTRL> __device__ __forceinline__ double lane_before(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false));
}

// Antennas b0 .. b1 - 1 (in column order) of channel a.c0 + cl, one set, into
// rout.  Eb, Mb: E' and the grids in LDS, two of each.
template <int P, int SET, bool WIDE, int KIND>
__device__ __forceinline__ void cov_fold_body(const CovFoldArgs& a, double2* const lds, double2* const rout, int cl,
                                              int b0, int b1) {
  using S = CovFold<P, WIDE, KIND>;
  constexpr int N = S::N, NT = S::NT, MAXA = S::MAXA, NV = S::NV, RS = S::RS, VS = S::VS, LR = S::LR, ES = S::ES, RU = S::RU;
  constexpr int NE = (NV * MAXA + NT - 1) / NT;
  constexpr int GB = 2;                 // steps whose reads are in flight together
  constexpr int NB = WIDE || (P == 2 && SET == 0) ? 1 : 2;   // antennas b per step
  constexpr bool XY = SET >= (WIDE ? 2 : 1);
  constexpr bool YYSET = WIDE && SET == 1;                   // YY alone
  constexpr bool PAIR = !WIDE && !XY;                        // each half of the units has a grid of its own
  const int tid = threadIdx.x, lane = tid & 63;
  const int c = a.c0 + cl;
  const int A = a.n_ant, ap = a.ap;
  const int n_it = (b1 - b0 + NB - 1) / NB;
  double2 *const Eb = lds, *const Mb = lds + 2 * NV * ES;
  // in the constant address space: uniform indices load through the scalar
  // cache, off the vector memory counter that the prefetch of V waits on
  using ConstAnt = const __attribute__((address_space(4))) CovAnt;
  ConstAnt* ants = (ConstAnt*)(a.ants + (int64_t)c * A);
  using ConstGain = const __attribute__((address_space(4))) float2;
  ConstGain* gains = (ConstGain*)(a.gains + (int64_t)c * P * A);

  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  CovProgHead head = a.head[c * S::NW + wave];
  head.steps = __builtin_amdgcn_readfirstlane(head.steps);
  head.ends = __builtin_amdgcn_readfirstlane(head.ends);
  const CovProgLane<S::STEPS, S::SLOTS> prog =
      reinterpret_cast<const CovProgLane<S::STEPS, S::SLOTS>*>(a.prog)[(int64_t)(c * S::NW + wave) * 64 + lane];
  // E' offsets unpacked (opaque: else they are unpacked at every step), where
  // there are registers for it
  constexpr bool UNPACK = KIND == kCovPlain || (WIDE && KIND == kCovMany);
  uint32_t eoff[UNPACK ? S::STEPS : 1];
  if constexpr (UNPACK) {
#pragma unroll
    for (int i = 0; i < S::STEPS; ++i) {
      eoff[i] = i & 1 ? prog.e[i / 2] >> 16 : prog.e[i / 2] & 0xFFFFu;
      asm volatile("" : "+v"(eoff[i]));
    }
  }
  const int row_lo = __builtin_amdgcn_readfirstlane(head.row_lo), row_hi = __builtin_amdgcn_readfirstlane(head.row_hi);

  // staging: element e = tid + NT i of the columns of V; a wave's 64 are in
  // one column (ap is a multiple of 128), so that all but the place in the
  // column and the gain of a is uniform
  int vec[NE], sofs[NE];                // element i: its column, and its place less tid
  float2 ga[NE];                        // its gain
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int e = tid + NT * i;
    vec[i] = __builtin_amdgcn_readfirstlane((e >= ap) + (e >= 2 * ap));
    sofs[i] = vec[i] < NV ? __builtin_amdgcn_readfirstlane(NT * i - vec[i] * ap) : 0;
    const int ant = cov_ant(tid + sofs[i]);
    ga[i] = make_float2(0.f, 0.f);
    if (vec[i] < NV && ant < A) ga[i] = a.gains[((int64_t)c * P + (YYSET || (P == 2 && PAIR && vec[i] == 1))) * A + ant];
  }
  // a channel's planes of one split are below 2^23 bytes: a uniform base and
  // 32-bit offsets
  const int plane = ap * ap;
  const int64_t vsplit = (int64_t)CovShape<P>::NPROD * plane * sizeof(int2);
  const char* vc = reinterpret_cast<const char*>(a.v) + cl * a.n_split * vsplit;
  // V of a step: loaded two steps before it is staged, with the antennas it is of.
  // Steps past the range read the antennas that follow (in the table), unused:
  // every step issues the same loads, which can be counted and waited for alone
  struct Pre {
    int2 v[NE];
    int ant[NB];
    float2 gain[NB];                    // b's
  };
  Pre pre0, pre1;
  ConstAnt* next = ants + b0;           // the first antenna of the step fetched next,
  int nant[NB], nvoff[NB];              // already looked up
  auto lookup = [&]() {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      nant[j] = next[j].ant;
      nvoff[j] = next[j].voff;
    }
    next += NB;
  };
  auto fetch = [&](Pre& p) {
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int v = vec[i] < NV ? vec[i] : 0;
      const int pl = P == 1 ? 0 : XY ? 2 : WIDE ? SET : v;
      const uint32_t col = __builtin_amdgcn_readfirstlane(pl * plane + (v ? nvoff[NB - 1] : nvoff[0]));
      p.v[i] = *reinterpret_cast<const int2*>(vc + 8u * (col + sofs[i] + (vec[i] < NV ? tid : 0)));
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      // grid 1 of XX | YY is YY's
      p.ant[j] = nant[j];
      ConstGain& k = gains[(XY || YYSET || (P == 2 && PAIR && vec[0] == 1) ? A : 0) + nant[j]];
      p.gain[j] = make_float2(k.x, k.y);
    }
    lookup();
  };
  auto stage = [&](double2* E, const Pre& p) {
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int v = vec[i];
      if (v >= NV) continue;
      const int ant = cov_ant(tid + sofs[i]);
      if (ant >= A) continue;
      int2 val = p.v[i];
      // the a = b terms are added (or left out) by cov_image_kernel
      if ((v ? p.ant[NB - 1] : p.ant[0]) == ant) val = make_int2(0, 0);
      const float2 kb = v ? p.gain[NB - 1] : p.gain[0];
      const double2 g = make_double2(ga[i].x, ga[i].y), k = make_double2(kb.x, kb.y);
      const double2 h = make_double2(fma(g.x, k.x, g.y * k.y), fma(g.y, k.x, -(g.x * k.y)));
      const double x = val.x, y = val.y;
      E[v * ES + tid + sofs[i]] = make_double2(fma(h.x, x, -(h.y * y)), fma(h.x, y, h.y * x));
    }
  };
  // the grids of one step: MASK bit v set: grid v is made
  auto grid_some = [&](auto mask, const double2* E, double2* M) {
    constexpr int MASK = decltype(mask)::value;
    const char* eb = reinterpret_cast<const char*>(E);
    char* mb = reinterpret_cast<char*>(M);
    double2 s[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) s[v] = make_double2(0.0, 0.0);
    // opaque copies: unpacked here and not, into twice the registers, before
    // the loop over the range
    uint32_t n = head.steps, ends = head.ends;
    asm volatile("" : "+s"(n), "+s"(ends));
    int slot = 0;
    auto steps = [&](auto first) {
      constexpr int st = decltype(first)::value * GB;
      if (st >= (int)n) return false;
      double2 e[GB][NV];                 // a step past the last: a read of E'[0], weight 0
#pragma unroll
      for (int i = 0; i < GB; ++i) {
        uint32_t off;
        if constexpr (UNPACK) {
          off = eoff[st + i];
        } else {
          uint32_t ew = prog.e[(st + i) / 2];
          asm volatile("" : "+v"(ew));
          off = i & 1 ? ew >> 16 : ew & 0xFFFFu;
        }
        const double2* p = reinterpret_cast<const double2*>(eb + off);
#pragma unroll
        for (int v = 0; v < NV; ++v)
          if (MASK >> v & 1) e[i][v] = p[v * ES];
      }
#pragma unroll
      for (int i = 0; i < GB; ++i) {
        const double w = prog.w[st + i];
#pragma unroll
        for (int v = 0; v < NV; ++v)
          if (MASK >> v & 1) {
            s[v].x = fma(w, e[i][v].x, s[v].x);
            s[v].y = fma(w, e[i][v].y, s[v].y);
          }
        if (S::SLOTS > 1 && (ends >> (st + i) & 1)) { // uniform over the wave
          uint32_t cw = slot < 2 ? prog.cell[0] : prog.cell[S::SLOTS > 2 ? 1 : 0];
          asm volatile("" : "+v"(cw));
          double2* cell = reinterpret_cast<double2*>(mb + (slot & 1 ? cw >> 16 : cw & 0xFFFFu));
          ++slot;
#pragma unroll
          for (int v = 0; v < NV; ++v)
            if (MASK >> v & 1) {
              cell[v * VS] = s[v];
              s[v] = make_double2(0.0, 0.0);
            }
        }
      }
      return true;
    };
    static_while<S::STEPS / GB>(steps);
    if (S::SLOTS == 1) {
      double2* cell = reinterpret_cast<double2*>(mb + prog.cell[0]);
#pragma unroll
      for (int v = 0; v < NV; ++v)
        if (MASK >> v & 1) cell[v * VS] = s[v];
    }
  };
  int r0, r1;                           // first rows of the antennas gridded next
  auto grid = [&](const double2* E, double2* M) {
    if (head.steps == 0) return;
    // rows that a half plane reads: past b's first (a unit's last row wraps to 31
    // rows before it, row d = 32 to 30), or up to its last
    auto up = [&](int r) { return row_hi >= r || (WIDE && row_lo <= r - 30); };
    auto down = [&](int r) { return row_lo <= r + 2 || (WIDE && row_hi >= r + 32); };
    constexpr std::integral_constant<int, 1> one{};
    if constexpr (WIDE) {
      if (SET == 1 || SET == 3 ? down(r0) : up(r0)) grid_some(one, E, M);
    } else if constexpr (XY) {
      grid_some(std::integral_constant<int, 3>{}, E, M);
    } else {
      const bool need0 = up(r0), need1 = P == 1 ? up(r1) : down(r1);
      if (need0 && need1) grid_some(std::integral_constant<int, 3>{}, E, M);
      else if (need0) grid_some(one, E, M);
      else if (need1) grid_some(std::integral_constant<int, 2>{}, E, M);
    }
  };

  // fold: unit u, column ux; the unit covers rows dfirst .. dfirst + RU - 1 of d
  const int u = tid / LR, ux = tid % LR;
  const int hset = PAIR ? __builtin_amdgcn_readfirstlane(u / S::HU) : 0;
  const int dy0 = RU * (PAIR ? u % S::HU : u);
  // YY's half plane runs downwards: its units cover d = -(dy0 + RU - 1) .. -dy0
  const bool down = YYSET || (P == 2 && PAIR && hset);
  const int dfirst = down ? 1 - RU - dy0 : dy0 + (SET == 3 ? 32 : 0);
  auto row_of = [&](int d) { return 32 * hset + dy0 + (down ? RU - 1 - d : d); };
  double2 q[3][RU];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int d = 0; d < RU; ++d) q[i][d] = make_double2(0.0, 0.0);
  const int ucol = ux < S::W ? ux : S::W;
  int x0 = 0, xfirst = -1;
  // Q_0 one lane on into Q_1; the columns move down
  auto advance = [&]() {
#pragma unroll
    for (int d = 0; d < RU; ++d) {
      const double2 t = q[0][d];
      double2 sh;
      if constexpr (LR == N) {           // the lanes are the whole circle of d
        sh = make_double2(lane_before<0x13C>(t.x), lane_before<0x13C>(t.y));
      } else {                           // the last column's d has had its last term
        sh = make_double2(lane_before<0x138>(t.x), lane_before<0x138>(t.y));
        if (ux == 0) sh = make_double2(0.0, 0.0);
        if (ux == LR - 1) rout[row_of(d) * N + ((LR - 1 - x0) & (N - 1))] = t;
      }
      q[0][d] = make_double2(q[1][d].x + sh.x, q[1][d].y + sh.y);
      q[1][d] = q[2][d];
      q[2][d] = make_double2(0.0, 0.0);
    }
    ++x0;
  };
  constexpr int NC = XY ? NB : 1;       // antennas a thread folds per step
  struct Cur {
    int row, col;
    double wr[3], wc[3];
  } held[NC];                           // those of the step gridded now, folded in the next
  ConstAnt* at = ants + b0;
  auto load_ant = [&]() {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      ConstAnt& t = at[PAIR && P == 1 ? hset : j];
      held[j].row = t.row;
      held[j].col = t.col;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        held[j].wr[i] = t.wr[i];
        held[j].wc[i] = t.wc[i];
      }
    }
    at += NB;
  };
  auto load_rows = [&](ConstAnt* t) {
    r0 = t[0].row;
    r1 = t[NB - 1].row;
  };
  // the antennas held; left: how many of them exist
  auto fold = [&](int left, const double2* M) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int k = PAIR && P == 1 ? hset : j;
      if (NB == 2 && k >= left) return;
      const Cur& b = held[j];
      if (xfirst < 0) x0 = xfirst = b.col;
      while (x0 < b.col) advance();
      const double2* Mv = M + (PAIR ? hset : j) * VS + S::PADR * RS + ucol;
      const int s = ((b.row + dfirst + S::PADR) & (N - 1)) - S::PADR;
      if (s < S::R) {
        double2 z[RU];
#pragma unroll
        for (int r = 0; r < RU + 2; ++r) {
          const double2 m = Mv[(s + r) * RS];
#pragma unroll
          for (int d = 0; d < RU; ++d) {
            if (r == d) z[d] = make_double2(b.wr[0] * m.x, b.wr[0] * m.y);
            else if (r > d && r - d < 3) {
              z[d].x = fma(b.wr[r - d], m.x, z[d].x);
              z[d].y = fma(b.wr[r - d], m.y, z[d].y);
            }
          }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int d = 0; d < RU; ++d) {
            q[i][d].x = fma(b.wc[i], z[d].x, q[i][d].x);
            q[i][d].y = fma(b.wc[i], z[d].y, q[i][d].y);
          }
      }
      if constexpr (WIDE && !XY) {
        if (dy0 == 0) {                  // i times row d = 32 into row 0
          const int s2 = ((b.row + 32 + S::PADR) & (N - 1)) - S::PADR;
          if (s2 < S::R && s2 >= -2) {
            double2 z = make_double2(0.0, 0.0);
#pragma unroll
            for (int r = 0; r < 3; ++r) {
              z.x = fma(b.wr[r], Mv[(s2 + r) * RS].x, z.x);
              z.y = fma(b.wr[r], Mv[(s2 + r) * RS].y, z.y);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
              double2& q0 = q[i][YYSET ? RU - 1 : 0];
              q0.x = fma(-b.wc[i], z.y, q0.x);
              q0.y = fma(b.wc[i], z.x, q0.y);
            }
          }
        }
      }
    }
  };

  load_rows(at);
  lookup();
  fetch(pre0);
  fetch(pre1);
  __syncthreads();                      // the last range's last reads done
  for (int i = tid; i < 2 * (NV * ES + S::MSIZE); i += NT) lds[i] = make_double2(0.0, 0.0);
  __syncthreads();
  stage(Eb, pre0);
  fetch(pre0);
  __syncthreads();
  // step `it`: grid it, stage it + 1 from `p`, fetch it + 3 into it, fold it - 1.
  // Gridding first and ahead of the other waves' folding: LDS and vector ALU
  // are then wanted by different waves
  auto step = [&](int it, Pre& p) {
    __builtin_amdgcn_s_setprio(1);
    grid(Eb + (it & 1) * NV * ES, Mb + (it & 1) * S::MSIZE);
    __builtin_amdgcn_s_setprio(0);
    load_rows(at + NB);
    if (it > 0) fold(NB, Mb + ((it - 1) & 1) * S::MSIZE);   // a step that is not the last is full
    load_ant();
    if (it + 1 < n_it) stage(Eb + ((it + 1) & 1) * NV * ES, p);
    fetch(p);
    __syncthreads();
  };
  for (int it = 0; it < n_it; it += 2) {
    step(it, pre1);
    if (it + 1 < n_it) step(it + 1, pre0);
  }
  fold(b1 - b0 - NB * (n_it - 1), Mb + ((n_it - 1) & 1) * S::MSIZE);

  // Q_0 and Q_1 into Q_2, then every d the range has touched; zero elsewhere
  if (xfirst < 0) x0 = xfirst = 0;      // the second grid of a range of one antenna
  advance();
  advance();
#pragma unroll
  for (int d = 0; d < RU; ++d) {
    double2* o = rout + row_of(d) * N;
    o[(ux - x0) & (N - 1)] = q[0][d];
    if (LR < N && ux < LR - (x0 - xfirst)) o[(LR - xfirst + ux) & (N - 1)] = make_double2(0.0, 0.0);
  }
}

// A channel costs A passes of a grid per product, whatever T is, in float64
// throughout: R is summed before the transform, so that its rounding spreads over
// every pixel alike, and a pixel far below the peak would lose what a sum of
// squares keeps (in float32, 3e-9 of the largest possible pixel: up to 4 % of
// pixels 50 dB below a point source's peak, and negative power).
// A workgroup takes the antennas b of its range in column order.  Per b:
// E'[a] = g_a conj(g_b) V_ab is staged, gridded with the channel's program
// (held in registers for the whole range), and folded into R: a thread owns
// one aperture column and two rows of d, forms the row taps of M_b at its rows,
// and adds them, times the three column taps, to its sums Q_0 .. Q_2 of the
// aperture columns col .. col + 2.  When the next antenna starts at the next
// column, Q_0 moves one lane on into Q_1 (the same d), so a sum stays in
// registers until its last term and R is written once.
// Bound: the chain of a step (an antenna's gridding, staging and folding between
// two barriers; vector ALU 32 %, LDS 41 % of the cycles).  132 channels of 256
// dual-pol antennas: 235 us, the wide block's 461 (the direct kernels take 1173 at
// T = 1000 and 1752 at T = 1250).  On the way, at 128 channels: whole rows per
// wave instead of bands 260 against 244 us (wide 587 and 515); gridding at a raised
// priority 240 (469), as LDS and vector ALU are then wanted by different waves;
// antennas' table read by counted pointers, one step ahead, 224 (436); four
// steps' reads in flight instead of two 250, longest slots' waves relieved of
// staging and of the fold's busiest rows 244.  512 threads with four rows of d
// each spill (106 registers).
template <int P, bool WIDE, int KIND>
__global__ __launch_bounds__(1024) void cov_fold_kernel(CovFoldArgs a) {
  using S = CovFold<P, WIDE, KIND>;
  __shared__ __align__(16) double2 lds[2 * (S::NV * S::ES + S::MSIZE)];
  const int w = wg_range_index(blockIdx.x, a.W, 1);
  int64_t u = w * a.units / a.W;
  const int64_t u1 = (w + 1) * a.units / a.W;
  while (u < u1) {
    const int cg = (int)(u / a.n_ant), b0 = (int)(u % a.n_ant);
    const int b1 = (int)(b0 + (u1 - u) < a.n_ant ? b0 + (u1 - u) : a.n_ant);
    double2* r = a.r + (int64_t)(w + cg) * S::ROWS * S::N;
    if constexpr (P == 1) {
      cov_fold_body<P, 0, WIDE, KIND>(a, lds, r, cg, b0, b1);
    } else if constexpr (!WIDE) {
      cov_fold_body<P, 0, WIDE, KIND>(a, lds, r, cg, b0, b1);
      cov_fold_body<P, 1, WIDE, KIND>(a, lds, r + S::SROWS * S::N, cg, b0, b1);
    } else if (cg % 2 == 0) {
      cov_fold_body<P, 0, WIDE, KIND>(a, lds, r, cg / 2, b0, b1);
      cov_fold_body<P, 2, WIDE, KIND>(a, lds, r + S::SROWS * S::N, cg / 2, b0, b1);
    } else {
      cov_fold_body<P, 1, WIDE, KIND>(a, lds, r, cg / 2, b0, b1);
      cov_fold_body<P, 3, WIDE, KIND>(a, lds, r + S::SROWS * S::N, cg / 2, b0, b1);
    }
    u += b1 - b0;
  }
}

// 8-point transform, positive exponent, float64.
__device__ __forceinline__ void dft8_f64(double2 (&x)[8]) {
  constexpr double h = 0.70710678118654752440;
  auto bf = [](double2& p, double2& q) {
    const double2 t = p;
    p = make_double2(t.x + q.x, t.y + q.y);
    q = make_double2(t.x - q.x, t.y - q.y);
  };
  auto mul_i = [](double2& p) { p = make_double2(-p.y, p.x); };
  bf(x[0], x[4]); bf(x[1], x[5]); bf(x[2], x[6]); bf(x[3], x[7]);
  x[5] = make_double2(h * (x[5].x - x[5].y), h * (x[5].x + x[5].y));       // w8
  mul_i(x[6]);                                                              // w8^2
  x[7] = make_double2(h * (-x[7].x - x[7].y), h * (x[7].x - x[7].y));      // w8^3
  bf(x[0], x[2]); bf(x[1], x[3]); bf(x[4], x[6]); bf(x[5], x[7]);
  mul_i(x[3]);
  mul_i(x[7]);
  bf(x[0], x[1]); bf(x[2], x[3]); bf(x[4], x[5]); bf(x[6], x[7]);
  // bit-reversed order back to natural
  double2 t = x[1]; x[1] = x[4]; x[4] = t;
  t = x[3]; x[3] = x[6]; x[6] = t;
}

// In-place transforms of the 64 lines of a 64 x 64 plane in LDS: line l at
// p[l * ls], its points ps apart; 512 threads, eight per line (8 x 8).
__device__ __forceinline__ void lines64_f64(double2* p, int ls, int ps, const double2* w64, int tid) {
  double2* x = p + (tid >> 3) * ls;
  const int m = tid & 7;
  double2 v[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) v[n] = x[(m + 8 * n) * ps];
  dft8_f64(v);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const double2 w = w64[m * k];
    x[(m + 8 * k) * ps] = make_double2(v[k].x * w.x - v[k].y * w.y, v[k].x * w.y + v[k].y * w.x);
  }
  __syncthreads();
#pragma unroll
  for (int n = 0; n < 8; ++n) v[n] = x[(n + 8 * m) * ps];
  dft8_f64(v);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 8; ++k) x[(m + 8 * k) * ps] = v[k];
  __syncthreads();
}

struct CovImageArgs {
  const double2* r;         // cov_fold_kernel's output
  const int2* v;            // cov_corr_kernel's output, the splits added
  const float2* gains;      // [C][P][A]
  const CovAnt* ants;       // [C][A]
  double2* image;           // [C][4 or 1][64][64]
  int n_ant, ap;
  int c0, n_split, reset, transposed;
  int W;                    // the fold's workgroups and units
  int64_t units;
  int wide;                 // layout of r: CovFold<P, wide, ..>
  int autos;                // 1: leave the a = b terms out
};

// One workgroup per product (XX, XY, YY) of a channel: the ranges' slots summed in
// order, the a = b terms added, the plane transformed in float64 and the image
// written (fftshifted).  XX and YY stay apart (as the parts of one complex
// plane, the rounding of the one would show in the other).  The a = b terms,
// sum_a g_P conj(g_Q) V_aa (w_a autocorrelated), at R's 25 innermost offsets, are
// added here, so that leaving them out costs nothing.  Bound: latency (one pass
// over the slots).
template <int P>
__global__ __launch_bounds__(512) void cov_image_kernel(CovImageArgs a) {
  constexpr int N = 64, LS = N + 1, NPL = P == 2 ? 3 : 1;
  __shared__ double2 pl[N * LS];
  __shared__ double2 w64[N];
  __shared__ double2 asum[8][9];
  const int tid = threadIdx.x;
  const int cl = blockIdx.x / NPL, plane = blockIdx.x % NPL;   // XX, XY, YY
  if (tid < N) {
    double s, co;
    sincospi(tid / 32.0, &s, &co);
    w64[tid] = make_double2(co, s);
  }
  const int groups = a.wide ? CovFold<P, true, kCovPlain>::GROUPS : CovFold<P, false, kCovPlain>::GROUPS;
  const int rows = a.wide ? CovFold<P, true, kCovPlain>::ROWS : CovFold<P, false, kCovPlain>::ROWS;   // of a slot
  // NB sums over the slots of the channel's group g at once, so that their loads
  // are in flight together
  auto sums = [&](auto count, int g, auto at, auto* out) {
    constexpr int NB = decltype(count)::value;
    const int cg = cl * groups + g;
    const int w0 = cov_owner((int64_t)cg * a.n_ant, a.units, a.W);
    const int w1 = cov_owner((int64_t)(cg + 1) * a.n_ant - 1, a.units, a.W);
    const double2* r = a.r + (int64_t)(w0 + cg) * rows * N;
    int off[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      off[j] = at(j);
      out[j] = make_double2(0.0, 0.0);
    }
    for (int k = w0; k <= w1; ++k, r += rows * N) {
      double2 v[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) v[j] = r[off[j]];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        out[j].x += v[j].x;
        out[j].y += v[j].y;
      }
    }
  };
  if (!a.autos) {
    double2 t[9];                      // at the 3 x 3 offsets |dy|, |dx|
#pragma unroll
    for (int i = 0; i < 9; ++i) t[i] = make_double2(0.0, 0.0);
    const int c = a.c0 + cl;
    for (int i = tid; i < a.n_ant; i += 512) {
      const CovAnt w = a.ants[(int64_t)c * a.n_ant + i];
      const int64_t pp = (int64_t)a.ap * a.ap, o = (int64_t)cov_slot(w.ant) * (a.ap + 1);
      const int2* v = a.v + (int64_t)cl * a.n_split * CovShape<P>::NPROD * pp + o;
      const int2 v0 = v[(plane == 1 ? 2 : plane == 2 ? 1 : 0) * pp];
      const float2* g = a.gains + (int64_t)c * P * a.n_ant + w.ant;
      const float2 gp = g[plane == 2 ? a.n_ant : 0], gq = g[plane >= 1 ? a.n_ant : 0];
      const double gr = (double)gp.x * gq.x + (double)gp.y * gq.y, gi = (double)gp.y * gq.x - (double)gp.x * gq.y;
      const double2 h = make_double2(gr * v0.x - gi * v0.y, gr * v0.y + gi * v0.x);
      double ry[3], rx[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        ry[d] = rx[d] = 0.0;
#pragma unroll
        for (int j = 0; j + d < 3; ++j) {
          ry[d] += w.wr[j] * w.wr[j + d];
          rx[d] += w.wc[j] * w.wc[j + d];
        }
      }
#pragma unroll
      for (int d = 0; d < 9; ++d) {
        const double q = ry[d / 3] * rx[d % 3];
        t[d].x += q * h.x;
        t[d].y += q * h.y;
      }
    }
#pragma unroll
    for (int d = 0; d < 9; ++d) {
#pragma unroll
      for (int m = 32; m > 0; m >>= 1) {
        t[d].x += __shfl_xor(t[d].x, m);
        t[d].y += __shfl_xor(t[d].y, m);
      }
      if ((tid & 63) == 0) asum[tid >> 6][d] = t[d];
    }
  }
  if (plane == 1) {
    double2 x[8];
    if (a.wide) {                      // a half in either group
      sums(std::integral_constant<int, 4>{}, 0, [&](int j) { return 32 * N + tid + 512 * j; }, x);
      sums(std::integral_constant<int, 4>{}, 1, [&](int j) { return 32 * N + tid + 512 * j; }, x + 4);
    } else {
      sums(std::integral_constant<int, 8>{}, 0, [&](int j) { return 64 * N + tid + 512 * j; }, x);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = tid + 512 * j;
      pl[(i >> 6) * LS + (i & 63)] = x[j];
    }
  } else {
    // the upper half plane of XX or YY (held for -d: YY(-d) = conj YY(d)); at
    // P = 1, half the grid, two parts of XX
    const int g = plane == 2 && a.wide ? 1 : 0, row0 = plane == 2 && !a.wide ? 32 : 0;
    const double sign = plane == 2 ? -1.0 : 1.0;
    constexpr int H = P == 1 ? 8 : 4;
    const bool two = P == 1 && !a.wide;
    double2 x[H];
    sums(std::integral_constant<int, H>{}, g,
         [&](int j) {
           const int i = tid + 512 * (j & 3), dy = i >> 6, dx = i & 63;
           return (row0 + (two ? (j >> 2) * 32 : 0) + dy) * N + (plane == 2 ? (N - dx) & (N - 1) : dx);
         },
         x);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = tid + 512 * j, dy = i >> 6, dx = i & 63, mx = (N - dx) & (N - 1);
      if (two) x[j] = make_double2(x[j].x + x[H - 4 + j].x, x[j].y + x[H - 4 + j].y);
      if (dy) {
        pl[dy * LS + dx] = make_double2(x[j].x, sign * x[j].y);
        pl[(N - dy) * LS + mx] = make_double2(x[j].x, -sign * x[j].y);
      }
    }
    if (tid < N) {
      // rows 0 and 32: S(d) = R_0(d) + i R_32(d), each Hermitian in d
      const int dx = tid, mx = (N - dx) & (N - 1);
      double2 s[4];
      sums(std::integral_constant<int, 4>{}, g,
           [&](int j) { return (row0 + (two && j >= 2 ? 32 : 0)) * N + (j & 1 ? mx : dx); }, s);
      double2 p = s[0], m = s[1];
      if (two) {
        p = make_double2(p.x + s[2].x, p.y + s[2].y);
        m = make_double2(m.x + s[3].x, m.y + s[3].y);
      }
      pl[dx] = make_double2(0.5 * (p.x + m.x), 0.5 * (p.y - m.y));
      pl[32 * LS + dx] = make_double2(0.5 * (p.y + m.y), 0.5 * (m.x - p.x));
    }
  }
  if (!a.autos) {
    __syncthreads();
    if (tid < 25) {
      const int dy = tid / 5 - 2, dx = tid % 5 - 2, d = 3 * (dy < 0 ? -dy : dy) + (dx < 0 ? -dx : dx);
      double2* q = &pl[(dy & (N - 1)) * LS + (dx & (N - 1))];
      for (int w = 0; w < 8; ++w) {
        q->x += asum[w][d].x;
        q->y += asum[w][d].y;
      }
    }
  }
  __syncthreads();
  lines64_f64(pl, LS, 1, w64, tid);
  lines64_f64(pl, 1, LS, w64, tid);
  const int64_t npix = N * N;
  double2* img = a.image + (int64_t)(a.c0 + cl) * (P == 2 ? 4 : 1) * npix;
  for (int i = tid; i < N * N; i += 512) {
    const int qr = i >> 6, qc = i & 63;                       // pixel row, column
    const int kr = (qr + N / 2) & (N - 1), kc = (qc + N / 2) & (N - 1);
    const double2 z = a.transposed ? pl[kc * LS + kr] : pl[kr * LS + kc];
    auto put = [&](int prod, double2 v) {
      double2* o = img + prod * npix + i;
      if (!a.reset) {
        const double2 p = *o;
        v = make_double2(v.x + p.x, v.y + p.y);
      }
      *o = v;
    };
    if (plane == 1) {
      put(1, z);
      put(2, make_double2(z.x, -z.y));
    } else {
      // a sum of squares less its rounding: never below zero (NaN stays NaN)
      put(plane == 2 ? 3 : 0, make_double2(a.autos || !(z.x <= 0.0) ? z.x : 0.0, 0.0));
    }
  }
}

}  // namespace epic
