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
//   cov_fold_kernel   R of a share of a channel's antennas b (float32 sums, as
//                     the fused kernels' block sums);
//   cov_image_kernel  the shares summed, transformed and written in float64.
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
// T = 1000: 126 us (41 us of them, the covariances' 208 MB, whatever T is) =
// 1.1 POP/s of 8 operations per pair and sample; 8.9 vector instructions per
// matrix one, of which about 4 are free, so the two take turns (matrix pipes 25 %,
// vector ALU 31 % busy).
template <int P, bool VEC>
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
  const uint32_t loff = ant < a.n_ant ? (uint32_t)(pol * a.n_ant + ant) : 0u;
  const int nvalid = a.n_ant - ant;    // antennas of the four that exist
  const uint32_t lmask = nvalid >= 4 ? ~0u : nvalid <= 0 ? 0u : (1u << (8 * nvalid)) - 1u;
  const int n_stage = (int)((t_end - t_begin + kCovStage - 1) / kCovStage);
  auto load = [&](int k, uint32_t (&raw)[16]) {
    if (k >= n_stage) k = n_stage - 1;
    // past the end the last row again, cleared when it is staged
    const int last = n_row - 1 - (k * kCovStage + 16 * uwave);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint8_t* row = src + (k * kCovStage + 16 * uwave + (i < last ? i : last)) * tstride;
      if (VEC) {
        raw[i] = *reinterpret_cast<const uint32_t*>(row + loff);
      } else {
        raw[i] = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
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
        for (int i = 0; i < 4; ++i) in[i] = raw[4 * s + i] & (4 * s + i < rows ? lmask : 0u);
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

// Time splits of V added into the first, so that what follows reads one plane
// per product whatever the split (holding up to four in flight cost the fold and
// the gradient 11 to 29 spilled registers, reloaded behind the prefetch of V).
// Bound: HBM, one pass.  Only calls of few channels split.
__global__ static __launch_bounds__(256) void cov_sum_kernel(CovSumArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.total) return;
  const int64_t h = a.n / 2, cl = i / h;
  int4* v = reinterpret_cast<int4*>(a.v + cl * a.n_split * a.n) + i % h;
  int4 s = v[0];
  for (int k = 1; k < a.n_split; ++k) {
    const int4 x = v[k * h];
    s = make_int4(s.x + x.x, s.y + x.y, s.z + x.z, s.w + x.w);
  }
  v[0] = s;
}

// Antenna b of a channel, in the order the fold takes them (by column): its
// first tap's cell in the programs' (possibly transposed) aperture and its
// kernel as row and column factors.
struct __align__(16) CovAnt {
  int ant, row, col, pad0;
  float wr[4];              // weights of rows row .. row + 2
  float wc[4];              // weights of columns col .. col + 2
};

// Gridding program of the fold, per channel and wave: a wave grids RPW whole
// consecutive rows, its cells dealt to "slots" of 64 (one per lane) by number of
// entries, so that the lanes of a slot end together and a step is a read and
// the products, with no test per lane.  `ends` marks the steps that end a slot
// and store its cells; cells of no antenna are never written and stay zero.
// Padding reads a zero slot of E'.  Per lane: the cells' byte offsets and the
// steps' E' byte offsets, 16 bits each, and the steps' weights, all of it in
// registers for the whole share (a step read from memory in the loop would wait
// behind the prefetch of V).
constexpr int kCovSlots = 4;        // slots of a wave at most
struct CovProgHead {
  uint32_t row_lo, row_hi;          // aperture rows of the wave
  uint32_t steps, ends;
};
template <int STEPS> struct CovProgLane {
  uint32_t cell[kCovSlots / 2];
  uint32_t e[STEPS / 2];
  float w[STEPS];
};

struct CovFoldArgs {
  const int2* v;            // cov_corr_kernel's output, the splits added
  const float2* gains;      // [C][P][A]
  const CovProgHead* head;  // [C][waves]
  const void* prog;         // CovProgLane [C][waves][64]
  const CovAnt* ants;       // [C][A]
  float2* r;                // [channel - c0][chunk][CovFold rows][64]
  int n_ant, ap;
  int c0, n_split, n_chunk;
  int total;                // workgroups: channels * n_chunk
};

// Shape of the fold: NV aperture grids at a time (P = 2: the columns XX, YY and
// XY of one antenna b; P = 1: XX of two antennas), R rows and W columns each,
// lanes along the columns (LR lanes per row) and "units" of LR lanes along d's
// rows, four rows of d per group.  XX and YY need half of the plane of d
// (R(-d) = conj R(d)): rows 0 .. 31 for XX and 0 .. -31 for YY, row 32
// riding in row 0's imaginary part (both are Hermitian in d's column alone,
// which tells them apart).  Of M_b they read only the rows at or past b's first
// (XX) or up to its last (YY), so a wave grids for one b mostly one of the two.
// DENSE: more than 256 antennas, or more steps than the registers of the
// others hold.
// The wide block's grids need twice the LDS: one workgroup of 1024 threads per
// CU instead of two of 512 (16 waves either way).
template <int P, bool WIDE, bool DENSE> struct CovFold {
  static constexpr int N = 64, NT = WIDE ? 1024 : 512, NW = NT / 64;
  static constexpr int MAXA = DENSE ? 512 : 256;
  static constexpr int STEPS = DENSE && !WIDE ? 24 : 12;     // program steps of a wave at most
  static constexpr int NV = P == 2 ? 3 : 2;
  static constexpr int R = WIDE ? FusedShape<64>::HW : 32;   // rows of a grid
  static constexpr int W = WIDE ? 48 : 32;                   // columns of a grid
  static constexpr int RS = W + 1;                           // row stride; WIDE: column 48 stays zero
  static constexpr int PADR = 5;                             // zero rows around each grid
  static constexpr int VS = (R + PADR) * RS;                 // grid stride
  static constexpr int MSIZE = PADR * RS + NV * VS;
  static constexpr int LR = WIDE ? 64 : 32;
  static constexpr int UNITS = NT / LR;
  static constexpr int HG = 16 / UNITS;                      // half-plane groups per unit (XX | YY)
  static constexpr int FG = P == 2 ? 16 / UNITS : 0;         // full-plane groups per unit (XY)
  static constexpr int G = HG + FG;
  static constexpr int ROWS = P == 2 ? 128 : 64;             // rows of r: half planes, then XY
};

// Bound: LDS (gridding: about 2.25 reads of E' per cell and grid, gathered)
// and the vector ALU.  A channel costs A passes of three grids, whatever T is.
// The workgroup takes the antennas b of its share in column order.  Per b:
// E'[a] = g_a conj(g_b) V_ab is staged, gridded with the channel's program
// (held in registers for the whole share), and folded into R: a thread owns
// one aperture column and four rows of d per group, forms the row taps of M_b
// at its rows, and adds them, times the three column taps, to its sums Q_0 ..
// Q_2 of the aperture columns col .. col + 2.  When the next antenna starts at
// the next column, Q_0 moves one lane on into Q_1 (the same d), so a sum stays
// in registers until its last term and R is written once.
// 132 channels of 256 dual-pol antennas: 165 us (vector ALU 50 %, LDS 60 %; the
// direct kernel takes 1173 us at T = 1000); with the direct kernels' programs,
// whose lanes end their cells one by one, 340; with the steps past the eighth
// read from memory 418; with the antennas' table read by vector loads 338.
// The wide block: 305 us as one workgroup of 1024 threads, 349 as 512 threads and
// one grid buffer (direct: 1752 us at T = 1250).
// f(0), f(1), .. f(N - 1) with compile-time indices, until one returns false.
template <typename F, int... I>
__device__ __forceinline__ void static_while_impl(F&& f, std::integer_sequence<int, I...>) {
  (void)(f(std::integral_constant<int, I>{}) && ...);
}
template <int N, typename F> __device__ __forceinline__ void static_while(F&& f) {
  static_while_impl(f, std::make_integer_sequence<int, N>{});
}

template <int P, bool WIDE, bool DENSE>
__global__ __launch_bounds__((WIDE ? 1024 : 512), (DENSE && !WIDE ? 2 : 4)) void cov_fold_kernel(CovFoldArgs a) {
  using S = CovFold<P, WIDE, DENSE>;
  constexpr int N = S::N, NT = S::NT, MAXA = S::MAXA, kCovSteps = S::STEPS, NV = S::NV, RS = S::RS, VS = S::VS, LR = S::LR, G = S::G;
  constexpr int ESF = MAXA + 16;
  constexpr int NE = (NV * MAXA + NT - 1) / NT;
  constexpr int GB = 2;                 // steps whose reads are in flight together
  __shared__ __align__(16) float2 lds[2 * NV * ESF + 2 * S::MSIZE + P * MAXA];
  float2* const Eb = lds;
  float2* const Mb = lds + 2 * NV * ESF;
  float2* const Gl = Mb + 2 * S::MSIZE;       // the channel's gains
  const int tid = threadIdx.x, lane = tid & 63;
  const int logical = wg_range_index(blockIdx.x, a.total, 1);
  const int cl = logical / a.n_chunk, ch = logical % a.n_chunk, c = a.c0 + cl;
  const int A = a.n_ant, ap = a.ap;
  const int b0 = (int)((int64_t)ch * A / a.n_chunk), b1 = (int)((int64_t)(ch + 1) * A / a.n_chunk);
  const int n_it = P == 2 ? b1 - b0 : (b1 - b0 + 1) / 2;
  // in the constant address space: uniform indices load through the scalar
  // cache, off the vector memory counter that the prefetch of V waits on
  using ConstAnt = const __attribute__((address_space(4))) CovAnt;
  ConstAnt* ants = (ConstAnt*)(a.ants + (int64_t)c * A);

  for (int i = tid; i < 2 * NV * ESF + 2 * S::MSIZE; i += NT) lds[i] = make_float2(0.f, 0.f);
  for (int i = tid; i < P * A; i += NT) Gl[i < A ? i : MAXA + i - A] = a.gains[(int64_t)c * P * A + i];

  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const CovProgHead head = a.head[c * S::NW + wave];
  const CovProgLane<S::STEPS> prog =
      reinterpret_cast<const CovProgLane<S::STEPS>*>(a.prog)[(int64_t)(c * S::NW + wave) * 64 + lane];
  const int row_lo = head.row_lo, row_hi = head.row_hi;

  // staging: element e = tid + NT i of the NV columns of V; a wave's 64 are in
  // one column (ap is a multiple of 128), so that all but the place in the
  // column and the gain of a is uniform
  constexpr int NB = P == 2 ? 1 : NV;   // antennas b per step
  int vec[NE], sofs[NE];                // element i: its column, and its place less tid
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int e = tid + NT * i;
    vec[i] = __builtin_amdgcn_readfirstlane((e >= ap) + (e >= 2 * ap) + (e >= 3 * ap));
    sofs[i] = __builtin_amdgcn_readfirstlane(NT * i - vec[i] * ap);
    if (vec[i] >= NV) sofs[i] = 0;
  }
  // a channel's planes of one split are below 2^23 bytes: a uniform base and
  // 32-bit offsets
  const int plane = ap * ap;
  const int64_t vsplit = (int64_t)CovShape<P>::NPROD * plane * sizeof(int2);
  const char* vc = reinterpret_cast<const char*>(a.v) + cl * a.n_split * vsplit;
  // V of a step: loaded two steps before it is staged
  struct Pre {
    int2 v[NE];
    int b[NB];                          // antennas of the step (-1: none)
  };
  Pre pre0, pre1;
  int nextb[NB];                        // antennas of the next step to fetch
  auto lookup = [&](int it) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int bi = b0 + NB * it + j;
      nextb[j] = bi < b1 ? ants[bi].ant : -1;
    }
  };
  auto fetch = [&](int it, Pre& p) {
#pragma unroll
    for (int j = 0; j < NB; ++j) p.b[j] = nextb[j];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      // always loaded (past the columns or the share: some valid place, unused),
      // so that the loads in flight can be counted and each set waited for alone
      const int v = vec[i] < NV ? vec[i] : 0;
      const int b = NB == 1 ? p.b[0] : v ? p.b[NB - 1] : p.b[0];
      const uint32_t col = __builtin_amdgcn_readfirstlane((P == 2 ? v * plane : 0) + cov_slot(b < 0 ? 0 : b) * ap);
      const uint32_t off = 8u * (col + sofs[i] + (vec[i] < NV ? tid : 0));
      p.v[i] = *reinterpret_cast<const int2*>(vc + off);
    }
    lookup(it + 1);
  };
  auto stage = [&](float2* E, const Pre& p) {
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int v = vec[i];
      if (v >= NV) continue;
      const int b = NB == 1 ? p.b[0] : v ? p.b[NB - 1] : p.b[0];
      const int ant = cov_ant(tid + sofs[i]);
      if (ant >= A) continue;
      int2 val = p.v[i];
      // the a = b terms are added (or left out) by cov_image_kernel, in float64;
      // b < 0: the last step of a share at P = 1 may have one antenna only
      if (b == ant || b < 0) val = make_int2(0, 0);
      const int ga = P == 2 && v == 1 ? MAXA : 0, go = (P == 2 && v >= 1 ? MAXA : 0) + (b < 0 ? 0 : b);
      const float2 g = Gl[ga + ant], gb = Gl[go];
      const float2 h = make_float2(g.x * gb.x + g.y * gb.y, g.y * gb.x - g.x * gb.y);
      E[v * ESF + ant] = cmul(h, make_float2((float)val.x, (float)val.y));
    }
  };
  // the grids of one step: MASK bit v set: grid v is made
  auto grid_some = [&](auto mask, const float2* E, float2* M) {
    constexpr int MASK = decltype(mask)::value;
    const char* eb = reinterpret_cast<const char*>(E);
    char* mb = reinterpret_cast<char*>(M);
    float2 s[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) s[v] = make_float2(0.f, 0.f);
    // opaque copies: unpacked here and not, into twice the registers, before
    // the loop over the share
    uint32_t n = head.steps, ends = head.ends;
    asm volatile("" : "+s"(n), "+s"(ends));
    int slot = 0;
    auto steps = [&](auto first) {
      constexpr int st = decltype(first)::value * GB;
      if (st >= (int)n) return false;
      float2 e[GB][NV];                  // a step past the last: a read of E'[0], weight 0
#pragma unroll
      for (int i = 0; i < GB; ++i) {
        uint32_t ew = prog.e[(st + i) / 2];
        asm volatile("" : "+v"(ew));
        const uint32_t off = (st + i) & 1 ? ew >> 16 : ew & 0xFFFFu;
        const float2* p = reinterpret_cast<const float2*>(eb + off);
#pragma unroll
        for (int v = 0; v < NV; ++v)
          if (MASK >> v & 1) e[i][v] = p[v * ESF];
      }
#pragma unroll
      for (int i = 0; i < GB; ++i) {
        const float w = prog.w[st + i];
#pragma unroll
        for (int v = 0; v < NV; ++v)
          if (MASK >> v & 1) {
            s[v].x = fmaf(w, e[i][v].x, s[v].x);
            s[v].y = fmaf(w, e[i][v].y, s[v].y);
          }
        if (ends >> (st + i) & 1) { // uniform over the wave
          uint32_t cw = slot < 2 ? prog.cell[0] : prog.cell[1];
          asm volatile("" : "+v"(cw));
          float2* cell = reinterpret_cast<float2*>(mb + (slot & 1 ? cw >> 16 : cw & 0xFFFFu));
          ++slot;
#pragma unroll
          for (int v = 0; v < NV; ++v)
            if (MASK >> v & 1) {
              cell[v * VS] = s[v];
              s[v] = make_float2(0.f, 0.f);
            }
        }
      }
      return true;
    };
    static_while<kCovSteps / GB>(steps);
  };
  int r0 = 0, r1 = 0;                   // first rows of the antennas gridded next
  auto load_rows = [&](int it) {
    const int bi = b0 + NB * it;
    r0 = r1 = ants[bi < b1 ? bi : b0].row;
    if (NB == 2) r1 = ants[bi + 1 < b1 ? bi + 1 : b0].row;
  };
  auto grid = [&](const float2* E, float2* M) {
    if (head.steps == 0) return;
    const bool need0 = row_hi >= r0 || (WIDE && row_lo <= r0 - 30);
    const bool need1 = P == 1 ? row_hi >= r1 || (WIDE && row_lo <= r1 - 30)
                              : row_lo <= r1 + 2 || (WIDE && row_hi >= r1 + 32);
    constexpr int X = P == 2 ? 4 : 0;
    if (need0 && need1) grid_some(std::integral_constant<int, 3 | X>{}, E, M);
    else if (need0) grid_some(std::integral_constant<int, 1 | X>{}, E, M);
    else if (need1) grid_some(std::integral_constant<int, 2 | X>{}, E, M);
    else if (X) grid_some(std::integral_constant<int, 4>{}, E, M);
  };

  // fold: unit u, column ux; group k of the unit covers rows dy0 .. dy0 + 3 of
  // d of grid vec
  const int u = tid / LR, ux = tid % LR;
  const int hset = u >= S::UNITS / 2 ? 1 : 0, hu = u % (S::UNITS / 2);
  float2 q[G][3][4];
#pragma unroll
  for (int k = 0; k < G; ++k)
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int d = 0; d < 4; ++d) q[k][i][d] = make_float2(0.f, 0.f);
  const int ucol = ux < S::W ? ux : S::W;
  float2* const rout = a.r + (int64_t)logical * S::ROWS * N;
  auto dy0_of = [&](int k) { return k < S::HG ? 4 * (hu + k * (S::UNITS / 2)) : 4 * (u + (k - S::HG) * S::UNITS); };
  // grid 1's half plane runs downwards: its group covers d = -(dy0 + 3) .. -dy0
  auto dfirst_of = [&](int k) { return P == 2 && k < S::HG && hset ? -3 - dy0_of(k) : dy0_of(k); };
  auto row_of = [&](int k, int d) {
    return k < S::HG ? 32 * hset + dy0_of(k) + (P == 2 && hset ? 3 - d : d) : 64 + dy0_of(k) + d;
  };
  int x0 = 0, xfirst = -1;
  // Q_0 one lane on into Q_1; the columns move down
  auto advance = [&]() {
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const float2 t = q[k][0][d];
        float2 sh;
        if constexpr (LR == N) {         // the lanes are the whole circle of d
          sh.x = __shfl(t.x, (lane + 63) & 63);
          sh.y = __shfl(t.y, (lane + 63) & 63);
        } else {                         // the last column's d has had its last term
          sh.x = __shfl_up(t.x, 1, LR);
          sh.y = __shfl_up(t.y, 1, LR);
          if (ux == 0) sh = make_float2(0.f, 0.f);
          if (ux == LR - 1) rout[row_of(k, d) * N + ((LR - 1 - x0) & (N - 1))] = t;
        }
        q[k][0][d] = make_float2(q[k][1][d].x + sh.x, q[k][1][d].y + sh.y);
        q[k][1][d] = q[k][2][d];
        q[k][2][d] = make_float2(0.f, 0.f);
      }
    ++x0;
  };
  auto fold = [&](int it, const float2* M, const CovAnt& b) {
    if (P == 1 && __builtin_amdgcn_readfirstlane(b0 + 2 * it + hset) >= b1) return;
    if (xfirst < 0) x0 = xfirst = b.col;
    while (x0 < b.col) advance();
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const int vec = k < S::HG ? hset : 2;
      const int s = ((b.row + dfirst_of(k) + S::PADR) & (N - 1)) - S::PADR;
      if (s < S::R) {
        const float2* m = M + vec * VS + (s + S::PADR) * RS + ucol;
        float2 row[6];
#pragma unroll
        for (int r = 0; r < 6; ++r) row[r] = m[r * RS];
        float2 z[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          z[d].x = b.wr[0] * row[d].x;
          z[d].y = b.wr[0] * row[d].y;
#pragma unroll
          for (int j = 1; j < 3; ++j) {
            z[d].x = fmaf(b.wr[j], row[d + j].x, z[d].x);
            z[d].y = fmaf(b.wr[j], row[d + j].y, z[d].y);
          }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            q[k][i][d].x = fmaf(b.wc[i], z[d].x, q[k][i][d].x);
            q[k][i][d].y = fmaf(b.wc[i], z[d].y, q[k][i][d].y);
          }
      }
      if constexpr (WIDE) {
        if (k == 0 && hu == 0) {         // i times row d = 32 into row 0
          const int s2 = ((b.row + 32 + S::PADR) & (N - 1)) - S::PADR;
          if (s2 < S::R && s2 >= -2) {
            const float2* m = M + vec * VS + (s2 + S::PADR) * RS + ucol;
            float2 z = make_float2(0.f, 0.f);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
              z.x = fmaf(b.wr[j], m[j * RS].x, z.x);
              z.y = fmaf(b.wr[j], m[j * RS].y, z.y);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
              float2& q0 = P == 2 && hset ? q[0][i][3] : q[0][i][0];
              q0.x = fmaf(-b.wc[i], z.y, q0.x);
              q0.y = fmaf(b.wc[i], z.x, q0.y);
            }
          }
        }
      }
    }
  };

  CovAnt cur = {};
  auto load_ant = [&](int it) {
    const int bi = P == 2 ? b0 + it : __builtin_amdgcn_readfirstlane(b0 + 2 * it + hset);
    ConstAnt& t = ants[bi < A ? bi : A - 1];
    cur.row = t.row;
    cur.col = t.col;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      cur.wr[i] = t.wr[i];
      cur.wc[i] = t.wc[i];
    }
  };
  lookup(0);
  fetch(0, pre0);
  fetch(1, pre1);
  if (n_it > 0) {
    load_ant(0);
    load_rows(0);
  }
  __syncthreads();
  if (n_it > 0) stage(Eb, pre0);
  fetch(2, pre0);
  __syncthreads();
  // step `it`: grid it, stage it + 1 from `p`, fetch it + 3 into it
  auto step = [&](int it, Pre& p) {
    grid(Eb + (it & 1) * NV * ESF, Mb + (it & 1) * S::MSIZE);
    load_rows(it + 1);
    if (it + 1 < n_it) stage(Eb + ((it + 1) & 1) * NV * ESF, p);
    fetch(it + 3, p);
    if (it > 0) {                       // the previous antenna's grids, while this one's are made
      fold(it - 1, Mb + ((it - 1) & 1) * S::MSIZE, cur);
      load_ant(it);
    }
    __syncthreads();
  };
  for (int it = 0; it < n_it; it += 2) {
    step(it, pre1);
    if (it + 1 < n_it) step(it + 1, pre0);
  }
  if (n_it > 0) fold(n_it - 1, Mb + ((n_it - 1) & 1) * S::MSIZE, cur);

  // Q_0 and Q_1 into Q_2, then every d the share has touched; zero elsewhere
  if (xfirst < 0) xfirst = 0;
  advance();
  advance();
#pragma unroll
  for (int k = 0; k < G; ++k)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      float2* o = rout + row_of(k, d) * N;
      o[(ux - x0) & (N - 1)] = q[k][0][d];
      if (LR < N && ux < LR - (x0 - xfirst)) o[(LR - xfirst + ux) & (N - 1)] = make_float2(0.f, 0.f);
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
  const float2* r;          // [channel - c0][chunk][rows][64]
  const int2* v;            // cov_corr_kernel's output
  const float2* gains;      // [C][P][A]
  const CovAnt* ants;       // [C][A]
  double2* image;           // [C][4 or 1][64][64]
  int n_ant, ap;
  int c0, n_split, n_chunk, reset, transposed;
  int autos;                // 1: leave the a = b terms out
};

// One workgroup per product (XX, XY, YY) of a channel: the shares summed in
// share order, the a = b terms added, the plane transformed in float64 and the
// image written (fftshifted).  XX and YY stay apart (as the parts of one complex
// plane, the rounding of the one would show in the other).  The a = b terms, sum_a g_P conj(g_Q) V_aa (w_a autocorrelated),
// are by far the largest values of R, at its 25 innermost offsets: summed here
// in float64 rather than with the others in float32, they cost the image no
// accuracy (without this the error at 256 antennas, T = 1000, against 64 bits
// was three times larger).  Bound: latency (one pass over the shares).
template <int P>
__global__ __launch_bounds__(512) void cov_image_kernel(CovImageArgs a) {
  constexpr int N = 64, LS = N + 1, ROWS = CovFold<P, false, false>::ROWS, NPL = P == 2 ? 3 : 1;
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
  const float2* r = a.r + (int64_t)cl * a.n_chunk * ROWS * N;
  // NB sums over the shares at once, so that their loads are in flight together
  auto sums = [&](auto count, auto at, auto& out) {
    constexpr int NB = decltype(count)::value;
    int off[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      off[j] = at(j);
      out[j] = make_double2(0.0, 0.0);
    }
    for (int k = 0; k < a.n_chunk; ++k) {
      float2 v[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) v[j] = r[(int64_t)k * ROWS * N + off[j]];
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
          ry[d] += (double)w.wr[j] * w.wr[j + d];
          rx[d] += (double)w.wc[j] * w.wc[j + d];
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
    sums(std::integral_constant<int, 8>{}, [&](int j) { return 64 * N + tid + 512 * j; }, x);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = tid + 512 * j;
      pl[(i >> 6) * LS + (i & 63)] = x[j];
    }
  } else {
    // the upper half plane of XX or YY (held for -d: YY(-d) = conj YY(d)); at
    // P = 1 two shares of XX
    const int row0 = plane == 2 ? 32 : 0;
    const double sign = plane == 2 ? -1.0 : 1.0;
    constexpr int H = P == 1 ? 8 : 4;
    double2 x[H];
    sums(std::integral_constant<int, H>{},
         [&](int j) {
           const int i = tid + 512 * (j & 3), dy = i >> 6, dx = i & 63;
           return (row0 + (j >> 2) * 32 + dy) * N + (plane == 2 ? (N - dx) & (N - 1) : dx);
         },
         x);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = tid + 512 * j, dy = i >> 6, dx = i & 63, mx = (N - dx) & (N - 1);
      if (P == 1) x[j] = make_double2(x[j].x + x[H - 4 + j].x, x[j].y + x[H - 4 + j].y);
      if (dy) {
        pl[dy * LS + dx] = make_double2(x[j].x, sign * x[j].y);
        pl[(N - dy) * LS + mx] = make_double2(x[j].x, -sign * x[j].y);
      }
    }
    if (tid < N) {
      // rows 0 and 32: S(d) = R_0(d) + i R_32(d), each Hermitian in d
      const int dx = tid, mx = (N - dx) & (N - 1);
      double2 s[4];
      sums(std::integral_constant<int, 4>{},
           [&](int j) { return (row0 + (j >= 2 ? 32 : 0) * (P == 1)) * N + (j & 1 ? mx : dx); }, s);
      double2 p = s[0], m = s[1];
      if (P == 1) {
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
      put(plane == 2 ? 3 : 0, make_double2(z.x, 0.0));
    }
  }
}

}  // namespace epic
