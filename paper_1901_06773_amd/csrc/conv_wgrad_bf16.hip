// Weight gradient of a convolution with bf16 storage on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16):
//
//   dw[co][j] = sum_m dy[m][co] * X[m][j],   m = (img,p,q),  j = (r,t,ci), ci fastest,
//   X[m][j] = x[img, p*stride+r-pad, q*stride+t-pad, ci]  (zero in the padding)
//
// The instruction wants consecutive values of the reduction index m per lane, and memory is contiguous along channels.  Rows of
// m go from global memory straight into LDS as they lie (buffer_load ... lds, 16 bytes per lane), and the transposition is the
// LDS read's: ds_read_b64_tr_b16 hands every lane of a group of sixteen the four rows of one of sixteen channels.
//
// What bounds it.  A wave of 64 x 64 asks for twice the LDS bytes per product that its matrix instructions can wait for, so the large tiles are 128 x 64 a
// wave; a compute unit runs eight such waves, and as the parts of a gradient (and the scratch memory that holds them) are limited,
// they share one 256 x 128 tile, two groups of four waves that multiply every second 32 positions and add their sums at the end.  256->256 3x3 at
// 14x14, 512 images, takes 121 us with the sum of the parts (980 TFLOP/s), 96 (1230) where only the first chunks are loaded and then
// multiplied again and again: the matrix cores with the transposing reads, the epilogue and the sum (matrix instructions alone, in a loop on such
// data, hold 1650 to 1840).  Address arithmetic and loads stand among the matrix instructions (behind a barrier, before them: 148 us for 130).
// Against 128 x 128 tiles of 64 x 64 a wave, transposed in registers on their way into LDS (us, with the sum of the parts):
// 256->256 3x3 at 14x14, 512 images 192 -> 131; 512->512 3x3 at 7x7, 512 images 202 -> 133; 64->64 3x3 at 56x56, 128 images 106 -> 54;
// 512->128 1x1 at 28x28, 256 images 64 -> 60 (56 at the copy rate); 512->512 3x3 at 7x7, 16 images 26.4 -> 12.3.
#include <cmath>

#include "kernels.h"
#include "dtype.h"
#include "lds_load.h"
#include "side_wide.h"

namespace acc {
namespace {

typedef short v4s __attribute__((ext_vector_type(4)));

// A workgroup of KS groups of WM x WN waves owns a tile of 32*MB*WM output channels and 32*NB*WN columns of dw, a wave MB x NB
// blocks of 32 x 32; of every chunk of CK = BK*KS positions each group multiplies its BK.  NS LDS stages.
template <int WM_, int WN_, int KS_, int MB_, int NB_, int BK_, int NS_, int WPE_> struct WCfg {
  static constexpr int WM = WM_, WN = WN_, KS = KS_, MB = MB_, NB = NB_, BK = BK_, NS = NS_, WPE = WPE_;
  static constexpr int THREADS = 64 * WM * WN * KS, CK = BK * KS;
  static constexpr int BM = 32 * MB * WM, BN = 32 * NB * WN;
  static constexpr int PA = BM * 2, PB = BN * 2;                     // bytes of a staged row
  static constexpr int CA = BM / 8, CB = BN / 8;                     // 16-byte columns of a staged row
  static constexpr int RA = THREADS / CA, RB = THREADS / CB;         // rows that one load instruction of the workgroup fills
  static constexpr int AI = CK / RA, BI = CK / RB;
  static constexpr int A_BYTES = CK * PA, STAGE = CK * (PA + PB);
  static constexpr int MAIN = NS * STAGE;
  static constexpr int OUT = KS == 2 ? THREADS * MB * NB * 16 * 4 / 2 : THREADS * MB * NB * 16 * 4;
  static constexpr int LDS0 = MAIN > OUT ? MAIN : OUT, LDS = LDS0 > wide_scratch<bf16_t>(THREADS) ? LDS0 : wide_scratch<bf16_t>(THREADS);
  static_assert(AI > 0 && BI > 0 && AI * RA == CK && BI * RB == CK && RA % 4 == 0 && RB % 4 == 0, "whole rows, four at a time");
  static_assert(BK % 32 == 0, "an even number of steps of 16 positions");
  static_assert(KS >= 2 && NS >= 2, "the epilogue adds the groups' sums");
};

// PLAIN: 1x1 filters without stride or padding, row m is pixel m; else a thread follows the pixels of its rows.
struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

template <class C, bool PLAIN>
__global__ __launch_bounds__(C::THREADS, C::WPE) void wgrad_bf16_kernel(WgradGeom g, int Mrows, int J, int tiles_j, int tiles, int splits,
                                                                        int chunks_per_split, float* out, size_t split_stride, int main_grid) {
  __shared__ __attribute__((aligned(1024))) char lds[C::LDS];
  if ((int)blockIdx.x >= main_grid) {
    wide_side_jobs<bf16_t, C::THREADS>(g.side, FlipJob{g.flip_w, g.flip_wt, g.cout, g.cin, g.r, g.s}, (int)blockIdx.x - main_grid, lds);
    return;
  }
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int MB = C::MB, NB = C::NB, AI = C::AI, BI = C::BI, NS = C::NS, KS = C::KS;
  // every XCD takes a contiguous range of (part, tile): the tiles of a part find its rows in that XCD's L2
  const int per_xcd = main_grid >> 3;
  const int work = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (work >= tiles * splits) return;
  const int split = work / tiles, tile = work - split * tiles;
  const int tile_co = tile / tiles_j, tile_j = tile - tile_co * tiles_j;
  const int co0 = tile_co * C::BM, j0 = tile_j * C::BN;
  const int chunk_lo = split * chunks_per_split;
  const int n_chunks_all = (Mrows + C::CK - 1) / C::CK;
  const int mine = min(chunk_lo + chunks_per_split, n_chunks_all) - chunk_lo;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / (C::WM * C::WN), gw = wave - grp * (C::WM * C::WN);
  const int wm0 = (gw / C::WN) * 32 * MB, wn0 = (gw % C::WN) * 32 * NB;

  v16f acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  // ---- loads: the thread's 16-byte column of both operands and its rows a multiple of four apart (the permutation is the same)
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;           // beyond any descriptor range: reads as zero
  const int arow = tid / C::CA, acol = (tid % C::CA) ^ (row_xor<C::PA>(arow) << 2);
  const int brow = tid / C::CB, bcol = (tid % C::CB) ^ (row_xor<C::PB>(brow) << 2);
  const int jt = j0 + bcol * 8;                       // first of the thread's eight columns of dw
  const bool b_col_ok = jt < J;
  const int tap = (b_col_ok ? jt : 0) / g.cin, ci0 = (b_col_ok ? jt : 0) - tap * g.cin;
  const int kr = tap / g.s, kt = tap - kr * g.s;
  // (rows beyond the part read as zero: so do the loads that run ahead of its end)
  const int m_end = min((chunk_lo + mine) * C::CK, Mrows);
  const int a_lim = co0 + acol * 8 < g.cout ? m_end : 0, b_lim = b_col_ok ? m_end : 0;
  const uint32_t a_row = (uint32_t)g.cout * 2u, b_row = (uint32_t)g.cin * 2u;
  int a_m = chunk_lo * C::CK + arow, b_m = chunk_lo * C::CK + brow;
  uint32_t a_off = (uint32_t)a_m * a_row + (uint32_t)(co0 + acol * 8) * 2u;
  // pixel (by, bx) of the input that the thread's tap meets for each of its rows, and its byte offset; from chunk to chunk a row moves on by CK
  // positions = whole images, rows and columns of the output map, with one wrap of each at most
  const int gy = kr - g.pad, gx = kt - g.pad, pq = g.p * g.q;
  const int x_lim = g.q * g.stride + gx, y_lim = g.p * g.stride + gy, x_span = g.q * g.stride, y_span = g.p * g.stride;
  const int step_img = C::CK / pq, step_p = (C::CK - step_img * pq) / g.q, step_q = C::CK - step_img * pq - step_p * g.q;
  const int step_x = step_q * g.stride, step_y = step_p * g.stride;
  const uint32_t step_off = (uint32_t)(step_img * g.h * g.wd + step_y * g.wd + step_x) * b_row;
  const uint32_t wrap_x = (uint32_t)(g.stride * g.wd - x_span) * b_row, wrap_y = (uint32_t)((g.h - y_span) * g.wd) * b_row;
  uint32_t b_off[PLAIN ? 1 : BI];
  int by[PLAIN ? 1 : BI], bx[PLAIN ? 1 : BI];
  if constexpr (PLAIN) {
    b_off[0] = (uint32_t)b_m * b_row + (uint32_t)ci0 * 2u;
  } else {
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      const int m = b_m + C::RB * i, img = m / pq, rem = m - img * pq, p = rem / g.q;
      by[i] = p * g.stride + gy;
      bx[i] = (rem - p * g.q) * g.stride + gx;
      b_off[i] = (uint32_t)((img * g.h + by[i]) * g.wd + bx[i]) * b_row + (uint32_t)ci0 * 2u;
    }
  }
  const srsrc rs_a = descriptor(g.dy, (size_t)Mrows * g.cout * 2), rs_b = descriptor(g.x, (size_t)g.n_img * g.h * g.wd * g.cin * 2);
  const uint32_t lds0 = (uint32_t)(size_t)lds, lds_w = lds0 + wave * 1024;
  // load u of a chunk (first those of dy), which goes to the stage at `at`
  auto load = [&](int u, uint32_t at) {
    if (u < AI) {
      load_lds16(rs_a, a_m + C::RA * u < a_lim ? a_off + (uint32_t)(C::RA * u) * a_row : OUTSIDE, at + u * (C::THREADS * 16));
      if (u == AI - 1) {
        a_m += C::CK;
        a_off += (uint32_t)C::CK * a_row;
      }
      return;
    }
    const int i = u - AI;
    uint32_t voff;
    if constexpr (PLAIN) {
      voff = b_m + C::RB * i < b_lim ? b_off[0] + (uint32_t)(C::RB * i) * b_row : OUTSIDE;
      if (i == BI - 1) b_off[0] += (uint32_t)C::CK * b_row;
    } else {
      const bool in = ((unsigned)by[i] < (unsigned)g.h) & ((unsigned)bx[i] < (unsigned)g.wd) & (b_m + C::RB * i < b_lim);
      voff = in ? b_off[i] : OUTSIDE;
      bx[i] += step_x;
      const bool wx = bx[i] >= x_lim;
      bx[i] -= wx ? x_span : 0;
      by[i] += step_y + (wx ? g.stride : 0);
      const bool wy = by[i] >= y_lim;
      by[i] -= wy ? y_span : 0;
      b_off[i] += step_off + (wx ? wrap_x : 0u) + (wy ? wrap_y : 0u);
    }
    load_lds16(rs_b, voff, at + C::A_BYTES + i * (C::THREADS * 16));
    if (i == BI - 1) b_m += C::CK;
  };
  // ---- fragments.  Lane t of sixteen names four channels of row t/4 and receives rows 0..3 of channel t; a fragment wants
  // channel lane%32 and positions 8*(lane/32) .. +7: two such reads.
  const int t16 = lane & 15, frow = grp * C::BK + 8 * (lane >> 5) + (t16 >> 2), fcol = 32 * ((lane >> 4) & 1) + 8 * (t16 & 3);
  uint32_t a_at[MB], b_at[NB];
#pragma unroll
  for (int i = 0; i < MB; ++i) a_at[i] = frow * C::PA + (((wm0 / 32 + i) ^ row_xor<C::PA>(frow)) << 6) + fcol;
#pragma unroll
  for (int j = 0; j < NB; ++j) b_at[j] = C::A_BYTES + frow * C::PB + (((wn0 / 32 + j) ^ row_xor<C::PB>(frow)) << 6) + fcol;
  typedef __attribute__((address_space(3))) v4s* tr_ptr;
  auto* const lds3 = (__attribute__((address_space(3))) char*)lds;
  auto read_tr = [&](uint32_t at, int pitch4) {
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    const v2u lo = __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(lds3 + at)));
    const v2u hi = __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(lds3 + at + pitch4)));
    return v4u{lo.x, lo.y, hi.x, hi.y};
  };
  constexpr int NG = C::BK / 16;
  struct Frags { v4u a[MB], b[NB]; } F[2];
  auto rd = [&](Frags& f, uint32_t st, int g16) {
#pragma unroll
    for (int i = 0; i < MB; ++i) f.a[i] = read_tr(a_at[i] + st + g16 * 16 * C::PA, 4 * C::PA);
#pragma unroll
    for (int j = 0; j < NB; ++j) f.b[j] = read_tr(b_at[j] + st + g16 * 16 * C::PB, 4 * C::PB);
  };
  constexpr int L = AI + BI, MF = MB * NB, RD = 2 * (MB + NB);
  // MFMAs of one step; with LOADS the next chunk's loads and the arithmetic of their addresses among them
  auto mm = [&](const Frags& f, uint32_t at, auto loads) {
#pragma unroll
    for (int u = 0; u < MF; ++u) {
      acc[u / NB][u % NB] = mfma_bf16(f.a[u / NB], f.b[u % NB], acc[u / NB][u % NB]);
      if constexpr (decltype(loads)::value) {
#pragma unroll
        for (int l = u * L / MF; l < (u + 1) * L / MF; ++l) load(l, at);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // One chunk = BK/16 steps.  The reads of step s+1 are issued among the MFMAs of step s, and the last step's MFMAs are held back until
  // the next chunk's barrier has been passed and its first reads are on their way; a later chunk's loads are issued among them.
  auto chunk = [&](int stage, int to, auto first) {
    const uint32_t st = stage * C::STAGE, at = lds_w + to * C::STAGE;
    __builtin_amdgcn_sched_barrier(0);
    rd(F[0], st, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(first)::value) {
#pragma unroll
      for (int l = 0; l < L; ++l) load(l, at);
    } else {
      mm(F[1], at, Yes());
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s + 1 < NG; ++s) {
      rd(F[(s + 1) & 1], st, s + 1);
      mm(F[s & 1], 0, No());
#pragma unroll
      for (int u = 0; u < MF; ++u) {
        __builtin_amdgcn_sched_group_barrier(0x100, (RD + MF - 1) / MF, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    static_assert(NG % 2 == 0, "the held-back step is F[1]");
  };
  // What opens a chunk: this wave's loads of it have landed (those of the NS - 2 later ones may be on their way), then a barrier:
  // everybody's have, and everybody is done with the chunk before, whose stage the next loads overwrite.
  auto open = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    wait_loads<(NS - 2) * L>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
#pragma unroll
    for (int l = 0; l < L; ++l) load(l, lds_w + s * C::STAGE);
  open();
  chunk(0, NS - 1, Yes());
  int stage = 1, to = 0;
  for (int j = 1; j < mine; ++j) {
    open();
    chunk(stage, to, No());
    stage = stage + 1 == NS ? 0 : stage + 1;
    to = to + 1 == NS ? 0 : to + 1;
  }
  mm(F[1], 0, No());

  // ---- epilogue: register v of a lane holds output channel 8*(v/4) + 4*(lane/32) + v%4, column lane%32 of its block
  float* dst = out + (size_t)split * split_stride;
  auto store = [&](const v16f& c, int i, int j) {
    const int jcol = j0 + wn0 + 32 * j + (lane & 31);
    if (jcol >= J) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int co = co0 + wm0 + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      if (co < g.cout) dst[(size_t)co * J + jcol] = c[v];
    }
  };
  wait_loads<0>();                                   // (the loads that ran ahead write LDS too)
  __builtin_amdgcn_s_barrier();                      // every wave is done reading the last chunk
  asm volatile("" ::: "memory");
  typedef float v4f __attribute__((ext_vector_type(4)));
  v4f* red = reinterpret_cast<v4f*>(lds);            // [wave][block][register / 4][lane]
  auto put = [&](const v16f& c, int slot) {
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) red[(slot * 4 + q4) * 64 + lane] = v4f{c[4 * q4], c[4 * q4 + 1], c[4 * q4 + 2], c[4 * q4 + 3]};
  };
  auto add = [&](v16f& c, int slot) {
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const v4f o = red[(slot * 4 + q4) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) c[4 * q4 + e] += o[e];
    }
  };
  if constexpr (KS == 2) {                           // either group finishes half of the blocks
    constexpr int HB = MB / 2 * NB;
    const int mine_at = wave * HB, other_at = (wave ^ (C::WM * C::WN)) * HB;
    static_assert(MB % 2 == 0, "halves");
    if (grp == 0) {
#pragma unroll
      for (int i = 0; i < MB / 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) put(acc[MB / 2 + i][j], mine_at + i * NB + j);
    } else {
#pragma unroll
      for (int i = 0; i < MB / 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) put(acc[i][j], mine_at + i * NB + j);
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int i = 0; i < MB / 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          add(acc[i][j], other_at + i * NB + j);
          store(acc[i][j], i, j);
        }
    } else {
#pragma unroll
      for (int i = 0; i < MB / 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          add(acc[MB / 2 + i][j], other_at + i * NB + j);
          store(acc[MB / 2 + i][j], MB / 2 + i, j);
        }
    }
  } else {                                           // block b is finished by group b % KS, the groups' sums in pairs
    constexpr int W = C::WM * C::WN, BL = MB * NB;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) put(acc[i][j], wave * BL + i * NB + j);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int b = i * NB + j;
        if (b % KS != grp) continue;
        v16f part[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) {
#pragma unroll
          for (int v = 0; v < 16; ++v) part[k][v] = 0.f;
          add(part[k], (k * W + gw) * BL + b);
        }
#pragma unroll
        for (int d = KS / 2; d > 0; d /= 2)
#pragma unroll
          for (int k = 0; k < d; ++k) part[k] += part[k + d];
        store(part[0], i, j);
      }
  }
#else
  (void)Yes::value; (void)No::value;
#endif
}

typedef WCfg<2, 2, 2, 4, 2, 32, 3, 2> W256x128;        // 48 KB a stage, one workgroup of 512 threads per compute unit
typedef WCfg<2, 2, 2, 2, 4, 32, 3, 2> W128x256;
typedef WCfg<1, 1, 4, 2, 2, 32, 2, 2> W64x64;          // 32 KB a stage, two workgroups of 256 threads
typedef WCfg<1, 2, 2, 2, 2, 32, 3, 2> W64x128;         // 24 KB a stage, two of 256
typedef WCfg<2, 1, 2, 2, 2, 32, 3, 2> W128x64;

// Which tiling: the one with the smallest predicted time, in microseconds.  With the parts below, steps = chunks of a part and the workgroups of
// the busiest compute unit, per_cu of them at a time,
//   base + (compute^2 + memory^2)^(1/2) + per_mb_result * MB of all parts + (several parts: sum_base + sum_mb * MB written and read again),
//   compute = taps (filters larger than 1x1) + the sum over rounds of max(first + first_step * steps, r * (next + next_step * steps)),
//   memory = per_mb * MB of both operands, each once.
// Fitted to 239 shapes (the layers of the ResNets at minibatches 1 to 512 and random ones with widths in 8s, every tiling on each, replayed
// from a graph, six sets of tensors in turn): median errors of 5 to 7 %, the choice is within 1.8 % of the best on average, 19 % at most.  Against
// the one 128 x 128 tiling with its transposition in registers that was here before, none of them is slower, by 1.36 on average
// (1.02 to 2.2).  Without 256 x 128 the choice of the best would be slower by up to 4 %, without 128 x 256 10, 64 x 64 72, 64 x 128 19,
// 128 x 64 10; 128 x 128, 64 x 256 and 256 x 256, which the parts leave half of the chip, are worth 1 to 3 % of single shapes and aren't here.
struct Kind {
  const char *gathered, *plain;                        // what a probe is told: filters of any kind, 1x1 without stride or padding
  int bm, bn, ck, threads, per_cu;
  double base, first, first_step, next, next_step, taps, per_mb, sum_base, sum_mb, per_mb_result;
};
enum { K256x128 = 0, K128x256, K64x64, K64x128, K128x64, KINDS };
#define ACC_WN(N) "wgrad_bf16 " N, "wgrad_bf16 " N " plain"
#define ACC_WK(C) C::BM, C::BN, C::CK, C::THREADS
constexpr Kind kKinds[KINDS] = {
    {ACC_WN("256x128"), ACC_WK(W256x128), 1, 0.000, 4.685, 0.753, 0.600, 0.600, 1.314, 0.118, 2.606, 0.114, 0.165},
    {ACC_WN("128x256"), ACC_WK(W128x256), 1, 0.000, 5.140, 0.564, 0.000, 0.891, 1.829, 0.129, 2.807, 0.124, 0.161},
    {ACC_WN("64x64"), ACC_WK(W64x64), 2, 2.207, 0.080, 0.850, 1.053, 0.286, 0.881, 0.172, 1.680, 0.212, 0.247},
    {ACC_WN("64x128"), ACC_WK(W64x128), 2, 2.249, 0.000, 0.557, 0.581, 0.234, 1.185, 0.150, 1.886, 0.181, 0.240},
    {ACC_WN("128x64"), ACC_WK(W128x64), 2, 3.234, 0.065, 0.269, 0.070, 0.264, 0.768, 0.150, 2.219, 0.178, 0.178},
};
#undef ACC_WK
#undef ACC_WN

inline bool plain_filter(const WgradGeom& g) { return g.r == 1 && g.s == 1 && g.stride == 1 && g.pad == 0; }

WgradBf16Cfg cut(const Kind& k, long Mrows, int cout, long J, int max_splits) {
  WgradBf16Cfg c{};
  c.tiles_co = (int)((cout + k.bm - 1) / k.bm);
  c.tiles_j = (int)((J + k.bn - 1) / k.bn);
  const long tiles = (long)c.tiles_co * c.tiles_j, chunks = (Mrows + k.ck - 1) / k.ck;
  long splits = 256L * k.per_cu / tiles;               // one round of workgroups
  if (splits > chunks) splits = chunks;
  if (splits > max_splits) splits = max_splits;
  if (splits < 1) splits = 1;
  c.chunks_per_split = (int)((chunks + splits - 1) / splits);
  c.splits = (int)((chunks + c.chunks_per_split - 1) / c.chunks_per_split);
  return c;
}

double predicted_us(const Kind& k, const WgradBf16Cfg& c, long Mrows, long pixels, int cin, int cout, int taps) {
  const long work = (long)c.tiles_co * c.tiles_j * c.splits, round = 256L * k.per_cu;
  const double first = k.first + k.first_step * c.chunks_per_split, next = k.next + k.next_step * c.chunks_per_split;
  auto busy = [&](long r) { return r == 0 ? 0.0 : first > r * next ? first : r * next; };
  const double compute = (double)(work / round) * busy(k.per_cu) + busy((work % round + 255) / 256) + (taps > 1 ? k.taps : 0.0);
  // pixels that are read: all of the input or, by filters smaller than their stride, those under a tap
  const double under = (double)Mrows * taps, read = under < (double)pixels ? under : (double)pixels;
  const double memory = k.per_mb * 2e-6 * (read * cin + (double)Mrows * cout);
  const double parts = 4e-6 * c.splits * cout * taps * cin;
  return k.base + std::sqrt(compute * compute + memory * memory) + k.per_mb_result * parts + (c.splits > 1 ? k.sum_base + k.sum_mb * 2 * parts : 0.0);
}

}  // namespace

WgradBf16Cfg wgrad_bf16_choose(long Mrows, long pixels, int cin, int cout, int r, int s, int max_splits) {
  WgradBf16Cfg best{};
  double us = 0;
  for (int v = 0; v < KINDS; ++v) {
    WgradBf16Cfg c = cut(kKinds[v], Mrows, cout, (long)r * s * cin, max_splits);
    const double t = predicted_us(kKinds[v], c, Mrows, pixels, cin, cout, r * s);
    if (v > 0 && t >= us) continue;
    c.kind = v;
    best = c;
    us = t;
  }
  return best;
}

const char* wgrad_bf16_name(const WgradGeom& g, const WgradBf16Cfg& c) { return plain_filter(g) ? kKinds[c.kind].plain : kKinds[c.kind].gathered; }

hipError_t conv_wgrad_bf16(const WgradGeom& g, const WgradBf16Cfg& c, int Mrows, int J, float* out, size_t count, hipStream_t st) {
  const long work = (long)c.tiles_co * c.tiles_j * c.splits;
  const int threads = kKinds[c.kind].threads, tiles = c.tiles_co * c.tiles_j;
  const long side = wide_side_blocks(g.side, FlipJob{g.flip_w, g.flip_wt, g.cout, g.cin, g.r, g.s}, threads);
  const long main_grid = (work + 7) / 8 * 8;
  if (main_grid + side > (1L << 30)) return hipErrorInvalidValue;
  const bool plain = plain_filter(g);
  const dim3 grid((unsigned)(main_grid + side));
#define ACC_WB(C, G) hipLaunchKernelGGL((wgrad_bf16_kernel<C, G>), grid, dim3(C::THREADS), 0, st, g, Mrows, J, c.tiles_j, tiles, \
                                        c.splits, c.chunks_per_split, out, count, (int)main_grid)
#define ACC_WB2(K, C) case K: if (plain) ACC_WB(C, true); else ACC_WB(C, false); break
  switch (c.kind) {
    ACC_WB2(K256x128, W256x128);
    ACC_WB2(K128x256, W128x256);
    ACC_WB2(K64x64, W64x64);
    ACC_WB2(K64x128, W64x128);
    ACC_WB2(K128x64, W128x64);
    default: return hipErrorInvalidValue;
  }
#undef ACC_WB2
#undef ACC_WB
  return hipGetLastError();
}

}  // namespace acc
