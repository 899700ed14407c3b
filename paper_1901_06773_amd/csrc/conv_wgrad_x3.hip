// Weight gradient of a convolution for fp32 storage on the bf16 matrix cores (split3.h has the arithmetic):
//
//   dw[co][j] = sum_m dy[m][co] * X[m][j],   m = (img,p,q),  j = (r,t,ci), ci fastest,
//   X[m][j] = x[img, p*stride+r-pad, q*stride+t-pad, ci]  (zero in the padding)
//
// A workgroup of eight waves owns a 64*WT x 64*WT tile of dw and a range of m; each wave 64 x 64 (2 x 2
// blocks), KS = 8 / WT^2 groups of waves each take a part of the range, 16 values of m per step, and add up at
// the end.  The matrix instruction wants eight consecutive m of one channel per lane, memory is contiguous along
// channels: a thread fetches four rows of m, sixteen bytes (four channels) each, and the splitting packs pairs of
// rows, so the transposition costs nothing.  LDS planes are [64 rows][16 m] bf16 per block of 64 channels, row r
// holding channel 4 * (r % 16) + r / 16 (the four channels of a thread lie 16 rows apart, the threads of a write
// instruction on neighbouring rows: no bank conflicts); the tile comes out in that order and is put right when it is
// stored.  Pipeline as in conv_igemm_x3.hip: step j multiplied out of registers, j+1 read from LDS, j+2 split and
// stored, later loads issued.
//
// Bound: the vector instructions (104 per wave and step for the splitting, a few for the offsets, beside 24 matrix instructions; with half the matrix
// instructions left out 256->256 3x3 at 14x14, 41 images, takes 60 us instead of 68) and the parts, which are written and read
// once.  Offsets worked out 64 at a time (TABLE below) instead of by every lane for its own rows: 183 -> 109 vector instructions per step, that
// layer 67.2 -> 61.5 us, 512->512 3x3 at 7x7 83.0 -> 74.5, 128->128 3x3/2 at 55x55, 19 images 41.9 -> 39.4; 98 shapes 4 % on average.
// Measured against the fp32-instruction kernel this replaces, minibatch 41, reduction of the parts included:
// 256->256 3x3 at 14x14 115.7 -> 63.8 us, 128->128 3x3 at 28x28 96.1 -> 63.7, 512->512 3x3 at 7x7 117.8 -> 79.6, 256->1024
// 1x1 at 14x14 44.4 -> 35.5, 64->256 at 56x56 (minibatch 32) 42.9 -> 39.3; error against float64 6.2e-7 -> 3.6e-7 on the
// first of them, smaller on all.
#include "kernels.h"
#include "split3.h"
#include "side_wide.h"

namespace acc {
namespace {

template <int WT>
struct WDeep {
  static constexpr int KS = 8 / (WT * WT), GT = 64 * WT * WT;        // groups, threads of a group
  static constexpr int BLOCKS = 2 * WT, BPW = BLOCKS / (WT * WT);    // 64-channel blocks staged per step, by one wave
  static constexpr int PLANE = 64 * 32, BLOCK = 3 * PLANE, STAGE = BLOCKS * BLOCK;
  static constexpr int NST = GT == 64 ? 1 : 2;                       // a group of one wave needs no second stage: its LDS accesses keep their order
  static constexpr int MAIN = KS * NST * STAGE;
  static constexpr int NQ = KS < 4 ? KS : 4, BPQ = 4 / NQ;           // groups that finish blocks, blocks each
  static constexpr int RED = NQ * (KS - 1) * WT * WT * BPQ * 16 * 64 * 4;
  static constexpr int LDS = MAIN > RED ? MAIN : RED;
};

__device__ __forceinline__ int channel_of(int r) { return 4 * (r & 15) + (r >> 4); }   // of a block's row

// One 32 x 32 block over the positions [m_lo, m_hi) with the fp32 matrix instruction, operands straight from memory:
// for blocks whose split products are not finite (see split3.h).  co, j: the lane's row and column of dw.
__device__ __forceinline__ x3_v16f plain_wgrad_block(const WgradGeom& g, int co, int j, int J, int m_lo, int m_hi, int lane) {
  x3_v16f acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const bool co_ok = co < g.cout, j_ok = j < J;
  const int tap = (j_ok ? j : 0) / g.cin, ci = (j_ok ? j : 0) - tap * g.cin, kr = tap / g.s, kt = tap - kr * g.s;
  const float* dy = static_cast<const float*>(g.dy) + (co_ok ? co : 0);
  const float* x = static_cast<const float*>(g.x) + ci;
  const int pq = g.p * g.q;
#pragma unroll 1
  for (int mb = m_lo; mb < m_hi; mb += 2) {
    const int m = mb + (lane >> 5), mm = m < m_hi ? m : m_lo;
    const int img = mm / pq, rem = mm - img * pq, p = rem / g.q, q = rem - p * g.q;
    const int iy = p * g.stride + kr - g.pad, ix = q * g.stride + kt - g.pad;
    const bool in = m < m_hi && (unsigned)iy < (unsigned)g.h && (unsigned)ix < (unsigned)g.wd;
    float a = dy[(size_t)mm * g.cout], b = x[(size_t)(in ? (img * g.h + iy) * g.wd + ix : 0) * g.cin];
    a = co_ok && m < m_hi ? a : 0.f;
    b = j_ok && in ? b : 0.f;
#if defined(__HIP_DEVICE_COMPILE__)
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
#endif
  }
  return acc;
}

// How a thread finds its rows of x.  PLAIN: 1x1 filters without stride or padding, row m is pixel m.  TABLE: the wave's 64 channels lie in
// one filter tap; every fourth step its lanes work out the offsets of the next 64 positions, one each, and leave them in LDS, where a
// thread finds those of its four rows with one read.  LANES: several taps, every lane follows its own rows (some 60
// vector instructions per step and block).
enum { PLAIN = 0, TABLE, LANES };

template <int WT, int GATHER>
__global__ __launch_bounds__(512, 1) void wgrad_x3_kernel(WgradGeom g, int Mrows, int J, int tiles_j, int tiles, int splits,
                                                          int steps_per_split, float* out, size_t split_stride, int main_grid) {
  using D = WDeep<WT>;
  [[maybe_unused]] constexpr int KS = D::KS, GT = D::GT;
  constexpr int TAB = GATHER == TABLE ? 8 * D::BPW * 256 : 0;       // 64 offsets per wave and block that it stages
  __shared__ __attribute__((aligned(1024))) char lds[D::LDS + TAB];
  if ((int)blockIdx.x >= main_grid) {
    static_assert(D::LDS >= wide_scratch<float>(512), "side jobs");
    wide_side_jobs<float, 512>(g.side, FlipJob{g.flip_w, g.flip_wt, g.cout, g.cin, g.r, g.s}, (int)blockIdx.x - main_grid, lds);
    return;
  }
#if defined(__HIP_DEVICE_COMPILE__)
  // XCD-aware order: each XCD gets a contiguous range of (split, tile) pairs; the tiles of one split read
  // the same rows of x and dy and find them in that XCD's L2.
  const int per_xcd = main_grid >> 3;
  const int work = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (work >= tiles * splits) return;
  const int split = work / tiles, tile = work - split * tiles;
  const int tile_co = tile / tiles_j, tile_j = tile - tile_co * tiles_j;
  const int co0 = tile_co * (64 * WT), j0 = tile_j * (64 * WT);
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  const int grp = __builtin_amdgcn_readfirstlane(tid / GT);
  const int gw = __builtin_amdgcn_readfirstlane((tid >> 6) & (WT * WT - 1));   // wave of the group
  const int wm0 = (gw / WT) * 64, wn0 = (gw % WT) * 64;
  const int n_all = (Mrows + 15) >> 4, step_lo = split * steps_per_split;
  const int n_steps = min(step_lo + steps_per_split, n_all) - step_lo;         // of the workgroup, at least one
  const int first = step_lo + (int)((long)n_steps * grp / KS);
  const int mine = step_lo + (int)((long)n_steps * (grp + 1) / KS) - first, rounds = (n_steps + KS - 1) / KS;

  // ---- loads.  A thread stages, per block its wave is in charge of, rows 4*m4 .. +3 of the step, channels
  // 4*c4 .. +3 of the block.  Blocks 0 .. WT-1 are dy, WT .. 2*WT-1 are x; dy is gathered as a 1x1 convolution's
  // input would be, so that both run the same instructions.
  const int m4 = lane & 3, c4 = lane >> 2;
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;              // beyond any descriptor range: reads as zero
  constexpr int BPW = D::BPW;
  __amdgpu_buffer_rsrc_t rs[BPW];
  int m_lim[BPW];                                        // rows from here on read as zero (0: the thread's channels do not exist)
  uint32_t row_b[BPW], off[BPW];                         // bytes per position; offset of the thread's first row of the step loaded next
  // the gather: position (p, q) reads pixel (p*gs + gy, q*gs + gx) of a gh x gw image; what the offset gains where q, where p wraps
  int gh[BPW], gwd[BPW], gs[BPW], gy[BPW], gx[BPW];
  uint32_t wrap_q[BPW], wrap_p[BPW], ch_of[BPW];
  int m_next = first * 16 + m4 * 4;                      // the thread's first row of the step that is loaded next
  int p0 = 0, q0 = 0;
  const float inv_q = 1.0f / (float)g.q, inv_p = 1.0f / (float)g.p;
  const int pq = g.p * g.q, img0 = m_next / pq;
  {
    const int rem = m_next - img0 * pq;
    p0 = rem / g.q;
    q0 = rem - p0 * g.q;
  }
#pragma unroll
  for (int b = 0; b < BPW; ++b) {
    const int blk = BPW == 1 ? gw : b;
    const bool is_x = blk >= WT;                         // wave-uniform
    uint32_t ch;
    if (!is_x) {
      const int co = co0 + blk * 64 + c4 * 4;
      m_lim[b] = co < g.cout ? Mrows : 0;
      ch = (uint32_t)co * 4u;
      row_b[b] = (uint32_t)g.cout * 4u;
      gh[b] = g.p; gwd[b] = g.q; gs[b] = 1; gy[b] = gx[b] = 0;
    } else {
      const int j = j0 + (blk - WT) * 64 + c4 * 4, jj = j < J ? j : 0;
      const int tap = jj / g.cin, ci = jj - tap * g.cin, kr = tap / g.s;
      m_lim[b] = j < J ? Mrows : 0;
      ch = (uint32_t)ci * 4u;
      row_b[b] = (uint32_t)g.cin * 4u;
      gh[b] = g.h; gwd[b] = g.wd; gs[b] = g.stride; gy[b] = kr - g.pad; gx[b] = tap - kr * g.s - g.pad;
    }
    ch_of[b] = ch;
    // offsets modulo 2^32; one that is used lies inside the tensor
    off[b] = (uint32_t)((img0 * gh[b] + p0 * gs[b] + gy[b]) * gwd[b] + q0 * gs[b] + gx[b]) * row_b[b] + ch;
    wrap_q[b] = (uint32_t)(gs[b] * gwd[b] - g.q * gs[b]) * row_b[b];
    wrap_p[b] = (uint32_t)((gh[b] - g.p * gs[b]) * gwd[b]) * row_b[b];
    // (wave-uniform; said so explicitly, or the descriptor ends up in vector registers)
    const uint64_t px = reinterpret_cast<uint64_t>(g.x), pdy = reinterpret_cast<uint64_t>(g.dy), base = is_x ? px : pdy;
    const int bytes = (int)(uint32_t)(is_x ? (size_t)g.n_img * g.h * g.wd * g.cin * 4 : (size_t)Mrows * g.cout * 4);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base), hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    rs[b] = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((uint64_t)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
  }
  // TABLE: the lane's position of the 64 that are worked out next: its row, the input pixel (ty, tx) it reads and its offset without the channel;
  // 64 positions on = whole images, rows and columns, with one wrap of each at most
  constexpr int NTB = GATHER == TABLE ? BPW : 1;
  uint32_t* const tab = reinterpret_cast<uint32_t*>(lds + D::LDS) + (tid >> 6) * (BPW * 64);
  int tm = first * 16 + lane, turn = 0, tx[NTB], ty[NTB];
  uint32_t toff[NTB], ch_off[NTB];
  const int d_img = 64 / pq, d_p = (64 - d_img * pq) / g.q, d_q = 64 - d_img * pq - d_p * g.q;
  if constexpr (GATHER == TABLE) {
    const int img = tm / pq, rem = tm - img * pq, p = rem / g.q, q = rem - p * g.q;
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
      // (the same for the whole wave: one tap)
      gy[b] = __builtin_amdgcn_readfirstlane(gy[b]);
      gx[b] = __builtin_amdgcn_readfirstlane(gx[b]);
      ty[b] = p * gs[b] + gy[b];
      tx[b] = q * gs[b] + gx[b];
      toff[b] = (uint32_t)((img * gh[b] + ty[b]) * gwd[b] + tx[b]) * row_b[b];
      ch_off[b] = m_lim[b] ? ch_of[b] : OUTSIDE;
    }
  }
  // The offsets of the next 64 positions.  A lane reads what other lanes of its wave store here: LDS accesses of a wave happen in the order in
  // which they are issued, and the fences keep the compiler from issuing a read on the wrong side of the stores (they cost no instruction).
  auto same_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto fill = [&]() {
    same_order();                  // the reads of the 64 before
#pragma unroll
    for (int b = 0; b < NTB; ++b) {
      const bool in = ((unsigned)ty[b] < (unsigned)gh[b]) & ((unsigned)tx[b] < (unsigned)gwd[b]) & (tm < Mrows);
      tab[b * 64 + lane] = in ? toff[b] : OUTSIDE;
      tx[b] += d_q * gs[b];
      const bool wx = tx[b] >= g.q * gs[b] + gx[b];
      tx[b] -= wx ? g.q * gs[b] : 0;
      ty[b] += d_p * gs[b] + (wx ? gs[b] : 0);
      const bool wy = ty[b] >= g.p * gs[b] + gy[b];
      ty[b] -= wy ? g.p * gs[b] : 0;
      toff[b] += (uint32_t)((d_img * gh[b] + d_p * gs[b]) * gwd[b] + d_q * gs[b]) * row_b[b] + (wx ? wrap_q[b] : 0u) + (wy ? wrap_p[b] : 0u);
    }
    tm += 64;
    same_order();                  // the reads of these
  };
  constexpr int NR = BPW == 2 ? 1 : 2;                   // register sets of loads in flight
  struct Regs { x3_v4u v[BPW][4]; } R0, R1_;
  Regs& R1 = NR == 2 ? R1_ : R0;
  auto load = [&](Regs& R) {
    uint32_t voff[BPW][4];
    if constexpr (GATHER == TABLE) {
#pragma unroll
      for (int b = 0; b < BPW; ++b) {
        const x3_v4u t = *reinterpret_cast<const x3_v4u*>(tab + b * 64 + turn * 16 + m4 * 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) voff[b][u] = __builtin_elementwise_add_sat(t[u], ch_off[b]);     // what is outside stays there
      }
      turn = (turn + 1) & 3;
    } else if constexpr (GATHER == PLAIN) {
#pragma unroll
      for (int b = 0; b < BPW; ++b) {
        uint32_t o = off[b];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          voff[b][u] = m_next + u < m_lim[b] ? o : OUTSIDE;
          o += row_b[b];
        }
        off[b] += 16 * row_b[b];
      }
    } else {
      int p = p0, q = q0;
      uint32_t o[BPW];
#pragma unroll
      for (int b = 0; b < BPW; ++b) o[b] = off[b];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool wq = q + 1 == g.q, wp = wq & (p + 1 == g.p);
#pragma unroll
        for (int b = 0; b < BPW; ++b) {
          const int iy = __mul24(p, gs[b]) + gy[b], ix = __mul24(q, gs[b]) + gx[b];
          const bool in = ((unsigned)iy < (unsigned)gh[b]) & ((unsigned)ix < (unsigned)gwd[b]) & (m_next + u < m_lim[b]);
          voff[b][u] = in ? o[b] : OUTSIDE;
          o[b] += gs[b] * row_b[b] + (wq ? wrap_q[b] : 0u) + (wp ? wrap_p[b] : 0u);
        }
        q = wq ? 0 : q + 1;
        p = wp ? 0 : p + (wq ? 1 : 0);
      }
      // sixteen rows on: the numbers of rows and of images passed are small quotients, exact in float with
      // the half added (p, q <= 4096)
      const int xq = q0 + 16, nq = (int)(((float)xq + 0.5f) * inv_q);
      q0 = xq - nq * g.q;
      const int xp = p0 + nq, np = (int)(((float)xp + 0.5f) * inv_p);
      p0 = xp - np * g.p;
#pragma unroll
      for (int b = 0; b < BPW; ++b) off[b] += 16 * gs[b] * row_b[b] + (uint32_t)nq * wrap_q[b] + (uint32_t)np * wrap_p[b];
    }
#pragma unroll
    for (int b = 0; b < BPW; ++b)
#pragma unroll
      for (int u = 0; u < 4; ++u) R.v[b][u] = __builtin_amdgcn_raw_buffer_load_b128(rs[b], voff[b][u], 0, 0);
    m_next += 16;
  };
  auto prepare = [&]() {           // before load(): outside what is scheduled by hand
    if constexpr (GATHER == TABLE)
      if (turn == 0) fill();
  };
  // ---- split and store: channel e of the thread goes to row 16*e + c4, its four values of m side by side
  char* const lds_g = lds + grp * (D::NST * D::STAGE);
  const int st_at = (BPW == 1 ? gw * D::BLOCK : 0) + c4 * 32 + (((m4 >> 1) ^ ((c4 >> 3) & 1)) << 4) + (m4 & 1) * 8;
  auto store = [&](const Regs& R, int buf) {
    char* at = lds_g + (buf & (D::NST - 1)) * D::STAGE + st_at;
#pragma unroll
    for (int b = 0; b < BPW; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t h0, m0_, l0, h1, m1_, l1;
        x3_split(__uint_as_float(R.v[b][0][e]), __uint_as_float(R.v[b][1][e]), h0, m0_, l0);
        x3_split(__uint_as_float(R.v[b][2][e]), __uint_as_float(R.v[b][3][e]), h1, m1_, l1);
        char* a = at + b * D::BLOCK + e * (16 * 32);
        *reinterpret_cast<x3_v2u*>(a) = x3_v2u{h0, h1};
        *reinterpret_cast<x3_v2u*>(a + D::PLANE) = x3_v2u{m0_, m1_};
        *reinterpret_cast<x3_v2u*>(a + 2 * D::PLANE) = x3_v2u{l0, l1};
      }
  };
  // ---- fragments and products
  struct Frags { x3_v4u a[3][2], b[3][2]; } F0, F1;
  const int f_at = (lane & 31) * 32 + ((half ^ ((lane >> 3) & 1)) << 4);
  const int fa_at = (wm0 >> 6) * D::BLOCK + f_at, fb_at = (WT + (wn0 >> 6)) * D::BLOCK + f_at;
  auto read = [&](Frags& F, int buf) {
    const char* st = lds_g + (buf & (D::NST - 1)) * D::STAGE;
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        F.a[p][i] = *reinterpret_cast<const x3_v4u*>(st + fa_at + p * D::PLANE + i * (32 * 32));
        F.b[p][i] = *reinterpret_cast<const x3_v4u*>(st + fb_at + p * D::PLANE + i * (32 * 32));
      }
  };
  x3_v16f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto multiply = [&](const Frags& F) {
    x3_product<2, 0, 2, 2>(F.a, F.b, acc);
    x3_product<0, 2, 2, 2>(F.a, F.b, acc);
    x3_product<1, 1, 2, 2>(F.a, F.b, acc);
    x3_product<1, 0, 2, 2>(F.a, F.b, acc);
    x3_product<0, 1, 2, 2>(F.a, F.b, acc);
    x3_product<0, 0, 2, 2>(F.a, F.b, acc);
  };
  auto sync = [&]() {              // a group of one wave shares nothing with the others
    if constexpr (D::NST == 2) __syncthreads();
  };
  // Step j: fragments F multiplied, fragments of j+1 read from stage (j+1)&1 into G, step j+2 (in R) stored into
  // stage j&1, whose last reader was step j-1's read of j; its registers are loaded with step j+2+NR.
  auto step = [&](const Frags& F, Frags& G, Regs& R, int par) {
    prepare();
    __builtin_amdgcn_sched_barrier(0);
    read(G, par ^ 1);
    store(R, par);
    load(R);
    multiply(F);
    constexpr int V = (104 * BPW + (GATHER == PLAIN ? 12 : GATHER == TABLE ? 6 : 60) * BPW + 23) / 24;
#pragma unroll
    for (int u = 0; u < 24; ++u) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (u < 12) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
      if (u >= 12) __builtin_amdgcn_sched_group_barrier(0x200, BPW, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto fetch = [&](Regs& R) { prepare(); load(R); };
  if (mine > 0) fetch(R0);
  if (NR == 2 && mine > 1) fetch(R1);
  if (mine > 0) store(R0, 0);
  if (mine > NR) fetch(R0);
  sync();
  if (mine > 0) read(F0, 0);
  if (mine > 1) store(R1, 1);
  if (mine > NR + 1) fetch(R1);
  sync();
  int j = 0;
  for (; j + 4 + NR <= mine; j += 2) {   // steady state: every load and store unconditional
    step(F0, F1, R0, 0);
    sync();
    step(F1, F0, R1, 1);
    sync();
  }
  for (; j < rounds; j += 2) {
    if (j + 1 < mine) read(F1, 1);
    if (j + 2 < mine) store(R0, 0);
    if (j + 2 + NR < mine) fetch(R0);
    if (j < mine) multiply(F0);
    sync();
    if (j + 1 >= rounds) break;
    if (j + 2 < mine) read(F0, 0);
    if (j + 3 < mine) store(R1, 1);
    if (j + 3 + NR < mine) fetch(R1);
    if (j + 1 < mine) multiply(F1);
    sync();
  }
  // ---- group q < NQ adds up the blocks BPQ*q ... of all wave positions, the groups' sums in their order after its own
  constexpr int BLK = 16 * 64, PER = WT * WT * D::BPQ * BLK;      // floats of a block, of one (to, from) pair of groups
  float* const red = reinterpret_cast<float*>(lds) + gw * (D::BPQ * BLK) + lane;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < D::NQ; ++q) {
    if (q == grp) continue;
    float* to = red + (q * (KS - 1) + (grp < q ? grp : grp - 1)) * PER;
#pragma unroll
    for (int b = 0; b < D::BPQ; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) to[b * BLK + v * 64] = acc[(q * D::BPQ + b) >> 1][(q * D::BPQ + b) & 1][v];
  }
  __syncthreads();
  if (KS > D::NQ && grp >= D::NQ) return;
  x3_v16f c[1][D::BPQ];            // BPQ = 2: one row block, two column blocks; BPQ = 1: one block
#pragma unroll
  for (int q = 0; q < D::NQ; ++q)
    if (q == grp) {
#pragma unroll
      for (int b = 0; b < D::BPQ; ++b) c[0][b] = acc[(q * D::BPQ + b) >> 1][(q * D::BPQ + b) & 1];
    }
#pragma unroll
  for (int u = 0; u < KS - 1; ++u)
#pragma unroll
    for (int b = 0; b < D::BPQ; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) c[0][b][v] += red[(grp * (KS - 1) + u) * PER + b * BLK + v * 64];
  const int bi = (grp * D::BPQ) >> 1, bj = (grp * D::BPQ) & 1;    // first block: row block bi, column block bj
  if (x3_any_nonfinite<1, D::BPQ>(c)) {
    const int m_lo = step_lo * 16, m_hi = min(Mrows, (step_lo + n_steps) * 16);
#pragma unroll
    for (int b = 0; b < D::BPQ; ++b)
      c[0][b] = plain_wgrad_block(g, co0 + wm0 + channel_of(32 * bi + (lane & 31)), j0 + wn0 + channel_of(32 * (bj + b) + (lane & 31)), J, m_lo, m_hi, lane);
  } else {
#pragma unroll
    for (int b = 0; b < D::BPQ; ++b) c[0][b] *= kX3Unscale;
  }
  float* dst = out + (size_t)split * split_stride;
#pragma unroll
  for (int b = 0; b < D::BPQ; ++b) {
    const int jcol = j0 + wn0 + channel_of(32 * (bj + b) + (lane & 31));
    if (jcol >= J) continue;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int co = co0 + wm0 + channel_of(32 * bi + 8 * (v >> 2) + 4 * half + (v & 3));
      if (co < g.cout) dst[(size_t)co * J + jcol] = c[0][b][v];
    }
  }
#else
  (void)&plain_wgrad_block; (void)&channel_of;
#endif
}

}  // namespace

// How a weight gradient is cut, never a function of addresses or of the swap plan: the tile and the number of parts, up
// to max_splits, with the smallest predicted time,
//   rounds of 256 workgroups x (fixed + per step of a group) + 3 us for the reduction + 1 byte / 4 TB/s for every part
// written and read, with 7.0 + 1.05 us (128 x 128 tile) and 4.5 + 1.75 us (64 x 64, eight groups) as measured.  At least
// 16 steps per part (more parts of small layers gain little); at most 32 MiB together.
WgradX3Cfg wgrad_x3_choose(long Mrows, int cin, int cout, int r, int s, int max_splits) {
  const long J = (long)r * s * cin, steps = (Mrows + 15) / 16;
  WgradX3Cfg best{};
  double best_us = 0;
  for (int wt = 1; wt <= 2; ++wt) {
    const int ks = 8 / (wt * wt);
    const int tco = (cout + 64 * wt - 1) / (64 * wt);
    const long tj = (J + 64 * wt - 1) / (64 * wt), tiles = tco * tj;
    const double part_us = (double)cout * J * 4 * 2 / 4.0e6;       // a part is written and read once
    for (long want = 1; want <= 256 && want <= max_splits; ++want) {
      const long per = (steps + want - 1) / want, splits = (steps + per - 1) / per;
      if (splits != want) continue;
      if (splits > 1 && (per < 16 || splits * cout * J * 4 > (32L << 20))) break;
      const long rounds = (tiles * splits + 255) / 256;
      const double us = rounds * (wt == 2 ? 7.0 + 1.05 * ((per + ks - 1) / ks) : 4.5 + 1.75 * ((per + ks - 1) / ks)) +
                        (splits > 1 ? 3.0 + splits * part_us : 0.0);
      if (best.wt == 0 || us < best_us) {
        best_us = us;
        best = WgradX3Cfg{wt, tco, (int)tj, (int)splits, (int)per};
      }
    }
  }
  return best;
}

hipError_t conv_wgrad_x3(const WgradGeom& g, const WgradX3Cfg& c, int Mrows, int J, float* out, size_t count, hipStream_t st) {
  const long side_blocks = wide_side_blocks(g.side, FlipJob{g.flip_w, g.flip_wt, g.cout, g.cin, g.r, g.s}, 512);
  const int tiles = c.tiles_co * c.tiles_j, main_grid = (int)(((long)tiles * c.splits + 7) / 8 * 8);
  const dim3 grid((unsigned)(main_grid + side_blocks));
  const int gather = g.r == 1 && g.s == 1 && g.stride == 1 && g.pad == 0 ? PLAIN : g.cin % 64 == 0 || g.r * g.s == 1 ? TABLE : LANES;
#define ACC_WX3(W, P) hipLaunchKernelGGL((wgrad_x3_kernel<W, P>), grid, dim3(512), 0, st, g, Mrows, J, c.tiles_j, tiles, c.splits, \
                                         c.steps_per_split, out, count, main_grid)
  if (c.wt == 2) { if (gather == PLAIN) ACC_WX3(2, PLAIN); else if (gather == TABLE) ACC_WX3(2, TABLE); else ACC_WX3(2, LANES); }
  else { if (gather == PLAIN) ACC_WX3(1, PLAIN); else if (gather == TABLE) ACC_WX3(1, TABLE); else ACC_WX3(1, LANES); }
#undef ACC_WX3
  return hipGetLastError();
}

}  // namespace acc
