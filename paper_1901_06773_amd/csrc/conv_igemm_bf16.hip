// Implicit-GEMM convolution for bf16 storage on the bf16 matrix cores of gfx950
// (v_mfma_f32_32x32x16_bf16), forward pass and data gradient.
//
//   out[m][n] (+)= sum_k A[m][k] * W[n][k],   m = (img,p,q), k = (r,t,c)
//
// K-chunks of a GEMM row go from global memory straight into LDS (buffer_load ... lds), rows unpadded with their 16-byte
// columns permuted by the row number, zero fill by offsets outside the buffer descriptor.  LDS has 64 banks here: sixteen
// consecutive rows read at one column lie on different ones (with a permutation of eight rows every read took eight cycles
// instead of four).
//
// What bounds it.  The matrix cores sustain about 2.0 PFLOP/s; a wave that multiplies 64 x 64 from fragments in LDS asks for
// as many bytes of LDS, and a 128 x 128 tile for twice as many bytes of L2, as a 256 x 256 tile of eight waves of 128 x 64 does.
// Large layers therefore run tiles of 256 x 256, and what remains is the start and the end of a tile (one workgroup
// per compute unit: nobody computes while it stores) and the number of rounds.  Rows of a chunk are 128 bytes wherever LDS allows:
// with 64-byte rows L2 answers twice as many requests (256->256 3x3 at 14x14, 512 images, 256 x 256 tile: 1.33e7 against 0.67e7, 136
// against 126 us).  The taps of 64 channels run before the next 64 channels: rows are found in L2 again (134 -> 126 us).
// Few tiles: the values of K are dealt out to groups of waves, down to eight waves that share one 32 x 32 tile.
// Measured against one 128 x 128 kernel and a 64 x 64 one for the rest (us, six sets of tensors in turn): 256->256 3x3 at 14x14,
// 512 images 142.6 -> 126.2; 512->512 3x3 at 7x7, 512 images 131.9 -> 111.6; 2048->512 1x1 at 7x7, 512 images 77.6 -> 59.7;
// 256->1024 1x1 at 14x14, 512 images 109.2 -> 93.6; 512->512 3x3 at 7x7, 4 images 36.9 -> 14.2, 32 images 37.5 -> 22.8; channels that come
// in 8s (a per-element loader before): 72->72 3x3 at 28x28, 128 images 169 -> 29, 200->200 731 -> 110.
#include <cmath>
#include <type_traits>

#include "kernels.h"
#include "dtype.h"
#include "lds_load.h"
#include "side_wide.h"

namespace acc {
namespace {

struct RowPos {  // decoded GEMM row
  int pix;       // img * h * wd (pixel index of the image origin)
  int iy0, ix0;  // p*stride - pad, q*stride - pad
  int ok;
};

__device__ __forceinline__ RowPos decode_row(const ConvGeom& g, int m, int M) {
  RowPos rp;
  rp.ok = m < M;
  const int mm = rp.ok ? m : 0;
  const int pq = g.p * g.q;
  const int img = mm / pq;
  const int rem = mm - img * pq;
  const int p = rem / g.q;
  const int q = rem - p * g.q;
  rp.pix = img * g.h * g.wd;
  rp.iy0 = p * g.stride - g.pad;
  rp.ix0 = q * g.stride - g.pad - g.pad_dx;
  return rp;
}

__device__ __forceinline__ size_t out_row_offset(const ConvGeom& g, int m) {
  const int pq = g.p * g.q;
  const int img = m / pq;
  const int rem = m - img * pq;
  const int p = rem / g.q;
  const int q = rem - p * g.q;
  return ((size_t)(img * g.out_h + g.out_y0 + p * g.out_stride) * g.out_w + g.out_x0 + q * g.out_stride) * g.n_out;
}

// A workgroup of KS groups of WM x WN waves owns a tile of 32*MB*WM rows and 32*NB*WN columns, a wave MB x NB blocks of
// 32 x 32.  BK values of K per chunk, NS LDS stages per group.
template <int WM_, int WN_, int KS_, int MB_, int NB_, int BK_, int NS_, int WPE_> struct Cfg {
  static constexpr int WM = WM_, WN = WN_, KS = KS_, MB = MB_, NB = NB_, BK = BK_, NS = NS_, WPE = WPE_;
  static constexpr int GT = 64 * WM * WN, THREADS = GT * KS;         // threads of a group, of the workgroup
  static constexpr int BM = 32 * MB * WM, BN = 32 * NB * WN;
  // Loads among the matrix instructions of the tiles that have a compute unit to themselves and two stages: 256->256 3x3 at 14x14, 512
  // images 130 -> 125 us; smaller tiles, where other workgroups fill the gap, gain nothing.
  static constexpr bool SPREAD = KS == 1 && NS == 2 && THREADS == 512;
  static constexpr int ROWB = BK * 2, CPR = BK / 8;                  // bytes and 16-byte columns of a staged row
  static constexpr int RPP = GT / CPR, AI = BM / RPP, BI = BN / RPP; // rows one load instruction of a group fills; instructions
  static constexpr int A_BYTES = BM * ROWB, STAGE = (BM + BN) * ROWB;
  static constexpr int MAIN = KS * NS * STAGE;
  static constexpr int EPF = NB * 128 + 16;                          // bytes per row staged in fp32 by one wave (KS == 1)
  static constexpr int PITCH = BN + 4;                               // floats per row staged by a group (KS > 1)
  static constexpr int OUT = KS == 1 ? WM * WN * 32 * EPF : KS * BM * PITCH * 4;
  static constexpr int LDS0 = MAIN > OUT ? MAIN : OUT, LDS = LDS0 > wide_scratch<bf16_t>(THREADS) ? LDS0 : wide_scratch<bf16_t>(THREADS);
};

// One tile, its first row m0 and column n0; `lds`: C::LDS bytes.  KN (whole chunks): the filter is read as a data gradient finds it, g.w_kn[c][taps, the
// last first][n]: rows of a chunk are its 64 c, of BN columns, and the LDS read transposes (ds_read_b64_tr_b16 hands every lane
// of a group of sixteen the four rows of one of sixteen columns).  The same products in the same order.
template <class C, bool ACT, bool RAGGED, bool KN = false>
__device__ __forceinline__ void tile(const ConvGeom& g, int M, int K, int m0, int n0, char* lds) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int MB = C::MB, NB = C::NB, AI = C::AI, BI = C::BI, CPR = C::CPR, ROWB = C::ROWB, NS = C::NS, KS = C::KS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / C::GT);
  const int gt = KS == 1 ? tid : tid & (C::GT - 1);
  const int uwave = __builtin_amdgcn_readfirstlane(gt >> 6);
  const int wm0 = (uwave / C::WN) * 32 * MB, wn0 = (uwave % C::WN) * 32 * NB;

  v16f acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  // ---- loads: global memory straight into LDS, 16 bytes per lane, rows unpadded with their 16-byte columns permuted
  // by the row number (the lane fetches the column that belongs into its slot)
  const int n_chunks = (K + C::BK - 1) / C::BK;
  auto swz = [](int row) { return CPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3; };
  const int lrow = gt / CPR, lcol = (gt & (CPR - 1)) ^ swz(lrow);
  static_assert(C::RPP % 16 == 0, "the permutation repeats every sixteen rows");
  const int margin = g.pad * g.wd + g.pad + g.pad_dx; // pixels; the descriptor starts that far before the tensor
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;           // beyond any descriptor range: reads as zero
  uint32_t a_voff[AI], a_mask[AI], b_voff[BI];
  const bool plain = g.r == 1 && g.s == 1 && g.stride == 1 && g.pad == 0 && g.pad_dx == 0 && g.p == g.h && g.q == g.wd;
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int m = m0 + lrow + C::RPP * i;
    if (plain) {      // 1x1, stride 1, no padding: GEMM row m is pixel m
      a_voff[i] = (uint32_t)(m < M ? m : 0) * (uint32_t)(g.c * 2) + lcol * 16;
      a_mask[i] = m < M ? 1u : 0u;
      continue;
    }
    const RowPos rp = decode_row(g, m, M);
    a_voff[i] = (uint32_t)(rp.pix + rp.iy0 * g.wd + rp.ix0 + margin) * (uint32_t)(g.c * 2) + lcol * 16;
    uint32_t mask = 0;
    for (int kr = 0; kr < g.r; ++kr)
      for (int kt = 0; kt < g.s; ++kt) {
        const bool ok = rp.ok && (unsigned)(rp.iy0 + kr) < (unsigned)g.h && (unsigned)(rp.ix0 + kt) < (unsigned)g.wd;
        mask |= (ok ? 1u : 0u) << (kr * g.s + kt);
      }
    a_mask[i] = mask;
  }
  const int taps = g.r * g.s;
  const uint32_t row_n = (uint32_t)g.n_out * 2u;      // KN: bytes of one tap of one c
  // KN: the lane's 16-byte column of BN and its rows a multiple of four apart
  constexpr int PB = C::BN * 2, CB = C::BN / 8, RB = C::GT / CB;
  static_assert(!KN || (RB % 4 == 0 && BI * RB == C::BK), "whole rows, four at a time");
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    if constexpr (KN) {
      const int row = gt / CB, n = n0 + 8 * ((gt % CB) ^ (row_xor<PB>(row) << 2));
      b_voff[i] = n < g.n_out ? (uint32_t)(row + RB * i) * ((uint32_t)taps * row_n) + (uint32_t)n * 2u : OUTSIDE;
    } else {
      const int n = n0 + lrow + C::RPP * i;
      b_voff[i] = (uint32_t)(n < g.n_out ? n : 0) * (uint32_t)(K * 2) + lcol * 16;   // beyond n_out: filter 0, never stored
    }
  }
  const size_t margin_bytes = (size_t)margin * g.c * 2;
  const size_t a_bytes = margin_bytes + (size_t)g.n_img * g.h * g.wd * g.c * 2;
  __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(g.in)) - margin_bytes, 0, (int)(uint32_t)a_bytes, 0x00020000);
  __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(g.w), 0, (int)(uint32_t)((size_t)g.n_out * K * 2), 0x00020000);
  [[maybe_unused]] const srsrc kn_a = descriptor(static_cast<const char*>(g.in) - margin_bytes, a_bytes), kn_b = descriptor(g.w_kn, (size_t)g.n_out * K * 2);
  typedef __attribute__((address_space(3))) void* lds_ptr;
  char* const lds_g = lds + grp * (NS * C::STAGE);
  const uint32_t lds_w = (uint32_t)(size_t)lds_g + uwave * 1024;
  // the group's chunks, and where the next one to be loaded lies.  Whole chunks inside one tap (not RAGGED): the same for
  // all lanes; else every lane follows the 16-byte column it loads
  const int first = KS == 1 ? 0 : (int)((long)n_chunks * grp / KS);
  const int mine = KS == 1 ? n_chunks : (int)((long)n_chunks * (grp + 1) / KS) - first;
  const int rounds = KS == 1 ? n_chunks : (n_chunks + KS - 1) / KS;
  const int cols = g.c >> 3;                          // 16-byte columns of a pixel
  int tap, kt, col = 0, soff_b, toff;                 // toff: bytes from the row's first pixel
  if constexpr (RAGGED) {
    const int u = first * CPR + lcol;
    tap = u / cols;
    col = u - tap * cols;
    soff_b = first * ROWB;
  } else if constexpr (KS > 1) {                      // a group's own part of K, in the order of memory
    const int u = first * CPR;
    tap = u / cols;
    col = u - tap * cols;
    soff_b = first * ROWB;
  } else {                                            // the taps of 64 channels, then those of the next: rows stay in L2 between taps
    const int c0 = first / taps;
    tap = first - c0 * taps;
    soff_b = tap * g.c * 2 + c0 * ROWB;
    col = c0 * CPR;
  }
  {
    const int kr = tap / g.s;
    kt = tap - kr * g.s;
    toff = ((kr * g.wd + kt) * cols + col - (RAGGED ? lcol : 0)) * 16;
  }
  if constexpr (KN) soff_b = (col * 8 * taps + taps - 1 - tap) * (int)row_n;
  int left = (K >> 3) - first * CPR - lcol;           // RAGGED: columns of K from the lane's on
  const int row_jump = (g.wd - g.s) * g.c * 2;
  const int back_a = g.r * g.wd * g.c * 2 - ROWB, back_b = K * 2 - ROWB;
  constexpr int L = AI + BI, MF = MB * NB;
  // load u of the next chunk (first those of A), which goes to the stage at `at`; advance() when all have been issued
  auto load = [&](int u, uint32_t at) {
    const bool k_ok = !RAGGED || left > 0;
    if constexpr (KN) {                               // (all loads of such an instance, or none, are load_lds16's)
      if (u < AI) load_lds16(kn_a, ((a_mask[u] >> (tap & 31)) & 1u) != 0 ? a_voff[u] : OUTSIDE, (uint32_t)toff, at + u * (C::GT * 16));
      else load_lds16(kn_b, b_voff[u - AI], (uint32_t)soff_b, at + C::A_BYTES + (u - AI) * (C::GT * 16));
      return;
    }
    if (u < AI) {
      const bool ok = ((a_mask[u] >> (tap & 31)) & 1u) != 0 && k_ok;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_a, (lds_ptr)(size_t)(at + u * (C::GT * 16)), 16,
                                               ok ? a_voff[u] + (RAGGED ? (uint32_t)toff : 0u) : OUTSIDE, RAGGED ? 0 : toff, 0, 0);
    } else {
      const int i = u - AI;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_b, (lds_ptr)(size_t)(at + C::A_BYTES + i * (C::GT * 16)), 16, k_ok ? b_voff[i] : OUTSIDE,
                                               soff_b, 0, 0);
    }
  };
  auto advance = [&]() {
    if constexpr (RAGGED) {
      soff_b += ROWB;
      left -= CPR;
      col += CPR;
      const bool wrap = col >= cols;                  // (cols >= CPR: once at most)
      col -= wrap ? cols : 0;
      tap += wrap ? 1 : 0;
      kt += wrap ? 1 : 0;
      const bool down = kt == g.s;
      kt = down ? 0 : kt;
      toff += ROWB + (down ? row_jump : 0);           // the next tap of a filter row is the next pixel
    } else if constexpr (KS > 1) {
      soff_b += KN ? C::BK * taps * (int)row_n : ROWB;
      toff += ROWB;                                   // the next tap of a filter row is the next pixel
      if ((col += CPR) == cols) {
        col = 0;
        ++tap;
        if constexpr (KN) soff_b = (taps - 1 - tap) * (int)row_n;
        if (++kt == g.s) { kt = 0; toff += row_jump; }
      }
    } else {
      soff_b += KN ? -(int)row_n : g.c * 2;
      toff += g.c * 2;
      if (++kt == g.s) { kt = 0; toff += row_jump; }
      if (++tap == taps) { tap = 0; toff -= back_a; soff_b += KN ? (C::BK + 1) * taps * (int)row_n : -back_b; }
    }
  };
  auto issue = [&](int stage) {
#pragma unroll
    for (int u = 0; u < L; ++u) load(u, lds_w + stage * C::STAGE);
    advance();
  };
  // ---- fragments: 16-byte column c16 of a row sits in slot c16 ^ swz(row); the lane's blocks lie multiples of 32 rows apart
  constexpr int NG = C::BK / 16;
  const int ra = wm0 + (lane & 31), rb = wn0 + (lane & 31);
  const int xa = swz(ra), xb = swz(rb);
  struct Frags { v4u a[MB], b[NB]; } F[2];
  // KN: lane t of sixteen names four columns of row t/4 and receives rows 0..3 of column t; a fragment wants column lane%32 and eight rows: two reads
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(3))) v4s* tr_ptr;
  const int frow = 8 * (lane >> 5) + ((lane & 15) >> 2);
  [[maybe_unused]] int kn_at[NB];
  if constexpr (KN) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      kn_at[j] = C::A_BYTES + frow * PB + (((wn0 / 32 + j) ^ row_xor<PB>(frow)) << 6) + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
  }
  auto rd = [&](Frags& f, const char* st, int g8) {
    const int c16 = g8 * 2 + (lane >> 5);
    const char* as = st + ra * ROWB + ((c16 ^ xa) << 4);
    if constexpr (KN) {
#pragma unroll
      for (int i = 0; i < MB; ++i) f.a[i] = *reinterpret_cast<const v4u*>(as + i * 32 * ROWB);
      auto* const st3 = (__attribute__((address_space(3))) char*)const_cast<char*>(st);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const v2u lo = __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(st3 + kn_at[j] + g8 * 16 * PB)));
        const v2u hi = __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(st3 + kn_at[j] + g8 * 16 * PB + 4 * PB)));
        f.b[j] = v4u{lo.x, lo.y, hi.x, hi.y};
      }
      return;
    }
    const char* bs = st + C::A_BYTES + rb * ROWB + ((c16 ^ xb) << 4);
#pragma unroll
    for (int i = 0; i < MB; ++i) f.a[i] = *reinterpret_cast<const v4u*>(as + i * 32 * ROWB);
#pragma unroll
    for (int j = 0; j < NB; ++j) f.b[j] = *reinterpret_cast<const v4u*>(bs + j * 32 * ROWB);
  };
  auto mm = [&](const Frags& f) {
#pragma unroll
    for (int u = 0; u < MF; ++u) acc[u / NB][u % NB] = mfma_bf16(f.b[u % NB], f.a[u / NB], acc[u / NB][u % NB]);   // transposed block, see the epilogue
  };
  // One chunk = BK/16 groups of 16 values of K.  The reads of group g+1 are issued among the MFMAs of group g, and the last
  // group's MFMAs are held back until the next chunk's barrier has been passed and its first reads are on their way; the loads of a later
  // chunk are issued before or (SPREAD) among them: the matrix cores have work queued while the wave waits.
  auto groups = [&](const char* st) {
#pragma unroll
    for (int g8 = 0; g8 + 1 < NG; ++g8) {
      rd(F[(g8 + 1) & 1], st, g8 + 1);
      mm(F[g8 & 1]);
      constexpr int RD = MB + (KN ? 2 : 1) * NB;
#pragma unroll
      for (int u = 0; u < RD; ++u) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, MF / RD > 0 ? MF / RD : 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    static_assert(NG % 2 == 0, "the held-back group is F[1]");
  };
  auto chunk = [&](int stage, bool prev, bool more, int to) {
    const char* st = lds_g + stage * C::STAGE;
    __builtin_amdgcn_sched_barrier(0);
    rd(F[0], st, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (more) issue(to);
    if (prev) mm(F[1]);
    __builtin_amdgcn_sched_barrier(0);
    groups(st);
  };
  auto spread_chunk = [&](int stage, int to) {
    const char* st = lds_g + stage * C::STAGE;
    __builtin_amdgcn_sched_barrier(0);
    rd(F[0], st, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < MF; ++u) {
      acc[u / NB][u % NB] = mfma_bf16(F[1].b[u % NB], F[1].a[u / NB], acc[u / NB][u % NB]);
#pragma unroll
      for (int l = u * L / MF; l < (u + 1) * L / MF; ++l) load(l, lds_w + to * C::STAGE);
      __builtin_amdgcn_sched_barrier(0);
    }
    advance();
    __builtin_amdgcn_sched_barrier(0);
    groups(st);
  };
  // What opens chunk j: this wave's loads of chunk j have landed (those of later chunks may be on their way), and, where a
  // group has several waves, a barrier: everybody's have, and everybody is done with chunk j-1, whose stage the next loads overwrite.
  auto open = [&](int j) {
    __builtin_amdgcn_sched_barrier(0);
    const int later = mine - 1 - j;                   // chunks behind this one that can have been issued: NS - 2 at most
    if (NS > 3 && later >= 2) wait_loads<(NS > 3 ? 2 * L : 0)>();
    else if (NS > 2 && later >= 1) wait_loads<(NS > 2 ? L : 0)>();
    else wait_loads<0>();
    if constexpr (C::GT > 64) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(NS >= 2 && NS <= 4, "open() knows up to two later chunks");
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < mine) issue(s);
  if constexpr (C::SPREAD) {
    static_assert(KS == 1 && NS == 2, "the last chunk is the one without loads");
    open(0);
    chunk(0, false, mine > 1, 1);
    int j = 1;
    for (; j + 1 < mine; ++j) {
      open(j);
      spread_chunk(j & 1, (j & 1) ^ 1);
    }
    if (j < mine) {
      open(j);
      chunk(j & 1, true, false, 0);
    }
  } else {
    int stage = 0, to = NS - 1;
    for (int j = 0; j < rounds; ++j) {
      open(j);
      if (KS == 1 || j < mine) chunk(stage, j > 0, j + NS - 1 < mine, to);
      stage = stage + 1 == NS ? 0 : stage + 1;
      to = to + 1 == NS ? 0 : to + 1;
    }
  }
  if (KS == 1 || mine > 0) mm(F[1]);

  // Epilogue.  The blocks were accumulated transposed (filter fragment first): register v of a
  // lane holds output channel 8*(v/4) + 4*(lane/32) + v%4 of GEMM row lane%32 of its block, i.e.
  // four consecutive channels of one row per group of four registers.  They are staged in LDS and read back as whole rows:
  // eight channels per lane, one 16-byte store each.
  wait_loads<0>();
  __builtin_amdgcn_s_barrier();                      // every wave is done reading the last chunk
  asm volatile("" ::: "memory");
  const bool dense = g.out_stride == 1 && g.out_h == g.p && g.out_w == g.q;
  typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
  typedef float v2f __attribute__((ext_vector_type(2)));
  auto pack2 = [](float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{a, b}, v2bf));   // round to nearest even
  };
  auto place = [&](int m, int n) { return static_cast<bf16_t*>(g.out) + (dense ? (size_t)m * g.n_out : out_row_offset(g, m)) + n; };
  // eight fp32 results: bias and ReLU, or the old values, then one rounding
  auto finish = [&](float (&f)[8], bf16_t* o, const float (&bias8)[8]) {
    if constexpr (ACT) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        f[e] += bias8[e];
        if (g.relu) f[e] = fmaxf(f[e], 0.f);
      }
    } else if (g.accumulate) {
      const v4u old = *reinterpret_cast<const v4u*>(o);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        f[2 * w] += __uint_as_float(old[w] << 16);
        f[2 * w + 1] += __uint_as_float(old[w] & 0xffff0000u);
      }
    }
    v4u res;
#pragma unroll
    for (int w = 0; w < 4; ++w) res[w] = pack2(f[2 * w], f[2 * w + 1]);
    *reinterpret_cast<v4u*>(o) = res;
  };
  if constexpr (KS > 1) {
    // the groups' sums side by side in fp32; every thread adds up pieces of eight channels, the groups in their order
    float* red = reinterpret_cast<float*>(lds) + grp * (C::BM * C::PITCH);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const v16f& c = acc[i][j];
          *reinterpret_cast<float4*>(red + (wm0 + 32 * i + (lane & 31)) * C::PITCH + wn0 + 32 * j + 8 * q4 + 4 * (lane >> 5)) =
              make_float4(c[4 * q4], c[4 * q4 + 1], c[4 * q4 + 2], c[4 * q4 + 3]);
        }
    __syncthreads();
    constexpr int PPR = C::BN / 8;                   // pieces of a row
#pragma unroll
    for (int pc = tid; pc < C::BM * PPR; pc += C::THREADS) {
      const int row = pc / PPR, c8 = pc - row * PPR, m = m0 + row, n = n0 + 8 * c8;
      if (m >= M || n >= g.n_out) continue;          // (n_out is a multiple of 8: a piece is stored whole or not at all)
      const float* p = reinterpret_cast<const float*>(lds) + row * C::PITCH + 8 * c8;
      float f[8], bias8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      float part[KS][8];
#pragma unroll
      for (int u = 0; u < KS; ++u) {
        const float4 lo = *reinterpret_cast<const float4*>(p + u * (C::BM * C::PITCH)), hi = *reinterpret_cast<const float4*>(p + u * (C::BM * C::PITCH) + 4);
        part[u][0] = lo.x; part[u][1] = lo.y; part[u][2] = lo.z; part[u][3] = lo.w;
        part[u][4] = hi.x; part[u][5] = hi.y; part[u][6] = hi.z; part[u][7] = hi.w;
      }
#pragma unroll
      for (int d = KS / 2; d > 0; d /= 2)              // in pairs: the fewest roundings
#pragma unroll
        for (int u = 0; u < d; ++u)
#pragma unroll
          for (int e = 0; e < 8; ++e) part[u][e] += part[u + d][e];
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = part[0][e];
      if constexpr (ACT) {
        if (g.bias) {
#pragma unroll
          for (int e = 0; e < 8; ++e) bias8[e] = g.bias[n + e];
        }
      }
      finish(f, place(m, n), bias8);
    }
    return;
  }
  // One region per wave, 32 rows at a time.  Plain results are rounded to bf16 before staging; results that
  // get a bias and a ReLU, or are added to what the tensor holds, are staged in fp32, so that they are rounded once, after
  // the addition.
  char* stg = lds + uwave * (32 * C::EPF);
  constexpr int PPR = NB * 4, RPI = 64 / PPR, IT = 32 / RPI;      // pieces of a row, rows per instruction, instructions
  const int c8 = lane % PPR, prow = lane / PPR;
  const int n = n0 + wn0 + 8 * c8;
  const bool n_ok = n < g.n_out;                     // (n_out is a multiple of 8: a piece is stored whole or not at all)
  if (!ACT && !g.accumulate) {
    constexpr int EP = NB * 64 + 16;                 // bytes per staged row (rows on different banks)
#pragma unroll
    for (int i = 0; i < MB; ++i) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const v16f& c = acc[i][j];
          uint2 pk;
          pk.x = pack2(c[4 * q4], c[4 * q4 + 1]);
          pk.y = pack2(c[4 * q4 + 2], c[4 * q4 + 3]);
          *reinterpret_cast<uint2*>(stg + (lane & 31) * EP + (32 * j + 8 * q4 + 4 * (lane >> 5)) * 2) = pk;
        }
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int row = prow + RPI * it, m = m0 + wm0 + 32 * i + row;
        if (m >= M || !n_ok) continue;
        *reinterpret_cast<v4u*>(place(m, n)) = *reinterpret_cast<const v4u*>(stg + row * EP + c8 * 16);
      }
    }
    return;
  }
  float bias8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if constexpr (ACT) {
    if (g.bias && n_ok) {
#pragma unroll
      for (int e = 0; e < 8; ++e) bias8[e] = g.bias[n + e];
    }
  }
#pragma unroll
  for (int i = 0; i < MB; ++i) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const v16f& c = acc[i][j];
        *reinterpret_cast<float4*>(stg + (lane & 31) * C::EPF + (32 * j + 8 * q4 + 4 * (lane >> 5)) * 4) =
            make_float4(c[4 * q4], c[4 * q4 + 1], c[4 * q4 + 2], c[4 * q4 + 3]);
      }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int row = prow + RPI * it, m = m0 + wm0 + 32 * i + row;
      if (m >= M || !n_ok) continue;
      const float4 lo = *reinterpret_cast<const float4*>(stg + row * C::EPF + c8 * 32);
      const float4 hi = *reinterpret_cast<const float4*>(stg + row * C::EPF + c8 * 32 + 16);
      float f[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      finish(f, place(m, n), bias8);
    }
  }
#else
  (void)&decode_row; (void)&out_row_offset;
#endif
}

template <class C, bool ACT, bool RAGGED, bool KN>
__global__ __launch_bounds__(C::THREADS, C::WPE) void igemm_bf16_kernel(ConvGeom g, int M, int K, int n_tiles_n, int n_tiles, int main_grid) {
  __shared__ __attribute__((aligned(1024))) char lds[C::LDS];
  if ((int)blockIdx.x >= main_grid) {
    wide_side_jobs<bf16_t, C::THREADS>(g.side, g.flip, (int)blockIdx.x - main_grid, lds);
    return;
  }
  // XCD-aware tile order: each XCD gets a contiguous range of tiles (neighbours share operand rows in its L2)
  const int per_xcd = main_grid >> 3;
  const int at = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (at >= n_tiles) return;
  const int tile_m = at / n_tiles_n, tile_n = at - tile_m * n_tiles_n;
  tile<C, ACT, RAGGED, KN>(g, M, K, tile_m * C::BM, tile_n * C::BN, lds);
}

// Two heights of tiles in one launch: n_tiles of C in main_grid workgroups, then the rows from `m` on in `tiles` of T (as wide) in `grid` more.
struct Tail {
  int m, tiles, grid;
};
template <class C, class T, bool ACT, bool RAGGED, bool KN>
__global__ __launch_bounds__(C::THREADS, C::WPE) void igemm_bf16_tail_kernel(ConvGeom g, int M, int K, int n_tiles_n, int n_tiles, int main_grid, Tail tail) {
  __shared__ __attribute__((aligned(1024))) char lds[C::LDS > T::LDS ? C::LDS : T::LDS];
  const int id = (int)blockIdx.x - main_grid;
  if (id >= tail.grid) {
    wide_side_jobs<bf16_t, C::THREADS>(g.side, g.flip, id - tail.grid, lds);
    return;
  }
  if (id >= 0) {
    const int at = (id & 7) * (tail.grid >> 3) + (id >> 3);
    if (at >= tail.tiles) return;
    const int tile_m = at / n_tiles_n, tile_n = at - tile_m * n_tiles_n;
    tile<T, ACT, RAGGED, KN>(g, M, K, tail.m + tile_m * T::BM, tile_n * T::BN, lds);
    return;
  }
  const int at = (blockIdx.x & 7) * (main_grid >> 3) + (blockIdx.x >> 3);
  if (at >= n_tiles) return;
  const int tile_m = at / n_tiles_n, tile_n = at - tile_m * n_tiles_n;
  tile<C, ACT, RAGGED, KN>(g, M, K, tile_m * C::BM, tile_n * C::BN, lds);
}

// the launch was given the filter as a data gradient finds it, and only that
inline bool reads_kn(const ConvGeom& g) { return g.w_kn && !g.w; }

template <class C>
void launch(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe) {
  const int tm = (M + C::BM - 1) / C::BM, tn = (g.n_out + C::BN - 1) / C::BN, tiles = tm * tn, main_grid = (tiles + 7) / 8 * 8;
  const dim3 grid((unsigned)(main_grid + wide_side_blocks(g.side, g.flip, C::THREADS)));
  const bool ragged = g.c % C::BK != 0, act = g.bias || g.relu;
  if (probe->before) (void)hipEventRecord(probe->before, st);
#define ACC_BF16(...) hipLaunchKernelGGL((igemm_bf16_kernel<C, __VA_ARGS__>), grid, dim3(C::THREADS), 0, st, g, M, K, tn, tiles, main_grid)
  if (reads_kn(g)) ACC_BF16(false, false, true);
  else if (act) { if (ragged) ACC_BF16(true, true, false); else ACC_BF16(true, false, false); }
  else { if (ragged) ACC_BF16(false, true, false); else ACC_BF16(false, false, false); }
#undef ACC_BF16
  if (probe->after) (void)hipEventRecord(probe->after, st);
}

// the rows from tail_m (whole tiles of C) on in tiles of T
template <class C, class T>
void launch_tail(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe, int tail_m) {
  static_assert(T::BN == C::BN && T::THREADS == C::THREADS && T::BK == C::BK, "one launch");
  const int tn = (g.n_out + C::BN - 1) / C::BN, tiles = tail_m / C::BM * tn, main_grid = (tiles + 7) / 8 * 8;
  const int tail_tiles = (M - tail_m + T::BM - 1) / T::BM * tn;
  const Tail tail{tail_m, tail_tiles, (tail_tiles + 7) / 8 * 8};
  const dim3 grid((unsigned)(main_grid + tail.grid + wide_side_blocks(g.side, g.flip, C::THREADS)));
  const bool ragged = g.c % C::BK != 0, act = g.bias || g.relu;
  if (probe->before) (void)hipEventRecord(probe->before, st);
#define ACC_BF16(...) hipLaunchKernelGGL((igemm_bf16_tail_kernel<C, T, __VA_ARGS__>), grid, dim3(C::THREADS), 0, st, g, M, K, tn, tiles, main_grid, tail)
  if (reads_kn(g)) ACC_BF16(false, false, true);
  else if (act) { if (ragged) ACC_BF16(true, true, false); else ACC_BF16(true, false, false); }
  else { if (ragged) ACC_BF16(false, true, false); else ACC_BF16(false, false, false); }
#undef ACC_BF16
  if (probe->after) (void)hipEventRecord(probe->after, st);
}

typedef Cfg<2, 4, 1, 4, 2, 64, 2, 2> T256x256;
typedef Cfg<2, 4, 1, 2, 2, 64, 3, 2> T128x256;
typedef Cfg<2, 4, 1, 3, 2, 64, 2, 2> L192x256;         // the last rows behind tiles of 256 x 256
typedef Cfg<2, 4, 1, 1, 2, 64, 2, 2> L64x256;
typedef Cfg<2, 2, 1, 4, 2, 32, 3, 2> T256x128;
typedef Cfg<2, 2, 1, 2, 2, 64, 2, 2> T128x128;
typedef Cfg<2, 2, 1, 2, 1, 64, 2, 2> T128x64;
typedef Cfg<2, 2, 1, 1, 1, 64, 2, 2> T64x64;
typedef Cfg<2, 2, 1, 1, 1, 64, 4, 2> T64x64s4;         // four LDS stages: long reductions of few tiles
typedef Cfg<2, 1, 4, 1, 2, 64, 2, 2> T64x64k4;         // four groups of two waves
typedef Cfg<1, 1, 4, 2, 2, 32, 2, 1> T64x64k4n;        // four groups of one wave, chunks of 32 values
typedef Cfg<1, 1, 8, 1, 1, 32, 4, 2> T32x32k8;         // eight groups of one wave

// Which kernel: the one with the smallest predicted time, in microseconds.  With steps = chunks of K per group of waves, and tiles
// counted on the compute unit with the most,
//   base + (compute^2 + memory^2)^(1/2),           (256 x 256: tiles = the rounds of heights())
//   compute = one workgroup per compute unit: first + first_step * steps + (tiles - 1) * (next + next_step * steps),
//             several (r <= per_cu resident): the sum over rounds of max(first + first_step * steps, r * (next + next_step * steps)),
// taps more per tile for filters larger than 1x1, memory = per_mb_read * MB of both operands + per_mb_written * MB of the result,
// each once.  The constants are fitted to 420 launches (the layers of the ResNets at minibatches 1 to 512 and random ones with
// widths in 8s, every kernel on each, replayed from a graph, six sets of tensors in turn, so that large operands come from memory):
// median errors of 3 to 6 %, the choice is within 0.8 % of the best on average, 26 % at most.  Strided filters (137 more launches)
// within 1.1 % on average, 16 % at most; with the whole input counted for each of them 2 % and 33 %: 42x39 128->256 1x1/2,
// 125 images 16.9 -> 12.1 us, 56x56 128->128 3x3/2, 128 images 59.7 -> 53.7.
// What each is worth, over those and 138 more forward launches: without it the choice gets slower on average by, and is off the best by at
// most, 256 x 256 0.7 % and 26 %, 128 x 256 0.2 and 19, 128 x 128 0.9 and 45, 128 x 64 0.5 and 23, 64 x 64 0.7 and 18, its four stages 1.6 and 28,
// four pairs 0.3 and 20, four waves 0.1 and 34, 32 x 32 6 and 155; 256 x 128 is the only large one for fewer than 64 channels and
// worth nothing from there on.  A function of the shape and the alignment only.
struct Kind {
  const char* name;
  int bm, bn, ks, kc, per_cu;
  double base, first, first_step, next, next_step, taps, per_mb_read, per_mb_written;
};
enum { K256x256 = 0, K128x256, K256x128, K128x128, K128x64, K64x64, K64x64S4, K64x64K4, K64x64K4N, K32x32K8, KINDS };
constexpr Kind kKinds[KINDS] = {
    {"igemm_bf16 256x256", 256, 256, 1, 64, 1, 4.714, 0.0, 1.277, 1.809, 1.818, 2.416, 0.203, 0.223},
    {"igemm_bf16 128x256", 128, 256, 1, 64, 1, 3.027, 0.868, 0.730, 1.668, 0.954, 1.056, 0.189, 0.266},
    {"igemm_bf16 256x128", 256, 128, 1, 32, 2, 3.643, 0.662, 0.481, 0.621, 0.478, 1.509, 0.179, 0.267},
    {"igemm_bf16 128x128", 128, 128, 1, 64, 2, 2.311, 1.132, 0.623, 0.613, 0.487, 1.003, 0.169, 0.287},
    {"igemm_bf16 128x64", 128, 64, 1, 64, 3, 1.983, 0.954, 0.555, 0.914, 0.298, 0.569, 0.166, 0.171},
    {"igemm_bf16 64x64", 64, 64, 1, 64, 4, 2.097, 0.506, 0.484, 0.561, 0.176, 0.118, 0.161, 0.157},
    {"igemm_bf16 64x64, four stages", 64, 64, 1, 64, 2, 1.646, 1.345, 0.310, 0.850, 0.196, 0.472, 0.094, 0.332},
    {"igemm_bf16 64x64, four pairs", 64, 64, 4, 64, 1, 3.394, 0.0, 1.033, 2.060, 0.957, 1.338, 0.208, 0.249},
    {"igemm_bf16 64x64, four waves", 64, 64, 4, 32, 2, 2.286, 1.275, 0.586, 0.914, 0.503, 0.035, 0.136, 0.431},
    {"igemm_bf16 32x32, eight waves", 32, 32, 8, 32, 1, 0.0, 3.255, 0.543, 1.221, 0.487, 0.520, 0.271, 2.084},
};
// Tiles of 256 x 256 take a compute unit each, and in their last round most units may have none (392 tiles: 256 and 136).  The rows that don't
// fill a round run behind the others as tiles of 192 or 64 rows in the same launch, where that saves 3 % of the rounds or more, a round of 192 rows
// counted as 0.8 of one of 256, one of 64 as 0.4 (the half of the chip that runs a part round runs it faster).  us, 256 x 256
// alone -> with lower tiles: 256->256 3x3 at 14x14, 512 images (256 + 182 x 192) 113 -> 106, at 28x28, 200 images (256 + 476 x 192) 173 -> 157;
// 128->256 3x3 at 28x28, 256 images (768 + 64 x 64) 130 -> 118; 1024->512 1x1 at 28x28, 128 images (768 + 64 x 64) 127 -> 116.
// Measured with every split of up to four rounds on 299 forward launches of 2 to 47 rounds (layers of the ResNets at minibatches of 32 to 512,
// random 1x1 and 3x3 ones): 214 are split, 1.09 times as fast on average (0.96 once, else 1.001 to 1.26), and all within 0.7 % of the best split on
// average, 6 % at most.  Splits that save less than 3 % gained 0.5 % on average and lost up to 4 (85 launches, 20 slower: long launches drift apart
// and have no last round).  The weights may lie anywhere from 0.7 and 0.3 to 0.8 and 0.45; below 0.78, three rounds of 192 come before two
// of 256 and one of 64: 51 launches differ, 0.95 to 1.06, by nothing on average.
// Layers that wait for memory keep one height (22 of them would be 1.06 times as fast with lower tiles, 0.97 to 1.17).
struct Heights {
  int low, rows;                                         // height of the lower tiles (0: none), rows of the higher ones
  double rounds;
};
Heights heights(long M, long N) {
  const long tn = (N + 255) / 256, all = (M + 255) / 256 * tn, plain = (all + 255) / 256;
  Heights best{0, 0, (double)plain};
  for (long full = plain - 1; full >= 1 && full >= plain - 3; --full) {
    const long rows = full * 256 / tn * 256, rest = M - rows;
    if (rows <= 0 || rest <= 0) continue;
    const long r192 = ((rest + 191) / 192 * tn + 255) / 256, r64 = ((rest + 63) / 64 * tn + 255) / 256;
    if (r192 <= 3 && full + 0.8 * r192 < best.rounds - 0.05) best = Heights{192, (int)rows, full + 0.8 * r192};
    if (r64 == 1 && full + 0.4 < best.rounds - 0.05) best = Heights{64, (int)rows, full + 0.4};
  }
  return best.rounds > 0.97 * (double)plain ? Heights{0, 0, (double)plain} : best;
}
double memory_us(const Kind& k, const ConvGeom& g, long M, long K) {
  // pixels that are read: all of the input, or, by strided filters smaller than their stride, those under a tap; chunks of 32 values (half
  // lines of memory) find nothing again that a tap of a strided filter has read before
  const double taps = (double)M * g.r * g.s, in = (double)g.n_img * g.h * g.wd, pixels = g.stride > 1 && (taps < in || k.kc == 32) ? taps : in;
  const double read = 2e-6 * (pixels * g.c + (double)g.n_out * K), written = 2e-6 * (double)M * g.n_out;
  return k.per_mb_read * read + k.per_mb_written * written;
}
double compute_us(const Kind& k, const ConvGeom& g, long M, long K, bool lower) {
  const long tiles = ((M + k.bm - 1) / k.bm) * ((g.n_out + k.bn - 1) / k.bn), steps = ((K + k.kc - 1) / k.kc + k.ks - 1) / k.ks;
  const long whole = (tiles + 255) / 256;                // tiles of the busiest compute unit
  const double most = lower ? heights(M, g.n_out).rounds : (double)whole;
  const double first = k.first + k.first_step * steps, next = k.next + k.next_step * steps, more = g.r * g.s > 1 ? k.taps * most : 0;
  auto round = [&](long r) { return r == 0 ? 0.0 : first > r * next ? first : r * next; };
  return more + (k.per_cu == 1 ? first + (most - 1) * next : (whole / k.per_cu) * round(k.per_cu) + round(whole % k.per_cu));
}
// whether a launch of 256 x 256 tiles may have lower ones: it does not wait for memory
bool lower_tiles(const Kind& k, const ConvGeom& g, long M, long K) {
  return k.bm == 256 && k.bn == 256 && memory_us(k, g, M, K) <= compute_us(k, g, M, K, false);
}
double predicted_us(const Kind& k, const ConvGeom& g, long M, long K) {
  const double compute = compute_us(k, g, M, K, lower_tiles(k, g, M, K)), memory = memory_us(k, g, M, K);
  return k.base + std::sqrt(compute * compute + memory * memory);
}
int best_kind(const ConvGeom& g, long M, long K) {
  int best = -1;
  double us = 0;
  for (int v = 0; v < KINDS; ++v) {
    if (g.c < kKinds[v].kc) continue;                    // a chunk spans two taps at most
    const double t = predicted_us(kKinds[v], g, M, K);
    if (best < 0 || t < us) { best = v; us = t; }
  }
  return best;
}

}  // namespace

bool conv_igemm_bf16_takes(const ConvGeom& g, long M, long K) {
  if (g.dtype != DT_BF16) return false;
  // channels that come in 8s, at least a chunk of 32 of them, at most 32 taps, both operands within 32-bit byte ranges
  // (the last bytes stay free for the offset that stands for "outside"), 16-byte aligned tensors and rows of the result; no fused
  // batch-norm sums (those belong to fp32 storage)
  const long margin_px = (long)g.pad * g.wd + g.pad + g.pad_dx;
  if (g.c % 8 != 0 || g.c < 32 || g.r * g.s > 32 || g.n_out % 8 != 0 || g.stats || g.bnb.sums) return false;
  if ((margin_px + (long)g.n_img * g.h * g.wd) * g.c * 2 > 0xFFFFFF00L || (long)g.n_out * K * 2 > 0xFFFFFF00L) return false;
  if ((reinterpret_cast<uintptr_t>(g.in) & 15) || (reinterpret_cast<uintptr_t>(g.w) & 15) ||
      (reinterpret_cast<uintptr_t>(g.out) & 15)) return false;
  // the filter as it lies: whole chunks of the kernel that will run, nothing fused behind, its offsets within 30 bits
  if (reads_kn(g) && ((long)g.n_out * K * 2 >= (1L << 30) || (reinterpret_cast<uintptr_t>(g.w_kn) & 15) || g.bias || g.relu || g.c % kKinds[best_kind(g, M, K)].kc != 0)) return false;
  return ((M + 31) / 32) * ((g.n_out + 31) / 32) <= (1L << 30);
}

hipError_t conv_igemm_bf16(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe) {
  if (g.side.count && (!g.side.part || !g.side.dw || g.side.splits < 1)) return hipErrorInvalidValue;
  if ((g.bias || g.relu) && g.accumulate) return hipErrorInvalidValue;
  if (g.flip.wt && (!g.flip.w || g.flip.cout <= 0 || g.flip.cin <= 0 || g.flip.r <= 0 || g.flip.s <= 0)) return hipErrorInvalidValue;
  if (wide_side_blocks(g.side, g.flip, 256) > (1L << 30) - 8) return hipErrorInvalidValue;
  const int kind = best_kind(g, M, K);
  probe->variant = V_IGEMM_BF16;
  probe->kernel = kKinds[kind].name;
  Heights h{0, 0, 0};
  if (kind == K256x256 && lower_tiles(kKinds[kind], g, M, K)) h = heights(M, g.n_out);
  if (h.low) probe->kernel = h.low == 192 ? "igemm_bf16 256x256 and 192x256" : "igemm_bf16 256x256 and 64x256";
  if (probe->dry) return hipSuccess;
  switch (kind) {
    case K256x256:
      if (h.low == 192) launch_tail<T256x256, L192x256>(g, M, K, st, probe, h.rows);
      else if (h.low == 64) launch_tail<T256x256, L64x256>(g, M, K, st, probe, h.rows);
      else launch<T256x256>(g, M, K, st, probe);
      break;
    case K128x256: launch<T128x256>(g, M, K, st, probe); break;
    case K256x128: launch<T256x128>(g, M, K, st, probe); break;
    case K128x128: launch<T128x128>(g, M, K, st, probe); break;
    case K128x64: launch<T128x64>(g, M, K, st, probe); break;
    case K64x64: launch<T64x64>(g, M, K, st, probe); break;
    case K64x64S4: launch<T64x64s4>(g, M, K, st, probe); break;
    case K64x64K4: launch<T64x64k4>(g, M, K, st, probe); break;
    case K64x64K4N: launch<T64x64k4n>(g, M, K, st, probe); break;
    default: launch<T32x32k8>(g, M, K, st, probe); break;
  }
  return hipGetLastError();
}

}  // namespace acc
