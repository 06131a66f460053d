// Batches of more than 64 tokens (prompts, evaluation windows): both products
// of a layer as tiled matrix-core products over every row of the pass.
//
// pf_pack_kernel    the call input in row blocks, and the route of each row.
// pf_gateup_kernel  p = SiLU(h W_gate) (h W_up), each row under its own route
//                   and keep rule (Eq. 1, 2, 4-5, 13): BM rows by NT columns
//                   of both projections per workgroup.
// pf_down_kernel    partial y over one chunk of d_ff: BM rows by BN columns.
// The partials are added in chunk order by dense_glue_kernel.
//
// At 64 rows a pass is bound by the weight stream (235 MB of W_gate and W_up
// per pass at the Llama-3.1-8B shape); more rows per pass reuse every weight
// byte until the matrix cores are the bound.  A workgroup of 8 wavefronts
// walks k in steps of 32 through rings of LDS stages that are loaded by
// buffer loads writing LDS.  The MFMA operands of step s + 1 are read from
// LDS under the products of step s, so a step starts with its products right
// after the barrier.  A stage is refilled one barrier after the products
// that used its last operands.
//
// Bound: the matrix cores, after the weight stream.  1000 rows of a
// Llama-3.1-8B layer (352 Gflop): 16 passes of 64 rows take 1276 us, a call here
// 336 us (1.05 Pflop/s; a large library product reaches 1.18).  Its launches,
// each under rocprofv3, where they take longer than in a row of calls: rows into
// blocks 6 us, gate/up 234, down 114, second stage 13.  Without its loads the
// gate/up loop takes 169 us.
//
// Layouts.  The left operands (h, p) are kept in row blocks: 16 rows by 32 k,
// 1 KB, the blocks of 16 rows in k order; chunk q (16 bytes) of row r sits at
// q ^ pf_swz(r) of the row's 64 bytes, so that a load of a block is 1 KB in a
// row and the 16-byte LDS reads of a wavefront (16 rows at one k) fall in
// distinct banks.  W_gate_T and W_up_T rows are staged 64 k (a 128-byte line)
// at a time, chunk q of row r at q ^ (r & 7): half lines double the requests
// on the L2, which then bounds the product (gate/up 280 us with h and the
// weights in 64-byte pieces).  W_down rows are staged 32 at a time, BN columns each;
// the pair of chunks of columns 16 c .. 16 c + 15 of row r sits at pair
// c ^ pf_kswz(r), so that the transposing LDS reads (ds_read_b64_tr_b16: 4
// rows x 16 columns per 16 lanes) fall in distinct banks.
#pragma once

#include <type_traits>

#include "dense.hpp"

namespace sats {

constexpr int kPfThreads = 512;  // 8 wavefronts
constexpr int kPfKC = 32;        // k per step

// transposed operand of a k-row tile (pitch bytes per row): columns 16 ct ..
// 16 ct + 15, this lane's column l16, rows 8 g .. 8 g + 7.  Of each group of
// 16 lanes, lane i reads 4 columns 4 (i % 4) .. of row i / 4 and receives
// column i of the 4 rows.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ int pf_kswz(int r) { return (r & 3) | (((r >> 3) & 1) << 2); }
__device__ __forceinline__ bf16x8 pf_krow_operand(uint8_t *tile, int pitch, int ct, int g, int l16) {
  s16x4 v[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = 8 * g + 4 * h + (l16 >> 2);
    v[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4 *)(tile + r * pitch + (ct ^ pf_kswz(r)) * 32 + (l16 & 3) * 8));
  }
  const s16x8 b = {v[0][0], v[0][1], v[0][2], v[0][3], v[1][0], v[1][1], v[1][2], v[1][3]};
  return __builtin_bit_cast(bf16x8, b);
}
// operand of a row block: row r of the block's 16, k = 8 g .. 8 g + 7
__device__ __forceinline__ bf16x8 pf_block_operand(const uint8_t *blk, int r, int g) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(blk + r * 64 + (g ^ pf_swz(r)) * 16));
}

struct PfArgs {
  const uint16_t *A;      // row blocks of h (gate/up) or p (down); float32 data for the float32 kernels
  const uint16_t *Wg, *Wu;  // gate/up: [N][K] each (the same)
  const uint16_t *Wd;     // down: [K][N] (the same)
  uint16_t *P;            // gate/up: row blocks of p
  size_t pterm;           // split p: elements from one term's row blocks to the next's (P, A)
  float *part;            // down: partials [ks][n][N]
  const float *thr;       // layer threshold, or null (base path for every row)
  const uint8_t *gbase;   // base-path flag of each row (gate/up; allocated to whole tiles of 256)
  const uint8_t *x;       // up to 64 rows, first layer: the call input [n][K] in place of A
  const int32_t *ids;     // up to 64 rows: the flags are looked up in the kernel
  const uint8_t *lut;
  int route_mode;
  uint8_t *keep_out;      // optional [n][N] keep flags
  uint16_t *kept;         // few float32 rows: bit c mod 16 of word c / 16 is set where some row keeps
                          // column c (written by gate/up for down, which reads up to 32 words of 32 past the last)
  int n, K, N;            // rows; reduction length; output columns
  int mtiles, units;      // row tiles; column tiles (times k chunks, down)
  int ks, kchunk;         // down: k chunks and their length (a multiple of 32)
  float *cal_g;           // calibration: g in float32, [n][N] ...
  uint16_t *cal_ph, *cal_pl;  // ... and p as two bf16 terms (hi = rne(p), lo = rne(p - hi))
  const uint16_t *ext;    // PF_LORA: row blocks of the further k of h; B_gate^T and B_up_T [N][rank]
  const uint16_t *BgT, *BuT;
  int rank;
};

// The rows of x in row blocks (rows past n and k past d zero), the base-path
// flags, and the inspection copies of both.  A wavefront per block.
struct PfPackArgs {
  const uint8_t *x;       // [n] rows of `bytes` bytes (a multiple of 16)
  uint8_t *A;             // row blocks, or null
  uint8_t *gbase;         // [n], or null
  const int32_t *ids;
  const uint8_t *lut;
  int route_mode;
  int n, bytes;
  uint8_t *route_out;     // optional [n]
  uint8_t *layer_in;      // optional copy of x
};
__global__ __launch_bounds__(kThreads) void pf_pack_kernel(PfPackArgs a) {
  const int lane = threadIdx.x & 63;
  const int nb = (a.bytes + 63) / 64;
  const int b = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);  // block: row tile b / nb, k block b % nb
  if (b >= (a.n + 15) / 16 * nb) return;
  const int r = lane >> 2, m = b / nb * 16 + r, k = b % nb * 64 + 16 * ((lane & 3) ^ pf_swz(r));
  u32x4 v = {0u, 0u, 0u, 0u};
  if (m < a.n && k < a.bytes) {
    v = *reinterpret_cast<const u32x4 *>(a.x + (size_t)m * a.bytes + k);
    if (a.layer_in) *reinterpret_cast<u32x4 *>(a.layer_in + (size_t)m * a.bytes + k) = v;
  }
  if (a.A) *reinterpret_cast<u32x4 *>(a.A + (size_t)b * 1024 + 16 * lane) = v;
  if (b % nb == 0 && (lane & 3) == 0 && m < a.n && (a.gbase || a.route_out)) {
    const uint8_t base = (uint8_t)token_is_base(a.route_mode, a.ids, a.lut, m);
    if (a.gbase) a.gbase[m] = base;
    if (a.route_out) a.route_out[m] = base;
  }
}

// Workgroup b (on XCD b mod 8) takes row tile j % mtiles of unit 8 (j /
// mtiles) + b % 8, j = b / 8: the row tiles of a unit run side by side on one
// XCD, whose L2 then reads the unit's weights from memory once.
__device__ __forceinline__ bool pf_tile(const PfArgs &a, int &mt, int &unit) {
  const int j = blockIdx.x >> 3;
  mt = j % a.mtiles;
  unit = (j / a.mtiles) * 8 + (blockIdx.x & 7);
  return unit < a.units;
}

// Waits until at most VM of this wavefront's loads are outstanding, then
// meets the other wavefronts (its LDS reads may still be under way: the
// buffer refilled next holds operands already used).
template <int VM> __device__ __forceinline__ void pf_barrier() {
  static_assert(VM >= 0 && VM < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (15 << 8) | ((VM >> 4) << 14));
  __builtin_amdgcn_s_barrier();
}

// 16 bytes per lane from base + voff + soff of the buffer into LDS at dst +
// 16 * lane; a lane whose voff is kDenseOffNone reads zeros (soff is the
// same for the wavefront, so a step costs no address arithmetic per lane)
__device__ __forceinline__ void pf_dma(__amdgpu_buffer_rsrc_t r, uint8_t *dst, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)dst, 16, (int)voff, (int)soff, 0, 0);
}

// Sums of split shapes are folded: the accumulators of four steps (128 k) are
// added to a second set and restart at zero.  A float32 sum over 4096 k in one
// accumulator is about four times further from 64 bits than the compacted
// kernels' (64 lanes of 64 terms each), which those shapes take otherwise;
// folded, it is as near.
template <int MT, int CT> __device__ __forceinline__ void pf_fold(f32x4v (&sum)[MT][CT], f32x4v (&acc)[MT][CT]) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      sum[i][j] += acc[i][j];
      acc[i][j] = f32x4v{0.f, 0.f, 0.f, 0.f};
    }
}

// Eight columns of p as three bf16 terms, 16 bytes of each term's row blocks.  A term
// is the leading 8 bits of what is left, cut off and not rounded: three of them hold
// the 24 bits of p, none leaves the range, and an infinite p has no remainder.
__device__ __forceinline__ void pf_store_terms(uint16_t *o, size_t pterm, float (&v)[8]) {
#pragma unroll
  for (int h = 0; h < 3; ++h) {
    u32x4 b;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t t = __float_as_uint(v[k]) & 0xffff0000u;
      if (k & 1)
        b[k / 2] |= t;
      else
        b[k / 2] = t >> 16;
      if (h < 2) {
        const float rest = v[k] - __uint_as_float(t);
        v[k] = h > 0 || fabsf(v[k]) < INFINITY ? rest : 0.0f;
      }
    }
    *reinterpret_cast<u32x4 *>(o + h * pterm) = b;
  }
}

// The ring buffers are an array per stage: the compiler then knows which
// stage a pending load writes and adds no wait of its own before the LDS
// reads of another (it tells at most 8 apart).

// ---------------------------------------------------------------- gate/up

// BM = 256: wavefront w takes rows 64 (w / 2) .. + 63 and all NT columns of
// W_gate (w even) or W_up (w odd).  BM = 128: rows 64 (w / 4) .. + 63 and
// half of the columns.  The rings hold 4 stages of h (32 k) and WR of the
// weights (64 k, used by steps 2 j and 2 j + 1).
// MODE: how p leaves the kernel.
enum { PF_P16 = 0,   // rounded to bf16
       PF_SPLIT = 1,  // three bf16 terms whose sum is p
       PF_CAL = 2,    // calibration: g in float32, and p as two terms, without the keep rule
       PF_LORA = 3 }; // as PF_P16, with 4 R further k for the adapters (K a multiple of 64): rows of
                      // h continue with [hi | lo] of s (h A_gate) and of s (h A_up), W_gate rows with
                      // B_gate twice and zeros, W_up rows with zeros and B_up twice, so that the adapter
                      // terms are in the sums before SiLU and the keep rule
template <int BM, int NT, int MODE>
__global__ __launch_bounds__(kPfThreads, 2) void pf_gateup_kernel(PfArgs a) {
  constexpr bool CAL = MODE == PF_CAL;
  constexpr int WPG = 8 / (BM / 64);           // wavefronts per 64-row group
  constexpr int CW = NT / (WPG / 2);           // columns per wavefront
  constexpr int MT = 4, CT = CW / 16;          // its 16 x 16 tiles
  constexpr int IA = BM / 128;                 // 1 KB loads per wavefront: a stage of h ...
  constexpr int IW = 2 * NT / 64;              // ... and of the weights (8 rows each)
  constexpr int SA = BM * 64, SW = IW * 8192;  // stage bytes
  constexpr int WR = 4 * SA + 4 * SW <= 160 * 1024 ? 4 : 3;
  static_assert(4 * SA + WR * SW <= 160 * 1024 && CT * 16 == CW && NT % 32 == 0, "rings and tile shapes");
  __shared__ __attribute__((aligned(1024))) uint8_t a0[SA], a1[SA], a2[SA], a3[SA], w0[SW], w1[SW], w2[SW],
      w3[WR > 3 ? SW : 16];
  auto abuf = [&](int i) -> uint8_t * { return (i &= 3) == 0 ? a0 : i == 1 ? a1 : i == 2 ? a2 : a3; };
  auto wbuf = [&](int i) -> uint8_t * { return (i %= WR) == 0 ? w0 : i == 1 ? w1 : i == 2 ? w2 : w3; };
  int mt0, unit;
  if (!pf_tile(a, mt0, unit)) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const int m0 = mt0 * BM, n0 = unit * NT;
  constexpr bool LORA = MODE == PF_LORA;
  const int K = a.K, N = a.N, S0 = (K + kPfKC - 1) / kPfKC;
  const int R4 = LORA ? 4 * a.rank : 0, SE = (R4 + kPfKC - 1) / kPfKC, S = S0 + SE;  // steps: of K, of the adapters, all
  const int grp = w / WPG, mat = (w % WPG) / (WPG / 2), half = w % (WPG / 2);
  (void)R4;
  // base-path flags of the rows this lane finishes (see the epilogue), four to a word
  const int lm0 = 64 * grp + (mat ? 0 : 32);
  uint32_t base4[MT / 2];
#pragma unroll
  for (int i = 0; i < MT / 2; ++i)
    base4[i] = CAL ? 0u : *reinterpret_cast<const uint32_t *>(a.gbase + m0 + lm0 + 16 * i + 4 * g);
  const int rows16 = (a.n + 15) / 16;
  const __amdgpu_buffer_rsrc_t rsa = dense_rsrc(a.A, (uint32_t)((size_t)rows16 * S0 * 1024));
  const uint32_t wbytes = (uint32_t)((size_t)N * K * 2);
  // h: load i = w + 8 q of a stage is row block m0 / 16 + i at the stage's k (past the last row: zeros)
  uint32_t aoff[IA], aext[IA];
#pragma unroll
  for (int q = 0; q < IA; ++q) {
    const int rb = m0 / 16 + w + 8 * q;
    aoff[q] = rb < rows16 ? (uint32_t)rb * (uint32_t)S0 * 1024u + 16u * lane : kDenseOffNone;
    aext[q] = rb < rows16 ? (uint32_t)rb * (uint32_t)SE * 1024u + 16u * lane : kDenseOffNone;
  }
  // weights: load i = w + 8 q of a stage is rows 8 i .. 8 i + 7 of [W_gate | W_up], 128 bytes each
  const int lr = lane >> 3, lq = (lane & 7) ^ lr;
  uint32_t woff[IW], wext[IW];
#pragma unroll
  for (int q = 0; q < IW; ++q) {
    const int row = 8 * (w + 8 * q) + lr, c = n0 + (row < NT ? row : row - NT);
    woff[q] = row < 2 * NT && c < N ? (uint32_t)(((size_t)c * K + 8 * lq) * 2) : kDenseOffNone;
    wext[q] = LORA && c < N ? (uint32_t)c * (uint32_t)a.rank * 2u : kDenseOffNone;
  }
  auto issue_a = [&](uint8_t *buf, int s) {
    const bool e = LORA && s >= S0;  // (scalar selects, no branch: see the ring buffers)
#pragma unroll
    for (int q = 0; q < IA; ++q)
      if constexpr (LORA)
        pf_dma(dense_rsrc(e ? a.ext : a.A, (uint32_t)(rows16 * (e ? SE : S0)) * 1024u), buf + (w + 8 * q) * 1024,
               s < S ? (e ? aext[q] : aoff[q]) : kDenseOffNone, (uint32_t)(e ? s - S0 : s) * 1024u);
      else
        pf_dma(rsa, buf + (w + 8 * q) * 1024, s < S ? aoff[q] : kDenseOffNone, (uint32_t)s * 1024u);
  };
  auto issue_w = [&](uint8_t *buf, int j) {
    const bool v = 64 * j + 8 * lq < K;
    const bool e = LORA && 2 * j >= S0;
    const int ke = 64 * (j - S0 / 2) + 8 * lq;  // the lane's k among the further ones
#pragma unroll
    for (int q = 0; q < IW; ++q) {
      const int i = w + 8 * q;
      const bool up = i >= NT / 8;
      if constexpr (LORA) {
        const bool on = ke < R4 && (ke >= R4 / 2) == up && wext[q] != kDenseOffNone;
        pf_dma(dense_rsrc(e ? (up ? a.BuT : a.BgT) : (up ? a.Wu : a.Wg), e ? (uint32_t)N * (uint32_t)a.rank * 2u : wbytes),
               buf + i * 1024, e ? (on ? wext[q] + 2u * (uint32_t)(ke & (a.rank - 1)) : kDenseOffNone)
                                 : (v ? woff[q] : kDenseOffNone),
               e ? 0u : (uint32_t)j * 128u);
      } else {
        pf_dma(dense_rsrc(up ? a.Wu : a.Wg, wbytes), buf + i * 1024, v ? woff[q] : kDenseOffNone, (uint32_t)j * 128u);
      }
    }
  };
  bf16x8 oa0[MT], oa1[MT], ob[CT];  // operands: h of even and of odd steps, weights
  auto load_a = [&](const uint8_t *buf, int t) { return pf_block_operand(buf + (4 * grp + t) * 1024, l16, g); };
  auto load_b = [&](const uint8_t *buf, int t, int h) {  // k half h of the stage
    const int r = mat * NT + half * CW + 16 * t + l16;
    return __builtin_bit_cast(bf16x8,
                              *reinterpret_cast<const u32x4 *>(buf + r * 128 + ((4 * h + g) ^ (r & 7)) * 16));
  };
  f32x4v acc[MT][CT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[i][j] = f32x4v{0.f, 0.f, 0.f, 0.f};
  constexpr bool FOLD = MODE == PF_SPLIT;
  static_assert(!FOLD || CT <= 4, "registers of the second set");
  f32x4v sum[FOLD ? MT : 1][FOLD ? CT : 1] = {};
  // the order of the loop's loads, from 2 WR - 2 steps before the first
#pragma unroll
  for (int s = 2 - 2 * WR; s < 0; ++s) {
    if (s + 3 >= 0) issue_a(abuf(s + 3), s + 3);
    if (s % 2 == 0) issue_w(wbuf(s / 2 + WR - 1), s / 2 + WR - 1);
  }
  pf_barrier<2 * IA + IW>();
#pragma unroll
  for (int t = 0; t < MT; ++t) oa0[t] = load_a(a0, t);
#pragma unroll
  for (int t = 0; t < CT; ++t) ob[t] = load_b(w0, t, 0);
  // step s: the stages of step s + 1 have landed, and every wavefront is done
  // with the products of step s - 1; the stages it used last are refilled,
  // and the operands of step s + 1 are read under the products (a weight
  // operand once its last product is issued, into the same registers)
  auto step = [&](int s, int p, bf16x8(&xa)[MT], bf16x8(&ya)[MT]) {  // s = p modulo the round
    pf_barrier<IA + IW>();
    issue_a(abuf(p + 3), s + 3);
    if (p % 2 == 0) issue_w(wbuf(p / 2 + WR - 1), s / 2 + WR - 1);
    const uint8_t *an = abuf(p + 1), *wn = wbuf((p + 1) / 2);
#pragma unroll
    for (int t = 0; t < MT; ++t) ya[t] = load_a(an, t);
#pragma unroll
    for (int j = 0; j < CT; ++j) {
#pragma unroll
      for (int i = 0; i < MT; ++i) acc[i][j] = mfma16(xa[i], ob[j], acc[i][j]);
      ob[j] = load_b(wn, j, (p + 1) & 1);
    }
#pragma unroll
    for (int i = 0; i < MT * CT; ++i) {  // a product, and an LDS read beside the first ones and the last of a column
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i < MT || i % MT == MT - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
  };
  constexpr int U = WR == 3 ? 12 : 8;  // steps of a round: whole turns of both rings
  for (int s0 = 0; s0 < S; s0 += U) {
    step(s0, 0, oa0, oa1);
    step(s0 + 1, 1, oa1, oa0);
    step(s0 + 2, 2, oa0, oa1);
    step(s0 + 3, 3, oa1, oa0);
    if constexpr (FOLD) pf_fold(sum, acc);
    step(s0 + 4, 4, oa0, oa1);
    step(s0 + 5, 5, oa1, oa0);
    step(s0 + 6, 6, oa0, oa1);
    step(s0 + 7, 7, oa1, oa0);
    if constexpr (FOLD) pf_fold(sum, acc);
    if constexpr (U > 8) {
      step(s0 + 8, 8, oa0, oa1);
      step(s0 + 9, 9, oa1, oa0);
      step(s0 + 10, 10, oa0, oa1);
      step(s0 + 11, 11, oa1, oa0);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);  // the zero-filling loads past the range land too
  if constexpr (FOLD)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) acc[i][j] = sum[i][j];
  __syncthreads();
  // epilogue: the wavefronts of W_gate and W_up of the same rows and columns
  // (a pair) trade half of their tiles through LDS, lane to lane: the W_up
  // one finishes row tiles 0 and 1, the W_gate one 2 and 3
  const int pair = grp * (WPG / 2) + half;  // 4 pairs
  static_assert(MT / 2 * CT * 1024 <= SA && MT * CT * 1024 <= SW, "the exchange fits the stage buffers");
  uint8_t *xw = pair == 0 ? w0 : pair == 1 ? w1 : pair == 2 ? w2 : a0;   // SiLU inputs for the W_up wavefront
  uint8_t *xu = pair == 3 ? a1 : xw + MT / 2 * CT * 1024;               // h W_up for the W_gate wavefront
  f32x4v *xo = reinterpret_cast<f32x4v *>(mat ? xu : xw) + lane;
  uint8_t *xi = mat ? xw : xu;
  f32x4v own[MT / 2][CT];  // (moved, not selected by index: the accumulators stay in registers)
  if (mat) {
#pragma unroll
    for (int i = 0; i < MT / 2; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) xo[(i * CT + j) * 64] = acc[i + MT / 2][j], own[i][j] = acc[i][j];
  } else {
#pragma unroll
    for (int i = 0; i < MT / 2; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) xo[(i * CT + j) * 64] = acc[i][j], own[i][j] = acc[i + MT / 2][j];
  }
  __syncthreads();
  const float thr = !CAL && a.thr ? *a.thr : 0.0f;
  const int c0 = n0 + half * CW;
  uint64_t kept = 0;  // bit 4 (i CT + j) + r
#pragma unroll
  for (int i = 0; i < MT / 2; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      const int t = i * CT + j;
      const f32x4v o = reinterpret_cast<const f32x4v *>(xi)[t * 64 + lane];
      const f32x4v av = mat ? o : own[i][j], uv = mat ? own[i][j] : o;
      float pk[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float gv = silu(av[r]), pv = gv * uv[r];
        if constexpr (CAL) {
          const int m = m0 + lm0 + 16 * i + 4 * g + r, c = c0 + 16 * j + l16;
          if (m < a.n && c < N) {
            const uint16_t hi = f32_to_bf16(pv);
            const size_t e = (size_t)m * N + c;
            a.cal_g[e] = gv;
            a.cal_ph[e] = hi;
            a.cal_pl[e] = f32_to_bf16(pv - bf16_to_f32(hi));
          }
        } else {
          const bool keep = ((base4[i] >> (8 * r)) & 0xffu) || fabsf(gv) >= thr;
          kept |= (uint64_t)keep << ((4 * t + r) & 63);
          pk[r] = keep ? pv : 0.0f;
        }
      }
      // the tile as 16 rows of 16 columns, over the part of the exchange already read
      if constexpr (!CAL)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (MODE == PF_SPLIT)
            *reinterpret_cast<float *>(xi + t * 1024 + (4 * g + r) * 64 + l16 * 4) = pk[r];
          else
            *reinterpret_cast<uint16_t *>(xi + t * 512 + (4 * g + r) * 32 + l16 * 2) = f32_to_bf16(pk[r]);
        }
    }
  if constexpr (CAL) return;
  // 16 bytes (a row's 8 columns) per lane and store: lane (row r, chunk q) of tile t
  const int nbp = (N + kPfKC - 1) / kPfKC;  // k blocks of a row block of p
#pragma unroll
  for (int e = 0; e < MT / 2 * CT / 2; ++e) {
    const int t = 2 * e + (lane & 1), r = (lane >> 2), q = (lane >> 1) & 1;
    const int m = m0 + lm0 + 16 * (t / CT) + r, c = c0 + 16 * (t % CT) + 8 * q;
    uint16_t *o = a.P + ((size_t)(m >> 4) * nbp + (c >> 5)) * 512 + r * 32 + (((c >> 3) & 3) ^ pf_swz(r)) * 8;
    if constexpr (MODE == PF_SPLIT) {
      float v[8];
      *reinterpret_cast<f32x4v *>(v) = *reinterpret_cast<const f32x4v *>(xi + t * 1024 + r * 64 + q * 32);
      *reinterpret_cast<f32x4v *>(v + 4) = *reinterpret_cast<const f32x4v *>(xi + t * 1024 + r * 64 + q * 32 + 16);
      if (m < a.n && c < N) pf_store_terms(o, a.pterm, v);
    } else {
      const u32x4 v = *reinterpret_cast<const u32x4 *>(xi + t * 512 + r * 32 + q * 16);
      if (m < a.n && c < N) *reinterpret_cast<u32x4 *>(o) = v;
    }
  }
  if (a.keep_out)
    for (int b = 0; b < MT / 2 * CT * 4; ++b) {
      const int t = b >> 2, m = m0 + lm0 + 16 * (t / CT) + 4 * g + (b & 3), c = c0 + 16 * (t % CT) + l16;
      if (m < a.n && c < N) a.keep_out[(size_t)m * N + c] = (uint8_t)((kept >> b) & 1);
    }
}

// ---------------------------------------------------------------- down

// Wavefront w takes rows (BM / WM) (w / WN) .. and columns (BN / WN) (w % WN)
// .. of the tile; unit u is column tile u / ks and k chunk u % ks.
// SPLIT: p comes as three bf16 terms, each multiplied with the same W_down
// operands (a stage holds the terms' blocks; tiles of 128 rows, for the LDS
// they take).  With two terms (16 bits of p) the sums were 4e-6 from those of
// float32 p, and roundings of the next layer's input that fell the other way
// moved a two-layer result by up to half its own rounding error; with three
// the two agree.
template <int BM, int BN, bool SPLIT>
__global__ __launch_bounds__(kPfThreads, 2) void pf_down_kernel(PfArgs a) {
  constexpr int WM = BM == 256 && BN == 128 ? 4 : 2, WN = 8 / WM;
  constexpr int MT = BM / WM / 16, CT = BN / WN / 16;
  constexpr int NP = SPLIT ? 3 : 1;            // terms of p
  constexpr int IA = BM / 128, IW = BN / 128;  // 1 KB loads per wavefront and stage: a term of p, W_down
  constexpr int SA = BM * 64, SB = SA + BN * 64, SL = SPLIT ? 2 * SA : 16;  // stage bytes; further terms of p apart
  static_assert(!SPLIT || BM == 128, "LDS of a stage");
  constexpr int R = SPLIT ? 4 : SB <= 16 * 1024 ? 8 : SB <= 24 * 1024 ? 6 : 4;
  constexpr int PB = BN * 2, RPL = 1024 / PB;  // W_down tile: bytes per row, rows per load
  __shared__ __attribute__((aligned(1024))) uint8_t rg0[SB], rg1[SB], rg2[SB], rg3[SB],
      rg4[R > 4 ? SB : 16], rg5[R > 4 ? SB : 16], rg6[R > 6 ? SB : 16], rg7[R > 6 ? SB : 16], l0[SL], l1[SL], l2[SL],
      l3[SL];
  auto rb = [&](int i) -> uint8_t * {  // stage buffer i mod R
    i %= R;
    return i == 0 ? rg0 : i == 1 ? rg1 : i == 2 ? rg2 : i == 3 ? rg3 : i == 4 ? rg4 : i == 5 ? rg5 : i == 6 ? rg6 : rg7;
  };
  auto lb = [&](int i) -> uint8_t * { return (i %= R) == 0 ? l0 : i == 1 ? l1 : i == 2 ? l2 : l3; };
  (void)lb;
  int mt0, unit;
  if (!pf_tile(a, mt0, unit)) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const int kc = unit % a.ks, m0 = mt0 * BM, n0 = (unit / a.ks) * BN;
  const int K = a.K, N = a.N;
  const int kb = kc * a.kchunk, ke = min(K, kb + a.kchunk);
  const int S = ke > kb ? (ke - kb + kPfKC - 1) / kPfKC : 0;
  const int wm = w / WN, wn = w % WN;
  const int rows16 = (a.n + 15) / 16, nbp = (K + kPfKC - 1) / kPfKC;
  const uint32_t pbytes = (uint32_t)((size_t)rows16 * nbp * 1024);
  const __amdgpu_buffer_rsrc_t rsw = dense_rsrc(a.Wd, (uint32_t)((size_t)K * N * 2));
  // p: chunk q of each row holds k = 8 q .. of the block; chunks at or past ke are read as zeros
  const int aq = 8 * ((lane & 3) ^ pf_swz(lane >> 2));
  uint32_t aoff[IA], woff[IW];
  const int wr = lane / (PB / 16);  // W_down: row of the lane's piece within the load
#pragma unroll
  for (int q = 0; q < IA; ++q) {
    const int b = m0 / 16 + w + 8 * q;
    aoff[q] = b < rows16 ? ((uint32_t)b * (uint32_t)nbp + (uint32_t)(kb / kPfKC)) * 1024u + 16u * lane : kDenseOffNone;
  }
#pragma unroll
  for (int q = 0; q < IW; ++q) {
    const int r = (w + 8 * q) * RPL + wr, p = lane % (PB / 16), c = n0 + 8 * (((p >> 1) ^ pf_kswz(r)) * 2 + (p & 1));
    woff[q] = c < N ? (uint32_t)(((size_t)(kb + r) * N + c) * 2) : kDenseOffNone;
  }
  auto issue = [&](uint8_t *buf, uint8_t *lo, int s) {
    const int left = ke - kb - s * kPfKC;  // k of the chunk from this step on
#pragma unroll
    for (int q = 0; q < NP * IA; ++q)
      pf_dma(dense_rsrc(a.A + (q / IA) * a.pterm, pbytes),
             (q < IA ? buf : lo + (q / IA - 1) * SA) + (w + 8 * (q % IA)) * 1024,
             aq < left ? aoff[q % IA] : kDenseOffNone, (uint32_t)s * 1024u);
#pragma unroll
    for (int q = 0; q < IW; ++q)
      pf_dma(rsw, buf + SA + (w + 8 * q) * 1024, wr + (w + 8 * q) * RPL < left ? woff[q] : kDenseOffNone,
             (uint32_t)s * (uint32_t)(kPfKC * 2 * N));
  };
  bf16x8 oa[MT], ob0[CT], ob1[CT];  // operands: p, W_down of even and of odd steps
  auto load_a = [&](const uint8_t *buf, int t) { return pf_block_operand(buf + (wm * MT + t) * 1024, l16, g); };
  auto load_b = [&](uint8_t *buf, int t) { return pf_krow_operand(buf + SA, PB, wn * CT + t, g, l16); };
  f32x4v acc[MT][CT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[i][j] = f32x4v{0.f, 0.f, 0.f, 0.f};
  f32x4v sum[SPLIT ? MT : 1][SPLIT ? CT : 1] = {};
#pragma unroll
  for (int s = 0; s < R - 1; ++s) issue(rb(s), lb(s), s);
  constexpr int IS = NP * IA + IW;  // loads of a stage
  pf_barrier<(R - 2) * IS>();
#pragma unroll
  for (int t = 0; t < MT; ++t) oa[t] = load_a(rg0, t);
#pragma unroll
  for (int t = 0; t < CT; ++t) ob0[t] = load_b(rg0, t);
  // (opaque: against a constant offset the compiler sees that the loads of
  // the second term write elsewhere, finds none it knows to write here, and
  // waits for all)
  int third = SA;
  asm volatile("" : "+s"(third));
  // products of the p operands held with xb, each p operand replaced by the
  // one at `nxt` once its last product is issued
  auto prod = [&](const uint8_t *nxt, bf16x8(&xb)[CT], auto reads) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
#pragma unroll
      for (int j = 0; j < CT; ++j) acc[i][j] = mfma16(oa[i], xb[j], acc[i][j]);
      oa[i] = load_a(nxt, i);
    }
#pragma unroll
    for (int i = 0; i < MT * CT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i < reads.value || i % CT == CT - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
  };
  // step s, as in the gate/up kernel (with split p the first two terms' products
  // come before the barrier: they need nothing of stage s + 1)
  auto step = [&](int s, int p, bf16x8(&xb)[CT], bf16x8(&yb)[CT]) {
    if constexpr (SPLIT) {
      prod(lb(p), xb, std::integral_constant<int, 0>{});
      prod(lb(p) + third, xb, std::integral_constant<int, 0>{});
    }
    pf_barrier<(R - 3) * IS>();
    issue(rb(p + R - 1), lb(p + R - 1), s + R - 1);
#pragma unroll
    for (int t = 0; t < CT; ++t) yb[t] = load_b(rb(p + 1), t);
    prod(rb(p + 1), xb, std::integral_constant<int, 2 * CT>{});
  };
  for (int s0 = 0; s0 < S; s0 += R) {
    step(s0, 0, ob0, ob1);
    step(s0 + 1, 1, ob1, ob0);
    step(s0 + 2, 2, ob0, ob1);
    step(s0 + 3, 3, ob1, ob0);
    if constexpr (R > 4) {
      step(s0 + 4, 4, ob0, ob1);
      step(s0 + 5, 5, ob1, ob0);
    }
    if constexpr (R > 6) {
      step(s0 + 6, 6, ob0, ob1);
      step(s0 + 7, 7, ob1, ob0);
    }
    if constexpr (SPLIT) pf_fold(sum, acc);
  }
  __builtin_amdgcn_s_waitcnt(0);
  if constexpr (SPLIT)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) acc[i][j] = sum[i][j];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + (wm * MT + i) * 16 + 4 * g + r;
      if (m >= a.n) continue;
      float *o = a.part + ((size_t)kc * a.n + m) * N + n0 + wn * CT * 16 + l16;
#pragma unroll
      for (int j = 0; j < CT; ++j)
        if (n0 + (wn * CT + j) * 16 + l16 < N) o[16 * j] = acc[i][j][r];
    }
}

// ---------------------------------------------------------------- up to 64 rows

// The same products for at most 16 MT <= 64 rows, for split shapes and for
// float32, where the weights' stream and the latency of a short loop are the
// bound: stages of 128 bytes of each weight row (64 k, float32: 32), every
// wavefront 16 columns of all rows, and enough workgroups to spread short
// matrices over the chip (the tiles of 128 rows above put 7 tokens of a 1024 x
// 2730 layer on 43 workgroups: gate/up 14.8 and down 8.1 us; here 8.2 and
// 5.1, rocprofv3).  Grid: column tiles (times k chunks).  Slots of a stage that nothing
// needs are read as zeros without a memory access.
//
// float32 products are v_mfma_f32_16x16x4_f32, four to a 64-byte block of 16
// k: a lane holds k = 4 g .. 4 g + 3 of its row or column (one 16-byte LDS
// read), and product i takes element i of both operands, so each k meets
// itself.  The compacted kernels they replace form every product on the
// vector units, 4 tokens a tile, and read the weights once a tile (16 tokens
// of a Qwen3-8B layer: 550 us, here 117 to 120: 604 MB at 5.1 TB/s).

// Every stage sums into accumulators of its own, which the next stage adds to
// the total under its products; what each of those additions rounds off is summed
// apart and added at the end (sm_total): only the sums within a stage carry rounding.
// Plain folds of 64 k left float32 results 1.4 times as far from 64 bits as the
// compacted kernels'; these are as near or nearer (1.9e-7 to 2.1e-7 of a layer's
// output, there 2.0e-7 to 3.4e-7).  The total is a plain sum, so an overflow stays
// an infinity; the part rounded off is then meaningless (inf - inf) and left out.
// (Kahan's form, with the compensation in the next addend, takes as many operations,
// but an infinite total turns into NaN; guarded there it cost up to 8 %.)
template <int MT> __device__ __forceinline__ void sm_fold(f32x4v (&sum)[MT], f32x4v (&off)[MT], const f32x4v (&acc)[MT]) {
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const f32x4v t = sum[i] + acc[i];
    off[i] += acc[i] - (t - sum[i]);
    sum[i] = t;
  }
}
template <int MT> __device__ __forceinline__ void sm_total(f32x4v (&sum)[MT], const f32x4v (&off)[MT]) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (fabsf(sum[i][r]) < INFINITY) sum[i][r] += off[i][r];
}

// acc[i] = (first) or += the block product of row tile i (operand x[i]) and b
template <typename T, int MT>
__device__ __forceinline__ void sm_mfma(const u32x4 (&x)[MT], const u32x4 &b, f32x4v (&acc)[MT], bool first) {
  const f32x4v zero = {0.f, 0.f, 0.f, 0.f};
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
      acc[i] = mfma16(__builtin_bit_cast(bf16x8, x[i]), __builtin_bit_cast(bf16x8, b), first ? zero : acc[i]);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < MT; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x[i][e]), __uint_as_float(b[e]),
                                                      first && e == 0 ? zero : acc[i], 0, 0, 0);
  }
}
__device__ __forceinline__ u32x4 sm_block_operand(const uint8_t *blk, int r, int g) {
  return *reinterpret_cast<const u32x4 *>(blk + r * 64 + (g ^ pf_swz(r)) * 16);
}

// Columns [nt b, nt b + nt) of both projections: wavefronts 0-3 W_gate, 4-7 W_up.
// KEPT: the launch also writes a.kept (float32, one row tile: see sm_down_kernel).
template <typename T, int MT, bool KEPT = false>
__global__ __launch_bounds__(kPfThreads, 2) void sm_gateup_kernel(PfArgs a, int nt) {
  static_assert(!KEPT || (sizeof(T) == 4 && MT == 1), "16 flags per tile");
  constexpr int SW = 16 * 1024, SB = SW + 8 * 1024, R = 6;  // W_gate and W_up 8 KB each, h
  __shared__ __attribute__((aligned(1024))) uint8_t rg0[SB], rg1[SB], rg2[SB], rg3[SB], rg4[SB], rg5[SB];
  auto rb = [&](int i) -> uint8_t * {
    return (i %= R) == 0 ? rg0 : i == 1 ? rg1 : i == 2 ? rg2 : i == 3 ? rg3 : i == 4 ? rg4 : rg5;
  };
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15, mat = w >> 2, ct = w & 3;
  const int K = a.K, N = a.N, n0 = blockIdx.x * nt;
  constexpr int E = sizeof(T), KB = 64 / E;  // bytes of an element, k of a block
  const int nb = (K + KB - 1) / KB, S = (nb + 1) / 2;
  const int rid = route_id(a.route_mode, a.ids, a.n, lane);  // of row `lane`
  const int rows16 = (a.n + 15) / 16;
  const uint32_t wbytes = (uint32_t)((size_t)N * K * E);
  const __amdgpu_buffer_rsrc_t rsg = dense_rsrc(a.Wg, wbytes), rsu = dense_rsrc(a.Wu, wbytes);
  // wavefront w: rows 8 w .. 8 w + 7 of each projection, and block w & 1 of row tile w / 2 of h
  const int lr = lane >> 3, lq = (lane & 7) ^ lr, row = 8 * w + lr;
  const uint32_t woff = row < nt && n0 + row < N ? (uint32_t)((size_t)(n0 + row) * K * E + 16 * lq) : kDenseOffNone;
  // (the call input is read as it is, a row's 64 bytes by four lanes, into the same LDS layout)
  const bool direct = a.x != nullptr;
  const int am = w / 2 * 16 + (lane >> 2), ak = 64 * (w & 1) + 16 * ((lane & 3) ^ pf_swz(lane >> 2));
  // (24-bit products and selects, no branch: a 64-bit multiply-add in a branch here took the
  // register that the id's load was still writing, and so waited for it before the first stage)
  const uint32_t adir = __umul24((uint32_t)am, (uint32_t)(K * E)) + (uint32_t)ak;
  const uint32_t ablk = (__umul24((uint32_t)(w / 2), (uint32_t)nb) + (uint32_t)(w & 1)) * 1024u + 16u * lane;
  const uint32_t aoff = (w / 2 < MT) & (am < a.n) ? (direct ? adir : ablk) : kDenseOffNone;
  const uint32_t astep = direct ? 128u : 2048u;
  const __amdgpu_buffer_rsrc_t rsa = dense_rsrc(direct ? (const void *)a.x : (const void *)a.A,
                                                direct ? (uint32_t)(a.n * K * E) : (uint32_t)(rows16 * nb * 1024));
  auto issue = [&](uint8_t *buf, int s) {
    const bool v = 128 * s + 16 * lq < K * E;
    pf_dma(rsg, buf + w * 1024, v ? woff : kDenseOffNone, (uint32_t)s * 128u);
    pf_dma(rsu, buf + 8192 + w * 1024, v ? woff : kDenseOffNone, (uint32_t)s * 128u);
    pf_dma(rsa, buf + SW + w * 1024, 128 * s + ak < K * E ? aoff : kDenseOffNone, (uint32_t)s * astep);
  };
  u32x4 oa0[2][MT], oa1[2][MT], ob0[2], ob1[2];  // operands of even and odd stages
  auto load = [&](const uint8_t *buf, u32x4(&xa)[2][MT], u32x4(&xb)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 16 * ct + l16;
      xb[h] = *reinterpret_cast<const u32x4 *>(buf + mat * 8192 + r * 128 + ((4 * h + g) ^ (r & 7)) * 16);
#pragma unroll
      for (int i = 0; i < MT; ++i) xa[h][i] = sm_block_operand(buf + SW + (2 * i + h) * 1024, l16, g);
    }
  };
  f32x4v acc0[MT] = {}, acc1[MT] = {}, sum[MT] = {}, off[MT] = {};  // stage sums (even, odd); total
#pragma unroll
  for (int s = 0; s < R - 1; ++s) issue(rb(s), s);
  const int rflag = route_flag(a.route_mode, a.lut, rid);
  pf_barrier<(R - 2) * 3 + 1>();
  load(rg0, oa0, ob0);
  // stage s: stage s + 1 has landed, every wavefront holds the operands of stage s
  auto step = [&](int s, int p, u32x4(&xa)[2][MT], u32x4(&xb)[2], u32x4(&ya)[2][MT], u32x4(&yb)[2],
                  f32x4v(&cur)[MT], const f32x4v(&prv)[MT]) {
    pf_barrier<(R - 3) * 3>();
    issue(rb(p + R - 1), s + R - 1);
    load(rb(p + 1), ya, yb);
#pragma unroll
    for (int h = 0; h < 2; ++h) sm_mfma<T, MT>(xa[h], xb[h], cur, h == 0);
    sm_fold(sum, off, prv);
    __builtin_amdgcn_sched_barrier(0);  // (the next step's reads stay there: registers)
  };
  for (int s0 = 0; s0 < S; s0 += R) {
    step(s0, 0, oa0, ob0, oa1, ob1, acc0, acc1);
    step(s0 + 1, 1, oa1, ob1, oa0, ob0, acc1, acc0);
    step(s0 + 2, 2, oa0, ob0, oa1, ob1, acc0, acc1);
    step(s0 + 3, 3, oa1, ob1, oa0, ob0, acc1, acc0);
    step(s0 + 4, 4, oa0, ob0, oa1, ob1, acc0, acc1);
    step(s0 + 5, 5, oa1, ob1, oa0, ob0, acc1, acc0);
  }
  sm_fold(sum, off, acc1);  // (rounds end on an odd stage)
  sm_total(sum, off);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // epilogue: SiLU lane to lane to the wavefront of W_up, p through LDS to 16-byte stores of its terms
  uint8_t *xt = rg0 + ct * MT * 1024;
  if (mat == 0) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      f32x4v v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = silu(sum[i][r]);
      reinterpret_cast<f32x4v *>(xt)[i * 64 + lane] = v;
    }
  }
  __syncthreads();
  if (mat == 0 || 16 * ct >= nt) return;
  const float thr = a.thr ? *a.thr : 0.0f;
  const int flag = a.route_mode == ROUTE_BASE || rflag != 0;
  const int c0 = n0 + 16 * ct;
  bool any = false;  // KEPT: some row keeps column c0 + l16
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const f32x4v gv = reinterpret_cast<const f32x4v *>(xt)[i * 64 + lane];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 16 * i + 4 * g + r, c = c0 + l16;
      const bool keep = __shfl(flag, m, 64) || fabsf(gv[r]) >= thr;
      if constexpr (KEPT) any = any || (keep && m < a.n);
      *reinterpret_cast<float *>(xt + i * 1024 + (4 * g + r) * 64 + l16 * 4) = keep ? gv[r] * sum[i][r] : 0.0f;
      if (a.keep_out && m < a.n && c < N) a.keep_out[(size_t)m * N + c] = (uint8_t)keep;
    }
  }
  if constexpr (E == 4) {  // a tile is a row block: lane's row and 4 columns
    if constexpr (KEPT) {
      uint64_t b = __ballot(any);
      b |= b >> 32;
      b |= b >> 16;
      if (lane == 0 && c0 < N) a.kept[c0 >> 4] = (uint16_t)b;
    }
    const int r = lane >> 2, q = lane & 3, nbp = (N + 15) / 16;
#pragma unroll
    for (int i = 0; i < MT; ++i)
      if (16 * i + r < a.n && c0 + 4 * q < N)
        *reinterpret_cast<u32x4 *>(reinterpret_cast<uint8_t *>(a.P) + ((size_t)i * nbp + (c0 >> 4)) * 1024 + r * 64 +
                                   (q ^ pf_swz(r)) * 16) =
            *reinterpret_cast<const u32x4 *>(xt + i * 1024 + r * 64 + q * 16);
  } else {
    // lane: row, half of the tile's columns (8), and one of two row tiles
    const int nbp = (N + kPfKC - 1) / kPfKC;
#pragma unroll
    for (int i0 = 0; i0 < MT; i0 += 2) {
      const int i = i0 + (lane & 1), r = lane >> 2, q = (lane >> 1) & 1, m = 16 * i + r, c = c0 + 8 * q;
      if (i >= MT || m >= a.n || c >= N) continue;
      float v[8];
      *reinterpret_cast<f32x4v *>(v) = *reinterpret_cast<const f32x4v *>(xt + i * 1024 + r * 64 + q * 32);
      *reinterpret_cast<f32x4v *>(v + 4) = *reinterpret_cast<const f32x4v *>(xt + i * 1024 + r * 64 + q * 32 + 16);
      pf_store_terms(a.P + ((size_t)i * nbp + (c >> 5)) * 512 + r * 32 + (((c >> 3) & 3) ^ pf_swz(r)) * 8, a.pterm, v);
    }
  }
}

typedef const __attribute__((address_space(4))) uint32_t *ConstWords;  // not written during the kernel

// 128 columns of one k chunk: wavefront w columns 16 w .. 16 w + 15.  A stage
// holds 16 KB of W_down (64 rows, float32: 32) and the blocks of p of its k:
// three terms of two blocks per row tile (float32: one).
//
// FLAGS: W_down rows that no row of the batch keeps are not read (as in
// dense_down_kernel and the compacted kernels) but for the first two stages,
// which are on their way while the flags come.  A stage's rows are one word of
// flags, loaded a round of R stages ahead.
template <typename T, int MT, bool FLAGS = false>
__global__ __launch_bounds__(kPfThreads, 2) void sm_down_kernel(PfArgs a) {
  static_assert(!FLAGS || sizeof(T) == 4, "a word of flags per stage of 32 rows");
  constexpr int E = sizeof(T), KB = 64 / E, KS = 2 * KB, NP = E == 2 ? 3 : 1;  // k of a block and a stage; terms of p
  constexpr int IP = (2 * NP * MT + 7) / 8;                  // loads of p per wavefront and stage (2 NP MT KB)
  constexpr int SW = 16 * 1024, SB = SW + IP * 8 * 1024, R = SB <= 24 * 1024 ? 6 : 4, IS = 2 + IP;
  constexpr int RPL = 1024 / (128 * E);                      // rows of W_down per load
  __shared__ __attribute__((aligned(1024))) uint8_t rg0[SB], rg1[SB], rg2[SB], rg3[SB], rg4[R > 4 ? SB : 16],
      rg5[R > 4 ? SB : 16];
  auto rb = [&](int i) -> uint8_t * {
    return (i %= R) == 0 ? rg0 : i == 1 ? rg1 : i == 2 ? rg2 : i == 3 ? rg3 : i == 4 ? rg4 : rg5;
  };
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const int K = a.K, N = a.N, kc = blockIdx.x % a.ks, n0 = blockIdx.x / a.ks * 128;
  const int kb = kc * a.kchunk, ke = min(K, kb + a.kchunk);
  const int S = ke > kb ? (ke - kb + KS - 1) / KS : 0;
  const int rows16 = (a.n + 15) / 16, nbp = (K + KB - 1) / KB;
  const __amdgpu_buffer_rsrc_t rsw = dense_rsrc(a.Wd, (uint32_t)((size_t)K * N * E));
  const uint32_t pbytes = (uint32_t)(rows16 * nbp * 1024);
  // W_down: load q of wavefront w is rows RPL (w + 8 q) .. of the stage, 128 columns each.
  // bf16: the pair of chunks of 16 columns swizzled by pf_kswz; float32: the 64 bytes of
  // 16 columns by the row's group of four, so that the four rows a wavefront's 4-byte
  // LDS read takes (k = i, 4 + i, ..) fall in distinct banks
  const int wr = RPL * w + lane / (64 / RPL), wp = lane % (64 / RPL);
  uint32_t woff[2], aoff[IP];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = wr + 8 * RPL * q;
    const int c = n0 + (E == 2 ? 8 * (((wp >> 1) ^ pf_kswz(r)) * 2 + (wp & 1)) : 16 * ((wp >> 2) ^ ((r >> 2) & 3)) + 4 * (wp & 3));
    woff[q] = c < N ? (uint32_t)(((size_t)(kb + r) * N + c) * E) : kDenseOffNone;
  }
  // p: load i = w + 8 q is term i / (2 MT), row tile (i / 2) % MT, block i & 1 of the stage
  const int aq = 16 / E * ((lane & 3) ^ pf_swz(lane >> 2)) + KB * (w & 1);
#pragma unroll
  for (int q = 0; q < IP; ++q) {
    const int i = w + 8 * q, t = i / 2 % MT;
    aoff[q] = i < 2 * NP * MT && t < rows16 ? (uint32_t)((t * nbp + kb / KB + (i & 1)) * 1024 + 16 * lane) : kDenseOffNone;
  }
  // flags of the rows of stages s .. s + R - 1 (scalar loads, which the waits for the
  // stages' loads do not count; those past the last column are not looked at: `left`)
  const ConstWords fw = (ConstWords)(uintptr_t)a.kept + kb / KS;
  auto flags = [&](uint32_t(&f)[FLAGS ? R : 1], int s) {
    if constexpr (FLAGS)
#pragma unroll
      for (int i = 0; i < R; ++i) f[i] = fw[s + i];
  };
  auto issue = [&](uint8_t *buf, int s, uint32_t f) {
    const int left = ke - kb - KS * s;
#pragma unroll
    for (int q = 0; q < 2; ++q)
      pf_dma(rsw, buf + (w + 8 * q) * 1024,
             wr + 8 * RPL * q < left && (!FLAGS || (f >> (wr + 8 * RPL * q & 31) & 1u)) ? woff[q] : kDenseOffNone,
             (uint32_t)s * (uint32_t)(KS * E * N));
#pragma unroll
    for (int q = 0; q < IP; ++q)
      pf_dma(dense_rsrc(a.A + min((w + 8 * q) / (2 * MT), NP - 1) * a.pterm, pbytes), buf + SW + (w + 8 * q) * 1024,
             aq < left ? aoff[q] : kDenseOffNone, (uint32_t)s * 2048u);
  };
  f32x4v acc0[MT] = {}, acc1[MT] = {}, sum[MT] = {}, off[MT] = {};  // stage sums (even, odd); total
#pragma unroll
  for (int s = 0; s < 2; ++s) issue(rb(s), s, ~0u);
  uint32_t fl[FLAGS ? R : 1], fn[FLAGS ? R : 1];  // of the stages that this round and the next one load
  flags(fn, 0);
#pragma unroll
  for (int s = 2; s < R - 1; ++s) issue(rb(s), s, FLAGS ? fn[FLAGS ? s : 0] : ~0u);
  flags(fl, R - 1);
  // (operands read where they are used: a chunk has few stages)
  auto step = [&](int s, int p, f32x4v(&cur)[MT], const f32x4v(&prv)[MT]) {
    pf_barrier<(R - 2) * IS>();
    issue(rb(p + R - 1), s + R - 1, FLAGS ? fl[FLAGS ? p : 0] : ~0u);
    uint8_t *buf = rb(p);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 b;
      if constexpr (E == 2) {
        b = __builtin_bit_cast(u32x4, pf_krow_operand(buf + h * 8192, 256, w, g, l16));
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          b[i] = *reinterpret_cast<const uint32_t *>(buf + (16 * h + 4 * g + i) * 512 + (w ^ g) * 64 + l16 * 4);
      }
#pragma unroll
      for (int t = 0; t < NP; ++t) {
        u32x4 x[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) x[i] = sm_block_operand(buf + SW + ((t * MT + i) * 2 + h) * 1024, l16, g);
        sm_mfma<T, MT>(x, b, cur, h == 0 && t == 0);
      }
    }
    sm_fold(sum, off, prv);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int s0 = 0; s0 < S; s0 += R) {
    flags(fn, s0 + 2 * R - 1);
    step(s0, 0, acc0, acc1);
    step(s0 + 1, 1, acc1, acc0);
    step(s0 + 2, 2, acc0, acc1);
    step(s0 + 3, 3, acc1, acc0);
    if constexpr (R > 4) {
      step(s0 + 4, 4, acc0, acc1);
      step(s0 + 5, 5, acc1, acc0);
    }
    if constexpr (FLAGS)
#pragma unroll
      for (int i = 0; i < R; ++i) fl[i] = fn[i];
  }
  sm_fold(sum, off, acc1);  // (rounds end on an odd stage)
  sm_total(sum, off);
  __builtin_amdgcn_s_waitcnt(0);
  const int c = n0 + 16 * w + l16;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 16 * i + 4 * g + r;
      if (m < a.n && c < N) a.part[((size_t)kc * a.n + m) * N + c] = sum[i][r];
    }
}

}  // namespace sats
