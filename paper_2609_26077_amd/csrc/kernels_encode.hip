// Fused operand combine + block quantization (the encoder of Assumption 1).
//
// One workgroup owns a tile of TR "rows" x TL contracted positions of the
// sub-block grid (TL = 128, or 64 / 32 for the B side's narrow tiles at
// depths 2 / 3) and produces the codes and scales of every flattened term
// for that tile.  A rows are rows of A's sub-blocks; B rows are columns of
// B's sub-blocks, so both outputs have the contracted axis last.
//
//   1. stage: the tile of all 4^l sub-blocks is read from HBM (coalesced)
//      into LDS as fp32, laid out [block][row][l] with the contracted axis
//      contiguous (the B side transposes on the way in);
//   2. combine: every lane of a wave works on one term (the term's nonzero
//      coefficients sit in scalar registers) and forms x = sum_b c_b a_b over
//      them in ascending b, as separate fp32 multiplies and adds, for a run of
//      consecutive contracted positions of one row: 16 at depths 1 and 2
//      (one 16-byte store of codes), 4 at depth 3 (whose 64 sub-blocks leave
//      no room in LDS for rows enough to fill a wave with 16-position runs);
//   3. quantize: the block maximum over `block` consecutive positions is
//      reduced across the lanes that hold it, the rule gives the scale, and
//      the lane casts its values and stores their codes.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.h"
#include "internal.h"

namespace fmm {

namespace {

// One operand side's coefficient tables: the nonzero entries of every term in
// ascending block order (offsets, entries; read at depth 1) and the dense
// flattened rows, T x 4^l fp32 with zeros (read at depths 2 and 3, and at depth 1
// by the weight-block encoder).
struct SideTab {
  const int32_t *off;
  const CoefEntry *ent;
  const float *dense;
  EncodePattern pat;     // depth 3
};
inline SideTab a_tab(const DeviceTables &t) { return {t.a_off, t.a_ent, t.u_dense, t.u_pat}; }
inline SideTab b_tab(const DeviceTables &t) { return {t.b_off, t.b_ent, t.v_dense, t.v_pat}; }

// The coefficient of block b of a dense row spread one block per lane (b uniform).
__device__ __forceinline__ float lane_coef(float c, int b) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c), b));
}

// Takes the lowest set bit of a uniform mask (the next nonzero block in
// ascending order) or, once the mask is empty, repeats `prev`.
__device__ __forceinline__ int next_block(uint64_t &mask, int prev) {
  if (mask == 0) return prev;
  const int b = __builtin_ctzll(mask);
  mask &= mask - 1;
  return b;
}

constexpr int kTL = 128;            // contracted positions per tile (>= every block size)
constexpr int kStride = kTL + 4;    // LDS row stride in floats: 33 16-byte slots, odd, so
                                    // 16-byte accesses of 16 lanes in 4 consecutive rows x
                                    // 4 slots, or in 16 consecutive rows, hit 16 distinct
                                    // bank groups

// Tile geometry.  VEC = contracted positions per lane (16 at depths 1-2, 4 at
// depth 3).  At depth 1 the B side takes 32 columns (its rows of B are read as
// 128-byte segments) with eight waves (two terms at once), the A side 8 rows
// with two waves that
// split the terms between them (8-row tiles leave room for more workgroups
// per CU than 16-row ones and measured 5-7% faster).  The
// NARROW form (depth 2, B side, blocks of 16 and 32) takes 16 columns x 64
// positions instead of 8 x 128, so B's rows are read as 64-byte segments
// rather than 32-byte ones and a wave writes whole 64-byte code runs.
constexpr int kA1Rows = 8, kA1Threads = 128;   // depth-1 A-side tile rows and threads
constexpr int kB1Rows = 32, kB1Threads = 512;  // depth-1 B-side tile rows (columns of B) and threads
constexpr int kB1NThreads = 256;                // threads of its narrow (64-position) form
constexpr int kB3Rows = 8;          // depth-3 B-side tile rows (columns of B), 32 positions each, at blocks <= 32

// CAP: a realization of another shape, staged as up to CAP blocks of a grid
// known at run time (0: the 2^l x 2^l grid of <2,2,2> at depth l).
template <int DEPTH, int VEC, int SIDE, bool NARROW = false, int CAP = 0>
struct Tile {
  static constexpr int nblk = CAP ? CAP : 1 << (2 * DEPTH);
  static constexpr int TL = NARROW ? (DEPTH == 3 ? 256 / kB3Rows : 64) : kTL;   // contracted positions per tile
  static constexpr int stride = TL + 4;                   // LDS row stride in floats (an odd number of 16-byte slots)
  static constexpr int TR = NARROW ? (DEPTH == 3 ? kB3Rows : DEPTH == 1 ? kB1Rows : 16) : VEC == 16 ? (DEPTH == 1 ? (SIDE == 1 ? kB1Rows : kA1Rows) : 8) : (DEPTH == 3 ? 2 : 64 / nblk);
  // depth 1: 128 (A) or 512 (B) threads; depths 2 and 3 deal the terms out to
  // sixteen waves, which with two workgroups per CU keeps eight waves per SIMD
  static constexpr int threads = DEPTH == 1 ? (SIDE == 0 ? kA1Threads : NARROW ? kB1NThreads : kB1Threads) : 1024;
  static constexpr int lds_floats = nblk * TR * stride;   // 33.8 (A) / 67.6 (B; 34.8 narrow), 67.6 (69.6 narrow), 67.6 KB
  static_assert(lds_floats * 4 <= 160 * 1024, "the tile fits in LDS");
  static_assert(!NARROW || (DEPTH <= 2 && SIDE == 1 && VEC == 16) || (DEPTH == 3 && SIDE == 1 && VEC == 4),
                "the narrow tiles are B sides'");
};

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
// The same permutation of a 32-bit pattern.  Maxima of non-negative finite
// floats are taken on their bit patterns, which order like the unsigned
// integers: one unsigned maximum with the permutation folded in per step.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// Read the tile into LDS ([block][row][l], row stride TL + 4 floats).  Every
// load is issued before the first LDS write, so the workgroup waits for HBM
// once, not once per element.  The fp32 operands are read exactly once, so
// the loads are nontemporal (they do not displace the codes, which the
// sub-product kernel reads next, from the caches), except where a tile takes
// only part of each cache line (B tiles narrower than 32 columns).  Positions
// outside the operand read as zero.
// GEN: a realization of another shape, whose A grid is gm x gk and B grid
// gk x gn (at most NB blocks; the others are neither read nor used).
typedef float f4v __attribute__((ext_vector_type(4)));

template <int SIDE, int NB, int TR, int NT, int TL = kTL, bool GEN = false>
__device__ __forceinline__ void stage_tile(float *lds, const float *__restrict__ src, const Problem &pb,
                                           int64_t bt, int64_t row0, int64_t l0, int t) {
  constexpr int nc = NB == 4 ? 2 : NB == 16 ? 4 : 8;
  // blocks per grid row (A: gk columns of A's grid; B: gn) and blocks in all
  const int n = GEN ? (SIDE == 0 ? pb.gk : pb.gn) : nc;
  const int nbr = GEN ? (SIDE == 0 ? pb.gm * pb.gk : pb.gk * pb.gn) : NB;
  constexpr int kStr = TL + 4;
  constexpr int kPer = NB * TR * (TL / 4) / NT;       // float4s per thread
  static_assert(NB * TR * (TL / 4) % NT == 0, "the tile splits evenly over the threads");
  const int64_t rows = SIDE == 0 ? pb.mp : pb.np;
  const int64_t kp = pb.kp;
  float4 stage[kPer];
  if (SIDE == 0) {
    // A (M x K): block b = I n + J holds rows I m' + p, columns J k' + l.
    const float *Ab = src + bt * pb.M * pb.K;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int e = t + NT * k;
      const int b = e / (TR * (TL / 4));
      const int rem = e % (TR * (TL / 4));
      const int64_t p = row0 + rem / (TL / 4), l = l0 + 4 * (rem % (TL / 4));
      stage[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      if ((!GEN || b < nbr) && p < rows && l < kp) {
        const int I = b / n, J = b % n;
        const f4v x = __builtin_nontemporal_load(reinterpret_cast<const f4v *>(Ab + (I * pb.mp + p) * pb.K + J * kp + l));
        stage[k] = make_float4(x.x, x.y, x.z, x.w);
      }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int e = t + NT * k;
      const int b = e / (TR * (TL / 4));
      const int rem = e % (TR * (TL / 4));
      *reinterpret_cast<float4 *>(lds + (b * TR + rem / (TL / 4)) * kStr + 4 * (rem % (TL / 4))) = stage[k];
    }
  } else {
    // B (K x N): block b = J n + K holds rows J k' + l, columns K n' + q;
    // lanes run along q so each of the four loads is coalesced.
    const float *Bb = src + bt * pb.K * pb.N;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int e = t + NT * k;
      const int b = e / (TR * (TL / 4));
      const int rem = e % (TR * (TL / 4));
      const int64_t qq = row0 + rem % TR, l = l0 + 4 * (rem / TR);
      stage[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      if ((!GEN || b < nbr) && qq < rows && l < kp) {
        const int J = b / n, Kb = b % n;
        const float *p = Bb + (J * kp + l) * pb.N + Kb * pb.np + qq;
        if constexpr (TR < 32) {
          // tiles narrower than 32 columns read each 128-byte line of B in
          // parts, the rest by the tiles of the neighbouring columns, which
          // run at the same time on the same XCD: keep the lines in L2
          stage[k].x = p[0];
          stage[k].y = p[pb.N];
          stage[k].z = p[2 * pb.N];
          stage[k].w = p[3 * pb.N];
        } else {
          stage[k].x = __builtin_nontemporal_load(p);
          stage[k].y = __builtin_nontemporal_load(p + pb.N);
          stage[k].z = __builtin_nontemporal_load(p + 2 * pb.N);
          stage[k].w = __builtin_nontemporal_load(p + 3 * pb.N);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int e = t + NT * k;
      const int b = e / (TR * (TL / 4));
      const int rem = e % (TR * (TL / 4));
      *reinterpret_cast<float4 *>(lds + (b * TR + rem % TR) * kStr + 4 * (rem / TR)) = stage[k];
    }
  }
}

// Where the results of a run of positions starting at (p, l) go inside one
// term's plane (the same for every term, so computed once per lane):
//   codes : row-major p k' + l, or (large-tile plans) the 256-row x 64-byte
//           tile image, chunk c of tile row t at c ^ ((t >> 2) & 3)
//   scales: row-major p kblocks + kb, or (large-tile plans) K-block-major,
//           E8M0 bytes with rows permuted inside each 256-row tile (row
//           128 wm + 32 i + r at byte 4 (32 wm + r) + i of the tile), fp32
//           values in row order
//   128 x 128 tiles: codes as the 128-row x 128-byte tile image (chunk c of
//           tile row t at c ^ (t & 7) ^ ((t >> 3) & 1)); scales 4 bytes per
//           tile row and 128-byte step (blocks 0, 2, 1, 3 at block 32; the
//           one block repeated at block 128), 8 at block 16 (blocks 0, 2, 4,
//           6, then 1, 3, 5, 7)
// `lead`: this run starts its block (its lane stores the block's scale).
struct Out {
  int64_t code, scale;
  bool valid, leader;
};
__device__ __forceinline__ Out out_of(const Problem &pb, int64_t rows, int64_t p, int64_t l, bool lead) {
  Out o;
  const int64_t kp = pb.kp;
  o.valid = p < rows && l < kp;
  o.leader = o.valid && lead;
  const int64_t kb = l / pb.block;
  if (pb.layout == FMM_LAYOUT_TILE256x64) {
    const int64_t t = p & 255, c = (l >> 4) & 3;
    o.code = ((((p >> 8) * (kp >> 6) + (l >> 6)) << 14) + t * 64 + 16 * (c ^ ((t >> 2) & 3)) + (l & 15));
    o.scale = kb * rows + (pb.scale_bytes == 4 ? p : ((p & ~int64_t(255)) | ((((p >> 7) & 1) * 32 + (p & 31)) * 4 + ((p >> 5) & 3))));
  } else if (pb.layout == FMM_LAYOUT_TILE128x128) {
    const int64_t t = p & 127, c = (l >> 4) & 7, tile = (p >> 7) * (kp >> 7) + (l >> 7);
    o.code = (tile << 14) + t * 128 + 16 * (c ^ (t & 7) ^ ((t >> 3) & 1)) + (l & 15);
    if (pb.block == 16) {
      const int64_t b = (l >> 4) & 7;                      // block of the step
      o.scale = tile * 1024 + t * 8 + 4 * (b & 1) + (b >> 1);
    } else {
      const int64_t kq = (l >> 5) & 3;                     // block of the step (block 32)
      o.scale = tile * 512 + t * 4 + (pb.block == 32 ? ((kq & 1) << 1) | (kq >> 1) : 0);
    }
  } else {
    o.code = p * kp + l;
    o.scale = p * pb.kblocks + kb;
  }
  return o;
}

// elements of scales per (batch, term) plane (the 128 x 128 layout keeps 4
// bytes per row and step, 8 at block 16)
__device__ __forceinline__ int64_t scale_plane_of(const Problem &pb, int64_t rows) {
  return pb.layout == FMM_LAYOUT_TILE128x128 ? rows * (pb.kp / 128) * (pb.block == 16 ? 8 : 4)
                                              : rows * pb.kblocks;
}

__device__ __forceinline__ void store_scale(const Problem &pb, uint8_t *scales, int64_t at, uint32_t stored) {
  if (pb.scale_bytes == 4)
    reinterpret_cast<uint32_t *>(scales)[at] = stored;
  else if (pb.layout == FMM_LAYOUT_TILE128x128 && pb.block == 128)
    *reinterpret_cast<uint32_t *>(scales + at) = stored * 0x01010101u;
  else
    scales[at] = (uint8_t)stored;
}

// ---------------------------------------------------------------------------
// Depths 1 and 2: 16 positions per lane.
//
// A wave covers 8 rows x 128 positions of one term: lane = 32 h + 4 r + c'
// holds row r, positions 16 (4 h + c') .. +15, so a 16-lane group reads 4
// rows x 4 slots (conflict-free at the odd stride) and a block of 32 is a lane
// pair (lane, lane ^ 1), a block of 128 the quad plus its partner 32 lanes on
// (the narrow tiles: 16 rows x 64 positions, lane = 4 r + c').  The waves that
// cover a tile's rows work on one term and the workgroup's wave groups take
// the terms in turn: depth 1 A 8 rows (one wave per term, two terms at once),
// B 32 rows (four waves per term, two terms at once); depth 2 one wave per
// term, sixteen terms at once.
// ---------------------------------------------------------------------------
// MODE 0 is the plain encoder.
// MODE 2 (FMM_FLAG_B_BF16 without FMM_FLAG_B_BLOCK128, B side at depth 1) rounds
// the combinations to bfloat16 first.
// MODE 3 measures the operand-side rounding energy of an encoding already in
// the workspace (Appendix D, eq. D.1): it forms x_r exactly as the encoder
// does, decodes the stored codes and scales to xhat_r (exact in binary64),
// and writes each wave's sum of (xhat - x)^2 and of x^2 per term to
// aux[((bt * tiles + tile) * waves + wave) * T + r][2] (binary64, lanes summed
// in a fixed butterfly order).
__device__ __forceinline__ float bf16_round(float x) {
  // nearest bfloat16, ties to even (finite x; a carry past the largest
  // finite value gives infinity, as the definition does)
  uint32_t b = __float_as_uint(x);
  b += 0x7fffu + ((b >> 16) & 1u);
  return __uint_as_float(b & 0xffff0000u);
}

// The plain depth-2 B-side encoder at blocks of 16 and 32 takes the narrow tile.
constexpr bool narrow_b(int side, int depth, int bs, int mode) {
  return side == 1 && depth == 2 && bs <= 32 && mode == 0;
}

// The work of one workgroup of NT threads: tile bx of nbx (of product bt) of one side.
template <int SIDE, int DEPTH, int BS, bool F32, int MODE, int CAP, bool N1, int NT>
__device__ __forceinline__ void encode16_tile(float *lds, const float *__restrict__ src, const Problem &pb, const SideTab &cf,
                                              uint8_t *__restrict__ codes, uint8_t *__restrict__ scales, int64_t tiles_l,
                                              void *__restrict__ aux, unsigned bx, unsigned nbx, int64_t bt) {
  static_assert(MODE == 0 || MODE == 3 || (MODE == 2 && SIDE == 1 && DEPTH == 1), "bfloat16 combinations: B side, depth 1");
  static_assert(CAP == 0 || (MODE == 0 && (DEPTH == 1 || CAP == 16)), "other shapes: the plain encoder");
  constexpr bool GEN = CAP != 0;
  using TT = Tile<DEPTH, 16, SIDE, narrow_b(SIDE, DEPTH, BS, MODE) || N1, CAP>;
  constexpr int TR = TT::TR, NB = TT::nblk, TL = TT::TL, STR = TT::stride;
  constexpr int RPW = 64 * 16 / TL;         // rows per wave: 8, or 16 in the narrow tile
  constexpr int WPT = TR / RPW;             // waves per term (1 (A), 4 (B) or 2 (narrow B) at depth 1, 1 at depth 2)
  constexpr int TSTEP = NT / 64 / WPT;      // terms a workgroup works on at once

  const int t = threadIdx.x;
  // depth-1 B side: the column tile varies fastest over the workgroups, so
  // neighbouring workgroups read adjacent 128-byte pieces of the same rows of
  // B at about the same time (the narrower tiles of depths 2 and 3 instead
  // rely on the neighbouring columns' tile running on the same XCD)
  const int64_t tiles_r = nbx / tiles_l;
  constexpr bool qfast = SIDE == 1 && DEPTH == 1 && MODE != 3;
  const int64_t row0 = (qfast ? bx % tiles_r : bx / tiles_l) * TR;
  const int64_t l0 = (qfast ? bx / tiles_r : bx % tiles_l) * TL;
  const int64_t rows = SIDE == 0 ? pb.mp : pb.np;
  stage_tile<SIDE, NB, TR, NT, TL, GEN>(lds, src, pb, bt, row0, l0, t);
  __syncthreads();

  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // 16-position run of the row and the row: lane = 32 h + 4 r + c' (run 4 h + c'),
  // or in the narrow tile lane = 4 r + c' (run c')
  const int ch = TL == 64 ? (lane & 3) : ((lane >> 5) << 2) | (lane & 3);
  const int row = RPW * (wave % WPT) + (TL == 64 ? (lane >> 2) : ((lane >> 2) & 7));
  const float *lrow = lds + row * STR + 16 * ch;
  const bool lead = BS == 16 ? true : BS == 32 ? (ch & 1) == 0 : ch == 0;
  const Out o = out_of(pb, rows, row0 + row, l0 + 16 * ch, lead);
  const int64_t code_plane = rows * pb.kp;
  const int64_t scale_plane = scale_plane_of(pb, rows);
  const int64_t T = pb.T;

  // depth 2: the term's dense coefficient row (block b in lane b) is loaded
  // one term ahead by a vector load, so the term loop never waits on scalar
  // memory; its nonzero blocks come from the wave's ballot in ascending order
  float cnext = 0.0f;
  if constexpr (DEPTH >= 2) {
    const int64_t rf = wave / WPT;
    if (rf < T && lane < NB) cnext = cf.dense[rf * NB + lane];
  }
  for (int64_t r = wave / WPT; r < T; r += TSTEP) {
    // x = sum_b c_b a_b in ascending b: products and sums rounded separately
    float x[16];
    if constexpr (DEPTH >= 2) {
      const float c = cnext;
      if (r + TSTEP < T && lane < NB) cnext = cf.dense[(r + TSTEP) * NB + lane];
      uint64_t mask = __ballot(c != 0.0f);
      if (mask == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = 0.0f;
      }
      bool first = true;
      while (mask != 0) {
        // two blocks per pass (the second repeats the first when there is none)
        const int b0 = next_block(mask, 0);
        const bool two = mask != 0;
        const int b1 = next_block(mask, b0);
        const float4 *p0 = reinterpret_cast<const float4 *>(lrow + b0 * (TR * STR));
        const float4 *p1 = reinterpret_cast<const float4 *>(lrow + b1 * (TR * STR));
        const float4 v[8] = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
        const float c0 = lane_coef(c, b0), c1 = lane_coef(c, b1);
        const float *a = reinterpret_cast<const float *>(v);
        if (first) {
#pragma unroll
          for (int i = 0; i < 16; ++i) x[i] = __fmul_rn(c0, a[i]);
        } else {
#pragma unroll
          for (int i = 0; i < 16; ++i) x[i] = __fadd_rn(x[i], __fmul_rn(c0, a[i]));
        }
        first = false;
        if (two) {
#pragma unroll
          for (int i = 0; i < 16; ++i) x[i] = __fadd_rn(x[i], __fmul_rn(c1, a[16 + i]));
        }
      }
    } else {
      const int beg = __builtin_amdgcn_readfirstlane(cf.off[r]);
      const int nc = __builtin_amdgcn_readfirstlane(cf.off[r + 1]) - beg;
      CoefEntry ce[NB];
#pragma unroll
      for (int e = 0; e < NB; ++e)
        if (e < nc) ce[e] = cf.ent[beg + e];
      if (nc == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = 0.0f;
      }
#pragma unroll
      for (int e = 0; e < NB; ++e) {
        if (e < nc) {
          const float4 *p = reinterpret_cast<const float4 *>(lrow + ce[e].block * (TR * STR));
          const float4 v0 = p[0], v1 = p[1], v2 = p[2], v3 = p[3];
          const float a[16] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w,
                               v2.x, v2.y, v2.z, v2.w, v3.x, v3.y, v3.z, v3.w};
          const float c = ce[e].coef;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float pr = __fmul_rn(c, a[i]);
            x[i] = e == 0 ? pr : __fadd_rn(x[i], pr);
          }
        }
      }
    }
    if constexpr (MODE == 3) {
      double e2 = 0.0, x2 = 0.0;
      if (o.valid) {
        const int64_t plane = bt * T + r;
        const uint4 cw = *reinterpret_cast<const uint4 *>(codes + plane * code_plane + o.code);
        const double sc = pb.scale_bytes == 4
                              ? (double)__uint_as_float(reinterpret_cast<const uint32_t *>(scales)[plane * scale_plane + o.scale])
                              : ldexp(1.0, (int)scales[plane * scale_plane + o.scale] - 127);
        const int cwv[4] = {(int)cw.x, (int)cw.y, (int)cw.z, (int)cw.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float d0 = __builtin_amdgcn_cvt_f32_fp8(cwv[j], 0), d1 = __builtin_amdgcn_cvt_f32_fp8(cwv[j], 1);
          const float d2 = __builtin_amdgcn_cvt_f32_fp8(cwv[j], 2), d3 = __builtin_amdgcn_cvt_f32_fp8(cwv[j], 3);
          const float dec[4] = {d0, d1, d2, d3};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double xv = (double)x[4 * j + i];
            const double dv = (double)dec[i] * sc - xv;
            e2 += dv * dv;
            x2 += xv * xv;
          }
        }
      }
#pragma unroll
      for (int sh = 32; sh >= 1; sh >>= 1) {
        e2 += __shfl_xor(e2, sh, 64);
        x2 += __shfl_xor(x2, sh, 64);
      }
      if (lane == 0) {
        double *pp = reinterpret_cast<double *>(aux) +
                     ((((int64_t)bt * nbx + bx) * (NT / 64) + wave) * T + r) * 2;
        pp[0] = e2;
        pp[1] = x2;
      }
      continue;
    }
    if constexpr (MODE == 2) {
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = bf16_round(x[i]);
    }
    // block maximum: the lane's 16, then across the lanes of its block
    float m = fmaxf(fabsf(x[0]), fabsf(x[1]));
#pragma unroll
    for (int i = 2; i < 16; ++i) m = fmaxf(m, fabsf(x[i]));
    if (BS >= 32) {
      uint32_t mb = __float_as_uint(m);                       // m >= 0
      mb = max(mb, dpp_u<0xB1>(mb));                          // quad_perm [1, 0, 3, 2]
      if (BS == 128) {
        mb = max(mb, dpp_u<0x4E>(mb));                        // quad_perm [2, 3, 0, 1]
        mb = max(mb, (uint32_t)__shfl_xor((int)mb, 32, 64));
      }
      m = __uint_as_float(mb);
    }
    uint32_t w[4];
    uint32_t stored;
    if constexpr (F32) {
      const dev::Scale sc = dev::block_scale(m, dev::RULE_FP32_AMAX);
      stored = sc.stored;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        w[j] = dev::e4m3_pack4(dev::div_by(x[4 * j], sc.div, sc.inv), dev::div_by(x[4 * j + 1], sc.div, sc.inv),
                               dev::div_by(x[4 * j + 2], sc.div, sc.inv), dev::div_by(x[4 * j + 3], sc.div, sc.inv));
    } else {
      // a power-of-two rule (the ceiling or the OCP one)
      const dev::Scale sc = dev::block_scale(m, pb.rule == dev::RULE_POW2_CEIL ? dev::RULE_POW2_CEIL
                                                                                : dev::RULE_POW2_OCP);
      stored = sc.stored;
      const float s = __uint_as_float(sc.stored << 23);     // 2^e (stored = e + 127)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        w[j] = dev::e4m3_pack4_pow2(x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3], s);
    }
    const int64_t plane = bt * T + r;
    if (o.valid)
      *reinterpret_cast<uint4 *>(codes + plane * code_plane + o.code) = make_uint4(w[0], w[1], w[2], w[3]);
    if (o.leader) store_scale(pb, scales, plane * scale_plane + o.scale, stored);
  }
}

template <int SIDE, int DEPTH, int BS, bool F32, int MODE, int CAP = 0, bool N1 = false>
__global__ __launch_bounds__((Tile<DEPTH, 16, SIDE, narrow_b(SIDE, DEPTH, BS, MODE) || N1>::threads)) void encode16_kernel(
    const float *__restrict__ src, Problem pb, SideTab cf, uint8_t *__restrict__ codes, uint8_t *__restrict__ scales,
    int64_t tiles_l, void *__restrict__ aux) {
  using TT = Tile<DEPTH, 16, SIDE, narrow_b(SIDE, DEPTH, BS, MODE) || N1, CAP>;
  __shared__ float4 lds4[TT::lds_floats / 4];
  encode16_tile<SIDE, DEPTH, BS, F32, MODE, CAP, N1, TT::threads>(reinterpret_cast<float *>(lds4), src, pb, cf, codes,
                                                                  scales, tiles_l, aux, blockIdx.x, gridDim.x, blockIdx.y);
}

// Both sides of a <2,2,2> plan in one launch: workgroups 0 .. tiles[0] - 1 of a
// product encode A, the rest B.  A small encode is two launches of about 5 us
// that read a few megabytes each; in one launch the sides run side by side
// (us, separate / one launch: 256^3 11.8 / 8.0, 1024^3 11.9 / 7.8, 100 of
// 256^3 22.8 / 20.7, 4096^3 45.9 / 43.1; depth 2 1024^3 19.1 / 10.6, 4096^3
// 71.5 / 62.5, 8192^3 286 / 274; one_launch has where it pays).  Both sides then
// have one workgroup size:
// at depth 1 256 threads (A's four waves each take every fourth term; B on
// the narrow tile) at blocks 16 and 32, 512 at block 128; at depth 2 1024, as
// each has by itself.  Alternating the sides' workgroups: up to 9% slower.
struct PairArgs {
  const float *src[2];
  SideTab cf[2];
  uint8_t *codes[2], *scales[2];
  int64_t tiles_l[2];
  unsigned tiles[2];           // workgroups per product and side
};

template <int DEPTH, int BS>
constexpr bool pair_n1() { return DEPTH == 1 && BS <= 32; }
template <int DEPTH, int BS>
constexpr int pair_threads() { return DEPTH == 2 ? 1024 : pair_n1<DEPTH, BS>() ? kB1NThreads : kB1Threads; }

template <int DEPTH, int BS, bool F32, int CAP = 0>
__global__ __launch_bounds__((pair_threads<DEPTH, BS>())) void encode_pair_kernel(Problem pb, PairArgs g) {
  constexpr bool N1 = pair_n1<DEPTH, BS>();
  constexpr int NT = pair_threads<DEPTH, BS>();
  using TA = Tile<DEPTH, 16, 0, false, CAP>;
  using TB = Tile<DEPTH, 16, 1, narrow_b(1, DEPTH, BS, 0) || N1, CAP>;
  __shared__ float4 lds4[(TA::lds_floats > TB::lds_floats ? TA::lds_floats : TB::lds_floats) / 4];
  float *lds = reinterpret_cast<float *>(lds4);
  if (blockIdx.x < g.tiles[0])
    encode16_tile<0, DEPTH, BS, F32, 0, CAP, false, NT>(lds, g.src[0], pb, g.cf[0], g.codes[0], g.scales[0], g.tiles_l[0],
                                                      nullptr, blockIdx.x, g.tiles[0], blockIdx.y);
  else
    encode16_tile<1, DEPTH, BS, F32, 0, CAP, N1, NT>(lds, g.src[1], pb, g.cf[1], g.codes[1], g.scales[1], g.tiles_l[1],
                                                   nullptr, blockIdx.x - g.tiles[0], g.tiles[1], blockIdx.y);
}

// ---------------------------------------------------------------------------
// Depth 3: 4 positions per lane (2 rows x 128 positions per tile, or on the B
// side at blocks 16 and 32 8 rows x 32 positions; 64 items of one term per
// wave).
// ---------------------------------------------------------------------------
// Maximum over each group of GL aligned lanes (GL = block / 4: 4, 8 or 32),
// every lane receiving its group's maximum: quad permutations (xor 1, xor 2),
// then the half-row and row mirrors, then across the two rows of 32 lanes.
// Taken on the bit patterns of non-negative finite values (equal to the
// floating-point maximum), one unsigned maximum per step.
template <int GL>
__device__ __forceinline__ uint32_t group_max_bits(uint32_t m) {
  m = max(m, dpp_u<0xB1>(m));                         // quad_perm [1, 0, 3, 2]
  m = max(m, dpp_u<0x4E>(m));                         // quad_perm [2, 3, 0, 1]
  if (GL >= 8) m = max(m, dpp_u<0x141>(m));           // row_half_mirror: lane i <- 7 - i within 8
  if (GL >= 16) m = max(m, dpp_u<0x140>(m));          // row_mirror: lane i <- 15 - i within 16
  if (GL >= 32) m = max(m, (uint32_t)__shfl_xor((int)m, 16, 64));
  return m;
}

// Scale and codes of a lane's 4 values of a block whose maximum is m: the
// fp32 rule rounds the quotient to nearest (div_by), the power-of-two rules scale
// exactly inside the conversion.
template <bool F32>
__device__ __forceinline__ uint32_t quantize4(const Problem &pb, float m, float x0, float x1, float x2, float x3,
                                              uint32_t &stored) {
  if constexpr (F32) {
    const dev::Scale sc = dev::block_scale(m, dev::RULE_FP32_AMAX);
    stored = sc.stored;
    return dev::e4m3_pack4(dev::div_by(x0, sc.div, sc.inv), dev::div_by(x1, sc.div, sc.inv), dev::div_by(x2, sc.div, sc.inv),
                           dev::div_by(x3, sc.div, sc.inv));
  } else {
    const dev::Scale sc =
        dev::block_scale(m, pb.rule == dev::RULE_POW2_CEIL ? dev::RULE_POW2_CEIL : dev::RULE_POW2_OCP);
    stored = sc.stored;
    return dev::e4m3_pack4_pow2(x0, x1, x2, x3, __uint_as_float(sc.stored << 23));
  }
}

// One block's contributions to the seven terms of a group whose inner column
// COL follows pattern PAT: each class's product once, then one addition or
// subtraction a term, as x + fl32(c a) has it bit for bit (c's sign moves
// through the product and the sum exactly).
template <int PAT, int COL>
__device__ __forceinline__ void add_column(float (&x)[8][4], const float4 &v, const float (&c)[8], int b) {
#pragma unroll
  for (int cls = 0; cls < 2; ++cls) {
    if (pattern_members(PAT, COL, cls) == 0) continue;
    const float cb = lane_coef(c[pattern_lead(PAT, COL, cls)], b);
    const float p0 = __fmul_rn(cb, v.x), p1 = __fmul_rn(cb, v.y), p2 = __fmul_rn(cb, v.z), p3 = __fmul_rn(cb, v.w);
#pragma unroll
    for (int j = 0; j < kPatternRows; ++j) {
      if (!(pattern_members(PAT, COL, cls) >> j & 1)) continue;
      const bool minus = pattern_minus(PAT, COL, cls) >> j & 1;
      x[j][0] = minus ? __fsub_rn(x[j][0], p0) : __fadd_rn(x[j][0], p0);
      x[j][1] = minus ? __fsub_rn(x[j][1], p1) : __fadd_rn(x[j][1], p1);
      x[j][2] = minus ? __fsub_rn(x[j][2], p2) : __fadd_rn(x[j][2], p2);
      x[j][3] = minus ? __fsub_rn(x[j][3], p3) : __fadd_rn(x[j][3], p3);
    }
  }
}

constexpr bool narrow_b3(int side, int bs) { return side == 1 && bs <= 256 / kB3Rows; }

// PAT: the side's coefficients follow that EncodePattern (0: any coefficients).
template <int SIDE, int BS, bool F32, bool GEN = false, int PAT = 0>
__global__ __launch_bounds__((Tile<3, 4, SIDE, narrow_b3(SIDE, BS)>::threads), 8) void encode4_kernel(
    const float *__restrict__ src, Problem pb, SideTab cf, uint8_t *__restrict__ codes, uint8_t *__restrict__ scales,
    int64_t tiles_l) {
  using TT = Tile<3, 4, SIDE, narrow_b3(SIDE, BS)>;
  constexpr int TR = TT::TR, NT = TT::threads, TL = TT::TL, STR = TT::stride;
  constexpr int P = TR * (TL / 4);           // positions (row, 4 consecutive l) per term
  static_assert(P == 64 && TT::nblk == 64, "a wave's 64 items are one term's tile; lane b holds block b's coefficient");
  __shared__ float4 lds4[TT::lds_floats / 4];
  float *lds = reinterpret_cast<float *>(lds4);

  const int t = threadIdx.x;
  const int64_t bt = blockIdx.y;
  const int64_t row0 = (blockIdx.x / tiles_l) * TR;
  const int64_t l0 = (blockIdx.x % tiles_l) * TL;
  const int64_t rows = SIDE == 0 ? pb.mp : pb.np;
  stage_tile<SIDE, TT::nblk, TR, NT, TL, GEN>(lds, src, pb, bt, row0, l0, t);
  __syncthreads();

  const int64_t T = pb.T;
  constexpr int GL = BS / 4;                 // lanes per block
  const int pos = t % P;
  const int row = pos / (TL / 4), c4 = pos % (TL / 4);
  static_assert(BS <= TL, "a block lies in one row of the tile");
  const Out o = out_of(pb, rows, row0 + row, l0 + 4 * c4, (c4 % GL) == 0);
  // a lane's offsets inside a (batch, term) plane fit in 32 bits
  const uint32_t o_code = (uint32_t)o.code, o_scale = (uint32_t)o.scale;
  const bool o_valid = o.valid, o_leader = o.leader;
  const int64_t code_plane = rows * pb.kp;
  const int64_t scale_plane = scale_plane_of(pb, rows);
  const float *lrow = lds + row * STR + 4 * c4;
  // A wave takes a group of up to kG consecutive terms at once: at depth 3 the
  // R terms that share their two outer digits (T* flattened: 17 nonzero
  // blocks per term on average, 26 in the union of a group of 7), so each
  // block is read from LDS once per group rather than once per term.  Every
  // term's x = sum_b c_b a_b still runs over its own nonzero blocks in
  // ascending b with products and sums rounded separately, its first block
  // giving x = c a.  The terms' dense coefficient rows (block b in lane b)
  // give each term's nonzero blocks by a ballot; their union is walked in
  // ascending order.
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // Whole rounds of groups (every wave one group per round) go first; the
  // terms left over are taken one per wave, which keeps the waves' loads
  // within one term of each other (343 terms in groups of 7: 48 groups in
  // three rounds, then 7 single terms).
  constexpr int WSTEP = NT / 64;
  constexpr int kG = 8;
  const int G = GEN ? kG : pb.R;             // R <= 8 at <2,2,2>
  const int64_t nfull = ((T + G - 1) / G / WSTEP) * WSTEP;      // groups taken in whole rounds
  const int64_t tail0 = nfull * G < T ? nfull * G : T;          // the first term taken alone
  const int64_t units = nfull + (T - tail0);
  int64_t u = wave;
  if constexpr (PAT != 0) {
    // Whole rounds under a known pattern: a group's terms draw on an outer
    // block all or none, and its two inner blocks of one inner row sit side by
    // side, so the walk in ascending block order needs no test per term, and a
    // product shared by a class's terms is formed once: per outer block
    // 7 x 4 multiplications and 18 x 4 additions for T* (4 x 4 and 12 x 4 for
    // Strassen) against 18 x 8 operations and 28 tests (12 x 8).  The arithmetic
    // bounds this kernel (us, 8192^3: T* 1066 -> 778, Strassen 679 -> 559; T*
    // 16384x8192x16384 2035 -> 1430, 2048x7168x2048 274 -> 174; codes identical).
    for (; u < nfull; u += WSTEP) {
      const int64_t g0 = u * kPatternRows;
      float c[kG];
#pragma unroll
      for (int j = 0; j < kG; ++j) c[j] = 0.0f;
#pragma unroll
      for (int j : {0, 1, 4}) c[j] = cf.dense[(g0 + cf.pat.perm[j]) * 64 + lane];
      // outer blocks in use: row 0 has the inner corner block in both patterns
      const uint64_t outer = __ballot(c[0] != 0.0f);
      float x[kG][4];
#pragma unroll
      for (int j = 0; j < kG; ++j) x[j][0] = x[j][1] = x[j][2] = x[j][3] = -0.0f;
      // block b = 16 P + 8 p + 2 Q + q of outer rows P, outer columns Q, inner (p, q)
      for (int P = 0; P < 4; ++P) {
        const uint32_t qs = (uint32_t)(outer >> (16 * P)) & 0x55u;
        uint32_t rest = qs;
        while (rest != 0) {
          const int b = 16 * P + __builtin_ctz(rest);
          rest &= rest - 1;
          const float *pv = lrow + b * (TR * STR);
          const float4 v0 = *reinterpret_cast<const float4 *>(pv), v1 = *reinterpret_cast<const float4 *>(pv + TR * STR);
          add_column<PAT, 0>(x, v0, c, b);
          add_column<PAT, 1>(x, v1, c, b + 1);
        }
        rest = qs;
        while (rest != 0) {
          const int b = 16 * P + 8 + __builtin_ctz(rest);
          rest &= rest - 1;
          const float *pv = lrow + b * (TR * STR);
          const float4 v0 = *reinterpret_cast<const float4 *>(pv), v1 = *reinterpret_cast<const float4 *>(pv + TR * STR);
          add_column<PAT, 2>(x, v0, c, b);
          add_column<PAT, 3>(x, v1, c, b + 1);
        }
      }
#pragma unroll
      for (int j = 0; j < kPatternRows; ++j) {
        if (outer == 0) x[j][0] = x[j][1] = x[j][2] = x[j][3] = 0.0f;
        const float mx = __uint_as_float(group_max_bits<GL>(__float_as_uint(
            fmaxf(fmaxf(fabsf(x[j][0]), fabsf(x[j][1])), fmaxf(fabsf(x[j][2]), fabsf(x[j][3]))))));
        uint32_t stored;
        const uint32_t w = quantize4<F32>(pb, mx, x[j][0], x[j][1], x[j][2], x[j][3], stored);
        const int64_t plane = bt * T + g0 + cf.pat.perm[j];      // uniform
        if (o_valid) *reinterpret_cast<uint32_t *>(codes + plane * code_plane + o_code) = w;
        if (o_leader) store_scale(pb, scales, plane * scale_plane + o_scale, stored);
      }
    }
  }
  for (; u < units; u += WSTEP) {
    const int64_t g0 = u < nfull ? u * G : tail0 + (u - nfull);
    const int gn = u < nfull ? (int)(T - g0 < G ? T - g0 : G) : 1;
    float c[kG];
#pragma unroll
    for (int j = 0; j < kG; ++j) c[j] = j < gn ? cf.dense[(g0 + j) * 64 + lane] : 0.0f;
    uint64_t m[kG];
    uint64_t uni = 0;
#pragma unroll
    for (int j = 0; j < kG; ++j) {
      m[j] = __ballot(c[j] != 0.0f);
      uni |= m[j];
    }
    // accumulators start at -0: -0 + t = t exactly for every t, so a term's
    // first block gives x = c a as the definition does; a term without
    // nonzero blocks ends at +0
    float x[kG][4];
#pragma unroll
    for (int j = 0; j < kG; ++j) x[j][0] = x[j][1] = x[j][2] = x[j][3] = -0.0f;
    if (uni != 0) {
      // the next block's values are read while this block's are used
      int b = __builtin_ctzll(uni);
      uni &= uni - 1;
      float4 v = *reinterpret_cast<const float4 *>(lrow + b * (TR * STR));
      while (true) {
        const bool more = uni != 0;
        const int bn = more ? __builtin_ctzll(uni) : b;
        uni &= uni - 1;
        const float4 vn = *reinterpret_cast<const float4 *>(lrow + bn * (TR * STR));
#pragma unroll
        for (int j = 0; j < kG; ++j) {
          if ((m[j] >> b) & 1) {
            const float cb = lane_coef(c[j], b);
            x[j][0] = __fadd_rn(x[j][0], __fmul_rn(cb, v.x));
            x[j][1] = __fadd_rn(x[j][1], __fmul_rn(cb, v.y));
            x[j][2] = __fadd_rn(x[j][2], __fmul_rn(cb, v.z));
            x[j][3] = __fadd_rn(x[j][3], __fmul_rn(cb, v.w));
          }
        }
        if (!more) break;
        b = bn;
        v = vn;
      }
    }
#pragma unroll
    for (int j = 0; j < kG; ++j)
      if (m[j] == 0) x[j][0] = x[j][1] = x[j][2] = x[j][3] = 0.0f;
#pragma unroll
    for (int j = 0; j < kG; ++j) {
      if (j < gn) {
        const float mx = __uint_as_float(group_max_bits<GL>(__float_as_uint(
            fmaxf(fmaxf(fabsf(x[j][0]), fabsf(x[j][1])), fmaxf(fabsf(x[j][2]), fabsf(x[j][3]))))));
        uint32_t stored;
        const uint32_t w = quantize4<F32>(pb, mx, x[j][0], x[j][1], x[j][2], x[j][3], stored);
        const int64_t plane = bt * T + g0 + j;      // uniform
        if (o_valid) *reinterpret_cast<uint32_t *>(codes + plane * code_plane + o_code) = w;
        if (o_leader) store_scale(pb, scales, plane * scale_plane + o_scale, stored);
      }
    }
  }
}

// N1: the depth-1 B side's narrow tile (32 columns x 64 positions, 256
// threads), taken on the 256 x 64 tile layout at blocks 16 and 32: each lane
// quad writes a whole 64-byte image row, and the half-size tile lets four
// workgroups share a CU (8192^3 T* encode 149 -> 143.5 us, codes identical).
template <int SIDE, int DEPTH, int BS, bool F32, int MODE = 0, int CAP = 0, bool N1 = false>
hipError_t launch16(const Problem &pb, const float *src, const SideTab &cf,
                    uint8_t *codes, uint8_t *scales, hipStream_t st, void *aux = nullptr) {
  if constexpr (SIDE == 1 && DEPTH == 1 && MODE == 0 && CAP == 0 && BS <= 32 && !N1) {
    if (pb.layout == FMM_LAYOUT_TILE256x64)
      return launch16<SIDE, DEPTH, BS, F32, MODE, CAP, true>(pb, src, cf, codes, scales, st, aux);
  }
  using TT = Tile<DEPTH, 16, SIDE, narrow_b(SIDE, DEPTH, BS, MODE) || N1, CAP>;
  const int64_t rows = SIDE == 0 ? pb.mp : pb.np;
  const int64_t tiles_l = (pb.kp + TT::TL - 1) / TT::TL;
  const int64_t tiles_r = (rows + TT::TR - 1) / TT::TR;
  const dim3 grid((unsigned)(tiles_l * tiles_r), (unsigned)pb.batch);
  hipLaunchKernelGGL((encode16_kernel<SIDE, DEPTH, BS, F32, MODE, CAP, N1>), grid, dim3(TT::threads), 0, st, src, pb, cf,
                     codes, scales, tiles_l, aux);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// B side with 128-row scale blocks (FMM_FLAG_B_BLOCK128, depth 1), optionally of
// bfloat16-rounded combinations (FMM_FLAG_B_BF16).
//
// A scale covers 128 columns of B x `block` positions, so a workgroup holds the
// four sub-blocks' 128 columns x TL positions (TL = 128 at block 128, else 64) in
// registers: a thread has 16 positions of one column of each (64 values; 256 KB a
// workgroup at block 128, more than LDS), read once, a wave's load one 256-byte
// row segment.  Per term every wave reduces the maximum of its 64 columns x 16
// positions, the workgroup's waves meet at one barrier (the maxima's slots
// alternate by term, so no second one is needed), and each thread quantizes its
// run.  Where the tiles leave CUs idle, several workgroups share a tile's terms
// (298x256x1102 19.8 us in the two passes below, 20.9 in one workgroup a tile, 10.3
// now; 2048^3 32.0, 27.5, 19.3).  HBM bounds it, and at block 128 the one workgroup a CU holds, which loads
// and computes in turn.  Two passes over B, the first for the maxima alone, and
// a pass clearing these took (encode of both sides, us, before / now): 8192^3
// fp32 scales at block 128 230 / 196, power-of-two scales at block 128 224 / 165, at
// block 32 223 / 147; 4096^3 block 128 69.5 / 49.7; 512^3 block 128 23.9 / 12.0.
// ---------------------------------------------------------------------------
template <int BS>
constexpr int rows128_tl() { return BS == 128 ? 128 : 64; }

template <int BS, bool F32>
__global__ __launch_bounds__(8 * rows128_tl<BS>(), 4) void encode_rows128_kernel(
    const float *__restrict__ src, Problem pb, SideTab cf, uint8_t *__restrict__ codes, uint8_t *__restrict__ scales) {
  constexpr int TL = rows128_tl<BS>(), NW = TL / 8;      // waves: 2 c + column half for run c
  constexpr int GW = 2 * BS / 16;                        // consecutive waves that share a block
  __shared__ uint32_t red[2][NW];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t tiles_r = (pb.np + 127) / 128, bt = blockIdx.y;
  // (the column tile varies fastest: neighbours read adjacent pieces of the same rows of B)
  const int64_t col = (blockIdx.x % tiles_r) * 128 + 64 * (wave & 1) + lane;
  const int64_t l = (blockIdx.x / tiles_r) * TL + 16 * (wave >> 1);
  const Out o = out_of(pb, pb.np, col, l, (l % BS) == 0);
  // every load unconditional, so that all are in flight together: threads past
  // an edge read the last column or run again and take no part in the maxima
  float a[4][16];
  const float *Bb = src + bt * pb.K * pb.N + (l < pb.kp ? l : pb.kp - 16) * pb.N + (col < pb.np ? col : pb.np - 1);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const float *p = Bb + (b >> 1) * pb.kp * pb.N + (b & 1) * pb.np;
#pragma unroll
    for (int i = 0; i < 16; ++i) a[b][i] = __builtin_nontemporal_load(p + i * pb.N);
  }
  // the T x 4 coefficients, one a lane (T <= 8), so that no term waits on scalar memory
  const float coef = lane < 4 * (int)pb.T ? cf.dense[lane] : 0.0f;
  const int64_t code_plane = pb.np * pb.kp, scale_plane = scale_plane_of(pb, pb.np);
  int slot = 0;
  for (int r = blockIdx.z; r < (int)pb.T; r += gridDim.z, slot ^= 1) {
    // x = sum_b c_b a_b in ascending b, products and sums rounded separately; -0 + t = t
    float x[16];
    bool any = false;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = -0.0f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const float c = lane_coef(coef, 4 * r + b);
      if (c != 0.0f) {
        any = true;
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = __fadd_rn(x[i], __fmul_rn(c, a[b][i]));
      }
    }
    if (!any) {
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = 0.0f;
    }
    if (pb.b_bf16) {
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = bf16_round(x[i]);
    }
    float m = fmaxf(fabsf(x[0]), fabsf(x[1]));
#pragma unroll
    for (int i = 2; i < 16; ++i) m = fmaxf(m, fabsf(x[i]));
    uint32_t mb = group_max_bits<32>(o.valid ? __float_as_uint(m) : 0u);
    mb = max(mb, (uint32_t)__shfl_xor((int)mb, 32, 64));
    if (lane == 0) red[slot][wave] = mb;
    __syncthreads();
    const uint32_t *rd = red[slot] + (wave & ~(GW - 1));
    mb = rd[0];
#pragma unroll
    for (int k = 1; k < GW; ++k) mb = max(mb, rd[k]);
    m = __uint_as_float(mb);
    uint32_t w[4];
    uint32_t stored;
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = quantize4<F32>(pb, m, x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3], stored);
    const int64_t plane = bt * pb.T + r;
    if (o.valid) *reinterpret_cast<uint4 *>(codes + plane * code_plane + o.code) = make_uint4(w[0], w[1], w[2], w[3]);
    if (o.leader) store_scale(pb, scales, plane * scale_plane + o.scale, stored);
  }
}

// B side with the weight-side deployment granularity (depth 1).
template <int BS, bool F32>
hipError_t launch_b_deploy(const Problem &pb, const float *src, const SideTab &cf,
                           uint8_t *codes, uint8_t *scales, hipStream_t st) {
  if (pb.b_rows == 1) return launch16<1, 1, BS, F32, 2>(pb, src, cf, codes, scales, st);
  constexpr int TL = rows128_tl<BS>();
  // few workgroups: each tile's terms over several of them, which load it again
  const int64_t tiles = ((pb.np + 127) / 128) * ((pb.kp + TL - 1) / TL);
  const int64_t z = std::min<int64_t>(std::max<int64_t>(pb.ncu / (tiles * pb.batch), 1), pb.T);
  const dim3 grid((unsigned)tiles, (unsigned)pb.batch, (unsigned)z);
  hipLaunchKernelGGL((encode_rows128_kernel<BS, F32>), grid, dim3(8 * TL), 0, st, src, pb, cf, codes, scales);
  return hipGetLastError();
}

hipError_t launch_b_deploy_any(const Problem &pb, const float *src, const SideTab &cf,
                               uint8_t *codes, uint8_t *scales, hipStream_t st) {
  const bool f32 = pb.rule == dev::RULE_FP32_AMAX;
  switch (pb.block) {
    case 16: return f32 ? launch_b_deploy<16, true>(pb, src, cf, codes, scales, st)
                        : launch_b_deploy<16, false>(pb, src, cf, codes, scales, st);
    case 32: return f32 ? launch_b_deploy<32, true>(pb, src, cf, codes, scales, st)
                        : launch_b_deploy<32, false>(pb, src, cf, codes, scales, st);
    case 128: return f32 ? launch_b_deploy<128, true>(pb, src, cf, codes, scales, st)
                         : launch_b_deploy<128, false>(pb, src, cf, codes, scales, st);
  }
  return hipErrorInvalidValue;
}

template <int SIDE, int DEPTH, int CAP = 0>
hipError_t launch_wide(const Problem &pb, const float *src, const SideTab &cf,
                       uint8_t *codes, uint8_t *scales, hipStream_t st) {
  const bool f32 = pb.rule == dev::RULE_FP32_AMAX;
  switch (pb.block) {
    case 16: return f32 ? launch16<SIDE, DEPTH, 16, true, 0, CAP>(pb, src, cf, codes, scales, st)
                        : launch16<SIDE, DEPTH, 16, false, 0, CAP>(pb, src, cf, codes, scales, st);
    case 32: return f32 ? launch16<SIDE, DEPTH, 32, true, 0, CAP>(pb, src, cf, codes, scales, st)
                        : launch16<SIDE, DEPTH, 32, false, 0, CAP>(pb, src, cf, codes, scales, st);
    case 128: return f32 ? launch16<SIDE, DEPTH, 128, true, 0, CAP>(pb, src, cf, codes, scales, st)
                         : launch16<SIDE, DEPTH, 128, false, 0, CAP>(pb, src, cf, codes, scales, st);
  }
  return hipErrorInvalidValue;
}

// 4 positions per lane over a grid of up to 64 blocks (depth 3, or GEN)
template <int SIDE, int BS, bool GEN>
hipError_t launch4(const Problem &pb, const float *src, const SideTab &cf, uint8_t *codes, uint8_t *scales, hipStream_t st) {
  using TT = Tile<3, 4, SIDE, narrow_b3(SIDE, BS)>;
  const int64_t rows = SIDE == 0 ? pb.mp : pb.np;
  const int64_t tiles_l = (pb.kp + TT::TL - 1) / TT::TL;
  const int64_t tiles_r = (rows + TT::TR - 1) / TT::TR;
  const dim3 grid((unsigned)(tiles_l * tiles_r), (unsigned)pb.batch), blk(TT::threads);
  const bool f32 = pb.rule == dev::RULE_FP32_AMAX;
#define FMM_ENCODE4(F32, PAT) \
  hipLaunchKernelGGL((encode4_kernel<SIDE, BS, F32, GEN, PAT>), grid, blk, 0, st, src, pb, cf, codes, scales, tiles_l)
  if constexpr (!GEN) {
    if (cf.pat.id != 0) {
      if (cf.pat.id == 1 && f32) FMM_ENCODE4(true, 1);
      else if (cf.pat.id == 1) FMM_ENCODE4(false, 1);
      else if (f32) FMM_ENCODE4(true, 2);
      else FMM_ENCODE4(false, 2);
      return hipGetLastError();
    }
  }
  if (f32) FMM_ENCODE4(true, 0);
  else FMM_ENCODE4(false, 0);
#undef FMM_ENCODE4
  return hipGetLastError();
}

template <int SIDE, bool GEN = false>
hipError_t launch_narrow4(const Problem &pb, const float *src, const SideTab &cf,
                          uint8_t *codes, uint8_t *scales, hipStream_t st) {
  switch (pb.block) {
    case 16: return launch4<SIDE, 16, GEN>(pb, src, cf, codes, scales, st);
    case 32: return launch4<SIDE, 32, GEN>(pb, src, cf, codes, scales, st);
    case 128: return launch4<SIDE, 128, GEN>(pb, src, cf, codes, scales, st);
  }
  return hipErrorInvalidValue;
}

template <int SIDE>
hipError_t launch_side(const Problem &pb, const float *src, const SideTab &cf,
                       uint8_t *codes, uint8_t *scales, hipStream_t st) {
  if (pb.shaped) {
    // another shape: the depth-1 tile staging 4 or 8 blocks (the sizes that
    // keep as many bytes in flight per CU as the <2,2,2> encoder), the
    // depth-2 tile (16 positions per lane, 16 waves) over up to 16 blocks,
    // the depth-3 one (4 per lane) over up to 64
    const int nb = SIDE == 0 ? pb.gm * pb.gk : pb.gk * pb.gn;
    if (nb <= 4) return launch_wide<SIDE, 1, 4>(pb, src, cf, codes, scales, st);
    if (nb <= 8) return launch_wide<SIDE, 1, 8>(pb, src, cf, codes, scales, st);
    if (nb <= 16) return launch_wide<SIDE, 2, 16>(pb, src, cf, codes, scales, st);
    return launch_narrow4<SIDE, true>(pb, src, cf, codes, scales, st);
  }
  switch (pb.depth) {
    case 1: return launch_wide<SIDE, 1>(pb, src, cf, codes, scales, st);
    case 2: return launch_wide<SIDE, 2>(pb, src, cf, codes, scales, st);
    case 3: return launch_narrow4<SIDE>(pb, src, cf, codes, scales, st);
  }
  return hipErrorInvalidValue;
}

// ---- operand-side rounding energy (MODE 3) ----------------------------------

// One side's noise partials: slot ((bt * tiles + tile) * waves + wave) * T + r
// holds term r's sums over the rows of that wave, written for the terms the
// wave works on (r mod step = wave / wpt; MODE 3 of encode16_kernel).
struct NoiseSide {
  const double *partial;
  int64_t tiles;
  int waves, wpt, step;
};

// tiles of one product's side, and waves per workgroup, of MODE 3
template <int SIDE>
int64_t noise_tiles(const Problem &pb) {
  const int64_t rows = SIDE == 0 ? pb.mp : pb.np;
  const int64_t tr = pb.depth == 1 ? Tile<1, 16, SIDE>::TR : Tile<2, 16, SIDE>::TR;
  return ((pb.kp + kTL - 1) / kTL) * ((rows + tr - 1) / tr);
}
template <int SIDE>
int noise_waves(const Problem &pb) {
  return (pb.depth == 1 ? Tile<1, 16, SIDE>::threads : Tile<2, 16, SIDE>::threads) / 64;
}
template <int SIDE>
int64_t noise_slots(const Problem &pb) {
  return pb.batch * noise_tiles<SIDE>(pb) * noise_waves<SIDE>(pb) * pb.T;
}
template <int SIDE>
NoiseSide noise_side(const Problem &pb, const double *partial) {
  NoiseSide s;
  s.partial = partial;
  s.tiles = noise_tiles<SIDE>(pb);
  s.waves = noise_waves<SIDE>(pb);
  // waves that share a term's rows (8 each), as encode16_kernel's WPT
  s.wpt = (pb.depth == 1 ? Tile<1, 16, SIDE>::TR : Tile<2, 16, SIDE>::TR) / 8;
  s.step = s.waves / s.wpt;
  return s;
}

template <int SIDE, int DEPTH>
hipError_t launch_noise_side(const Problem &pb, const float *src, const SideTab &cf,
                             const uint8_t *codes, const uint8_t *scales, double *partial, hipStream_t st) {
  uint8_t *c = const_cast<uint8_t *>(codes), *sc = const_cast<uint8_t *>(scales);
  const bool f32 = pb.rule == dev::RULE_FP32_AMAX;
  switch (pb.block) {
    case 16: return f32 ? launch16<SIDE, DEPTH, 16, true, 3>(pb, src, cf, c, sc, st, partial)
                        : launch16<SIDE, DEPTH, 16, false, 3>(pb, src, cf, c, sc, st, partial);
    case 32: return f32 ? launch16<SIDE, DEPTH, 32, true, 3>(pb, src, cf, c, sc, st, partial)
                        : launch16<SIDE, DEPTH, 32, false, 3>(pb, src, cf, c, sc, st, partial);
    case 128: return f32 ? launch16<SIDE, DEPTH, 128, true, 3>(pb, src, cf, c, sc, st, partial)
                         : launch16<SIDE, DEPTH, 128, false, 3>(pb, src, cf, c, sc, st, partial);
  }
  return hipErrorInvalidValue;
}

// out[(bt * 2 + side) * T + r][q]: W waves of a workgroup per (term, side,
// product) sum the term's slots, thread t taking slots t, t + 64 W, .. in that
// order, then the lanes by a fixed butterfly and the waves in order.  Four waves,
// or one where no term has more than 256 slots.  (A thread per output walking
// every slot, and a pass that cleared the slots nobody writes, took 448 us for two
// 2048 x 1024 x 1536 products, four waves 3.8; the whole measurement of 1000
// products of 64^3 57 us, 64 with four waves for a few slots each, 52 with one.)
template <int W>
__global__ __launch_bounds__(256) void noise_reduce_kernel(NoiseSide a, NoiseSide b, double *__restrict__ out, int64_t T,
                                                           int64_t total) {
  const int t = threadIdx.x % (64 * W), part = threadIdx.x / (64 * W);
  const int64_t i = (int64_t)blockIdx.x * (4 / W) + part;      // (bt, side, r); uniform over a wave
  if (i >= total) return;                                      // (W = 4: never)
  const int64_t r = i % T, side = i / T % 2, bt = i / T / 2;
  const NoiseSide s = side == 0 ? a : b;
  const int w0 = s.wpt * (int)(r % s.step);
  const int64_t n = s.tiles * s.wpt;
  double e2 = 0.0, x2 = 0.0;
  for (int64_t k = t; k < n; k += 64 * W) {
    const int64_t tile = k / s.wpt;
    const int64_t slot = ((bt * s.tiles + tile) * s.waves + w0 + (k - tile * s.wpt)) * T + r;
    e2 += s.partial[2 * slot];
    x2 += s.partial[2 * slot + 1];
  }
#pragma unroll
  for (int sh = 32; sh >= 1; sh >>= 1) {
    e2 += __shfl_xor(e2, sh, 64);
    x2 += __shfl_xor(x2, sh, 64);
  }
  double *o = out + 2 * i;
  if constexpr (W == 1) {
    if (t == 0) {
      o[0] = e2;
      o[1] = x2;
    }
  } else {
    __shared__ double se[4], sx[4];
    if ((t & 63) == 0) {
      se[t >> 6] = e2;
      sx[t >> 6] = x2;
    }
    __syncthreads();
    if (t == 0) {
      o[0] = ((se[0] + se[1]) + se[2]) + se[3];
      o[1] = ((sx[0] + sx[1]) + sx[2]) + sx[3];
    }
  }
}

}  // namespace

size_t encode_noise_scratch_bytes(const Problem &pb) {
  if (pb.depth > 2) return 0;
  return (size_t)(noise_slots<0>(pb) + noise_slots<1>(pb)) * 2 * sizeof(double);
}

int launch_encode_noise(const Problem &pb, const DeviceTables &tab, const float *A, const float *B,
                        const uint8_t *ws, const Workspace &wl, double *out, void *scratch, void *stream) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (pb.batch == 0 || pb.T == 0) return hipSuccess;
  double *pa = reinterpret_cast<double *>(scratch);
  double *pbp = pa + noise_slots<0>(pb) * 2;
  hipError_t e;
  if (pb.M > 0 && pb.K > 0) {
    e = pb.depth == 1 ? launch_noise_side<0, 1>(pb, A, a_tab(tab), ws + wl.a_codes, ws + wl.a_scales, pa, st)
                      : launch_noise_side<0, 2>(pb, A, a_tab(tab), ws + wl.a_codes, ws + wl.a_scales, pa, st);
    if (e != hipSuccess) return e;
  }
  if (pb.N > 0 && pb.K > 0) {
    e = pb.depth == 1 ? launch_noise_side<1, 1>(pb, B, b_tab(tab), ws + wl.b_codes, ws + wl.b_scales, pbp, st)
                      : launch_noise_side<1, 2>(pb, B, b_tab(tab), ws + wl.b_codes, ws + wl.b_scales, pbp, st);
    if (e != hipSuccess) return e;
  }
  const NoiseSide na = noise_side<0>(pb, pa), nb = noise_side<1>(pb, pbp);
  const int64_t total = pb.batch * 2 * pb.T;
  if (std::max(na.tiles * na.wpt, nb.tiles * nb.wpt) <= 256)
    hipLaunchKernelGGL(noise_reduce_kernel<1>, dim3((unsigned)((total + 3) / 4)), dim3(256), 0, st, na, nb, out, pb.T, total);
  else
    hipLaunchKernelGGL(noise_reduce_kernel<4>, dim3((unsigned)total), dim3(256), 0, st, na, nb, out, pb.T, total);
  return hipGetLastError();
}


namespace {

template <int DEPTH, int BS, bool F32, int CAP>
hipError_t launch_pair(const Problem &pb, PairArgs &g, hipStream_t st) {
  using TA = Tile<DEPTH, 16, 0, false, CAP>;
  using TB = Tile<DEPTH, 16, 1, narrow_b(1, DEPTH, BS, 0) || pair_n1<DEPTH, BS>(), CAP>;
  auto tiles = [](int64_t n, int64_t t) { return (n + t - 1) / t; };
  g.tiles_l[0] = tiles(pb.kp, TA::TL);
  g.tiles_l[1] = tiles(pb.kp, TB::TL);
  g.tiles[0] = (unsigned)(g.tiles_l[0] * tiles(pb.mp, TA::TR));
  g.tiles[1] = (unsigned)(g.tiles_l[1] * tiles(pb.np, TB::TR));
  const dim3 grid(g.tiles[0] + g.tiles[1], (unsigned)pb.batch);
  hipLaunchKernelGGL((encode_pair_kernel<DEPTH, BS, F32, CAP>), grid, dim3(pair_threads<DEPTH, BS>()), 0, st, pb, g);
  return hipGetLastError();
}

template <int DEPTH, int CAP = 0>
hipError_t launch_pair_any(const Problem &pb, PairArgs &g, hipStream_t st) {
  const bool f32 = pb.rule == dev::RULE_FP32_AMAX;
  switch (pb.block) {
    case 16: return f32 ? launch_pair<DEPTH, 16, true, CAP>(pb, g, st) : launch_pair<DEPTH, 16, false, CAP>(pb, g, st);
    case 32: return f32 ? launch_pair<DEPTH, 32, true, CAP>(pb, g, st) : launch_pair<DEPTH, 32, false, CAP>(pb, g, st);
    case 128: return f32 ? launch_pair<DEPTH, 128, true, CAP>(pb, g, st) : launch_pair<DEPTH, 128, false, CAP>(pb, g, st);
  }
  return hipErrorInvalidValue;
}

// When both sides go in one launch, which saves a launch's latency and fills the
// chip better where a side has few workgroups, but gives the sides one workgroup
// size and LDS footprint (us, separate / one launch below).
// Depth 1: A's best workgroup is two waves with a tile of 16 KB, nine to a CU; in
// the shared launch, where B's tile sets the LDS, fewer of A's tiles are in
// flight, so A's tile count decides. Blocks 16 and 32, up to 4608 (A of M x K,
// its tiles): 3132x4928 (3920) 33.0 / 30.2, 4096x5632 (5630) 37.3 / 39.3, 7180x4672
// (8530) 57.6 / 64.2, 343 of 1636x64 (35300) 114 / 165; block 128, two of whose
// workgroups fill a CU, up to 1280: 6226x512 (780) 15.0 / 12.8, 4 of 4348x256 (1090)
// 20.8 / 15.4, 3084x1536 (1160) 18.1 / 16.1, 3090x2304 (1750) 18.8 / 20.9, 7 of 1024x1024 (1790) 17.9 / 20.7, 113
// of 110x512 (1580) 16.9 / 27.5, 5734x3328 (4670) 31.0 / 38.8. Many bytes gain nothing
// (whole tiles counted): 302 MB 87.9 / 91.9, 537 MB 143 / 154 (block 32), 134 MB
// 59.4 / 61.6, 497 of 20x256 by 256x90 (81 MB) 31.0 / 37.9 (block 128).
// Depth 2, whose sides have one workgroup size by themselves: always (8192^3 286 /
// 274, 1024^3 19.1 / 10.6, 180 of 768^3 393 / 348, 404 of 1024x512x1024 1056 / 969, 38 of
// 636x3392x4028 1836 / 1699) but for large batches of products of 1 to 2 MiB (190 of
// 512^3 186 / 199, 405 372 / 412, 810 of 256x512x256 358 / 387; 71 of 512^3 73 / 63, 324 of
// 640x512x640 356 / 356, 1621 of 256^3 404 / 370) and, past 1 GiB, of some 6 to 18 (99 of
// 1024x2048x1024 736 / 804, 220 of 528x2048x300 777 / 813, 266 of 1288x1664x224 1739 /
// 1813; 203 of 1024x512x2048, 6 MiB, 881 / 782, 137 of 1368x1536x2104, 20, 1695 / 1582).
// Other shapes, on the sixteen-wave tiles over up to 16 blocks: always where
// both sides stage them anyway (more than 8 blocks; <3,3,3;27> 5 MB 14.0 / 8.1,
// 302 MB 186 / 180). Smaller grids trade their wider depth-1 tiles for it:
// with four blocks and more a side up to 128 MiB, at block 128 32, an A of four
// blocks beyond 24 only beside a B as large (<2,2,3;11> block 32, A + B: 8 + 13 MB
// 24.4 / 15.6, 24 + 177 90.2 / 85.1, 38 + 113 65.1 / 63.8, 38 + 14 25.4 / 27.5,
// 88 + 33 52.2 / 60.0, 88 + 66 63.9 / 69.0; block 128: 21 MB 23.7 / 17.3, 37 MB
// 24.2 / 21.9, 86 MB 45.1 / 52.1); with fewer, of which a tile
// holds little, by their tiles of 1024 positions per block, up to 1792, at block 128
// 768 (block 32: <3,1,3;9> 1660 tiles 14.6 / 15.0, 2560 18.5 / 21.3, 5250 32.2 / 42.3,
// <1,2,4;8> 1030 14.2 / 10.5, 6900 37.5 / 54.4; block 128: <3,1,3;9> 1030 13.3 / 9.8,
// 3000 24.9 / 31.6, <1,2,4;8> 770 16.6 / 11.3, 960 14.8 / 19.9, 1160 15.2 / 19.2).
bool one_launch(const Problem &pb) {
  if (pb.b_rows > 1 || pb.b_bf16 || pb.depth > 2) return false;
  constexpr int64_t MiB = int64_t(1) << 20;
  auto up = [](int64_t n, int64_t t) { return (n + t - 1) / t * t; };
  const int64_t each = 4 * (pb.M * pb.K + pb.K * pb.N), bytes = pb.batch * each;
  const bool wide = pb.block == 128;
  if (pb.shaped) {
    const int na = pb.gm * pb.gk, nb = pb.gk * pb.gn;
    if (na > 16 || nb > 16) return false;
    if (na < 4 || nb < 4) return pb.batch * pb.kp * (pb.mp + pb.np) <= (wide ? 768 : 1792) * 1024;
    const int64_t a = 4 * pb.batch * pb.M * pb.K;
    return (na > 8 && nb > 8) || (bytes <= (wide ? 32 : 128) * MiB && (na > 4 || a <= 24 * MiB || 2 * a <= bytes));
  }
  if (pb.depth == 2) {
    // (1024 threads a tile of at least 8 rows x 64 positions, fewer than 2^32 on the axis)
    if ((up(pb.mp, 8) + up(pb.np, 8)) / 8 * (up(pb.kp, 64) / 64) >= int64_t(1) << 22) return false;
    return !(bytes > 256 * MiB && each >= MiB && each <= 9 * MiB / 4) &&
           !(bytes > 1024 * MiB && each >= 25 * MiB / 4 && each <= 18 * MiB);
  }
  using TA = Tile<1, 16, 0>;
  const int64_t a = pb.batch * up(pb.mp, TA::TR) * up(pb.kp, TA::TL);       // positions of A's tiles
  const int64_t b = pb.batch * up(pb.np, kB1Rows) * up(pb.kp, wide ? 128 : 64);
  return a <= (wide ? 1280 : 4608) * TA::TR * TA::TL && 16 * (a + b) <= (wide ? 64 : 192) * MiB;
}

}  // namespace

int launch_encode(const Problem &pb, const DeviceTables &tab, const float *A, const float *B,
                  uint8_t *ws, const Workspace &wl, void *stream) {
  if (pb.batch == 0 || pb.M == 0 || pb.N == 0 || pb.K == 0) return hipSuccess;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (one_launch(pb)) {
    PairArgs g;
    g.src[0] = A; g.src[1] = B;
    g.cf[0] = a_tab(tab); g.cf[1] = b_tab(tab);
    g.codes[0] = ws + wl.a_codes; g.codes[1] = ws + wl.b_codes;
    g.scales[0] = ws + wl.a_scales; g.scales[1] = ws + wl.b_scales;
    if (pb.shaped) return launch_pair_any<2, 16>(pb, g, st);
    return pb.depth == 1 ? launch_pair_any<1>(pb, g, st) : launch_pair_any<2>(pb, g, st);
  }
  hipError_t e = launch_side<0>(pb, A, a_tab(tab), ws + wl.a_codes, ws + wl.a_scales, st);
  if (e != hipSuccess) return e;
  if (pb.b_rows > 1 || pb.b_bf16)
    return launch_b_deploy_any(pb, B, b_tab(tab), ws + wl.b_codes, ws + wl.b_scales, st);
  return launch_side<1>(pb, B, b_tab(tab), ws + wl.b_codes, ws + wl.b_scales, st);
}

}  // namespace fmm
