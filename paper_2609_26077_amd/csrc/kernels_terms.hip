// Sub-products and W-combine with one wave per inner term, for products that
// are too small or too ragged for the 128 x 128 and 256-row tiles.
//
// A workgroup of eight waves owns a small tile (32 TA rows x 32 TB columns)
// of the m' x n' grid, one outer term and one product.  Wave w runs the whole
// K loop of inner term r_i = w, so the R <= 8 terms that the fused kernels
// walk one behind the other run side by side; then the waves exchange their
// P_r through LDS and form the four quadrants sum_r w[r][q] P_r, ascending r,
// one fused multiply-add per nonzero weight (the order of the other paths).
//
// Small products are bound by latency: a 256^3 product is one 128 x 128 tile,
// whose workgroup waited for seven terms' transfers in turn while 255 CUs had
// nothing to do.  Here the operands go from L2 straight into the fragment
// registers (the next step's loads in flight under the current step's matrix
// instructions), with no LDS staging and no barrier before the exchange.
// Ragged plans (FMM_LAYOUT_ROWS) take the same kernel: a lane addresses its
// own row, rows past the end repeat the last one (their outputs are not
// stored) and 16-byte chunks past k' read as zero.
//
// Operand forms, by plan:
//   MX      E8M0 scales, blocks 32 and 128: v_mfma_scale_f32_32x32x64_f8f6f4
//   DQ      E8M0 scales, exact-dot flag or block 16: each code converted to
//           bf16 with its block's power of two, v_mfma_f32_32x32x16_bf16.
//           (The tiled 64-edge forms spill 8 to 10 of their 256 registers.)
//           The exponents enter one lower on both sides (so that no code
//           overflows at the largest scale, 2^120) and P_r is multiplied by 4.
//           In the tiled layout the instructions accumulate over the whole
//           contracted axis, as the 128 x 128 kernel's do; in the row layout
//           each block (at block 16 each two: an instruction spans both) is
//           summed by itself and added to the fp32 accumulator.
//           (The matrix core truncates what falls below its accumulator's last
//           bit at every instruction: over k' = 4096 with rows scaled over four
//           decades the error against 64 bits is 2.0e-7 of |C| by blocks of
//           128 and 4.8e-7 in one accumulation, over 256 8.3e-8 either way.)
//   PROMOTE fp32 scales: codes to bf16 at scale 1, each block's partial sum
//           times sA sB (formed for the 32 x 32 tile by one
//           v_mfma_f32_32x32x2_f32: sA and sB in the first contracted position,
//           zeros in the second) into the fp32 accumulator
#include <hip/hip_runtime.h>

#include <cmath>

#include "device.h"
#include "internal.h"

namespace fmm {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
using dev::dequant8;
using dev::e8m0_at;
using dev::v8bf;

enum { MX = 0, DQ = 1, PROMOTE = 2 };

constexpr int kThreads = 512;
constexpr int kStep = 128;          // contracted bytes per step

struct TermArgs {
  const uint8_t *xa, *xb, *sa, *sb;
  float *out;                       // C (depth 1) or partial products (depth >= 2)
  const float *w;                   // R x 4 base decoder weights (zero-padded)
  int64_t mp, np, kp, kblocks, T, To, M, N;
  int64_t first;                    // this launch's first (product, outer term, tile) item
  int R, depth, tiles_m, tiles_n;
};

// One side's operand of one wave: NT row tiles of 32 rows.
template <int LAYOUT, int MODE, int BS, int NT>
struct Side {
  static constexpr bool BLOCKS = MODE == PROMOTE || (MODE == DQ && LAYOUT == FMM_LAYOUT_ROWS);   // each block summed by itself
  static constexpr bool PIECES = MODE == PROMOTE && BS == 16;   // 8-byte pieces, one block per instruction
  static constexpr int NSC = MODE == PROMOTE ? kStep / BS : 1;  // scale words a lane holds per step
  const uint8_t *row[NT];      // the lane's row of each tile (its first step)
  const uint8_t *scale[NT];    // its scales
  uint32_t x;                  // the row's chunk swizzle (tiled layout; rows 32 apart share it)

  struct Frag {
    v8i v[2][NT];              // substep s: bytes 64 s + 16 h and 64 s + 32 + 16 h (16 each) of the row
    uint32_t sc[NT][NSC];
  };

  __device__ __forceinline__ void init(const TermArgs &g, const uint8_t *codes, const uint8_t *scales, int64_t rows,
                                       int64_t plane, int64_t row0, int r32) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int64_t p0 = row0 + 32 * i + r32, p = p0 < rows ? p0 : rows - 1;
      if constexpr (LAYOUT == FMM_LAYOUT_TILE128x128) {
        const int64_t tile = (plane * (rows / 128) + p / 128) * (g.kp / 128);
        row[i] = codes + tile * 16384 + (p & 127) * 128;
        scale[i] = scales + (tile * 128 + (p & 127)) * (BS == 16 ? 8 : 4);
      } else {
        row[i] = codes + (plane * rows + p) * g.kp;
        scale[i] = scales + (plane * rows + p) * g.kblocks * (MODE == PROMOTE ? 4 : 1);
      }
    }
    x = (uint32_t)((r32 & 7) ^ ((r32 >> 3) & 1));
  }

  // the fragments and scales of step ks
  __device__ __forceinline__ void load(const TermArgs &g, int ks, int h, Frag &f) const {
    if constexpr (LAYOUT == FMM_LAYOUT_TILE128x128) {
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const uint8_t *p = row[i] + (int64_t)ks * 16384;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint4 q = *reinterpret_cast<const uint4 *>(p + 16 * ((uint32_t)(2 * c + h) ^ x));
          put(f.v[c >> 1][i], c & 1, q);
        }
        const uint8_t *s = scale[i] + (int64_t)ks * (128 * (BS == 16 ? 8 : 4));
        if constexpr (MODE == MX) f.sc[i][0] = *reinterpret_cast<const uint16_t *>(s + 2 * h);
        else if constexpr (BS == 16) f.sc[i][0] = *reinterpret_cast<const uint32_t *>(s + 4 * h);
        else f.sc[i][0] = *reinterpret_cast<const uint32_t *>(s);
      }
    } else {
      const int64_t k0 = (int64_t)ks * kStep;
      const int left = (int)(g.kp - k0 < kStep ? g.kp - k0 : kStep);   // bytes of this step (a multiple of 16)
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const uint8_t *p = row[i] + k0;
        if constexpr (PIECES) {
#pragma unroll
          for (int b = 0; b < 8; ++b) {
            uint2 q = make_uint2(0, 0);
            if (16 * b < left) q = *reinterpret_cast<const uint2 *>(p + 16 * b + 8 * h);
            f.v[b >> 2][i][2 * (b & 3)] = (int)q.x;
            f.v[b >> 2][i][2 * (b & 3) + 1] = (int)q.y;
          }
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            uint4 q = make_uint4(0, 0, 0, 0);
            if (16 * (2 * c + h) < left) q = *reinterpret_cast<const uint4 *>(p + 16 * (2 * c + h));
            put(f.v[c >> 1][i], c & 1, q);
          }
        }
        const int kb0 = (int)(k0 / BS), nb = (int)g.kblocks - kb0;     // the step's first block, blocks left
        if constexpr (MODE == PROMOTE) {
          const float *s = reinterpret_cast<const float *>(scale[i]) + kb0;
#pragma unroll
          for (int b = 0; b < NSC; ++b) f.sc[i][b] = h == 0 && b < nb ? __float_as_uint(s[b]) : 0u;
        } else {
          // E8M0 bytes: MX those of the lane's own instruction halves, DQ (block 16: the
          // lane half's own) in the order of the instructions (127 = 1 past the end)
          const uint8_t *s = scale[i] + kb0;
          auto at = [&](int b) -> uint32_t { return b < nb ? s[b] : 127u; };
          if constexpr (BS == 128) f.sc[i][0] = s[0] * 0x01010101u;
          else if constexpr (MODE == MX) f.sc[i][0] = at(h) | at(2 + h) << 8;
          else if constexpr (BS == 32) f.sc[i][0] = at(0) | at(1) << 8 | at(2) << 16 | at(3) << 24;
          else f.sc[i][0] = at(h) | at(2 + h) << 8 | at(4 + h) << 16 | at(6 + h) << 24;
        }
      }
    }
    if constexpr (MODE == DQ) {
#pragma unroll
      for (int i = 0; i < NT; ++i) f.sc[i][0] -= 0x01010101u;      // bytes are at least 79: no borrow
    }
  }

  static __device__ __forceinline__ void put(v8i &v, int half, uint4 q) {
    v[4 * half] = (int)q.x; v[4 * half + 1] = (int)q.y; v[4 * half + 2] = (int)q.z; v[4 * half + 3] = (int)q.w;
  }
};

template <int LAYOUT, int MODE, int BS, int TA, int TB>
__global__ __launch_bounds__(kThreads, (TA * TB == 1 && MODE != PROMOTE ? 4 : 2)) void gemm_terms_kernel(TermArgs g) {
  using SA = Side<LAYOUT, MODE, BS, TA>;
  using SB = Side<LAYOUT, MODE, BS, TB>;
  __shared__ float lds[8][TA * TB][16][64];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r32 = lane & 31, h = lane >> 5;

  // Workgroups are dispatched round-robin over the eight XCDs: XCD x takes a
  // contiguous range of the (product, outer term, tile) items, so the tiles of
  // one item read its codes through one L2.
  int tm, tn;
  int64_t ro, bt;
  {
    const int64_t G = gridDim.x, L = blockIdx.x, x = L & 7;
    const int64_t id = g.first + x * (G >> 3) + min(x, G & 7) + (L >> 3);
    const int ntiles = g.tiles_m * g.tiles_n;
    const int64_t item = id / ntiles;
    const int tile = (int)(id - item * ntiles);
    constexpr int GM = 8;                                 // groups of eight tile rows
    const int per_group = GM * g.tiles_n, group = tile / per_group, first_m = group * GM;
    const int gm = min(g.tiles_m - first_m, GM), in = tile - group * per_group;
    tm = first_m + in % gm;
    tn = in / gm;
    ro = item % g.To;
    bt = item / g.To;
  }
  const int64_t pm0 = (int64_t)tm * (32 * TA), pn0 = (int64_t)tn * (32 * TB);

  if (wave < g.R) {
    const int64_t plane = bt * g.T + ro * g.R + wave;
    SA a;
    SB b;
    a.init(g, g.xa, g.sa, g.mp, plane, pm0, r32);
    b.init(g, g.xb, g.sb, g.np, plane, pn0, r32);
    v16f acc[TA][TB];
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j) acc[i][j] = (v16f){};

    auto mul = [&](const typename SA::Frag &fa, const typename SB::Frag &fb) {
      if constexpr (MODE == MX) {
#define FMM_MX_SUB(S)                                                                                   \
  _Pragma("unroll") for (int i = 0; i < TA; ++i) _Pragma("unroll") for (int j = 0; j < TB; ++j)         \
      acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa.v[S][i], fb.v[S][j], acc[i][j], 0, \
                                                                  0, S, (int)fa.sc[i][0], S, (int)fb.sc[j][0])
        FMM_MX_SUB(0);
        FMM_MX_SUB(1);
#undef FMM_MX_SUB
      } else if constexpr (!SA::BLOCKS) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int c = u >> 1, d = 4 * c + 2 * (u & 1);
            const int byte = BS == 16 ? 2 * s + c : BS == 32 ? 2 * c + s : 0;
            v8bf va[TA], vb[TB];
#pragma unroll
            for (int i = 0; i < TA; ++i) va[i] = dequant8(fa.v[s][i][d], fa.v[s][i][d + 1], e8m0_at(fa.sc[i][0], byte));
#pragma unroll
            for (int j = 0; j < TB; ++j) vb[j] = dequant8(fb.v[s][j][d], fb.v[s][j][d + 1], e8m0_at(fb.sc[j][0], byte));
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
              for (int j = 0; j < TB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], vb[j], acc[i][j], 0, 0, 0);
          }
      } else {
        constexpr int PER = MODE == DQ && BS == 16 ? 2 : BS / 16;   // instructions per sum
        v16f part[TA][TB];
#pragma unroll
        for (int n = 0; n < 8; ++n) {
          const int s = n >> 2, u = n & 3;
          const int d = SA::PIECES ? 2 * u : 4 * (u >> 1) + 2 * (u & 1);
          const int blk = n / PER;
          auto scale_of = [&](const uint32_t *sc) { return MODE == PROMOTE ? 1.0f : e8m0_at(sc[0], blk); };
          v8bf va[TA], vb[TB];
#pragma unroll
          for (int i = 0; i < TA; ++i) va[i] = dequant8(fa.v[s][i][d], fa.v[s][i][d + 1], scale_of(fa.sc[i]));
#pragma unroll
          for (int j = 0; j < TB; ++j) vb[j] = dequant8(fb.v[s][j][d], fb.v[s][j][d + 1], scale_of(fb.sc[j]));
#pragma unroll
          for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j)
              part[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], vb[j], n % PER == 0 ? (v16f){} : part[i][j], 0, 0, 0);
          if (n % PER == PER - 1) {
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
              for (int j = 0; j < TB; ++j) {
                if constexpr (MODE == DQ) {
#pragma unroll
                  for (int e = 0; e < 16; ++e) acc[i][j][e] = __fadd_rn(acc[i][j][e], part[i][j][e]);
                  continue;
                }
                const v16f s2 = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa.sc[i][blk]), __uint_as_float(fb.sc[j][blk]),
                                                                     (v16f){}, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = __fmaf_rn(s2[e], part[i][j][e], acc[i][j][e]);
              }
          }
        }
      }
    };

    const int nk = (int)((g.kp + kStep - 1) / kStep);
    if constexpr (SA::BLOCKS && TA * TB > 1) {
      // two accumulator sets leave no registers for a second fragment set
      for (int ks = 0; ks < nk; ++ks) {
        typename SA::Frag fa;
        typename SB::Frag fb;
        a.load(g, ks, h, fa);
        b.load(g, ks, h, fb);
        mul(fa, fb);
      }
    } else {
      typename SA::Frag fa0, fa1;
      typename SB::Frag fb0, fb1;
      if (nk > 0) {
        a.load(g, 0, h, fa0);
        b.load(g, 0, h, fb0);
      }
      for (int ks = 0; ks < nk; ks += 2) {
        if (ks + 1 < nk) {
          a.load(g, ks + 1, h, fa1);
          b.load(g, ks + 1, h, fb1);
        }
        mul(fa0, fb0);
        if (ks + 1 < nk) {
          if (ks + 2 < nk) {
            a.load(g, ks + 2, h, fa0);
            b.load(g, ks + 2, h, fb0);
          }
          mul(fa1, fb1);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) lds[wave][i * TB + j][e][lane] = MODE == DQ ? 4.0f * acc[i][j][e] : acc[i][j][e];
  }
  __syncthreads();

  // register e of a 32 x 32 tile: row 8 (e / 4) + 4 h + e % 4, column lane % 32
  const int64_t ld = g.depth == 1 ? g.N : g.To * 4 * g.np;
  constexpr int ROWS_E = TA * TB * 16;
#pragma unroll
  for (int k = 0; k < ROWS_E / 8; ++k) {
    const int idx = wave + 8 * k, tile = idx >> 4, e = idx & 15;
    float q[4] = {0.f, 0.f, 0.f, 0.f};
    for (int r = 0; r < g.R; ++r) {
      const float p = lds[r][tile][e][lane];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float wq = g.w[4 * r + c];
        if (wq != 0.0f) q[c] = __fmaf_rn(wq, p, q[c]);
      }
    }
    const int64_t row = pm0 + 32 * (tile / TB) + 8 * (e >> 2) + 4 * h + (e & 3), col = pn0 + 32 * (tile % TB) + r32;
    if (row < g.mp && col < g.np) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float *o = g.depth == 1 ? g.out + bt * g.M * g.N + ((c & 1) * g.mp + row) * ld + (c >> 1) * g.np + col
                                : g.out + (bt * g.mp + row) * ld + (ro * 4 + c) * g.np + col;
        *o = q[c];
      }
    }
  }
}

template <int LAYOUT, int MODE, int BS>
hipError_t launch_edge(const TermArgs &args, int64_t batch, hipStream_t st, int edge) {
  TermArgs g = args;
  const int64_t t = edge;
  g.tiles_m = (int)((g.mp + t - 1) / t);
  g.tiles_n = (int)((g.np + t - 1) / t);
  // HIP takes fewer than 2^32 threads on a grid axis: more workgroups than that
  // (8.4 million: tens of GB of small products) go in several launches
  constexpr int64_t kMaxGrid = (int64_t(1) << 32) / kThreads - 8;
  const int64_t items = (int64_t)g.tiles_m * g.tiles_n * g.To * batch;
  for (g.first = 0; g.first < items; g.first += kMaxGrid) {
    const dim3 grid((unsigned)(items - g.first < kMaxGrid ? items - g.first : kMaxGrid));
    if (edge == 32) hipLaunchKernelGGL((gemm_terms_kernel<LAYOUT, MODE, BS, 1, 1>), grid, dim3(kThreads), 0, st, g);
    else hipLaunchKernelGGL((gemm_terms_kernel<LAYOUT, MODE, BS, 2, 2>), grid, dim3(kThreads), 0, st, g);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Which products take this kernel, by the number of workgroups n32 and n64
// (tiles of 32 or 64 rows and columns, times outer terms, times products) and
// n128 of the 128 x 128 tiles.
//
// Tiled layout (E8M0 scales): while the 128 x 128 tiles fill less than a third
// of the chip.  One round of those takes R (0.66 k'/128 + 2.1) us whatever
// their number, this kernel's 32-edge tiles about 4 + n32 (0.0075 + 0.0027
// k'/128) us, so they meet near n32 = 16 n128 = 1280 at every k' (us, this
// kernel against 128 x 128 tiles: 256^3 n32 = 16 7.5 / 13.8, 1024 12.6 / 14.8,
// 1600 20.4 / 15.9; 512^3 64 7.4 / 18.2, 1024 14.9 / 19.2, 2048 27.7 / 21.5;
// 1024^3 256 7.7 / 26.7, 1024 21 / 28, 2048 39 / 32).  64-edge tiles
// halve the bytes per flop but hold a CU each: a round takes 10 + 2 k'/128 us, less than the
// 32-edge tiles from n32 = 768 on (2048x1024x2048: 18.9 / 20.5, 2048^3 one
// more step in k': 26 / 33), and only the first round is worth it.
//
// Row layout, fp32 scales at blocks 16 and 32: 64-edge tiles from 560 32-edge tiles
// per round of them on (k' 2048 2000x2000: 828 / 453; k' 128 127x127, 2800 of them:
// 1036 / 754; k' 8192 100x2000: 200 / 411).
//
// Row layout otherwise: the least of three fitted times, of this kernel on either
// tile and of the 128 x 128 kernels, gemm_mx_kernel and at block 128
// gemm_promote_kernel (at blocks 16 and 32 its like lost to this kernel at every
// size measured). Rounds r32, r64 and r128 are the workgroups over the CUs; several
// 32-edge workgroups share a CU and start as others end, 64-edge ones hold a CU each
// (their time goes by whole rounds and, with L2 shared, by the tiles), a round of
// 128 x 128 tiles walks its R terms in turn:
//   t32 = r32 (a + b nk)    t64 = r64 (c + d nk) + ceil(r64) (e + f nk)
//   t128 = R ceil(r128) (g + h nk)         us, nk = k' / 128 rounded up
// The per-term kernel's lanes read rows k' apart straight from L2: at k' a multiple
// of 256 or 1024 their codes and short rows of scales (blocks 16 and 32) meet on few
// of its channels, 1.3 and 1.65 times on 32-edge tiles, 1.15 and 1.3 on 64-edge ones;
// block 128 shows 1.15 from k' 3072 on.
// Fitted to 3400 plans of k' 32 .. 2200, 40 .. 6000 tiles of 128 and depths 1 to 3,
// then t32 raised by 4% and t128 by 2 to 4% (the costlier mistakes); on another 1000
// the choice is on average 1% off the best. Measured, us, 32 / 64 / 128 edge (k', m' x
// n', r128):
//   fp8, block 32   96 387x579 9.8 351 / 420 / 383; 160 203x503 1.5 68 / 91 / 105;
//                   928 263x559 8.6 1192 / 905 / 1400; 2048 2000x2000 1.0 592 / 331 / 300
//   fp8, block 128  128 1144x1576 3.2 167 / 165 / 143; 256 2439x52 0.9 40 / 36 / 56;
//                   2048 2000x2000 1.0 446 / 259 / 295
//   exact-dot, 128  128 112x226 11.3 685 / 633 / 521; 128 35x610 1.1 33 / 36 / 72;
//                   256 106x86 20.5 1307 / 1513 / 1312; 2048 2000x2000 1.0 449 / 271 / 324
//   fp32 scales, 128  128 128x128 10.5 855 / 641 / 462; 128 1326x123 0.95 69 / 53 / 45;
//                   256 512x768 4.6 488 / 342 / 304; 2048 2000x2000 1.0 534 / 296 / 328
struct EdgeTimes {
  double a, b, c, d, e, f, g, h;    // g = 0: no 128 x 128 kernel
};
EdgeTimes edge_times(const Problem &pb) {
  const bool wide = pb.block == 128;
  if (pb.scale_bytes == 4) return {2.75, 2.1, 1.75, 1.9, 7.0, 2.5, 2.75, 2.75};
  if (pb.exact_dot && wide) return {2.05, 1.83, 2.15, 1.0, 6.9, 2.9, 2.65, 2.65};
  if (pb.exact_dot || pb.block == 16) return {1.1, 2.15, 1.1, 2.6, 5.2, 3.5, 0, 0};
  if (wide) return {1.85, 1.8, 0.95, 2.1, 7.6, 1.65, 2.25, 2.4};
  return {1.25, 1.5, 1.5, 1.65, 5.3, 2.15, 2.05, 2.5};
}

}  // namespace

int terms_edge(const Problem &pb) {
  auto count = [&](int64_t e) { return ((pb.mp + e - 1) / e) * ((pb.np + e - 1) / e) * pb.To * pb.batch; };
  const int64_t n32 = count(32), n64 = count(64), n128 = count(128), ncu = pb.ncu;
  if (pb.layout == FMM_LAYOUT_TILE128x128) {
    if (16 * n128 > 5 * ncu) return 0;
    return n32 > 3 * ncu && n64 <= ncu ? 64 : 32;
  }
  const double r32 = (double)n32 / ncu, r64 = (double)n64 / ncu;
  if (pb.scale_bytes == 4 && pb.block != 128) return r32 > 35.0 / 16 * std::ceil(r64) ? 64 : 32;
  const EdgeTimes t = edge_times(pb);
  const double nk = (double)((pb.kp + kStep - 1) / kStep);
  const bool far = pb.block == 128 && pb.kp >= 3072, even = pb.block < 128 && pb.kp % 256 == 0, most = even && pb.kp % 1024 == 0;
  const double t32 = (most ? 1.65 : even ? 1.3 : far ? 1.15 : 1.0) * r32 * (t.a + t.b * nk);
  const double t64 = (most ? 1.3 : even || far ? 1.15 : 1.0) * (r64 * (t.c + t.d * nk) + std::ceil(r64) * (t.e + t.f * nk));
  const double t128 = pb.R * std::ceil((double)n128 / ncu) * (t.g + t.h * nk);
  if (t.g > 0 && t128 < t32 && t128 < t64) return 0;
  return t64 < t32 ? 64 : 32;
}

int launch_products_terms(const Problem &pb, const DeviceTables &tab, const uint8_t *ws, const Workspace &wl,
                          float *C, int edge, void *stream) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  TermArgs g;
  g.xa = ws + wl.a_codes; g.xb = ws + wl.b_codes;
  g.sa = ws + wl.a_scales; g.sb = ws + wl.b_scales;
  g.out = pb.depth == 1 ? C : reinterpret_cast<float *>(const_cast<uint8_t *>(ws) + wl.partial);
  g.w = tab.w_inner;
  g.mp = pb.mp; g.np = pb.np; g.kp = pb.kp; g.kblocks = pb.kblocks;
  g.T = pb.T; g.To = pb.To; g.M = pb.M; g.N = pb.N;
  g.R = pb.R; g.depth = pb.depth; g.tiles_m = g.tiles_n = 0; g.first = 0;
  const bool tiled = pb.layout == FMM_LAYOUT_TILE128x128;
#define FMM_TERMS(L, MODE, BS) return launch_edge<L, MODE, BS>(g, pb.batch, st, edge)
  if (pb.scale_bytes == 4) {
    if (pb.block == 16) FMM_TERMS(FMM_LAYOUT_ROWS, PROMOTE, 16);
    if (pb.block == 32) FMM_TERMS(FMM_LAYOUT_ROWS, PROMOTE, 32);
    FMM_TERMS(FMM_LAYOUT_ROWS, PROMOTE, 128);
  }
  if (pb.block == 16) {
    if (tiled) FMM_TERMS(FMM_LAYOUT_TILE128x128, DQ, 16);
    FMM_TERMS(FMM_LAYOUT_ROWS, DQ, 16);
  }
  if (pb.exact_dot) {
    if (tiled && pb.block == 32) FMM_TERMS(FMM_LAYOUT_TILE128x128, DQ, 32);
    if (tiled) FMM_TERMS(FMM_LAYOUT_TILE128x128, DQ, 128);
    if (pb.block == 32) FMM_TERMS(FMM_LAYOUT_ROWS, DQ, 32);
    FMM_TERMS(FMM_LAYOUT_ROWS, DQ, 128);
  }
  if (tiled && pb.block == 32) FMM_TERMS(FMM_LAYOUT_TILE128x128, MX, 32);
  if (tiled) FMM_TERMS(FMM_LAYOUT_TILE128x128, MX, 128);
  if (pb.block == 32) FMM_TERMS(FMM_LAYOUT_ROWS, MX, 32);
  FMM_TERMS(FMM_LAYOUT_ROWS, MX, 128);
#undef FMM_TERMS
}

}  // namespace fmm
