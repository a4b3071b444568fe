// Queue-driven peeling solver: routing where water runs in every direction,
// several receivers per cell (MFD masks, forward and adjoint) or one (D8 /
// D4 codes, adjoint).  Solves (I - W^T) q = r, or (I - W) rbar = qbar, on
// any acyclic routing (Section 2.1, Section 2.2; fractions as in Appendix A).
//
// A cell is computed ("peeled") once every cell that feeds it is final, by
// summing its inputs in neighbour order, so the result does not depend on
// the order in which cells become ready.  What bounds such a solve is the
// longest flow path (thousands of cells, one after another), not bytes or
// arithmetic: everything below shortens the time from one cell of a path to
// the next.
//
//   * One workgroup holds a tile of 32 x 64 cells in LDS: the fraction of
//     every edge between neighbours (one signed number per undirected edge,
//     since water crosses it one way only) and every cell's value.  A step
//     along a path inside the tile is then an LDS round trip.
//   * A lane holds one cell of every tile row: lane (2 r + c) mod 64 holds
//     cell (r, c) as bit r.  Which cells are final, and which inputs each
//     cell has, are then 32-bit masks per lane, the neighbours' masks are
//     lane rotations, all ready cells are found in about 30 vector
//     instructions, and each lane peels one of them per step.  The cells of a
//     row, of a column and of either diagonal lie in different lanes, so the
//     cells that become ready together mostly do too (with a lane per row a
//     step peeled 3 cells of a grid that drains along its columns).
//   * Values that cross tiles go through one 64-bit word per cell in device
//     memory (all ones = not final yet).  While one wavefront peels, another
//     polls the words of the cells around the tile that feed it, and a third
//     publishes the tile's own border cells and wakes the tiles they feed, so
//     the peeling wavefront never waits for memory.  The peeling wavefronts
//     of the workgroups on a compute unit run on different SIMDs.
//   * Tiles are actors on a device queue: a tile that is woken while idle is
//     queued, any workgroup takes it, loads it, peels until nothing is
//     ready, writes back what became final and lets go of it.  No workgroup
//     waits for another one to be resident, so any number of them makes
//     progress, and every wait is bounded.
//
// Measured (float32 water; the windowed wavefront sweep and, after 32 of its
// passes, an engine with grid-wide barriers did this before; both timed in
// turn in one run): filled 2048^2 MFD route 863 -> 3.9 ms; forward and gradient
// on a filled 1200 x 1601 grid 1028 -> 4.6; tilted 4096^2 adjoint 29.1 -> 13.4;
// 48 tiles of 64 to 2048 cells a side 72 -> 15.4.  Larger single grids, raw
// terrain: 8192^2 MFD 963 -> 6.3 ms, 20000^2 2441 -> 51, 30000^2 7624 -> 398.
// A step takes 0.35 to 0.4 us (a chain of lane rotations, 17 LDS reads and a
// sum of eight products), a value's way to a tile already in LDS about 3 us,
// loading a tile 15 to 25 us.  Against that: with
// the peeling wavefronts left on one SIMD a step of three workgroups on a
// compute unit took 1.0 us; tiles let go after 2 polls without news instead
// of 32 were loaded up to 4 times as often (48 tiles: 30 ms); a queue for
// each XCD with blocks of neighbouring tiles was slower throughout (raw
// 4096^2 1.7 -> 16 ms: neighbours were in LDS together less often, and a
// value's way was no shorter).  The tile is 32 x 64 because a row of it is
// then two full lines of every input, and because three such tiles with
// float32 fractions fill a compute unit's LDS (53 KB each).
//
// Arithmetic: float64 sums.  For float32 results the fractions are float32,
// t_j = (s_j / s_max)^p by the hardware log2 and exp2 and f_j = t_j / sum t
// (cells with slopes outside 2^-60 to 2^60: from float64 drops and quotients);
// a cell passes on its water times 2 - sum f (float64), which makes up for
// the rounding of its fractions to first order, as in the row sweep.  For
// float64 results the fractions are float64 (slope_log2(), slope_exp2()).
#include <limits.h>
#include <math.h>

#include <type_traits>

#include "fr_queue.hpp"
#include "fr_slopes.hpp"

namespace fr {
namespace {

constexpr int PT = 256;                // threads per workgroup
constexpr int TR = PEEL_ROWS;
constexpr uint64_t OPEN = ~0ull;       // word of a cell that is not final
// Phases of the wavefronts' roles.
constexpr int PH_RUN = 0, PH_STOP = 1;
// Full polls of the surrounding cells without news before an idle tile is
// let go: while other tiles are queued, and while none is.
constexpr int LINGER_BUSY = 32, LINGER_IDLE = 96;
__device__ constexpr float kInvSqrt2f = 0x1.6a09e6p-1f;

__device__ __forceinline__ uint32_t l_ld(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void l_st(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// LDS operations of one wavefront are performed in issue order; this keeps
// the compiler from moving data across the words that announce it.
__device__ __forceinline__ void fence() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }
__device__ __forceinline__ uint64_t ballot(bool p) { return (uint64_t)__builtin_amdgcn_ballot_w64(p); }
// x of lane - 1 / lane + 1 (mod 64).
__device__ __forceinline__ uint32_t from_below(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x13C, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t from_above(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x134, 0xF, 0xF, false);
}

__device__ __forceinline__ double bitsd(uint64_t w) { return __longlong_as_double((long long)w); }
__device__ __forceinline__ uint64_t dword(double v) {
  // A result whose upper half has those bits (a NaN) gives way to another NaN.
  const uint64_t w = (uint64_t)__double_as_longlong(v);
  const uint32_t hi = (uint32_t)(w >> 32);
  return ((uint64_t)(hi == ~0u ? 0x7FF80000u : hi) << 32) | (uint32_t)w;
}

// A tile in LDS.  Rows and columns -1 and TR / TC are the cells around the
// tile.  Edge (cell, k) with k = 4 (right), 5, 6, 7 (lower left, below, lower
// right) is kept at that cell: positive when water runs from the cell along
// k, negative against it; the value is the fraction of the giving cell.
template <typename F>
struct Tile {
  static constexpr int TC = peel_cols(sizeof(F) == 8);
  static constexpr int W = TC + 2;          // row pitch, from column -1 on
  static constexpr int PLANE = (TR + 1) * W;  // one direction's edges, from row -1 on (right edges: from row 0)
  F edge[4 * PLANE - W];
  union {
    double g[TR + 2][W];           // final: what the cell passes on; not final: its source term
    struct {                       // while fractions are computed:
      float z[TR + 4][TC + 4];     // elevations from row, column -2 on,
      uint8_t code[TR + 2][W];     // codes from row, column -1 on
    };
    uint8_t mask[11][64][4];       // while masks are built: a byte per wavefront and lane
  };
  uint32_t done[64];               // final cells per lane (while loading: per row, two words)
  uint32_t wait[64];               // cells with an input from outside that is not final, per lane
  uint32_t phase, polls, queue_empty;
  uint32_t gaps;                   // float64 fractions: some cell exchanges nothing with a neighbour
  int32_t tile, cmd;
  int32_t simd[5];                 // the wavefronts' SIMDs, the workgroup's slot
};
static_assert(sizeof(Tile<float>) <= 53760, "three float tiles per compute unit");
static_assert(sizeof(Tile<double>) <= 81920, "two float64 tiles per compute unit");

// Which lane holds cell (r, c), as bit r; the column of lane l's bit r.
__device__ __forceinline__ int lane_at(int r, int c) { return (2 * r + c) & 63; }
__device__ __forceinline__ int col_at(int l, int r) { return (l - 2 * r) & 63; }

// A cell's place in the arrays of pitch W, for addresses that differ from
// direction to direction by constants.
template <typename F>
__device__ __forceinline__ int place(int r, int c) {
  return (r + 1) * Tile<F>::W + c + 1;
}
// The edge word of the cell at place `at` along k; one of the edge's two
// cells lies in the tile.  For k < 4 it is the neighbour's edge 7 - k.
template <typename F>
__device__ __forceinline__ F* edge_at(Tile<F>& T, int at, int k) {
  constexpr int W = Tile<F>::W;
  F* first = T.edge + (at - W - 1);
  return k >= 4 ? first + ((k - 4) * Tile<F>::PLANE + 1)
                : first + ((3 - k) * Tile<F>::PLANE + nb_dr(k) * W + nb_dc(k) + 1);
}
// Fraction that runs from that cell along k (negative: toward it).
template <typename F>
__device__ __forceinline__ F out_at(Tile<F>& T, int at, int k) {
  const F w = *edge_at(T, at, k);
  return k < 4 ? -w : w;
}
template <typename F>
__device__ __forceinline__ F out_at(Tile<F>& T, int r, int c, int k) {
  return out_at(T, place<F>(r, c), k);
}

template <typename F>
__device__ __forceinline__ bool in_tile(int r, int c) {
  return (unsigned)r < (unsigned)TR && (unsigned)c < (unsigned)Tile<F>::TC;
}

// Wakes tile t: queues it when it was idle.
__device__ __forceinline__ void wake(const TileQueue& Q, uint32_t t) {
  if (atomicOr(Q.state + t, ST_PENDING) == 0u) push_tile(Q, t);
}

// Out-fractions of the cell at place `at` (its validated mask m over the 8
// neighbours at elevations zk), those of the mask `put` written to its edges.
template <typename F>
__device__ __forceinline__ void put_fractions(Tile<F>& T, int at, uint32_t put, uint32_t m, float zc,
                                              const float (&zk)[8], double p);
template <>
__device__ __forceinline__ void put_fractions<float>(Tile<float>& T, int at, uint32_t put, uint32_t m, float zc,
                                                     const float (&zk)[8], double p) {
  const float pf = (float)p;
  float s[8], smax = 0.0f, smin = INFINITY;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float drop = zc - zk[k];
    s[k] = ((m >> k) & 1u) ? (nb_diag(k) ? drop * kInvSqrt2f : drop) : 0.0f;
    smax = fmaxf(smax, s[k]);
    smin = fminf(smin, ((m >> k) & 1u) ? s[k] : INFINITY);
  }
  if (smin < SLOPE_LO || smax > SLOPE_HI) {
    wide_weights(zc, zk, m, 0xA5u, pf, s);
  } else {
    const float ism = smax > 0.0f ? __builtin_amdgcn_rcpf(smax) : 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      // s / smax, its rounding corrected once (the steepest gives 1 exactly).
      const float q = s[k] * ism;
      const float x = fmaf(fmaf(-q, smax, s[k]), ism, q);
      s[k] = ((m >> k) & 1u) ? __builtin_amdgcn_exp2f(pf * __builtin_amdgcn_logf(x)) : 0.0f;
    }
  }
  float sum = 0.0f;
#pragma unroll
  for (int k = 0; k < 8; ++k) sum += s[k];
  const float is = sum > 0.0f ? __builtin_amdgcn_rcpf(sum) : 0.0f;
  put &= m;
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if ((put >> k) & 1u) *edge_at(T, at, k) = k < 4 ? -(s[k] * is) : s[k] * is;
}
template <>
__device__ __forceinline__ void put_fractions<double>(Tile<double>& T, int at, uint32_t put, uint32_t m, float zc,
                                                      const float (&zk)[8], double p) {
  double s[8], sum = 0.0;
  if (p <= 500.0) {
    // Relative to the highest drop's binade: the steepest power is at least
    // 2^(-1.5 p).
    int e = INT_MIN;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      s[k] = (double)zc - (double)zk[k];
      const int ek = __builtin_amdgcn_frexp_exp(s[k]);
      e = ((m >> k) & 1u) && ek > e ? ek : e;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      double l, ll;
      slope_log2(s[k], nb_diag(k), e, l, ll);
      s[k] = ((m >> k) & 1u) ? slope_exp2(l, ll, p) : 0.0;
      sum += s[k];
    }
  } else {
    // Relative to the steepest slope (2% slower in all).
    double sl[8], top = -INFINITY, topl = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      slope_log2((double)zc - (double)zk[k], nb_diag(k), 0, s[k], sl[k]);
      const bool higher = ((m >> k) & 1u) && (s[k] > top || (s[k] == top && sl[k] > topl));
      top = higher ? s[k] : top;
      topl = higher ? sl[k] : topl;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const double d = s[k] - top, b = d - s[k];
      const double dl = ((s[k] - (d - b)) - (top + b)) + (sl[k] - topl);
      s[k] = ((m >> k) & 1u) ? slope_exp2(d, dl, p) : 0.0;
      sum += s[k];
    }
  }
  const double is = sum > 0.0 ? 1.0 / sum : 0.0;
  put &= m;
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if ((put >> k) & 1u) *edge_at(T, at, k) = k < 4 ? -(s[k] * is) : s[k] * is;
}

// RK_SINGLE: codes of one receiver, all of a cell's water runs there (F =
// float, fractions +-1).  VK: the precision of the result.  BATCH: the codes
// are found here, from the elevations, by the grid's rule (single receivers
// run as fractions of 1, whose correction is 1).
template <int RK, bool ADJ, int VK, bool BATCH, typename F>
__device__ __forceinline__ void peel_tile(const PeelGrid& P, const TileQueue& Q, Tile<F>& T, const int32_t tile) {
  constexpr bool CORRECT = RK == RK_MULTI && VK == VK_FF;
  constexpr bool ELEV = RK == RK_MULTI;  // elevations are read
  constexpr int TC = Tile<F>::TC;
  // The thread index, opaque to the compiler: what is derived from it is
  // computed anew for each tile instead of held in registers across tiles.
  int tid = (int)threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int32_t tr = tile / P.ntc, tc = tile - tr * P.ntc;
  const int64_t nr = P.nrows, nc = P.ncols;
  const int64_t r0 = (int64_t)tr * TR, c0 = (int64_t)tc * TC;
  const uint32_t id = (uint32_t)(P.tile0 + tile);

  // -------------------------------------------------------------- load
  // Every load is issued before the first is waited for; those off the grid
  // read its nearest cell and are replaced after (behind a branch each would
  // be waited for).  This thread's own cells: row 8 wave + i, column lane.
  constexpr int ZN = (TR + 4) * (TC + 4), ZU = (ZN + PT - 1) / PT;
  constexpr int CN = (TR + 2) * (TC + 2), CU = (CN + PT - 1) / PT;
  const int oc = lane, or0 = 8 * wave;
  const bool column = oc < TC;
  const int32_t rlast = (int32_t)(nr - 1 - r0 < TR + 1 ? nr - 1 - r0 : TR + 1);  // last row and column on the grid
  const int32_t clast = (int32_t)(nc - 1 - c0 < TC + 1 ? nc - 1 - c0 : TC + 1);  // (from the tile's first)
  const int32_t rfirst = tr > 0 ? -2 : 0, cfirst = tc > 0 ? -2 : 0;
  const int64_t cell0 = r0 * nc + c0;
  auto near = [&](int r, int c) -> int64_t {
    const int32_t rr = r < rfirst ? rfirst : (r > rlast ? rlast : r), cc = c < cfirst ? cfirst : (c > clast ? clast : c);
    return cell0 + (int64_t)rr * nc + cc;
  };
  auto on_grid = [&](int r, int c) -> bool { return r >= rfirst && r <= rlast && c >= cfirst && c <= clast; };
  uint64_t word[8];
  uint64_t raw[8];  // source terms as loaded
  bool nonfinite = false, badcode = false, cycle = false;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int64_t at = near(or0 + i, oc);
    word[i] = ld64(P.word + at);
    if (P.src64) raw[i] = (uint64_t)__double_as_longlong(P.src64[at]);
    else raw[i] = P.src32 ? __float_as_uint(P.src32[at]) : 0x3F800000u;
  }
  float zv[ELEV ? ZU : 1];
  if (ELEV) {
#pragma unroll
    for (int j = 0; j < ZU; ++j) {
      const int i = tid + j * PT;
      zv[j] = P.z[near(i / (TC + 4) - 2, i % (TC + 4) - 2)];
    }
  }
  uint8_t cv[BATCH ? 1 : CU];
  if (!BATCH) {
#pragma unroll
    for (int j = 0; j < CU; ++j) {
      const int i = tid + j * PT;
      cv[j] = P.code[near(i / (TC + 2) - 1, i % (TC + 2) - 1)];
    }
  }
  {
    // The four edge arrays.
    uint64_t* w = reinterpret_cast<uint64_t*>(&T);
    for (int i = tid; i < (int)(sizeof(T.edge) / 8); i += PT) w[i] = 0ull;
  }
  if (ELEV) {
#pragma unroll
    for (int j = 0; j < ZU; ++j) {
      const int i = tid + j * PT;
      if (i < ZN) (&T.z[0][0])[i] = on_grid(i / (TC + 4) - 2, i % (TC + 4) - 2) ? zv[j] : INFINITY;
    }
  }
  if (!BATCH) {
#pragma unroll
    for (int j = 0; j < CU; ++j) {
      const int i = tid + j * PT;
      if (i < CN) (&T.code[0][0])[i] = cv[j];
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    // Cells off the grid count as final.
    const int r = or0 + i;
    if (!column || !on_grid(r, oc)) word[i] = 0;
    const uint64_t b = ballot(word[i] != OPEN);
    if (lane < 2) T.done[2 * r + lane] = (uint32_t)(b >> (32 * lane));
  }
  if (tid == 0) {
    T.phase = PH_RUN;
    T.polls = 0;
    T.queue_empty = 0;
    T.gaps = 0;
  }
  __syncthreads();

  // --------------------------------------------------------- fractions
#pragma unroll 1
  for (int i = tid; i < CN; i += PT) {
    const int r = i / (TC + 2) - 1, c = i % (TC + 2) - 1;
    const int64_t y = r0 + r, x = c0 + c;
    if (!on_grid(r, c)) continue;
    const bool own = in_tile<F>(r, c);
    // The edges with a cell in the tile, by direction.
    const int at = place<F>(r, c);
    uint32_t put = 0xFFu;
    if (!own) {
      const uint32_t cols = (c >= 1 && c <= TC ? 0x29u : 0u) | (c >= 0 && c < TC ? 0x42u : 0u) |
                            (c >= -1 && c < TC - 1 ? 0x94u : 0u);
      const uint32_t rows = (r >= 1 && r <= TR ? 0x07u : 0u) | (r >= 0 && r < TR ? 0x18u : 0u) |
                            (r >= -1 && r < TR - 1 ? 0xE0u : 0u);
      put = cols & rows;
    }
    float zc = 0.0f, zk[8];
    uint32_t code, lower = 0;
    if (ELEV) {
      zc = T.z[r + 2][c + 2];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        zk[k] = T.z[r + 2 + nb_dr(k)][c + 2 + nb_dc(k)];
        lower |= zk[k] < zc ? 1u << k : 0u;  // off the grid: +inf, never lower
      }
      nonfinite |= own && !isfinite(zc);
    }
    if (BATCH) {
      code = P.rule == FR_MFD ? lower : (P.rule == FR_D4 ? route_code<FR_D4>(zc, zk) : route_code<FR_D8>(zc, zk));
      if (own && P.code_out) P.code_out[y * nc + x] = (uint8_t)code;
    } else {
      code = T.code[r + 1][c + 1];
    }
    if (RK == RK_SINGLE || (BATCH && P.rule != FR_MFD)) {
      if (code > 7u) {
        badcode |= own && code != SINK;
        continue;
      }
      if (!BATCH) {
        const int kr = (int)code < 3 ? -1 : ((int)code < 5 ? 0 : 1);
        const int kc = (code == 0u || code == 3u || code == 5u) ? -1 : ((code == 1u || code == 6u) ? 0 : 1);
        const int64_t yy = y + kr, xx = x + kc;
        if (yy < 0 || yy >= nr || xx < 0 || xx >= nc) {
          badcode |= own;
          continue;
        }
        if (P.code[yy * nc + xx] == 7u - code) {
          // Two cells that drain into each other (an edge carries one way).
          cycle |= own;
          continue;
        }
      }
      #pragma unroll
      for (int k = 0; k < 8; ++k)
        if ((int)code == k && ((put >> k) & 1u)) *edge_at(T, at, k) = k < 4 ? (F)-1 : (F)1;
    } else {
      // Only strictly lower cells of the grid can receive: whatever the
      // codes say, the routing solved is acyclic.
      badcode |= own && (code & ~lower) != 0u;
      put_fractions<F>(T, at, put, code & lower, zc, zk, P.p);
    }
  }
  __syncthreads();

  // ------------------------------------------------------------- masks
  // Wavefront w finds rows 8 w to 8 w + 7 of every lane: bytes w of the
  // lane's masks.  mask[8]: inputs from outside the tile; [9]: final; [10]:
  // feeds a cell outside.
  {
    uint32_t m[11] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    bool gap = false;
#pragma unroll 1
    for (int i = 0; i < 8; ++i) {
      const int r = 8 * wave + i, c = col_at(lane, r);
      if (c >= TC) {
        m[9] |= 1u << i;
        continue;
      }
      const int at = place<F>(r, c);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const F o = out_at(T, at, k);
        const uint32_t b = (ADJ ? o > (F)0 : o < (F)0) ? 1u << i : 0u;
        const bool inside = in_tile<F>(r + nb_dr(k), c + nb_dc(k));
        m[k] |= inside ? b : 0u;
        m[8] |= inside ? 0u : b;
        m[10] |= !inside && (ADJ ? o < (F)0 : o > (F)0) ? 1u << i : 0u;
        if (sizeof(F) == 8) gap |= o == (F)0 && on_grid(r, c) && on_grid(r + nb_dr(k), c + nb_dc(k));
      }
      m[9] |= ((T.done[2 * r + (c >> 5)] >> (c & 31)) & 1u) << i;
    }
#pragma unroll
    for (int k = 0; k < 11; ++k) T.mask[k][lane][wave] = (uint8_t)m[k];
    if (gap) l_st(&T.gaps, 1u);
  }
  __syncthreads();
  // Roles: the peeling wavefront is the one on SIMD (workgroup slot mod 4).
  int lw = 0;
  for (int w = 3; w >= 0; --w)
    if (T.simd[w] == T.simd[4]) lw = w;
  const int role = __builtin_amdgcn_readfirstlane((wave - lw) & 3);
  uint32_t in[8];
  uint32_t done = 0, feeder = 0;
  if (role == 0) {
    auto whole = [&](int k) -> uint32_t { return *reinterpret_cast<const uint32_t*>(&T.mask[k][lane][0]); };
#pragma unroll
    for (int k = 0; k < 8; ++k) in[k] = whole(k);
    T.wait[lane] = whole(8);
    done = whole(9);
    feeder = whole(10);
    T.done[lane] = done;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = or0 + i;
    double v = P.src64 ? bitsd(raw[i]) : (double)__uint_as_float((uint32_t)raw[i]);
    // A source the result's type cannot hold counts as non-finite.
    if (VK == VK_FF ? !isfinite((float)v) : !isfinite(v)) {
      nonfinite = true;
      v = 0.0;
    }
    if (column) T.g[r + 1][oc + 1] = word[i] != OPEN ? bitsd(word[i]) : v;
  }
  // The cells around the tile pass nothing on until they are known.
  for (int i = tid; i < 2 * (TC + 2) + 2 * TR; i += PT) {
    if (i < TC + 2) T.g[0][i] = 0.0;
    else if (i < 2 * (TC + 2)) T.g[TR + 1][i - (TC + 2)] = 0.0;
    else if (i < 2 * (TC + 2) + TR) T.g[i - 2 * (TC + 2) + 1][0] = 0.0;
    else T.g[i - 2 * (TC + 2) - TR + 1][TC + 1] = 0.0;
  }
  if (Q.status) {
    if (ballot(badcode) && lane == 0) atomicCAS(Q.status, 0, FR_ERR_BADCODE);
    if (ballot(nonfinite) && lane == 0) atomicCAS(Q.status, 0, FR_ERR_NONFINITE);
    if (ballot(cycle) && lane == 0) atomicCAS(Q.status, 0, FR_ERR_NOTDAG);
  }
  // Border cells published so far: final ones of columns 0 and TC - 1 (lane =
  // row) and of rows 0 and TR - 1 (lane = column).
  const auto border_done = [&]() -> uint32_t {
    const int rr = lane & 31;
    return ((l_ld(&T.done[lane_at(rr, 0)]) >> rr) & 1u) | (((l_ld(&T.done[lane_at(rr, TC - 1)]) >> rr) & 1u) << 1) |
           ((l_ld(&T.done[lane_at(0, lane)]) & 1u) << 2) | ((l_ld(&T.done[lane_at(TR - 1, lane)]) >> 31) << 3);
  };
  uint32_t published = role == 1 ? border_done() : 0u;
  __syncthreads();

  // ------------------------------------------------------------- roles
  for (;;) {
    if (role == 0) {
      // Peeling.
      __builtin_amdgcn_s_setprio(3);
      uint32_t idle_from = 0;
      bool idle = false;
      uint32_t outside = l_ld(&T.wait[lane]);
      // GAPS: some neighbours exchange nothing (equal heights).  In float64
      // such a neighbour, once overflowed, would add 0 * inf; a branch behind
      // the sum costs 5%, so tiles without such cells have a loop without it.
      auto peel = [&](auto gaps) __attribute__((always_inline)) {
        constexpr bool GAPS = decltype(gaps)::value;
        for (;;) {
          const uint32_t a1 = from_below(done), a2 = from_below(a1), a3 = from_below(a2);
          const uint32_t b1 = from_above(done), b2 = from_above(b1), b3 = from_above(b2);
          uint32_t wait = outside;
          wait |= in[0] & ~(a3 << 1);
          wait |= in[1] & ~(a2 << 1);
          wait |= in[2] & ~(a1 << 1);
          wait |= in[3] & ~a1;
          wait |= in[4] & ~b1;
          wait |= in[5] & ~(b1 >> 1);
          wait |= in[6] & ~(b2 >> 1);
          wait |= in[7] & ~(b3 >> 1);
          // Read now, used in the next step.
          outside = l_ld(&T.wait[lane]);
          fence();
          const uint32_t ready = ~(done | wait);
          if (ballot(ready != 0u) == 0ull) {
            if (ballot(done != ~0u) == 0ull) break;
            // Nothing ready: wait for cells around the tile, for a few polls.
            const uint32_t polls = l_ld(&T.polls);
            if (!idle) {
              idle = true;
              idle_from = polls;
            } else if (polls - idle_from > (uint32_t)(l_ld(&T.queue_empty) ? LINGER_IDLE : LINGER_BUSY)) {
              break;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
          }
          idle = false;
          if (ready != 0u) {
            const int r = __builtin_ctz(ready), c = col_at(lane, r);
            const int at = place<F>(r, c);
            double* g0 = &T.g[0][0] + (at - Tile<F>::W - 1);  // the upper left neighbour
            F o[8];
            double gk[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              o[k] = out_at(T, at, k);
              gk[k] = g0[(nb_dr(k) + 1) * Tile<F>::W + nb_dc(k) + 1];
            }
            double& gc = g0[Tile<F>::W + 1];
            double v = 0.0, give = 0.0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              if (RK == RK_SINGLE) {
                v = (ADJ ? o[k] : -o[k]) > (F)0 ? gk[k] : v;  // one input
                continue;
              }
              const double ok = (double)o[k];
              v = fma(fmax(ADJ ? ok : -ok, 0.0), gk[k], v);
              if (CORRECT) give += fmax(ok, 0.0);
            }
            if (GAPS && !isfinite(v)) {
              // The inputs alone.
              v = 0.0;
#pragma unroll
              for (int k = 0; k < 8; ++k) {
                const double ok = (double)o[k], w = fmax(ADJ ? ok : -ok, 0.0);
                if (w > 0.0) v = fma(w, gk[k], v);
              }
            }
            const double fix = CORRECT && give > 0.0 ? 2.0 - give : 1.0;
            const double own = gc;
            const double q = ADJ && CORRECT ? fma(v, fix, own) : own + v;
            gc = !ADJ && CORRECT ? q * fix : q;
            done |= 1u << r;
            fence();
            l_st(&T.done[lane], done);
            const int64_t cell = cell0 + (int64_t)((uint32_t)r * (uint32_t)nc + (uint32_t)c);
            // Stored at once for the tiles that poll it; the publishing
            // wavefront stores it again, to know when it has arrived.
            if ((feeder >> r) & 1u) st64(P.word + cell, dword(gc));
            if (VK == VK_F64) P.out64[cell] = q;
            else if (!BATCH || P.out32) P.out32[cell] = (float)q;
            else P.cnt[cell] = (uint64_t)q;  // whole numbers below 2^31
          }
          fence();
        }
      };
      if (sizeof(F) == 8 && __builtin_amdgcn_readfirstlane((int)l_ld(&T.gaps)) != 0) peel(std::true_type{});
      else peel(std::false_type{});
      l_st(&T.phase, PH_STOP);
      __builtin_amdgcn_s_setprio(0);
    } else if (role == 1) {
      // Publishing: cells with an edge out of the tile along the way their
      // value goes are stored and the tiles they feed woken.
      const int r = lane & 31, cc = lane < TC ? lane : TC - 1;
      auto feeds = [&](int rr, int c, int k) -> bool {
        const F o = out_at(T, rr, c, k);
        return ADJ ? o < (F)0 : o > (F)0;
      };
      uint32_t feed = 0;  // as border_done()
      if (lane < TR) {
        feed |= feeds(r, 0, 0) || feeds(r, 0, 3) || feeds(r, 0, 5) ? 1u : 0u;
        feed |= feeds(r, TC - 1, 2) || feeds(r, TC - 1, 4) || feeds(r, TC - 1, 7) ? 2u : 0u;
      }
      if (lane < TC) {
        feed |= feeds(0, cc, 0) || feeds(0, cc, 1) || feeds(0, cc, 2) ? 4u : 0u;
        feed |= feeds(TR - 1, cc, 5) || feeds(TR - 1, cc, 6) || feeds(TR - 1, cc, 7) ? 8u : 0u;
      }
      const bool f0 = feeds(0, 0, 0), f2 = feeds(0, TC - 1, 2), f5 = feeds(TR - 1, 0, 5),
                 f7 = feeds(TR - 1, TC - 1, 7);
      uint32_t all_fed = 0;  // tiles this one feeds, by direction
      {
        const uint64_t t = ballot((feed & 4u) != 0u), b = ballot((feed & 8u) != 0u);
        if (t) all_fed |= 1u << 1;
        if (b) all_fed |= 1u << 6;
        if (ballot((feed & 1u) != 0u)) all_fed |= 1u << 3;
        if (ballot((feed & 2u) != 0u)) all_fed |= 1u << 4;
        if (f0) all_fed |= 1u << 0;
        if (f2) all_fed |= 1u << 2;
        if (f5) all_fed |= 1u << 5;
        if (f7) all_fed |= 1u << 7;
      }
      const auto half_done = [&]() -> bool { return __popcll(ballot(__popc(l_ld(&T.done[lane])) >= TR / 2)) >= 32; };
      bool foretold = half_done();
      uint32_t wk = 0;  // tiles to wake, by direction
      for (bool last = false; !last;) {
        last = l_ld(&T.phase) != PH_RUN;
        fence();
        const uint32_t now = border_done();
        fence();
        const uint32_t fresh = now & ~published & feed;
        published = now;
        if (ballot(fresh != 0u)) {
          if (fresh & 1u) st64(P.word + (r0 + r) * nc + c0, dword(T.g[r + 1][1]));
          if (fresh & 2u) st64(P.word + (r0 + r) * nc + c0 + TC - 1, dword(T.g[r + 1][TC]));
          if (fresh & 4u) st64(P.word + r0 * nc + c0 + cc, dword(T.g[1][cc + 1]));
          if (fresh & 8u) st64(P.word + (r0 + TR - 1) * nc + c0 + cc, dword(T.g[TR][cc + 1]));
          const uint64_t top = ballot((fresh & 4u) != 0u), bot = ballot((fresh & 8u) != 0u);
          if (top) wk |= 1u << 1;
          if (bot) wk |= 1u << 6;
          if (ballot((fresh & 1u) != 0u)) wk |= 1u << 3;
          if (ballot((fresh & 2u) != 0u)) wk |= 1u << 4;
          if ((top & 1u) && f0) wk |= 1u << 0;
          if (((top >> (TC - 1)) & 1u) && f2) wk |= 1u << 2;
          if ((bot & 1u) && f5) wk |= 1u << 5;
          if (((bot >> (TC - 1)) & 1u) && f7) wk |= 1u << 7;
        }
        // A tile that is half finished wakes those it feeds while workgroups
        // are idle, so that they are in LDS when it ends.
        if (!foretold && half_done()) {
          foretold = true;
          if (l_ld(&T.queue_empty)) wk |= all_fed;
        }
        // While other tiles are queued, tiles are woken once this one stops:
        // they find more to do then, and those in LDS see the words anyway.
        if (wk == 0u || !(last || l_ld(&T.queue_empty))) {
          __builtin_amdgcn_s_sleep(2);
          continue;
        }
        stores_done();
        if (lane < 8 && ((wk >> lane) & 1u)) {
          const int dr = lane < 3 ? -1 : (lane < 5 ? 0 : 1);
          const int dc = (lane == 0 || lane == 3 || lane == 5) ? -1 : ((lane == 1 || lane == 6) ? 0 : 1);
          const int32_t ur = tr + dr, uc = tc + dc;
          if (ur >= 0 && ur < P.ntr && uc >= 0 && uc < P.ntc) wake(Q, (uint32_t)(P.tile0 + ur * P.ntc + uc));
        }
        wk = 0;
      }
    } else {
      // Polling (two wavefronts, so that words are looked at twice as often):
      // cells of the columns beside the tile (lane - 1 = row), of the rows
      // above and below it (lane = column); and the cells of the tile that
      // wait for them (lane = row, lane = column).
      auto gives = [&](int rr, int c, int k) -> bool {  // toward a cell of the tile
        if (!in_tile<F>(rr + nb_dr(k), c + nb_dc(k))) return false;
        const F o = out_at(T, rr, c, k);
        return ADJ ? o < (F)0 : o > (F)0;
      };
      auto takes = [&](int rr, int c, int k) -> bool {
        const F o = out_at(T, rr, c, k);
        return ADJ ? o > (F)0 : o < (F)0;
      };
      const int r = lane - 1, c = lane;
      const bool side = lane < TR + 2, cap = lane < TC, edge = lane < TR;
      bool need[4] = {false, false, false, false};
      uint32_t takes4[4] = {0, 0, 0, 0};  // bits 0-2: from the lane before, this lane, the lane after
      if (side) {
        need[0] = gives(r, -1, 2) || gives(r, -1, 4) || gives(r, -1, 7);
        need[1] = gives(r, TC, 0) || gives(r, TC, 3) || gives(r, TC, 5);
      }
      if (edge) {
        takes4[0] = (takes(lane, 0, 0) ? 1u : 0u) | (takes(lane, 0, 3) ? 2u : 0u) | (takes(lane, 0, 5) ? 4u : 0u);
        takes4[1] = (takes(lane, TC - 1, 2) ? 1u : 0u) | (takes(lane, TC - 1, 4) ? 2u : 0u) |
                    (takes(lane, TC - 1, 7) ? 4u : 0u);
      }
      if (cap) {
        need[2] = gives(-1, c, 5) || gives(-1, c, 6) || gives(-1, c, 7);
        need[3] = gives(TR, c, 0) || gives(TR, c, 1) || gives(TR, c, 2);
        takes4[2] = (takes(0, c, 0) ? 1u : 0u) | (takes(0, c, 1) ? 2u : 0u) | (takes(0, c, 2) ? 4u : 0u);
        takes4[3] =
            (takes(TR - 1, c, 5) ? 1u : 0u) | (takes(TR - 1, c, 6) ? 2u : 0u) | (takes(TR - 1, c, 7) ? 4u : 0u);
      }
      const uint64_t* at[4];
      at[0] = P.word + (r0 + r) * nc + c0 - 1;
      at[1] = P.word + (r0 + r) * nc + c0 + TC;
      at[2] = P.word + (r0 - 1) * nc + c0 + c;
      at[3] = P.word + (r0 + TR) * nc + c0 + c;
      double* to[4];
      to[0] = &T.g[side ? lane : 0][0];
      to[1] = &T.g[side ? lane : 0][TC + 1];
      to[2] = &T.g[0][cap ? c + 1 : 0];
      to[3] = &T.g[TR + 1][cap ? c + 1 : 0];
      bool have[4] = {false, false, false, false};
      uint32_t polls = l_ld(&T.polls);
      while (l_ld(&T.phase) == PH_RUN) {
        uint64_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = need[i] ? ld64(at[i]) : OPEN;
        uint32_t head = 0, tail = 0;
        if (role == 2) {
          head = ld32(&Q.ctl->head);
          tail = ld32(&Q.ctl->tail);
        }
        bool news = false;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (w[i] != OPEN) {
            *to[i] = bitsd(w[i]);
            need[i] = false;
            have[i] = true;
            news = true;
          }
        if (ballot(news)) {
          const uint64_t hl = ballot(have[0]), hr = ballot(have[1]), ht = ballot(have[2]), hb = ballot(have[3]);
          // Which of its three cells outside a border cell has: the corners
          // above and below a column belong to the columns beside the tile.
          auto three = [&](uint64_t h, uint64_t before, uint64_t after) -> uint32_t {
            const uint64_t a = lane == 0 ? before : h >> (lane - 1);
            const uint64_t d = lane == TC - 1 ? after : h >> ((lane + 1) & 63);
            return ((uint32_t)a & 1u) | (((uint32_t)(h >> lane) & 1u) << 1) | (((uint32_t)d & 1u) << 2);
          };
          const bool wl = (takes4[0] & ~((uint32_t)(hl >> (lane & 31)) & 7u)) != 0u;
          const bool wr = (takes4[1] & ~((uint32_t)(hr >> (lane & 31)) & 7u)) != 0u;
          const bool wt = (takes4[2] & ~three(ht, hl, hr)) != 0u;
          const bool wb = (takes4[3] & ~three(hb, hl >> (TR + 1), hr >> (TR + 1))) != 0u;
          // A corner cell waits for both of its sides.
          const uint64_t bl = ballot(wl), br = ballot(wr), bt = ballot(wt), bb = ballot(wb);
          const bool l0 = lane == 0, l1 = lane == TR - 1, k1 = lane == TC - 1;
          const bool ul = !wl && !(l0 && (bt & 1u)) && !(l1 && (bb & 1u));
          const bool ur = !wr && !(l0 && ((bt >> (TC - 1)) & 1u)) && !(l1 && ((bb >> (TC - 1)) & 1u));
          const bool ut = !wt && !(l0 && (bl & 1u)) && !(k1 && (br & 1u));
          const bool ub = !wb && !(l0 && ((bl >> (TR - 1)) & 1u)) && !(k1 && ((br >> (TR - 1)) & 1u));
          fence();
          if (takes4[0] && ul) atomicAnd(&T.wait[lane_at(lane, 0)], ~(1u << (lane & 31)));
          if (takes4[1] && ur) atomicAnd(&T.wait[lane_at(lane, TC - 1)], ~(1u << (lane & 31)));
          if (takes4[2] && ut) atomicAnd(&T.wait[lane_at(0, lane)], ~1u);
          if (takes4[3] && ub) atomicAnd(&T.wait[lane_at(TR - 1, lane)], ~(1u << (TR - 1)));
          fence();
        }
        ++polls;
        if (role == 2 && lane == 0) {
          l_st(&T.queue_empty, (int32_t)(tail - head) <= 0 ? 1u : 0u);
          l_st(&T.polls, polls);
        }
      }
    }
    __syncthreads();

    // ---------------------------------------------------------- let go
    // Final cells that were not when the tile was loaded go back to memory
    // (a finished tile's only where the mass balance reads them).
    const bool all = ballot(T.done[lane] != ~0u) == 0ull;
    if (!all || P.keep) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = or0 + i;
        if (word[i] == OPEN && ((T.done[lane_at(r, oc)] >> r) & 1u)) {
          word[i] = dword(T.g[r + 1][oc + 1]);
          st64(P.word + (r0 + r) * nc + c0 + oc, word[i]);
        }
      }
    }
    stores_done();
    __syncthreads();
    if (tid == 0) {
      T.cmd = 0;
      if (all) {
        atomicExch(Q.state + id, ST_DONE);
        atomicSub(&Q.ctl->left, 1u);
      } else if (atomicCAS(Q.state + id, ST_RUNNING, 0u) != ST_RUNNING) {
        // Woken meanwhile: look around once more before letting go.
        atomicAnd(Q.state + id, ~ST_PENDING);
        T.cmd = 1;
        T.phase = PH_RUN;
      }
    }
    __syncthreads();
    if (T.cmd == 0) return;
  }
}

// SIMD of every wavefront and the workgroup's slot on its compute unit, from
// the hardware's wave identity register (bits 5:4, 19:16).
template <typename F>
__device__ __forceinline__ void note_simds(Tile<F>& T) {
  const uint32_t hw = __builtin_amdgcn_s_getreg((31 << 11) | 4);
  if ((threadIdx.x & 63) == 0) T.simd[threadIdx.x >> 6] = (int)((hw >> 4) & 3u);
  if (threadIdx.x == 0) T.simd[4] = (int)((hw >> 16) & 3u);
}

// Float fractions: three workgroups fit a compute unit's LDS, so three
// wavefronts a SIMD; float64 ones: two.
template <int RK, bool ADJ, int VK>
__global__ __launch_bounds__(PT, RK == RK_MULTI && VK == VK_F64 ? 2 : 3) void k_peel(PeelGrid P, TileQueue Q,
                                                                                     const int32_t* gate) {
  using F = typename PeelFrac<RK, VK>::T;
  if (gate && *gate == 0) return;
  __shared__ Tile<F> T;
  note_simds(T);
  for (;;) {
    if (threadIdx.x == 0) T.tile = take_tile(Q);
    __syncthreads();
    const int32_t t = T.tile;
    if (t < 0) return;
    peel_tile<RK, ADJ, VK, false, F>(P, Q, T, t);
    __syncthreads();
  }
}

// A batch's grids are solved in groups of about this many tiles a workgroup
// (as many groups as there are queues, at most).  In one queue the tiles'
// first turns of all grids come before any second one, and what is woken
// meanwhile waits behind them: 512 grids (286 thousand tiles, 768 workgroups)
// took 882 ms, in groups 177; 128 grids (65 thousand tiles) are one group, 38
// ms.
constexpr int32_t GROUP_TILES = 85;

__device__ __forceinline__ TileQueue group_queue(const PeelBatch* B, int g) {
  TileQueue Q = B->queue;
  Q.ring += 2 * (size_t)B->lo[g];
  Q.cap = 2u * (uint32_t)(B->lo[g + 1] - B->lo[g]);
  Q.ctl = const_cast<TileCtl*>(&B->ctl[g]);
  return Q;
}

// Many grids (float32 water, or counts of single receivers).
__global__ __launch_bounds__(PT, 3) void k_peel_batch(const PeelBatch* B) {
  __shared__ Tile<float> T;
  const PeelGrid* grids = B->grids;
  const int32_t ngrids = B->ngrids;
  note_simds(T);
  for (int g = 0; g < B->ngroups;) {
    const TileQueue Q = group_queue(B, g);
    if (threadIdx.x == 0) T.tile = Q.cap ? take_tile(Q) : -1;
    __syncthreads();
    const int32_t t = __builtin_amdgcn_readfirstlane(T.tile);
    __syncthreads();
    if (t < 0) {
      ++g;
      continue;
    }
    // The grid whose tiles hold tile t (grids in queue order).
    int lo = 0, hi = ngrids - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (grids[mid].tile0 <= t) lo = mid;
      else hi = mid - 1;
    }
    const PeelGrid P = grids[lo];
    peel_tile<RK_MULTI, false, VK_FF, true, float>(P, Q, T, t - P.tile0);
    __syncthreads();
  }
}

// Which end of the grid water leaves (the adjoint: reaches), by the mean
// elevation of two sampled rows: its tiles are queued first, from the last
// row of tiles or from the first.  Any order gives the same result.
__device__ bool last_rows_first(const PeelGrid& P, bool adjoint) {
  if (!P.z) return adjoint;
  const int64_t step = P.ncols / 64 + 1;
  float d = 0.0f;
  for (int64_t c = 0; c < P.ncols; c += step)
    d += P.z[(P.nrows - 1 - P.nrows / 4) * P.ncols + c] - P.z[(P.nrows / 4) * P.ncols + c];
  return (d > 0.0f) != adjoint;
}

// No cell final, every tile queued (tickets from tile0 - lo on, lo the queue's
// first tile; the ring's second half empty).  Thread i of n.
__device__ void open_grid(const PeelGrid& P, const TileQueue& Q, int32_t lo, bool adjoint, int64_t i0,
                          int64_t stride) {
  const int64_t n = P.nrows * P.ncols;
  for (int64_t i = i0; i < n; i += stride) P.word[i] = OPEN;
  const int32_t nt = P.ntr * P.ntc;
  if (i0 >= nt) return;
  const bool last = last_rows_first(P, adjoint);
  for (int64_t i = i0; i < nt; i += stride) {
    const uint32_t ticket = (uint32_t)(P.tile0 - lo + i);
    const uint32_t t = (uint32_t)(P.tile0 + (last ? nt - 1 - i : i));
    Q.ring[ticket] = ((uint64_t)ticket << 32) | (t + 1u);
    Q.ring[Q.cap / 2 + ticket] = 0ull;
    Q.state[t] = ST_PENDING;
  }
}

__global__ __launch_bounds__(256) void k_peel_init(PeelGrid P, TileQueue Q, int adjoint, const int32_t* gate) {
  if (gate && *gate == 0) return;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  open_grid(P, Q, 0, adjoint != 0, i0, (int64_t)gridDim.x * blockDim.x);
  if (i0 == 0) open_queue(Q, (uint32_t)(P.ntr * P.ntc));
}

constexpr int BATCH_FILL_BLOCKS = 32;  // workgroups per grid of a batch

__global__ __launch_bounds__(256) void k_peel_batch_init(const PeelBatch* B) {
  if ((int)blockIdx.x >= B->ngrids) return;
  const int g = B->grids[blockIdx.x].tile0 / B->span;
  open_grid(B->grids[blockIdx.x], group_queue(B, g), B->lo[g], false, (int64_t)blockIdx.y * blockDim.x + threadIdx.x,
            (int64_t)BATCH_FILL_BLOCKS * blockDim.x);
}

// Inclusive scan of x over the workgroup (blockDim.x = 1024).
__device__ int64_t scan_inc(int64_t x, int64_t* sh) {
  const int t = (int)threadIdx.x;
  sh[t] = x;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int64_t y = t >= o ? sh[t - o] : 0;
    __syncthreads();
    sh[t] += y;
    __syncthreads();
  }
  const int64_t v = sh[t];
  __syncthreads();
  return v;
}

// Set-up of a batch (one workgroup): the tiles' schedule, their grids in that
// order with their first tile, words and queue, all in the workspace, laid
// out as peel_batch_bytes() counts it.
__global__ __launch_bounds__(1024) void k_peel_batch_setup(const fr_tile* tiles, int32_t ntiles, int order,
                                                           int32_t limit, int32_t group, char* ws,
                                                           size_t ws_bytes, int32_t* status) {
  __shared__ int64_t sh[1024];
  __shared__ int bad_sh;
  PeelBatch* B = reinterpret_cast<PeelBatch*>(ws);
  PeelGrid* grids = reinterpret_cast<PeelGrid*>(ws + peel_align(sizeof(PeelBatch)));
  int32_t* sched = reinterpret_cast<int32_t*>(ws + peel_align(sizeof(PeelBatch)) +
                                              peel_align((size_t)ntiles * sizeof(PeelGrid)));
  const int t = (int)threadIdx.x;
  if (t == 0) bad_sh = 0;
  __syncthreads();
  // Schedule: given order, or more rows (cells) first, stable, by parallel
  // ranking.
  for (int i = t; i < ntiles; i += 1024) {
    const fr_tile& T = tiles[i];
    if (T.nrows < 1 || T.ncols < 1 || !T.z || (T.rule == FR_MFD && !T.q_out) ||
        (T.rule != FR_MFD && (T.q_out != nullptr) == (T.counts_out != nullptr)))
      bad_sh = 1;
    int rank = i;
    if (order != FR_ORDER_GIVEN && ntiles <= 16384) {
      rank = 0;
      const bool rows = order == FR_ORDER_ROWS_DESC;
      const int64_t ki = rows ? T.nrows : T.nrows * T.ncols;
      for (int j = 0; j < ntiles; ++j) {
        const int64_t kj = rows ? tiles[j].nrows : tiles[j].nrows * tiles[j].ncols;
        rank += (kj > ki || (kj == ki && j < i)) ? 1 : 0;
      }
    }
    sched[rank] = i;
  }
  __threadfence();
  __syncthreads();
  const bool bad = bad_sh != 0;
  size_t off = peel_batch_head_bytes(ntiles);
  int64_t tile0 = 0;
  for (int k0 = 0; !bad && k0 < ntiles; k0 += 1024) {
    const int k = k0 + t;
    PeelGrid G{};
    int64_t bytes = 0, nt = 0;
    if (k < ntiles) {
      const fr_tile T = tiles[sched[k]];
      G.nrows = T.nrows;
      G.ncols = T.ncols;
      G.ntr = (int32_t)((T.nrows + TR - 1) / TR);
      G.ntc = (int32_t)((T.ncols + peel_cols(false) - 1) / peel_cols(false));
      G.z = T.z;
      G.p = 1.1;
      G.src32 = T.rule == FR_MFD || T.q_out ? T.rain : nullptr;
      G.out32 = T.q_out;
      G.cnt = T.rule == FR_MFD || T.q_out ? nullptr : T.counts_out;
      G.code_out = T.code_out;
      G.rule = T.rule;
      bytes = (int64_t)peel_align((size_t)(T.nrows * T.ncols) * sizeof(uint64_t));
      if (batch_strips(T.ncols) > limit) {
        // Not routed on so few workgroups: an empty grid in the queue.
        if (status) atomicCAS(status, 0, FR_ERR_ARG);
        G.nrows = 0;
        G.ntr = 0;
      }
      nt = (int64_t)G.ntr * G.ntc;
    }
    const int64_t bi = scan_inc(bytes, sh), ti = scan_inc(nt, sh);
    if (k < ntiles) {
      G.word = reinterpret_cast<uint64_t*>(ws + off + (size_t)(bi - bytes));
      G.tile0 = (int32_t)(tile0 + ti - nt);
      grids[k] = G;
    }
    sh[t] = bi;
    __syncthreads();
    off += (size_t)sh[1023];
    __syncthreads();
    sh[t] = ti;
    __syncthreads();
    tile0 += sh[1023];
    __syncthreads();
  }
  if (t == 0) {
    TileQueue Q{};
    Q.cap = (uint32_t)(2 * tile0);
    Q.state = reinterpret_cast<uint32_t*>(ws + off);
    off += peel_align((size_t)tile0 * sizeof(uint32_t));
    Q.ring = reinterpret_cast<uint64_t*>(ws + off);
    off += peel_align((size_t)Q.cap * sizeof(uint64_t));
    Q.status = status;
    Q.stuck = FR_ERR_STALL;
    const bool fits = off <= ws_bytes && !bad;
    if (!fits && status) atomicCAS(status, 0, bad ? FR_ERR_ARG : FR_ERR_WORKSPACE);
    B->queue = Q;
    B->grids = grids;
    B->ngrids = fits ? ntiles : 0;
    B->span = (int32_t)(tile0 / (PEEL_GROUPS - 1) + 1);
    if (B->span < group) B->span = group;
    B->ngroups = fits ? (int32_t)(tile0 / B->span) + 1 : 0;
    for (int g = 0; g <= PEEL_GROUPS; ++g) B->lo[g] = (int32_t)tile0;
  }
  __threadfence();
  __syncthreads();
  // A group starts at its first grid; one without grids is empty and starts
  // where the next does.
  if (bad) return;
  const int32_t span = B->span;
  for (int k = t; k < ntiles; k += 1024) {
    const int32_t first = grids[k].tile0;
    const int g1 = first / span, g0 = k > 0 ? grids[k - 1].tile0 / span + 1 : 0;
    for (int g = g0; g <= g1; ++g) B->lo[g] = first;
  }
  __threadfence();
  __syncthreads();
  for (int g = t; g < B->ngroups; g += 1024) open_queue(group_queue(B, g), (uint32_t)(B->lo[g + 1] - B->lo[g]));
}

// Mass balance partials: {sum of the values of the sinks, sum of the source
// terms}, in a fixed order.
__global__ __launch_bounds__(256) void k_peel_mass(PeelGrid P, double* partial, const int32_t* gate) {
  if (gate && *gate == 0) return;
  const int64_t n = P.nrows * P.ncols;
  double s = 0.0, t = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    if (P.code[i] == 0) s += bitsd(P.word[i]);
    t += P.src64 ? P.src64[i] : (P.src32 ? (double)P.src32[i] : 1.0);
  }
  __shared__ double rs[256], rt[256];
  rs[threadIdx.x] = s;
  rt[threadIdx.x] = t;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      rs[threadIdx.x] += rs[threadIdx.x + w];
      rt[threadIdx.x] += rt[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = rs[0];
    partial[2 * blockIdx.x + 1] = rt[0];
  }
}

// Workgroups of a persistent launch: as many as can be resident at once.
template <typename K>
hipError_t resident(K* kernel, int64_t* out) {
  int dev = 0, cus = 0, per = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, PT, 0);
  if (e != hipSuccess) return e;
  if (per < 1 || cus < 1) return hipErrorLaunchFailure;
  *out = (int64_t)cus * per;
  return hipSuccess;
}

template <int RK, bool ADJ, int VK>
hipError_t peel_t(const PeelGrid& P, const TileQueue& Q, const int32_t* gate, hipStream_t s) {
  int64_t grid = 0;
  const hipError_t e = resident(k_peel<RK, ADJ, VK>, &grid);
  if (e != hipSuccess) return e;
  const int64_t nt = (int64_t)P.ntr * P.ntc;
  if (grid > nt) grid = nt;
  hipLaunchKernelGGL((k_peel<RK, ADJ, VK>), dim3((unsigned)grid), dim3(PT), 0, s, P, Q, gate);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_peel(RuleKind rk, bool adjoint, ValKind vk, const PeelGrid& P, const TileQueue& Q,
                       const int32_t* gate, hipStream_t s) {
  int64_t b = (P.nrows * P.ncols + 255) / 256;
  if (b > 4096) b = 4096;
  hipLaunchKernelGGL(k_peel_init, dim3((unsigned)b), dim3(256), 0, s, P, Q, adjoint ? 1 : 0, gate);
  if (rk == RK_SINGLE) {
    if (!adjoint) return hipErrorInvalidValue;
    return vk == VK_F64 ? peel_t<RK_SINGLE, true, VK_F64>(P, Q, gate, s)
                        : peel_t<RK_SINGLE, true, VK_FF>(P, Q, gate, s);
  }
  if (adjoint)
    return vk == VK_F64 ? peel_t<RK_MULTI, true, VK_F64>(P, Q, gate, s) : peel_t<RK_MULTI, true, VK_FF>(P, Q, gate, s);
  return vk == VK_F64 ? peel_t<RK_MULTI, false, VK_F64>(P, Q, gate, s) : peel_t<RK_MULTI, false, VK_FF>(P, Q, gate, s);
}

hipError_t launch_peel_mass(const PeelGrid& P, double* partial, int nblocks, double* out, const int32_t* gate,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_peel_mass, dim3(nblocks), dim3(256), 0, s, P, partial, gate);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_mass_final_if(partial, nblocks, out, gate, s);
}

hipError_t launch_peel_batch(const fr_tile* tiles_dev, int32_t ntiles, int order, int workers, int limit, int32_t* status,
                             char* ws, size_t ws_bytes, hipStream_t s) {
  int64_t grid = 0;
  const hipError_t e = resident(k_peel_batch, &grid);
  if (e != hipSuccess) return e;
  if (workers > 0 && grid > workers) grid = workers;
  hipLaunchKernelGGL(k_peel_batch_setup, dim3(1), dim3(1024), 0, s, tiles_dev, ntiles, order,
                     limit, (int32_t)(GROUP_TILES * grid), ws, ws_bytes, status);
  const PeelBatch* B = reinterpret_cast<const PeelBatch*>(ws);
  hipLaunchKernelGGL(k_peel_batch_init, dim3((unsigned)ntiles, BATCH_FILL_BLOCKS), dim3(256), 0, s, B);
  hipLaunchKernelGGL(k_peel_batch, dim3((unsigned)grid), dim3(PT), 0, s, B);
  return hipGetLastError();
}

}  // namespace fr
