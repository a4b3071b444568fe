// Depression filling on the GPU: the surface the priority-flood method
// produces (Section 4 fills the DEM that way before routing), computed by
// tiled relaxation instead of a global priority queue.
//
// The filled surface F solves F = z on the grid boundary and
//     F(c) = max(z(c), min over neighbours n of next(F(n)))
// elsewhere, next(x) being the next float32 above x (epsilon variant) or x.
// Starting from F = +inf inside, every update F(c) <- max(z(c), min(F(c),
// next(F(n)) ...)) can only lower F and never below the solution, so any
// order of updates, stale neighbour values included, ends at the solution;
// a state in which no update changes anything is the solution.
//
// The surface from above: what takes time is how often a tile has to be
// looked at again, and how many tiles a value crosses one after another.  From
// +inf inside, values first enter a basin by bad paths and are lowered again
// and again, and the middle of the grid is only reached after as many launches
// as tiles lie before it.  So coarser grids go first: a cell of one stands for
// FILL_STEP x FILL_STEP cells of the one before, its elevation is their
// largest plus FILL_STEP - 1 rises, and its surface, solved in the same way
// with FILL_STEP rises from cell to cell, lies on or above theirs: from any
// cell of a block a path inside the block reaches the next block of the
// coarse path, or the grid's boundary, in at most that many steps and never
// above the block's largest elevation.  Any start on or above the surface
// ends at it.
//
// Layout: one wavefront owns a tile of 62 x 62 cells and holds it, with its
// one-cell halo ring, as a 64 x 64 window of order-preserving uint32 keys (so
// min, max and next are integer operations, exact for subnormals): lane =
// window column while sweeping down and up the rows, lane = window row
// (after a transpose through LDS) while sweeping right and left.  Neighbours
// in other lanes arrive by DPP wavefront shifts; the halo lanes and steps are
// read once per launch and never updated, so no lane needs an edge case.
// Elevations stay in LDS, read in either orientation.  A tile repeats its
// four sweeps until one sweep changes nothing (or a round cap is reached),
// then writes its own cells back.  Launch k works through a list of the
// tiles with a cell that a tile's new values in launch k - 1 would lower (the
// first list: all tiles); the host stops once a list is empty.
//
// Measured (epsilon variant, 8 neighbours, untilted fractal): 8192^2 17.1 ->
// 6.4 ms (96 launches with work -> 53 on the grid, after 16 on each of the two
// coarser ones, which cost about 3 us each once a list is empty).  The first
// launches over all 17424 tiles of 8192^2 take 1.2 ms each (four 33 KB
// workgroups a compute unit), those of the chain's end about 40 us, one
// tile's time.
#include "fr_internal.hpp"

namespace fr {
namespace {

constexpr int FT = 64;                     // window side = wavefront width
constexpr uint32_t KEY_INF = 0xFF800000u;  // key of +inf
constexpr int FILL_ROUNDS = 256;           // sweep rounds per tile and launch
static_assert(FT == FILL_TILE + 2, "a window is a tile and its halo");

// Order-preserving map of float32 to uint32 (-0 read as +0) and back.  The
// negative numbers' keys lie one above their inverted bits, which closes the
// gap that -0 would leave: the next key is the next float32 everywhere.
__device__ __forceinline__ uint32_t fkey(float x) {
  uint32_t b = __float_as_uint(x);
  if (b == 0x80000000u) b = 0;
  return (b & 0x80000000u) ? ~b + 1u : (b | 0x80000000u);
}
__device__ __forceinline__ float fval(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~(k - 1u));
}

// Lane i receives x of lane i - 1, or of lane i + 1; the halo lanes at the
// wavefront's ends keep their own value (never used).
__device__ __forceinline__ uint32_t from_lower(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t from_upper(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x130, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }

// One sweep over steps 1..62 of the window, forward or backward; lanes 1..62
// update.  zk(s) is the elevation key of this lane's cell at step s.  Every
// cell is evaluated with all its neighbours, so a sweep that changes nothing
// has found a fixed point of the tile (for its halo).
template <bool C8, bool FWD, typename ZK>
__device__ __forceinline__ bool sweep(uint32_t (&f)[FT], bool inner, uint32_t inc, ZK zk) {
  bool changed = false;
  // New values to the compiler, which would otherwise keep the lane-shifted
  // copies of one sweep for the next.
#pragma unroll
  for (int s = 0; s < FT; ++s) asm volatile("" : "+v"(f[s]));
#pragma unroll
  for (int i = 1; i < FT - 1; ++i) {
    const int s = FWD ? i : FT - 1 - i;
    const uint32_t prev = f[s - 1], next = f[s + 1];
    uint32_t m = umin(prev, next);
    m = umin(m, umin(from_lower(f[s]), from_upper(f[s])));
    if (C8) {
      m = umin(m, umin(from_lower(prev), from_upper(prev)));
      m = umin(m, umin(from_lower(next), from_upper(next)));
    }
    // m <= KEY_INF, so m + inc cannot wrap; min with f (<= KEY_INF) keeps
    // every value a valid key.
    const uint32_t nv = umax(zk(s), umin(f[s], m + inc));
    const bool ch = inner && nv != f[s];
    changed |= ch;
    f[s] = ch ? nv : f[s];
  }
  return __any(changed);
}

// a[s] of lane l becomes a[l] of lane s (64 x 64 transpose through LDS).
__device__ __forceinline__ void transpose(uint32_t (&a)[FT], uint32_t (*sT)[FT + 1], int lane) {
  __syncthreads();
#pragma unroll
  for (int s = 0; s < FT; ++s) sT[s][lane] = a[s];
  __syncthreads();
#pragma unroll
  for (int s = 0; s < FT; ++s) a[s] = sT[lane][s];
}

// The halo cells that the window's values would lower, as tiles to wake: bit
// 3 (dr + 1) + dc + 1 of the neighbour at (dr, dc).  Column orientation.
template <bool C8, typename ZK>
__device__ __forceinline__ uint32_t lowered(uint32_t (&f)[FT], uint32_t inc, int lane, ZK zk) {
  const bool inner = lane >= 1 && lane <= FT - 2;
#pragma unroll
  for (int s = 0; s < FT; ++s) asm volatile("" : "+v"(f[s]));
  // The row above (s = 0) and below: from the tile's first and last row.
  auto row = [&](int s, int in) -> bool {
    const uint32_t a = from_lower(f[in]), b = from_upper(f[in]);
    uint32_t m = inner ? f[in] : KEY_INF;
    if (C8) m = umin(m, lane == 0 ? b : (lane == FT - 1 ? a : umin(a, b)));
    return f[s] > umax(zk(s), m + inc);
  };
  const uint64_t t = __ballot(row(0, 1)), b = __ballot(row(FT - 1, FT - 2));
  // The columns beside: lanes 0 and 63, from lanes 1 and 62.
  bool low = false;
#pragma unroll
  for (int s = 1; s < FT - 1; ++s) {
    uint32_t m = f[s];
    if (C8) m = umin(m, umin(s > 1 ? f[s - 1] : KEY_INF, s < FT - 2 ? f[s + 1] : KEY_INF));
    const uint32_t below = from_lower(m), above = from_upper(m);  // every lane takes part
    const uint32_t n = lane == 0 ? above : below;
    low |= f[s] > umax(zk(s), n + inc);
  }
  const uint64_t c = __ballot(low);
  const uint64_t mid = ~(1ull | (1ull << 63));
  return (uint32_t)(t & 1ull) | ((t & mid) ? 2u : 0u) | ((t >> 63) ? 4u : 0u) | ((c & 1ull) ? 8u : 0u) |
         ((c >> 63) ? 32u : 0u) | ((b & 1ull) ? 64u : 0u) | ((b & mid) ? 128u : 0u) | ((b >> 63) ? 256u : 0u);
}

// Level l + 1's elevations: the largest of each block, plus the rises from
// one of its cells to another.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_fill_coarse(FillLevel V, FillLevel W, uint32_t rises) {
  const int64_t n = W.nr * W.nc;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r0 = i / W.nc * FILL_STEP, c0 = i % W.nc * FILL_STEP;
    uint32_t m = 0;
    for (int r = 0; r < FILL_STEP; ++r) {
      const int64_t y = r0 + r < V.nr ? r0 + r : V.nr - 1;
#pragma unroll
      for (int c = 0; c < FILL_STEP; ++c) {
        const int64_t x = c0 + c < V.nc ? c0 + c : V.nc - 1;
        m = umax(m, FIRST ? fkey(V.z[y * V.nc + x]) : V.zk[y * V.nc + x]);
      }
    }
    W.zk[i] = umin(m, KEY_INF - rises) + rises;
  }
}

// The surface's start on level V: the elevations on the boundary, inside
// what the coarser level W gives (+inf without one); every tile queued.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_fill_init(FillLevel V, FillLevel W, bool coarse, FillState S,
                                                   int32_t* status) {
  bool bad = false;
  const int64_t n = V.nr * V.nc;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x, i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = i0; i < n; i += stride) {
    const int64_t r = i / V.nc, c = i - r * V.nc;
    const bool edge = r == 0 || c == 0 || r == V.nr - 1 || c == V.nc - 1;
    uint32_t k;
    if (FIRST) {
      const float v = V.z[i];
      bad |= !isfinite(v);
      k = fkey(v);
    } else {
      k = V.zk[i];
    }
    if (!edge) k = coarse ? umax(k, W.Fk[r / FILL_STEP * W.nc + c / FILL_STEP]) : KEY_INF;
    if (FIRST) V.F[i] = fval(k);
    else V.Fk[i] = k;
  }
  const int32_t nt = V.ntr * V.ntc;
  for (int64_t t = i0; t < nt; t += stride) {
    S.queued[t] = 0;
    S.list[t] = (int32_t)t;
  }
  if (i0 == 0) {
    S.nlist[0] = nt;
    S.nlist[1] = 0;
    S.nlist[2] = 0;
    *S.last = -1;
  }
  if (bad && status) atomicCAS(status, 0, FR_ERR_NONFINITE);
}

// Relaxes tile (tr, tc) until a sweep changes nothing or the round cap is hit
// and writes its cells back if any changed.  Returns lowered()'s bits, and
// bit 4 (the tile itself) for a stop at the round cap; 0x200 if any cell
// changed.
template <bool C8, bool FIRST>
__device__ __forceinline__ uint32_t fill_tile(const FillLevel& V, int32_t tr, int32_t tc, uint32_t (*sT)[FT + 1],
                                              uint32_t (*sZ)[FT + 1], int lane) {
  // Window row w is grid row wr0 + w; window column lane is grid column
  // wc0 + lane.  Cells off the grid are +inf with elevation +inf: they never
  // change and lower nothing.
  const int32_t wr0 = tr * FILL_TILE - 1, wc0 = tc * FILL_TILE - 1;
  const int32_t nr = (int32_t)V.nr, nc = (int32_t)V.nc;
  const int32_t col = wc0 + lane;
  const bool col_in = col >= 0 && col < nc;
  const int32_t ccol = col < 0 ? 0 : (col < nc ? col : nc - 1);
  const uint32_t* const Z = FIRST ? reinterpret_cast<const uint32_t*>(V.z) : V.zk;
  uint32_t* const F = FIRST ? reinterpret_cast<uint32_t*>(V.F) : V.Fk;
  uint32_t f[FT];
  __syncthreads();  // the previous tile's LDS reads are done
  // Unconditional loads at clamped addresses, all in flight together (behind
  // a condition each would be waited for).
  uint32_t z[FT];
  {
    const int64_t at = (int64_t)(wr0 < 0 ? 0 : wr0) * nc + ccol;
    const uint32_t *fp = F + at, *zp = Z + at;
#pragma unroll
    for (int s = 0; s < FT; ++s) {
      f[s] = *fp;
      z[s] = *zp;
      // The next row, as far as the grid goes (addresses opaque to the
      // compiler, which would compute and hold them all beforehand).
      const int32_t step = wr0 + s >= 0 && wr0 + s < nr - 1 ? nc : 0;
      fp += step;
      zp += step;
      if (s % 8 == 7) asm volatile("" : "+v"(fp), "+v"(zp));
    }
  }
#pragma unroll
  for (int s = 0; s < FT; ++s) {
    const int32_t row = wr0 + s;
    const bool in = col_in && row >= 0 && row < nr;
    f[s] = in ? (FIRST ? fkey(__uint_as_float(f[s])) : f[s]) : KEY_INF;
    sZ[s][lane] = in ? (FIRST ? fkey(__uint_as_float(z[s])) : z[s]) : KEY_INF;
  }
  const bool inner = lane >= 1 && lane <= FT - 2;
  const auto zcol = [&](int s) { return sZ[s][lane]; };
  const auto zrow = [&](int s) { return sZ[lane][s]; };
  bool any = false, capped = true;
  for (int round = 0; round < FILL_ROUNDS && capped; ++round) {
    // Column orientation: steps = window rows, lanes = window columns.
    __syncthreads();
    if (!sweep<C8, true>(f, inner, V.inc, zcol)) {
      capped = false;
      break;
    }
    any = true;
    if (!sweep<C8, false>(f, inner, V.inc, zcol)) {
      capped = false;
      break;
    }
    transpose(f, sT, lane);
    // Row orientation: steps = window columns, lanes = window rows.
    if (!sweep<C8, true>(f, inner, V.inc, zrow)) capped = false;
    if (capped && !sweep<C8, false>(f, inner, V.inc, zrow)) capped = false;
    transpose(f, sT, lane);
  }
  if (!any) return 0;
#pragma unroll
  for (int s = 1; s < FT - 1; ++s) {
    const int32_t row = wr0 + s;
    if (inner && col_in && row < nr) F[(int64_t)row * nc + col] = FIRST ? __float_as_uint(fval(f[s])) : f[s];
  }
  return lowered<C8>(f, V.inc, lane, zcol) | (capped ? 16u : 0u) | 0x200u;
}

// Launch k works through list k (built by launch k - 1) and builds list
// k + 1: the neighbours of every tile that its new values would lower a cell
// of, and the tile itself when it stopped at the round cap, each once
// (queued[] holds the latest launch a tile was queued for).  List k + 2's
// length is cleared here: launch k + 1 fills it, and list k - 1, which shares
// its slot, is spent.
template <bool C8, bool FIRST>
__global__ __launch_bounds__(FT) void k_fill_tile(FillLevel V, FillState S, int32_t k) {
  __shared__ uint32_t sT[FT][FT + 1];
  __shared__ uint32_t sZ[FT][FT + 1];  // [window row][window column]
  const int lane = threadIdx.x;
  const int32_t ntiles = V.ntr * V.ntc;
  const int32_t cur = k % 3, nxt = (k + 1) % 3;
  if (blockIdx.x == 0 && lane == 0) S.nlist[(k + 2) % 3] = 0;
  const int32_t n = S.nlist[cur];
  const int32_t* list = S.list + (size_t)cur * ntiles;
  int32_t* out = S.list + (size_t)nxt * ntiles;
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int32_t t = list[i];
    const int32_t tr = t / V.ntc, tc = t - tr * V.ntc;
    const uint32_t res = fill_tile<C8, FIRST>(V, tr, tc, sT, sZ, lane);
    if (res == 0) continue;
    if (lane < 9 && ((res >> lane) & 1u)) {
      const int32_t rr = tr + lane / 3 - 1, cc = tc + lane % 3 - 1;
      if (rr >= 0 && rr < V.ntr && cc >= 0 && cc < V.ntc) {
        const int32_t u = rr * V.ntc + cc;
        if (atomicMax(&S.queued[u], k + 1) < k + 1) out[atomicAdd(&S.nlist[nxt], 1)] = u;
      }
    }
    if (lane == 0) __hip_atomic_store(S.last, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

int blocks_for(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return (int)(b > 8192 ? 8192 : (b < 1 ? 1 : b));
}

}  // namespace

hipError_t launch_fill_coarse(const FillLevel& V, const FillLevel& W, bool c8, hipStream_t s) {
  const uint32_t rises = V.inc * (uint32_t)(c8 ? FILL_STEP - 1 : 2 * (FILL_STEP - 1));
  const dim3 grid(blocks_for(W.nr * W.nc)), block(256);
  if (V.z) hipLaunchKernelGGL((k_fill_coarse<true>), grid, block, 0, s, V, W, rises);
  else hipLaunchKernelGGL((k_fill_coarse<false>), grid, block, 0, s, V, W, rises);
  return hipGetLastError();
}

hipError_t launch_fill_init(const FillLevel& V, const FillLevel* W, const FillState& S, int32_t* status,
                            hipStream_t s) {
  const dim3 grid(blocks_for(V.nr * V.nc)), block(256);
  if (V.z) hipLaunchKernelGGL((k_fill_init<true>), grid, block, 0, s, V, W ? *W : V, W != nullptr, S, status);
  else hipLaunchKernelGGL((k_fill_init<false>), grid, block, 0, s, V, W ? *W : V, W != nullptr, S, status);
  return hipGetLastError();
}

hipError_t launch_fill_tiles(const FillLevel& V, bool c8, const FillState& S, int32_t k, hipStream_t s) {
  // Enough single-wavefront workgroups for every SIMD of the chip; each
  // walks the list with a grid stride.
  int64_t blocks = (int64_t)V.ntr * V.ntc;
  if (blocks > 2048) blocks = 2048;
  const dim3 grid((unsigned)blocks), block(FT);
  if (V.z) {
    if (c8) hipLaunchKernelGGL((k_fill_tile<true, true>), grid, block, 0, s, V, S, k);
    else hipLaunchKernelGGL((k_fill_tile<false, true>), grid, block, 0, s, V, S, k);
  } else {
    if (c8) hipLaunchKernelGGL((k_fill_tile<true, false>), grid, block, 0, s, V, S, k);
    else hipLaunchKernelGGL((k_fill_tile<false, false>), grid, block, 0, s, V, S, k);
  }
  return hipGetLastError();
}

}  // namespace fr
