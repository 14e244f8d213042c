// HIP kernels for the Ant Colony System hot path on gfx950 (MI355X).
//
// Method: Skinderowicz, "The GPU-based Parallel Ant Colony System" (JPDC
// 2016), Sec. 3.  The paper maps one ant to one 32-thread block and its 32
// candidates to the threads; here one ant owns one 64-wide wavefront, the
// candidates sit one per lane, and every decision of the ant (which branch of
// Eq. 1, which candidate, the fallback) is wave-uniform, so it runs on the
// scalar unit: reductions use DPP and permlane swaps (no LDS round trips),
// the winning lane's values are read with readlane, the Philox draws are
// scalar.  The visited set is a bitmap in LDS.
//
// Data layout (dense memory).  The static record of candidate k of city i
// and the pheromone of that directed entry share one 16-byte slot,
//   crec[i][k] = {j, d(i, j), eta^beta(d) bits, tau(i, j) bits},
// so one step reads one coalesced 16-byte load per lane.  The pheromone of a
// non-candidate entry (i, j) lives in tau[i][j] (n x ldn).  Every directed
// entry therefore has exactly one home; the fallback scan only reads
// non-candidate entries, because it runs only when every candidate is
// visited.
//
// Compiled with -ffp-contract=off: every float expression is the written
// sequence of IEEE operations; fmaf is used only for the pheromone maps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "acs_internal.hpp"
#include "acs_protocol.hpp"

namespace acs {
namespace {

constexpr uint32_t kNone = 0xffffffffu;
// fourth word of a buffer resource for untyped dword loads (gfx9 family)
constexpr int kBufWord3 = 0x00020000;
// cache policy of a buffer load that reads what the device's coherence point
// holds (sc1), for values other waves update during the launch
constexpr int kCoherent = 16;

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC 2011): ten rounds of the 4x32 S-box with
// multipliers 0xD2511F53 / 0xCD9E8D57, the key bumped by the Weyl constants
// 0x9E3779B9 / 0xBB67AE85 between rounds.  Counter = (step, ant, iteration,
// instance), key = the 64-bit seed.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
    const uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
    c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// Cost d_ij (Sec. 3) as TSPLIB EUC_2D made exact: s = dx*dx + dy*dy in
// double, d = the integer with (d - 1/2)^2 <= s < (d + 1/2)^2 (0 if s < 1/4).
// A handle's coordinates span less than 65536 each way, so sqrt(s) < 92682 and
// its fp32 approximation (the rounding of s and one ulp) is off by less than
// 0.02: its integer part is d, or d - 1 where sqrt(s) lies in the upper half
// before d or just above d, and one exact compare decides.
__device__ __forceinline__ uint32_t dist_of_square(double s) {
  const uint32_t d = (uint32_t)__builtin_amdgcn_sqrtf((float)s);
  const double h = d + 0.5;
  return d + (h * h <= s ? 1u : 0u);
}

__device__ __forceinline__ uint32_t exact_dist(double xi, double yi, double xj,
                                               double yj) {
  const double dx = xi - xj, dy = yi - yj;
  return dist_of_square(dx * dx + dy * dy);
}

// d(i, j) from the coordinates (the selective memory keeps no n x n matrix).
__device__ __forceinline__ uint32_t dist_xy(const Dev &D, int i, int j) {
  return exact_dist(D.xy[2 * i], D.xy[2 * i + 1], D.xy[2 * j], D.xy[2 * j + 1]);
}

template <typename T>
__device__ __forceinline__ T wave_min(T v) {
#pragma unroll
  for (int off = 32; off; off >>= 1) {
    const T o = __shfl_xor(v, off, 64);
    v = o < v ? o : v;
  }
  return v;
}

// Wave-wide unsigned max / min, all lanes active: quad and row permutations
// by DPP, then the row-pair and half-wave swaps of gfx950.  Returns the
// result as a wave-uniform value.
__device__ __forceinline__ uint32_t wave_umax_u(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(v, max((uint32_t)a[0], (uint32_t)a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  v = max(v, max((uint32_t)b[0], (uint32_t)b[1]));
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Maximum over lanes 0..31 (lanes 32..63 hold no candidate when cl <= 32),
// as a wave-uniform value.
__device__ __forceinline__ uint32_t half_umax_u(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(v, max((uint32_t)a[0], (uint32_t)a[1]));
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Wave-wide sum, every lane active (rare paths only: LDS permutes).
__device__ __forceinline__ uint32_t wave_sum_u(uint32_t v) {
#pragma unroll
  for (int off = 32; off; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off, 64);
  return v;
}

__device__ __forceinline__ uint32_t wave_umin_u(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = min(v, min((uint32_t)a[0], (uint32_t)a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  v = min(v, min((uint32_t)b[0], (uint32_t)b[1]));
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Marks city c visited in an LDS bitmap without waiting for the old word
// (LDS operations of a wave take effect in issue order, so the next read of
// the word sees the bit).
__device__ __forceinline__ void mark(uint32_t *vis, int c) {
  __hip_atomic_fetch_or(vis + (c >> 5), 1u << (c & 31), __ATOMIC_RELAXED,
                        __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ uint32_t rdlane(uint32_t v, int k) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, k);
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// v_writelane: lane k of the result is s (wave-uniform), the other lanes
// keep old.  The compiler exposes it only as the LLVM intrinsic.
extern "C" __device__ int acs_writelane_i32(int s, int k, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ uint32_t wrlane(uint32_t s, int k, uint32_t old) {
  return (uint32_t)acs_writelane_i32((int)s, k, (int)old);
}

// Maximum over lanes 0..L-1 (L = 16, 32 or 64) as a scalar: the row
// maxima by DPP, then one read per row.  Fewer instructions than a
// full-wave finish when only the scalar is needed.
template <int L>
__device__ __forceinline__ uint32_t rows_umax_s(uint32_t v) {
  static_assert(L == 16 || L == 32 || L == 64, "16, 32 or 64 lanes");
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
  if (L == 16) return rdlane(v, 0);
  const uint32_t m01 = max(rdlane(v, 0), rdlane(v, 16));
  if (L == 32) return m01;
  return max(m01, max(rdlane(v, 32), rdlane(v, 48)));
}

// A pointer read from memory (a batch's descriptors) is generic to the
// compiler, which makes flat accesses of it; they count as LDS operations too.
// These are all to global memory.
template <class T>
__device__ __forceinline__ T *as_global(T *p) {
  return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}
__device__ __forceinline__ Dev global_dev(const Dev &d) {
  Dev D = d;
  D.xy = as_global(d.xy);
  D.dist = as_global(d.dist);
  D.crec = as_global(d.crec);
  D.tau = as_global(d.tau);
  D.etad = as_global(d.etad);
  D.rpos = as_global(d.rpos);
  D.fpre = as_global(d.fpre);
  D.fbound = as_global(d.fbound);
  D.ctau = as_global(d.ctau);
  D.tours = as_global(d.tours);
  D.lens = as_global(d.lens);
  D.counters = as_global(d.counters);
  D.sync = as_global(d.sync);
  return D;
}

// Pheromone slot of candidate k in city u's record.
__device__ __forceinline__ float *cand_tau(const Dev &D, int u, int k) {
  return reinterpret_cast<float *>(const_cast<uint4 *>(D.crec) + (size_t)u * D.cl + k) + 3;
}

// Home of the directed entry (u, v): candidate slot k of u, or tau[u][v].
__device__ __forceinline__ float *home(const Dev &D, int u, int v, int k) {
  return k >= 0 ? cand_tau(D, u, k) : D.tau + (size_t)u * D.ldn + v;
}

// Home of the directed entry (u, v) while a construction with an updater
// wave runs: slot k of u's row of ctau, or tau[u][v].
__device__ __forceinline__ float *qhome(const Dev &D, int u, int v, int k) {
  return k >= 0 ? D.ctau + (size_t)u * D.cl + k : D.tau + (size_t)u * D.ldn + v;
}

// Agent-coherent read of one pheromone value (sees every CAS performed so
// far on the device, whichever XCD performed it).
__device__ __forceinline__ float tau_load(const float *p) {
  return __uint_as_float(__hip_atomic_load(reinterpret_cast<const unsigned int *>(p),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Local or global map x -> fma(a, x, b), applied atomically.  `seen` is the
// value the caller believes the entry holds; a failed compare-and-swap (the
// entry changed meanwhile) retries with the value it returned.  Returns the
// number of retries.
__device__ __forceinline__ uint32_t cas_apply(float *p, unsigned int seen, float a, float b) {
  unsigned int *q = reinterpret_cast<unsigned int *>(p);
  unsigned int old = seen;
  uint32_t retries = 0;
  while (true) {
    const unsigned int nw = __float_as_uint(fmaf(a, __uint_as_float(old), b));
    const unsigned int prev = atomicCAS(q, old, nw);
    if (prev == old) break;
    old = prev;
    ++retries;
  }
  return retries;
}

// Whether the local map leaves x unchanged (in fp32).  During a
// construction an entry only receives that map, so an entry read at such a
// value still holds it, and its update can be skipped without changing any
// result.
__device__ __forceinline__ bool map_fixed(float x, float a, float b) {
  return __float_as_uint(fmaf(a, x, b)) == __float_as_uint(x);
}

// The local map applied `times` times to the value with bits x.
__device__ __forceinline__ unsigned int map_times(unsigned int x, uint32_t times, float a,
                                                  float b) {
  for (uint32_t i = 0; i < times; ++i) {
    const unsigned int y = __float_as_uint(fmaf(a, __uint_as_float(x), b));
    if (y == x) break;
    x = y;
  }
  return x;
}

// Position of v in the candidate list of u (wave-uniform), or -1.
__device__ __forceinline__ int cand_pos(const Dev &D, int u, int v, int lane) {
  const int kl = lane < D.cl ? lane : D.cl - 1;
  const uint32_t j = D.crec[(size_t)u * D.cl + kl].x;
  const uint64_t b = __ballot(lane < D.cl && j == (uint32_t)v);
  return b ? (int)__ffsll((unsigned long long)b) - 1 : -1;
}

// Grid-wide barrier for a cooperative launch, in two levels that follow the
// chip: the blocks of one XCD share an L2, the XCDs meet beyond it.  A flag
// stored and polled inside one XCD takes about 730 cycles to be seen, one
// across XCDs about 1800, and every poller of a line pays again after each
// store to it.  So each block flags its arrival in its XCD's own list, the
// first block of the XCD (its leader) waits for those, tells every XCD by one
// store into that XCD's mailbox line, and every block waits on the mailbox
// of its own XCD.  With one flag line per block polled by every block, a
// barrier took 2700 cycles with 13 blocks, 5600 with 150 and 7300 with 256;
// this takes 2300 to 2500 at all of these.
//
// Every wave waits for its own memory operations first (the local updates
// are compare-and-swaps whose results have been consumed, so they are
// performed at the device's coherence point).  Readers after the barrier use
// agent-coherent loads for everything the updates touch, so no cache
// write-back or invalidation is needed.
//
// The waits are bounded: on exhaustion an error flag is raised, later waits no
// longer poll, and the kernel runs to its end.  (Epochs: see barrier_reached.)
//
// Dev::bflags holds, per XCD (8), a list of one arrival epoch per block of the
// grid and a mailbox of 8 epochs (one per XCD), in 128-byte lines of their
// own, then one word per block with its XCD, tagged by the iteration.
struct GridBar {       // the first wave's
  uint32_t *mine, *list, *box;
  uint32_t members, xcds;  // blocks of this XCD; mask of the XCDs in use
  bool leader;
};

__device__ __forceinline__ bool reached(const uint32_t *flag, uint32_t epoch) {
  return barrier_reached(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                         epoch);
}

// Polls until `done` holds on every lane of the wave; false when the wait
// gave up.  Once any block has given up, no later wait polls long either
// (looked at every 64th poll, so a poll costs the flag loads only).
template <class F>
__device__ __forceinline__ bool bounded_wait(const Dev &D, F done) {
  for (uint32_t spins = 0;; ++spins) {
    if (__ballot(!done()) == 0) return true;
    if ((spins & 63) == 63 &&
        __hip_atomic_load(D.sync + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
      return false;
    if (spins >= (D.wait_limit ? D.wait_limit : (1u << 22))) {
      if ((threadIdx.x & 63) == 0)
        __hip_atomic_store(D.sync + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
  }
}

// words of one XCD's list, and of its list and mailbox
__device__ __forceinline__ uint32_t xcd_list() { return (gridDim.x + 31) & ~31u; }
__device__ __forceinline__ uint32_t xcd_words() { return xcd_list() + 32; }

// Start of a cooperative kernel: every block publishes its XCD and counts the
// others of the same one.
__device__ __forceinline__ GridBar grid_join(const Dev &D, const Iter &A) {
  GridBar B{};
  if (threadIdx.x >= 64) return B;
  const uint32_t lane = threadIdx.x, G = gridDim.x, self = blockIdx.x;
  // HW_REG_XCC_ID, its low three bits
  const uint32_t x = (uint32_t)__builtin_amdgcn_s_getreg(20 | (2 << 11));
  uint32_t *tab = D.bflags + kXcds * xcd_words();
  const uint32_t tag = (A.it + 1) << 4 | 8;  // no other iteration's, nor a cleared word
  if (lane == 0)
    __hip_atomic_store(tab + self, tag | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t rank = 0, members = 0, xcds = 0;
  for (uint32_t b0 = 0; b0 < G; b0 += 64) {
    const uint32_t b = min(b0 + lane, G - 1);
    uint32_t v = 0;
    bounded_wait(D, [&]() {
      v = __hip_atomic_load(tab + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return (v & ~7u) == tag;
    });
    const uint32_t id = v & 7;
    const uint64_t same = __ballot(b0 + lane < G && id == x);
    members += (uint32_t)__popcll(same);
    if (self >= b0) {
      const uint32_t q = self - b0;
      rank += (uint32_t)__popcll(q >= 64 ? same : same & ((1ull << q) - 1));
    }
    for (uint32_t i = 0; i < kXcds; ++i)
      if (__ballot(b0 + lane < G && id == i)) xcds |= 1u << i;
  }
  B.list = D.bflags + x * xcd_words();
  B.box = B.list + xcd_list();
  B.mine = rank == 0 ? D.bflags + xcd_list() + x : B.list + rank;
  B.members = members;
  B.xcds = xcds;
  B.leader = rank == 0;
  return B;
}

__device__ __forceinline__ void grid_barrier_f(const Dev &D, const GridBar &B, uint32_t epoch) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x < 64) {
    const uint32_t lane = threadIdx.x;
    if (B.leader) {
      for (uint32_t b0 = 1; b0 < B.members; b0 += 64)
        bounded_wait(D, [&]() {
          return b0 + lane >= B.members || reached(B.list + b0 + lane, epoch);
        });
      // this XCD's entry of every XCD's mailbox
      if (lane < kXcds && ((B.xcds >> lane) & 1u))
        __hip_atomic_store(B.mine + lane * xcd_words(), epoch, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    } else if (lane == 0) {
      // read by a block that shares this L2: no write beyond it is needed
      __hip_atomic_store(B.mine, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    bounded_wait(D, [&]() {
      return lane >= kXcds || !((B.xcds >> lane) & 1u) || reached(B.box + lane, epoch);
    });
  }
  __syncthreads();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// ---------------------------------------------------------------------------
// Instance preparation kernels.
// ---------------------------------------------------------------------------
// Largest value of a block's lanes into *word.  The block reduces it in LDS
// first and skips the atomic when the word already holds as much: one atomic
// per wave on one address took 12.9 ms per 2 * 10^8 distances, about all of
// the kernel's time.
__device__ __forceinline__ void block_max_into(uint32_t v, uint32_t *word) {
  __shared__ uint32_t sm[16];
  v = wave_umax_u(v);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) v = max(v, sm[w]);
    if (v > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(word, v);
  }
}

// Rows r0 .. r0 + rows - 1 of the distance matrix, stored from the start of
// D.dist, and (dmax not null) the largest distance into *dmax.  A wave takes
// 512 columns of a row, eight per lane and one 16-byte store.
__global__ __launch_bounds__(256) void k_dist(Dev D, uint32_t *dmax, int r0, int rows) {
  const int j0 = 8 * (blockIdx.x * 64 + (threadIdx.x & 63));
  const int r = blockIdx.y * 4 + (threadIdx.x >> 6);
  const int i = r0 + r;
  uint32_t mx = 0;
  if (r < rows && i < D.n && j0 < D.ldn) {
    const double xi = D.xy[2 * i], yi = D.xy[2 * i + 1];
    const double2 *c = reinterpret_cast<const double2 *>(D.xy);
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = j0 + q;
      const double2 p = c[min(j, D.n - 1)];
      uint32_t d = j < D.n && j != i ? exact_dist(xi, yi, p.x, p.y) : 0u;
      mx = max(mx, d);
      d = min(d, 65535u);
      w[q >> 1] = q & 1 ? w[q >> 1] | d << 16 : d;
    }
    *reinterpret_cast<uint4 *>(const_cast<uint16_t *>(D.dist) + (size_t)r * D.ldn + j0) =
        make_uint4(w[0], w[1], w[2], w[3]);
  }
  if (dmax) block_max_into(mx, dmax);
}

// The largest distance of the instance without a matrix (selective memory):
// distances grow with their squares, so each thread keeps the largest square
// of its city against kDmaxRows others (read through the scalar cache) and
// takes one root.  Pairs are covered once, from the smaller index's side.
constexpr int kDmaxRows = 256;
__global__ __launch_bounds__(256) void k_dmax(Dev D, uint32_t *dmax) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  const int i0 = blockIdx.y * kDmaxRows;
  if (i0 > (int)(blockIdx.x * 256 + 255)) return;  // the whole block: no i < j
  const double2 *c = reinterpret_cast<const double2 *>(D.xy);
  const double2 p = c[min(j, D.n - 1)];
  const int i1 = min(i0 + kDmaxRows, D.n);
  double s = 0.0;
  for (int i = i0; i < i1; ++i) {
    const double dx = p.x - c[i].x, dy = p.y - c[i].y;
    s = fmax(s, dx * dx + dy * dy);
  }
  block_max_into(dist_of_square(s), dmax);
}

// The nearest cities of city r0 + blockIdx.x by (d, j), from its row of
// distances (D.dist holds rows r0 .. from its start): the cl candidates, and
// beyond them the fallback's prefix with the key of the city after it (dense;
// the eta^beta words follow with k_fill) or the extended list (selective
// memory).  One block per city: a histogram of the distances (1024 bins over
// the instance's range, refined to single distances when the bin of the K-th
// city is crowded) gives a threshold, the cities within it are gathered into
// LDS and each finds its rank among them.  Three passes over the row replace
// one pass per listed city, which took 13.7 ms for 2048 rows of n = 20000
// (now 0.031 ms) and 1.3 ms for all rows of n = 2392 (now 0.017 ms).
constexpr int kNearBins = 1024, kNearCap = 512;

__device__ __forceinline__ void near_emit(const Dev &D, int32_t *cand, int i, int rank,
                                          uint32_t key) {
  if (rank < D.cl) cand[(size_t)i * D.cl + rank] = (int32_t)(key & 0xffffu);
  if (D.xnn && rank < D.xl) const_cast<uint32_t *>(D.xnn)[(size_t)i * D.xl + rank] = key;
  if (D.fpre) {
    const int p = rank - D.cl;
    uint32_t *out = reinterpret_cast<uint32_t *>(const_cast<uint4 *>(D.fpre)) +
                    (size_t)i * 2 * kFpre;
    if (p >= 0 && p < kFpre) out[2 * p] = key;
    if (p == kFpre) const_cast<uint32_t *>(D.flim)[i] = key;
  }
}

__global__ __launch_bounds__(256) void k_near(Dev D, int32_t *cand, const uint32_t *dmax, int r0) {
  __shared__ uint32_t hist[kNearBins];
  __shared__ alignas(16) uint32_t keys[kNearCap];
  __shared__ uint32_t wsum[4], s_bin, s_before, s_count, s_fill;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int i = r0 + blockIdx.x, n = D.n;
  const uint16_t *row = D.dist + (size_t)blockIdx.x * D.ldn;
  const uint32_t K = (uint32_t)(D.fpre ? D.cl + kFpre + 1 : D.xnn ? max(D.cl, D.xl) : D.cl);
  const uint32_t dm = min(*dmax, 65535u);
  const int S = max(0, 22 - (int)__clz((int)max(dm, 1u)));  // dm >> S < 1024

  auto each = [&](auto f) {  // f(d, j) over the row's other cities
    for (int j0 = 8 * tid; j0 < n; j0 += 2048) {
      const uint4 v = *reinterpret_cast<const uint4 *>(row + j0);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int j = j0 + q;
        if (j < n && j != i) f((w[q >> 1] >> (16 * (q & 1))) & 0xffffu, (uint32_t)j);
      }
    }
  };
  // the bin where the running count from `before` reaches K: s_bin, the
  // count below it s_before and through it s_count
  auto find = [&](uint32_t before) {
    uint32_t h[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) sum += h[q] = hist[4 * tid + q];
    uint32_t inc = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t o = (uint32_t)__shfl_up((int)inc, off, 64);
      if (lane >= off) inc += o;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    uint32_t run = before + inc - sum;
    for (int w = 0; w < wv; ++w) run += wsum[w];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (run < K && run + h[q] >= K) {
        s_bin = (uint32_t)(4 * tid + q);
        s_before = run;
        s_count = run + h[q];
      }
      run += h[q];
    }
    __syncthreads();
  };

  for (int b = tid; b < kNearBins; b += 256) hist[b] = 0u;
  if (tid == 0) s_fill = 0u;
  __syncthreads();
  each([&](uint32_t d, uint32_t) { atomicAdd(&hist[d >> S], 1u); });
  __syncthreads();
  find(0u);
  uint32_t limit = ((s_bin + 1) << S) - 1u, count = s_count;
  if (count > (uint32_t)kNearCap && S > 0) {
    const uint32_t bin = s_bin, before = s_before;
    __syncthreads();
    for (int b = tid; b < kNearBins; b += 256) hist[b] = 0u;
    __syncthreads();
    each([&](uint32_t d, uint32_t) {
      if (d >> S == bin) atomicAdd(&hist[d & ((1u << S) - 1u)], 1u);
    });
    __syncthreads();
    find(before);
    limit = (bin << S) + s_bin;
    count = s_count;
  }
  if (count > (uint32_t)kNearCap) {
    // hundreds of cities at one distance: one pass per listed city
    if (wv > 0) return;
    int64_t last = -1;
    for (uint32_t k = 0; k < K; ++k) {
      int64_t best = INT64_MAX;
      for (int j = lane; j < n; j += 64) {
        if (j == i) continue;
        const int64_t key = ((int64_t)row[j] << 16) | j;
        if (key > last && key < best) best = key;
      }
      best = wave_min(best);
      if (lane == 0) near_emit(D, cand, i, (int)k, (uint32_t)best);
      last = best;
    }
    return;
  }
  each([&](uint32_t d, uint32_t j) {
    if (d <= limit) keys[atomicAdd(&s_fill, 1u)] = d << 16 | j;
  });
  __syncthreads();
  if (tid < 4 && count + tid < (uint32_t)kNearCap) keys[count + tid] = kNone;
  __syncthreads();
  for (uint32_t u = tid; u < count; u += 256) {
    const uint32_t key = keys[u];
    uint32_t rank = 0;
    for (uint32_t v = 0; v < count; v += 4) {
      const uint4 o = *reinterpret_cast<const uint4 *>(keys + v);
      rank += (o.x < key) + (o.y < key) + (o.z < key) + (o.w < key);
    }
    if (rank < K) near_emit(D, cand, i, (int)rank, key);
  }
}

// Uniform grid over the cities (selective memory): the fallback's search
// for the nearest unvisited city reads whole cells, nearest first.  Cell of a
// coordinate, clamped to the grid.
__device__ __forceinline__ int grid_cx(const Dev &D, double x) {
  return min(max((int)((x - D.gx0) * D.ginv), 0), D.gnx - 1);
}
__device__ __forceinline__ int grid_cy(const Dev &D, double y) {
  return min(max((int)((y - D.gy0) * D.ginv), 0), D.gny - 1);
}

__global__ __launch_bounds__(256) void k_grid_count(Dev D, int32_t *cnt) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= D.n) return;
  atomicAdd(&cnt[grid_cy(D, D.xy[2 * j + 1]) * D.gnx + grid_cx(D, D.xy[2 * j])], 1);
}

// Exclusive prefix sum of the counts into gstart (one block); cnt becomes
// the fill cursor (a copy of the starts).
__global__ __launch_bounds__(1024) void k_grid_scan(Dev D, int32_t *cnt) {
  __shared__ int32_t part[1024];
  const int cells = D.gnx * D.gny;
  const int per = (cells + 1023) / 1024;
  const int c0 = min(cells, (int)threadIdx.x * per), c1 = min(cells, c0 + per);
  int32_t sum = 0;
  for (int c = c0; c < c1; ++c) sum += cnt[c];
  part[threadIdx.x] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t run = 0;
    for (int i = 0; i < 1024; ++i) {
      const int32_t x = part[i];
      part[i] = run;
      run += x;
    }
  }
  __syncthreads();
  int32_t *gstart = const_cast<int32_t *>(D.gstart);
  int32_t run = part[threadIdx.x];
  for (int c = c0; c < c1; ++c) {
    const int32_t x = cnt[c];
    gstart[c] = run;
    cnt[c] = run;
    run += x;
  }
  if (threadIdx.x == 0) gstart[cells] = D.n;
}

// Cities into their cells (order inside a cell is immaterial: the search
// takes the least (d, j) over every city it reads).
__global__ __launch_bounds__(256) void k_grid_fill(Dev D, int32_t *cur) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= D.n) return;
  const double x = D.xy[2 * j], y = D.xy[2 * j + 1];
  const int p = atomicAdd(&cur[grid_cy(D, y) * D.gnx + grid_cx(D, x)], 1);
  const_cast<uint32_t *>(D.gcity)[p] = (uint32_t)j;
  const_cast<double2 *>(D.gxy)[p] = make_double2(x, y);
}

// Nearest-neighbour tour from city 0 (ties: lowest index), one block; its
// length L_nn defines tau0 = 1 / (n * L_nn).  A chain of n - 1 dependent
// choices, so what counts is one choice's latency: the first C neighbours of
// every city sit in LDS as 16-bit indices (as many of 16 as fit) and the first
// wave follows them alone, with LDS operations only and one store per 64
// cities.  Where they are all visited, it reads the first 16 from `near`
// (16-bit, n x 16, where C < 16: this block writes it first, so it comes from
// its L2), then the city's stored list (the candidates and the prefix, or the
// extended list), and only when that is used up too does the whole block scan
// every city.  The lists are sorted by (d, j), so the first unvisited city of
// one is the answer.  The order is left in D.best (not in use yet) and summed
// at the end by all threads.  With a block barrier and a row scan or a list
// read per choice, n = 2392 took 5.6 ms and n = 20000 14.1 ms; this takes
// 0.40 and 6.3 ms (0.16 us a choice).
constexpr int kNnList = 16;
template <bool NEAR>
__global__ __launch_bounds__(1024) void k_nn_tour(Dev D, const int32_t *cand, int C,
                                                  uint16_t *near, int64_t *lnn) {
  extern __shared__ uint16_t lst[];  // n x C
  __shared__ uint32_t vis[2048];
  __shared__ int64_t red[16];
  __shared__ int s_cur, s_step;
  const int tid = threadIdx.x, lane = tid & 63, n = D.n, cl = D.cl;
  const int have = D.xnn ? D.xl : cl;
  const int W = (n + 31) >> 5;
  auto listed = [&](int c, int k) {
    return D.xnn ? D.xnn[(size_t)c * D.xl + k] & 0xffffu : (uint32_t)cand[(size_t)c * cl + k];
  };
  for (int w = tid; w < W; w += 1024) vis[w] = 0;
  const int nl = min(kNnList, have);
  for (int e = tid; e < n * kNnList; e += 1024) {
    const int c = e / kNnList, k = e % kNnList;
    if (k >= nl) continue;
    const uint32_t j = listed(c, k);
    if (k < C) lst[c * C + k] = (uint16_t)j;
    if (NEAR) near[e] = (uint16_t)j;
  }
  __threadfence_block();
  __syncthreads();
  if (tid == 0) {
    vis[0] = 1u;
    s_cur = 0;
    s_step = 1;
  }
  __syncthreads();
  // lanes whose city j is unvisited
  auto open = [&](uint32_t j) -> uint64_t {
    return __ballot(((vis[j >> 5] >> (j & 31)) & 1u) == 0);
  };
  auto low = [](uint64_t m) { return (int)__ffsll((unsigned long long)m) - 1; };
  int buf = 0;  // the first wave's order, entry t on lane t % 64 (entry 0: city 0)
  while (true) {
    if (tid < 64) {
      int cur = uni(s_cur), t = uni(s_step);
      const int kc = min(lane, C - 1), kn = min(lane, nl - 1);
      const uint64_t mc = ~0ull >> (64 - C), mn = ~0ull >> (64 - nl);
      while (t < n) {
        // up to the next 64-boundary, by the lists in LDS (and L2)
        const int tend = min(n, (t | 63) + 1);
        bool out = false;
        do {
          const uint32_t j2 = NEAR ? near[cur * kNnList + kn] : 0u;
          const uint32_t j1 = lst[cur * C + kc];
          uint32_t j = j1;
          uint64_t ok = open(j1) & mc;
          if (NEAR && !ok) {
            j = j2;
            ok = open(j2) & mn;
          }
          if (!ok) {
            out = true;
            break;
          }
          const int k = low(ok);
          cur = (int)rdlane(j, k);
          // lane k marks its city, the others OR zeros
          __hip_atomic_fetch_or(vis + (j >> 5), lane == k ? 1u << (j & 31) : 0u,
                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          buf = (int)wrlane((uint32_t)cur, t & 63, (uint32_t)buf);
        } while (++t < tend);
        if (out) {
          int nxt = -1;
          for (int b0 = C; nxt < 0 && b0 < have; b0 += 64) {
            const uint32_t j = listed(cur, min(b0 + lane, have - 1));
            const uint64_t ok = open(j) & (have - b0 >= 64 ? ~0ull : ~(~0ull << (have - b0)));
            if (ok) nxt = (int)rdlane(j, low(ok));
          }
          if (nxt < 0 && D.fpre) {
            // lane l holds the prefix positions 2l and 2l + 1
            const uint4 pe = D.fpre[(size_t)cur * (kFpre / 2) + lane];
            const uint32_t j0 = pe.x & 0xffffu, j1 = pe.z & 0xffffu;
            const uint64_t o0 = open(j0), o1 = open(j1);
            if (o0 | o1) {
              const int k = low(o0 | o1);
              nxt = (int)rdlane((o0 >> lane) & 1u ? j0 : j1, k);
            }
          }
          if (nxt < 0) break;
          if (lane == 0) mark(vis, nxt);
          buf = (int)wrlane((uint32_t)nxt, t & 63, (uint32_t)buf);
          cur = nxt;
          ++t;
        }
        if ((t & 63) == 0) D.best[t - 64 + lane] = buf;
      }
      if (tid == 0) {
        s_cur = cur;
        s_step = t;
      }
    }
    __syncthreads();
    const int cur = s_cur, t = s_step;
    if (t >= n) break;
    int64_t best = INT64_MAX;
    for (int j = tid; j < n; j += 1024)
      if (!((vis[j >> 5] >> (j & 31)) & 1u)) {
        const uint32_t dj = D.dist ? D.dist[(size_t)cur * D.ldn + j] : dist_xy(D, cur, j);
        const int64_t key = ((int64_t)dj << 16) | j;
        best = key < best ? key : best;
      }
    best = wave_min(best);
    if (lane == 0) red[tid >> 6] = best;
    __syncthreads();
    if (tid < 64) {
      best = red[lane & 15];
      best = wave_min(best);
      const int nxt = (int)(best & 0xffff);
      buf = lane == (t & 63) ? nxt : buf;
      if (((t + 1) & 63) == 0) D.best[t - 63 + lane] = buf;
      if (tid == 0) {
        mark(vis, nxt);
        s_cur = nxt;
        s_step = t + 1;
      }
    }
    __syncthreads();
  }
  if (tid < (n & 63)) D.best[(n & ~63) + tid] = buf;
  // the order's stores are this block's own: visible after a fence
  __threadfence_block();
  __syncthreads();
  int64_t L = 0;
  for (int p = tid; p < n; p += 1024)
    L += dist_xy(D, D.best[p], D.best[p + 1 < n ? p + 1 : 0]);
#pragma unroll
  for (int off = 32; off; off >>= 1) L += __shfl_xor(L, off, 64);
  if (lane == 0) red[tid >> 6] = L;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 16; ++w) L += red[w];
    *lnn = L;
  }
}

// Candidate records: the last word is the initial pheromone tau0 (dense
// memory) or the candidate's grid cell (selective memory); and (dense memory)
// the reverse positions: for candidate k of city i (j =
// cand[i][k]), the position of i in j's candidate list, -1 if i is not a
// candidate of j.
__global__ __launch_bounds__(256) void k_crec(Dev D, const int32_t *cand, float tau0) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= D.n * D.cl) return;
  const int i = e / D.cl;
  const uint32_t c = (uint32_t)cand[e];
  const uint32_t d = dist_xy(D, i, (int)c);
  const uint32_t w = D.spm ? (uint32_t)(grid_cy(D, D.xy[2 * c + 1]) * D.gnx + grid_cx(D, D.xy[2 * c]))
                           : __float_as_uint(tau0);
  const_cast<uint4 *>(D.crec)[e] = make_uint4(c, d, __float_as_uint(D.eta_tab[d]), w);
  if (!D.rpos) return;
  int r = -1;
  for (int k = 0; k < D.cl && r < 0; ++k)
    if (cand[(size_t)c * D.cl + k] == i) r = k;
  const_cast<int8_t *>(D.rpos)[e] = (int8_t)r;
}

__global__ __launch_bounds__(256) void k_cand_out(Dev D, int32_t *out) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < D.n * D.cl) out[e] = (int32_t)D.crec[e].x;
}

// A construction with an updater wave keeps the candidate entries' live
// pheromone in ctau (a record's 32 values in one 128-byte line), so the
// records the ants load are not written while it runs.  Before it, ctau
// takes the records' values; after it, each record takes back the value of
// its edge's canonical home (itself, or the same edge's slot in the smaller
// city's record when each city lists the other; see apply_entries), and a
// candidate slot whose city is not listed back passes its value to the dense
// entry (v, u).  Compare-and-swap mode only; the unsynchronised mode has no
// canonical homes and copies each slot back as it is.
__device__ __forceinline__ void ctau_out_slot(const Dev &D, size_t e, bool canonical) {
  const int u = (int)(e / (size_t)D.cl);
  const int v = (int)D.crec[e].x, kr = (int)D.rpos[e];
  const float x = canonical && kr >= 0 && u > v ? D.ctau[(size_t)v * D.cl + kr] : D.ctau[e];
  const_cast<uint4 *>(D.crec)[e].w = __float_as_uint(x);
  if (canonical && kr < 0) D.tau[(size_t)v * D.ldn + u] = x;
}

__global__ __launch_bounds__(256) void k_ctau_in(Dev D) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e < (size_t)D.n * D.cl) D.ctau[e] = __uint_as_float(D.crec[e].w);
}

// Before a construction, the bound that lets the dense fallback stop at its
// prefix.  During a construction an entry only ever receives the local map
// f(x) = fmaf(a, x, b) of a value one of the edge's entries held (the two
// entries of an edge start equal in every mode whose updates copy between
// them), and f(x) <= x above the map's real fixed point b / (1 - a), f(x) <=
// that point rounded up below it.  So T = max(start values, the point with a
// margin) bounds every value an entry of row i beyond the prefix holds, and
// by monotone rounding fl(T * femax) bounds their weights tau * eta^beta.
__device__ __forceinline__ void far_bound_row(const Dev &D, const Iter &A, int i, int lane) {
  const int n = D.n;
  const uint32_t lim = D.flim[i];
  const float *trow = D.tau + (size_t)i * D.ldn;
  const uint16_t *drow = D.dist + (size_t)i * D.ldn;
  uint32_t mx = 0;
  for (int j0 = 8 * lane; j0 < n; j0 += 512) {
    const float4 a = *reinterpret_cast<const float4 *>(trow + j0);
    const float4 b = *reinterpret_cast<const float4 *>(trow + j0 + 4);
    const uint4 dd = *reinterpret_cast<const uint4 *>(drow + j0);
    const float t[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    const uint32_t dw[4] = {dd.x, dd.y, dd.z, dd.w};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = j0 + q;
      const uint32_t key = ((dw[q >> 1] >> (16 * (q & 1))) & 0xffffu) << 16 | (uint32_t)j;
      if (j < n && j != i && key >= lim) mx = max(mx, __float_as_uint(t[q]));
    }
  }
  mx = wave_umax_u(mx);
  if (lane == 0) {
    const double fix = (double)A.b_loc / (1.0 - (double)A.a_loc);
    const float hi = (float)(fix * (1.0 + 0x1p-20));
    D.fbound[i] = fmaxf(__uint_as_float(mx), hi) * D.femax[i];
  }
}

// ctau_rows: the wave of row i also copies that row's candidate pheromone
// into ctau (k_ctau_in's work, for a construction with an updater wave).
__global__ __launch_bounds__(256) void k_far_bound(Dev D, Iter A, int ctau_rows) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= D.n) return;
  if (ctau_rows && lane < D.cl)
    D.ctau[(size_t)i * D.cl + lane] = __uint_as_float(D.crec[(size_t)i * D.cl + lane].w);
  far_bound_row(D, A, i, lane);
}

// The same for every instance of a batch that has a prefix (blockIdx.y =
// instance).
__global__ __launch_bounds__(256) void k_far_bound_batch(const Dev *devs, const Iter *iters) {
  const Dev D = global_dev(devs[blockIdx.y]);
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (D.fpre && i < D.n) far_bound_row(D, iters[blockIdx.y], i, threadIdx.x & 63);
}

// The same for every instance of a batch (blockIdx.y = instance).
__global__ __launch_bounds__(256) void k_ctau_in_batch(const Dev *devs) {
  const Dev D = global_dev(devs[blockIdx.y]);
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e < (size_t)D.n * D.cl) D.ctau[e] = __uint_as_float(D.crec[e].w);
}

__global__ __launch_bounds__(256) void k_ctau_out_batch(const Dev *devs, int canonical) {
  const Dev D = global_dev(devs[blockIdx.y]);
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e < (size_t)D.n * D.cl) ctau_out_slot(D, e, canonical != 0);
}

// The initial pheromone and everything else that needs only the eta^beta
// table: eta^beta of every entry (dense memory: one load per city in the
// fallback scan instead of a distance load followed by a table lookup), the
// prefix's eta^beta words and, per city, the largest eta^beta from the city
// after the prefix on.  That is the eta^beta of this city's distance where
// the table never grows with the distance (eta_falls); else it is taken over
// the table from there to the largest distance.
__global__ __launch_bounds__(256) void k_fill(Dev D, float tau0, uint32_t dmax, int eta_falls) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t nd = (size_t)D.n * D.ldn;
  if (D.tau && e < nd) {
    D.tau[e] = tau0;
    const_cast<float *>(D.etad)[e] = D.eta_tab[D.dist[e]];
  }
  if (D.fpre && e < (size_t)D.n * kFpre) {
    uint32_t *w = reinterpret_cast<uint32_t *>(const_cast<uint4 *>(D.fpre)) + 2 * e;
    w[1] = __float_as_uint(D.eta_tab[w[0] >> 16]);
  }
  if (D.fpre && e < (size_t)D.n) {
    const uint32_t d = D.flim[e] >> 16;
    float mx = D.eta_tab[d];
    if (!eta_falls)
      for (uint32_t x = d + 1; x <= dmax; ++x) mx = fmaxf(mx, D.eta_tab[x]);
    const_cast<float *>(D.femax)[e] = mx;
  }
  if (D.spm && e < (size_t)D.n * D.spm_s) D.spm[e] = make_uint2(kNone, __float_as_uint(tau0));
  if (D.spm_tail && e < (size_t)D.n) {
    D.spm_tail[e] = (uint32_t)(D.spm_s - 1);
    D.upd_head[e] = -1;
  }
  if (D.ccnt && e < (size_t)D.n * D.cl) D.ccnt[e] = 0u;
  if (e == 0) {
    D.gstate[0] = -1;
    D.gstate[1] = -1;
    D.gstate[2] = -1;
    D.sync[0] = 0;
    D.sync[1] = 0;
  }
  if (e < 8) D.counters[e] = 0;
}

// ---------------------------------------------------------------------------
// One step of Alg. 2 for the ant of this wave (dense memory).  `rec` is lane
// k's record of the current city (lanes >= cl hold a copy of the last one).
// Wave-uniform result.
// ---------------------------------------------------------------------------
struct Pick {
  int next;    // chosen city
  int k;       // its candidate position, -1 for the fallback
  uint32_t d;  // d(cur, next)
  float tval;  // pheromone of the entry (cur, next) as read
  int kind;    // 0 greedy (Eq. 1), 1 roulette (Eq. 2), 2 fallback
};

// Candidate-set membership and weight of this lane's candidate.
struct Cand {
  bool unv;  // member of the candidate set (an unvisited neighbour)
  float w;   // tau * eta^beta, 0 for non-members
};

__device__ __forceinline__ Cand weigh(const Dev &D, const uint32_t *vis, int lane, uint4 rec) {
  // every lane holds a valid city (lanes >= cl repeat the last candidate), so
  // the bitmap read needs no branch
  const uint32_t word = vis[rec.x >> 5];
  Cand c;
  c.unv = (lane < D.cl) & !((word >> (rec.x & 31)) & 1u);
  // tau * eta^beta >= 0, so its bit pattern orders like the value
  c.w = c.unv ? __uint_as_float(rec.w) * __uint_as_float(rec.z) : 0.f;
  return c;
}

// Philox words of 64 consecutive steps, one step per lane: lane l holds the
// draw of step base + l.  Each step then reads its words with readlane.
__device__ __forceinline__ uint4 philox_batch(const Iter &A, int ant, int base, int lane) {
  return philox10(make_uint4((uint32_t)(base + lane), (uint32_t)ant, A.it, A.instance), A.key0,
                  A.key1);
}

// q24 and u24 of step t from the batch that holds it.
__device__ __forceinline__ uint2 draw_of(uint4 batch, int t) {
  return make_uint2(rdlane(batch.x, t & 63) >> 8, rdlane(batch.y, t & 63) >> 8);
}

// Eq. 1 over the candidate set: the wave-uniform candidate position chosen,
// or -1 when the candidate set is empty (Alg. 2 then falls back).
__device__ __forceinline__ int pick_candidate(const Iter &A, int lane, int cl, Cand c, uint2 q,
                                              int &kind) {
  const bool unv = c.unv;
  const float w = c.w;
  const uint64_t umask = __ballot(unv);
  if (!umask) return -1;
  int k;
  if (q.x < A.q0_24) {
    // exploitation: maximum of tau * eta^beta, lowest position
    const uint32_t mx = cl <= 32 ? half_umax_u(__float_as_uint(w)) : wave_umax_u(__float_as_uint(w));
    const uint64_t sel = __ballot(unv && __float_as_uint(w) == mx);
    k = (int)__ffsll((unsigned long long)sel) - 1;
    kind = 0;
  } else {
    // Eq. 2 by roulette: inclusive Hillis-Steele scan over the positions
    // (offsets 1, 2, 4, ... < cl), r = u * total, first member of the
    // candidate set whose prefix sum exceeds r
    float P = w;
    for (int off = 1; off < cl; off <<= 1) {
      const float o = __shfl_up(P, off, 64);
      if (lane >= off) P = P + o;
    }
    const float total = __uint_as_float(rdlane(__float_as_uint(P), cl - 1));
    const float r = ((float)q.y * 0x1p-24f) * total;
    const uint64_t sel = __ballot(unv && P > r);
    k = sel ? (int)__ffsll((unsigned long long)sel) - 1 : 63 - (int)__clzll((long long)umask);
    kind = 1;
  }
  return uni(k);
}

// The prefix of a city's fallback (D.fpre): two cities per lane, and the bound
// on every weight beyond them.
struct PrefixRow {
  uint4 e;
  float bound;
};
// Without a prefix (D.fpre null) the loads go to the first record and, by the
// buffer's bounds check, to a zero: no branch, so that a caller's loads in
// flight need no wait where paths meet.  (The bound is a vector load because
// LDS reads would have to wait for a scalar one in flight.)
__device__ __forceinline__ PrefixRow prefix_row(const Dev &D, int cur, int lane) {
  const uint4 *row = D.fpre ? D.fpre + (size_t)cur * (kFpre / 2) + lane : D.crec;
  const __amdgpu_buffer_rsrc_t brs =
      __builtin_amdgcn_make_buffer_rsrc(D.fbound, 0, D.fbound ? D.n * 4 : 0, kBufWord3);
  return PrefixRow{*row, __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(brs, cur * 4, 0, 0))};
}

// Alg. 2, empty candidate set: greedy over every unvisited city, ties ->
// lowest index.  With a prefix (D.fpre; pre: cur's, if loaded), the kFpre cities after
// the candidates come first, two per lane; when the best unvisited one beats
// D.fbound[cur] strictly, no city beyond the prefix can reach or tie it (the
// candidates are all visited), so it is the answer of the whole scan.
// Otherwise each lane scans eight consecutive cities per round, the loads of
// several rounds issued before the first is examined (at addresses clamped
// into the padded row, so that their number is fixed).  In the asynchronous
// kernels one round is ahead (registers set their occupancy); in the
// synchronous one (COHERENT) every step waits for the slowest ant, whose scan
// this is: three rounds at a time, by 16-byte coherent loads (eight 4-byte
// ones and one round ahead made the scan 28 k cycles at n = 2392).
template <bool COHERENT>
__device__ __forceinline__ Pick fallback_dense(const Dev &D, const uint32_t *vis, int cur,
                                               int lane, const PrefixRow *pre = nullptr,
                                               const float *tsrc = nullptr) {
  const int n = D.n;
  Pick p;
  const float *trow = (tsrc ? tsrc : D.tau) + (size_t)cur * D.ldn;
  if (D.fpre) {
    const uint4 pe = pre ? pre->e : D.fpre[(size_t)cur * (kFpre / 2) + lane];
    const float fb = pre ? pre->bound : D.fbound[cur];
    const uint32_t j0 = pe.x & 0xffffu, j1 = pe.z & 0xffffu;
    const float t0 = COHERENT ? tau_load(trow + j0) : trow[j0];
    const float t1 = COHERENT ? tau_load(trow + j1) : trow[j1];
    const bool u0 = !((vis[j0 >> 5] >> (j0 & 31)) & 1u);
    const bool u1 = !((vis[j1 >> 5] >> (j1 & 31)) & 1u);
    const float v0 = t0 * __uint_as_float(pe.y), v1 = t1 * __uint_as_float(pe.w);
    // this lane's best (largest weight, then lowest index)
    const bool second = u1 && (!u0 || v1 > v0 || (v1 == v0 && j1 < j0));
    const bool any = u0 || u1;
    const float bv = second ? v1 : v0;
    const uint32_t bj = second ? j1 : j0;
    // weights are >= 0, so their bit patterns order like the values
    const uint32_t mx = wave_umax_u(any ? __float_as_uint(bv) : 0u);
    if (mx > __float_as_uint(fb)) {
      const uint32_t jn = wave_umin_u(any && __float_as_uint(bv) == mx ? bj : kNone);
      const uint64_t own = __ballot(any && bj == jn);
      const int owner = uni((int)__ffsll((unsigned long long)own) - 1);
      p.k = -1;
      p.next = (int)jn;
      p.d = rdlane(second ? pe.z >> 16 : pe.x >> 16, owner);
      p.tval = __uint_as_float(rdlane(__float_as_uint(second ? t1 : t0), owner));
      p.kind = 2;
      return p;
    }
  }
  const float *erow = D.etad + (size_t)cur * D.ldn;
  const uint16_t *drow = D.dist + (size_t)cur * D.ldn;
  const int rounds = (n + 511) >> 9;
  float bv = 0.f, bt = 0.f;
  uint32_t bj = kNone, bd = 0;
  struct Round {
    float t[8], e[8];
    uint4 d;
  };
  const __amdgpu_buffer_rsrc_t trs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(trow), 0, D.ldn * (int)sizeof(float), kBufWord3);
  auto fetch = [&](int r, Round &x) {
    const int j = min(8 * lane + 512 * r, D.ldn - 8);
    if (COHERENT) {
      const auto a = __builtin_amdgcn_raw_buffer_load_b128(trs, 4 * j, 0, kCoherent);
      const auto b = __builtin_amdgcn_raw_buffer_load_b128(trs, 4 * j, 16, kCoherent);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        x.t[q] = __uint_as_float(a[q]);
        x.t[4 + q] = __uint_as_float(b[q]);
      }
    } else {
      const float4 a = *reinterpret_cast<const float4 *>(trow + j);
      const float4 b = *reinterpret_cast<const float4 *>(trow + j + 4);
      x.t[0] = a.x; x.t[1] = a.y; x.t[2] = a.z; x.t[3] = a.w;
      x.t[4] = b.x; x.t[5] = b.y; x.t[6] = b.z; x.t[7] = b.w;
    }
    const float4 a = *reinterpret_cast<const float4 *>(erow + j);
    const float4 b = *reinterpret_cast<const float4 *>(erow + j + 4);
    x.e[0] = a.x; x.e[1] = a.y; x.e[2] = a.z; x.e[3] = a.w;
    x.e[4] = b.x; x.e[5] = b.y; x.e[6] = b.z; x.e[7] = b.w;
    x.d = *reinterpret_cast<const uint4 *>(drow + j);
  };
  auto examine = [&](int r, const Round &x) {
    const int j0 = 8 * lane + 512 * r;
    uint32_t bits = (vis[min(j0, n - 1) >> 5] >> (j0 & 31)) & 0xffu;
    if (j0 >= n) bits = 0xffu;
    else if (j0 + 8 > n) bits |= (0xffu << (n - j0)) & 0xffu;
    const uint32_t dw[4] = {x.d.x, x.d.y, x.d.z, x.d.w};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float v = x.t[q] * x.e[q];
      if (!((bits >> q) & 1u) && (bj == kNone || v > bv)) {
        bv = v; bj = (uint32_t)(j0 + q); bt = x.t[q]; bd = (dw[q >> 1] >> (16 * (q & 1))) & 0xffffu;
      }
    }
  };
  if (COHERENT) {
    for (int r = 0; r < rounds; r += 3) {
      Round x[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) fetch(min(r + i, rounds - 1), x[i]);
      examine(r, x[0]);
#pragma unroll
      for (int i = 1; i < 3; ++i)
        if (r + i < rounds) examine(r + i, x[i]);
    }
  } else {
    Round cr;
    fetch(0, cr);
    for (int r = 0; r < rounds; ++r) {
      Round nr;
      fetch(min(r + 1, rounds - 1), nr);
      examine(r, cr);
      cr = nr;
    }
  }
  const uint32_t mx = wave_umax_u(bj == kNone ? 0u : __float_as_uint(bv));
  const uint32_t jn = wave_umin_u((bj != kNone && __float_as_uint(bv) == mx) ? bj : kNone);
  const uint64_t own = __ballot(bj == jn);
  const int owner = uni((int)__ffsll((unsigned long long)own) - 1);
  p.k = -1;
  p.next = (int)jn;
  p.d = rdlane(bd, owner);
  p.tval = __uint_as_float(rdlane(__float_as_uint(bt), owner));
  p.kind = 2;
  return p;
}

// The choice from the current city's records.
__device__ __forceinline__ Pick select_dense(const Dev &D, const Iter &A, const uint32_t *vis,
                                             int cur, int lane, uint4 rec, Cand c, uint2 q) {
  Pick p;
  const int k = pick_candidate(A, lane, D.cl, c, q, p.kind);
  if (k < 0) return fallback_dense<false>(D, vis, cur, lane);
  p.k = k;
  p.next = (int)rdlane(rec.x, k);
  p.d = rdlane(rec.y, k);
  p.tval = __uint_as_float(rdlane(rec.w, k));
  return p;
}

__device__ __forceinline__ void add_counters(const Dev &D, uint32_t greedy, uint32_t roul,
                                             uint32_t fb, uint64_t fbu, uint32_t retries) {
  atomicAdd(&D.counters[0], (unsigned long long)greedy);
  atomicAdd(&D.counters[1], (unsigned long long)roul);
  atomicAdd(&D.counters[2], (unsigned long long)fb);
  atomicAdd(&D.counters[5], (unsigned long long)fbu);
  atomicAdd(&D.counters[6], (unsigned long long)retries);
}

// Tour entries are collected 64 at a time in one register (lane t % 64 holds
// entry t) and written with one coalesced store per 64 steps.
__device__ __forceinline__ void tour_put(const Dev &D, int ant, int t, int lane, int city,
                                         int &buf) {
  buf = lane == (t & 63) ? city : buf;
  if ((t & 63) == 63 || t == D.n - 1) {
    const int base = t & ~63;
    if (lane <= (t & 63)) D.tours[(size_t)ant * D.n + base + lane] = buf;
  }
}

// ---------------------------------------------------------------------------
// Synchronous construction, dense memory: persistent cooperative kernel, one
// ant per wave.  Step t is
//   SELECT (reads only, from the pheromone at the start of the step)
//   | barrier | UPDATE (Eq. 3 on both entries of each crossing, by CAS)
//   | barrier.
// The map is the same for every crossing, so the order of the updates of one
// step does not change the result: an entry crossed k times gets f^k.
// With a local-update period above 1, a step without updates leaves the
// pheromone as it is, so it needs neither barrier; the closing edges wait for
// the last step's selections before they write.
//
// With a period of 1 the pheromone is double-buffered instead, which needs
// one barrier per step: buffer 0 is (candidate records' words, tau), buffer
// 1 is (ctau, tau2), and buffer 1 starts the construction as a copy of
// buffer 0 (k_sync_buf).  Step t selects from buffer t % 2, which holds every
// update of steps < t, and applies the crossings of steps t - 1 and t to
// buffer (t + 1) % 2, which then holds every update of steps < t + 1; nobody
// reads that buffer during step t, and the barrier at the end of the step
// separates its writes from step t + 1's reads and step t's reads from step
// t + 1's writes.  The closing edges go to buffer n % 2, the final one.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float *sync_home(const Dev &D, int buf, int u, int v, int k) {
  if (buf == 0) return home(D, u, v, k);
  return k >= 0 ? D.ctau + (size_t)u * D.cl + k : D.tau2 + (size_t)u * D.ldn + v;
}

__global__ __launch_bounds__(1024) void k_construct_sync_dense(Dev D, Iter A) {
  extern __shared__ uint32_t smem[];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int ant = uni(blockIdx.x * (blockDim.x >> 6) + wv);
  const bool active = ant < D.m;
  const int n = D.n, cl = D.cl;
  const int W = (n + 31) >> 5;
  const int kl = lane < cl ? lane : cl - 1;
  uint32_t *vis = smem + wv * W;
  const bool dbuf = A.lperiod == 1;
  const GridBar gbar = grid_join(D, A);

  for (int w = lane; w < W; w += 64) vis[w] = 0u;
  uint4 draws = philox_batch(A, ant, 0, lane);
  const int start = (int)__umulhi(rdlane(draws.z, 0), (uint32_t)n);
  if (lane == 0) vis[start >> 5] |= 1u << (start & 31);
  int tb = start;

  int cur = start;
  int64_t len = 0;
  uint32_t c_greedy = 0, c_roul = 0, c_fb = 0, c_retry = 0;
  uint64_t c_fbu = 0;
  uint32_t bar = 0;
  // the previous step's crossing (double-buffered schedule)
  int pu = -1, pv = -1, pk = -1, pk2 = -1;
  float pval = 0.f;
  // what does not change while the ants run is loaded before the barrier that
  // the city's pheromone has to wait for: its records, its positions in its
  // candidates' lists and its fallback's prefix
  uint4 rec = D.crec[(size_t)cur * cl + kl];
  int rpos = D.rpos[(size_t)cur * cl + kl];
  PrefixRow pre = prefix_row(D, cur, lane);
  for (int t = 1; t < n; ++t) {
    Pick p{};
    int k2 = -1;
    const int rb = dbuf ? (t & 1) : 0;
    if ((t & 63) == 0) draws = philox_batch(A, ant, t, lane);
    if (active) {
      const float *ct = rb == 0 ? cand_tau(D, cur, kl) : D.ctau + (size_t)cur * cl + kl;
      rec.w = __float_as_uint(tau_load(ct));
      const Cand c = weigh(D, vis, lane, rec);
      const int k = pick_candidate(A, lane, cl, c, draw_of(draws, t), p.kind);
      if (k >= 0) {
        p.k = k;
        p.next = (int)rdlane(rec.x, k);
        p.d = rdlane(rec.y, k);
        p.tval = __uint_as_float(rdlane(rec.w, k));
        k2 = (int)rdlane((uint32_t)rpos, k);
      } else {
        p = fallback_dense<true>(D, vis, cur, lane, &pre, rb == 0 ? D.tau : D.tau2);
        k2 = cand_pos(D, p.next, cur, lane);
      }
      rec = D.crec[(size_t)p.next * cl + kl];
      rpos = D.rpos[(size_t)p.next * cl + kl];
      pre = prefix_row(D, p.next, lane);
      c_greedy += p.kind == 0;
      c_roul += p.kind == 1;
      if (p.kind == 2) { ++c_fb; c_fbu += (uint64_t)(n - t); }
      if (lane == 0) mark(vis, p.next);
      tour_put(D, ant, t, lane, p.next, tb);
      len += p.d;
    }
    if (dbuf) {
      // crossings of steps t - 1 and t into buffer (t + 1) % 2: lanes 0 and
      // 1 the previous crossing's two entries, lanes 2 and 3 this one's
      if (active) {
        const int wb = rb ^ 1;
        float *h = nullptr;
        unsigned int seen = 0;
        if (lane < 2 && pu >= 0) {
          h = lane == 0 ? sync_home(D, wb, pu, pv, pk) : sync_home(D, wb, pv, pu, pk2);
          seen = __float_as_uint(pval);
        } else if (lane == 2 || lane == 3) {
          h = lane == 2 ? sync_home(D, wb, cur, p.next, p.k) : sync_home(D, wb, p.next, cur, k2);
          seen = __float_as_uint(p.tval);
        }
        // a value the map leaves unchanged stays so under the maps that reach
        // the entry in this step: the update changes nothing
        if (h && !map_fixed(__uint_as_float(seen), A.a_loc, A.b_loc))
          c_retry += cas_apply(h, seen, A.a_loc, A.b_loc);
        pu = cur;
        pv = p.next;
        pk = p.k;
        pk2 = k2;
        pval = p.tval;
      }
      grid_barrier_f(D, gbar, barrier_epoch(A.it, ++bar));
    } else if (t % A.lperiod == 0) {
      grid_barrier_f(D, gbar, barrier_epoch(A.it, ++bar));
      if (active) {
        float *h = lane == 0 ? home(D, cur, p.next, p.k) : home(D, p.next, cur, k2);
        if (lane < 2 && !map_fixed(p.tval, A.a_loc, A.b_loc))
          c_retry += cas_apply(h, __float_as_uint(p.tval), A.a_loc, A.b_loc);
      }
      if (t + 1 < n) grid_barrier_f(D, gbar, barrier_epoch(A.it, ++bar));
    }
    if (active) cur = p.next;
  }
  if (!dbuf && (n - 1) % A.lperiod != 0) grid_barrier_f(D, gbar, barrier_epoch(A.it, ++bar));
  if (active) {
    // closing edge: its length and, as the last step's crossings, its update
    len += D.dist[(size_t)cur * D.ldn + start];
    const int fb = dbuf ? (n & 1) : 0;
    const int k1 = cand_pos(D, cur, start, lane);
    const int k2 = cand_pos(D, start, cur, lane);
    float *h = lane == 0 ? sync_home(D, fb, cur, start, k1) : sync_home(D, fb, start, cur, k2);
    if (lane < 2) {
      const float seen = tau_load(h);
      c_retry += cas_apply(h, __float_as_uint(seen), A.a_loc, A.b_loc);
    }
    c_retry = (uint32_t)uni((int)(rdlane(c_retry, 0) + rdlane(c_retry, 1) + rdlane(c_retry, 2) +
                                  rdlane(c_retry, 3)));
    if (lane == 0) {
      D.lens[ant] = len;
      add_counters(D, c_greedy, c_roul, c_fb, c_fbu, c_retry);
    }
  }
}

// The same construction where the pheromone of all candidate entries fits a
// block's LDS: every block keeps its own copy and applies every ant's crossings
// to it, so a step needs neither a coherent read of the row nor a
// compare-and-swap on memory, whose retries on the edges that several ants
// cross (1800 cycles each across XCDs) and whose round trips made up most of
// a step.  What the blocks exchange is one word per ant and update step, the
// crossing, tagged with the step; a block goes on when it has read all m of
// them, so the words are the barrier too (two sets in turn: a block can be one
// update step ahead of another that still reads).  The host takes this kernel
// for up to 1024 ants in at most 64 blocks, one word per thread: that many
// blocks poll each other's lines in about 3000 cycles, while 250 need 7000, and
// a grid barrier before the words made it slower than the kernel above (n =
// 1500, m = n, cl = 16: 6.5 against 5.3 us per step).  The map is the same for
// all crossings, so their order inside a step does not matter.
//
// Entries of edges that are not in a candidate list (fallbacks, 2% of the
// steps) stay in memory, double-buffered: buffer b (0: tau, 1: tau2) is read,
// the crossings of this update step and of the previous one go to the other,
// before the ant's word is published.  The closing edges are one more
// exchange; their non-candidate entries go to the buffer last read.
//
// m = n, us per step: n = 198 5.6 -> 2.8, n = 1000 4.7 -> 3.1; 64 ants, n =
// 1000: 4.2 -> 2.4.  About 800 cycles of a step are the choice, the rest the
// words' way (a store and a load beyond the XCD) and their application.
//
// HALF: cl <= 32, the maximum over 32 lanes.
struct Crossing {
  int u, v, k, kr;  // edge, position of v in u's list and of u in v's (-1: none)
};
__device__ __forceinline__ uint64_t pack_crossing(int t, const Crossing &c) {
  return (uint64_t)t << 46 | (uint64_t)c.u << 30 | (uint64_t)c.v << 14 | (uint64_t)(c.k + 1) << 7 |
         (uint64_t)(c.kr + 1);
}
__device__ __forceinline__ Crossing unpack_crossing(uint64_t w) {
  return Crossing{(int)(w >> 30) & 0xffff, (int)(w >> 14) & 0xffff, (int)((w >> 7) & 127) - 1,
                  (int)(w & 127) - 1};
}

// A block barrier that orders LDS only: global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <bool HALF>
__global__ __launch_bounds__(1024) void k_construct_sync_lds(Dev D, Iter A) {
  extern __shared__ uint32_t smem[];  // n x cl pheromone, then the ants' bitmaps
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int ant = uni(blockIdx.x * (blockDim.x >> 6) + wv);
  const bool active = ant < D.m;
  const int n = D.n, cl = D.cl, m = D.m;
  const int W = (n + 31) >> 5;
  const int kl = lane < cl ? lane : cl - 1;
  uint32_t *vis = smem + n * cl + wv * W;
  const float al = A.a_loc, bl = A.b_loc;
  // a block's words of one set in a 128-byte line of their own
  const int apb = (int)(blockDim.x >> 6);
  unsigned long long *words = reinterpret_cast<unsigned long long *>(D.ctau);
  const size_t set_words = (size_t)kSyncMaxAnts * gridDim.x;
  // the word this thread reads
  const bool mine = (int)threadIdx.x < m;
  const size_t slot = (size_t)kSyncMaxAnts * (threadIdx.x / apb) + threadIdx.x % apb;
  __shared__ uint64_t s_word[kSyncMaxAnts];

  for (int e = threadIdx.x; e < n * cl; e += blockDim.x) smem[e] = D.crec[e].w;
  for (int w = lane; w < W; w += 64) vis[w] = 0u;
  __syncthreads();
  uint4 draws = philox_batch(A, ant, 0, lane);
  uint64_t greedy = __ballot((draws.x >> 8) < A.q0_24);  // the 64 steps' greedy draws
  const int start = (int)__umulhi(rdlane(draws.z, 0), (uint32_t)n);
  if (lane == 0) vis[start >> 5] |= 1u << (start & 31);
  int tb = start;

  const uint64_t clmask = cl >= 64 ? ~0ull : (1ull << cl) - 1;
  int cur = start;
  int64_t len = 0;
  uint32_t c_roul = 0, c_fb = 0, c_retry = 0;
  uint64_t c_fbu = 0;
  uint32_t upds = 0;                    // update steps so far; buffer upds & 1 is read
  uint32_t left = A.lperiod;            // steps to the next one
  Crossing last{-1, -1, 0, 0};          // of the previous update step
  float lval = 0.f;
  uint4 rec = D.crec[(size_t)cur * cl + kl];
  int8_t rpos = D.rpos[(size_t)cur * cl + kl];
  PrefixRow pre = prefix_row(D, cur, lane);
  for (int t = 1; t <= n; ++t) {
    Crossing x{cur, start, -1, -1};
    float val = 0.f;
    float *const rd = (upds & 1) ? D.tau2 : D.tau, *const wr = (upds & 1) ? D.tau : D.tau2;
    const int tl = t & 63;
    if (tl == 0) {
      draws = philox_batch(A, ant, t, lane);
      greedy = __ballot((draws.x >> 8) < A.q0_24);
    }
    if (active && t < n) {
      const uint32_t tau = smem[cur * cl + kl];
      const bool unv = !((vis[rec.x >> 5] >> (rec.x & 31)) & 1u);
      const uint64_t umask = __ballot(unv) & clmask;
      uint32_t d;
      if (umask) {
        const float w = unv ? __uint_as_float(tau) * __uint_as_float(rec.z) : 0.f;
        if ((greedy >> tl) & 1u) {
          // Eq. 1: maximum weight, lowest position
          const uint32_t wb = __float_as_uint(w);
          const uint32_t mx = rows_umax_s<HALF ? 32 : 64>(wb);
          x.k = (int)__builtin_ctzll(__ballot(wb == mx) & umask);
        } else {
          // Eq. 2 by roulette, as in pick_candidate
          float P = w;
          for (int off = 1; off < cl; off <<= 1) {
            const float o = __shfl_up(P, off, 64);
            if (lane >= off) P = P + o;
          }
          const float total = __uint_as_float(rdlane(__float_as_uint(P), cl - 1));
          const float r = ((float)(rdlane(draws.y, tl) >> 8) * 0x1p-24f) * total;
          const uint64_t sel = __ballot(P > r) & umask;
          x.k = sel ? (int)__builtin_ctzll(sel) : 63 - (int)__builtin_clzll(umask);
          ++c_roul;
        }
        x.v = (int)rdlane(rec.x, x.k);
        x.kr = (int)rdlane((uint32_t)(int)rpos, x.k);
        d = rdlane(rec.y, x.k);
        val = __uint_as_float(rdlane(tau, x.k));
      } else {
        const Pick p = fallback_dense<true>(D, vis, cur, lane, &pre, rd);
        x.v = p.next;
        x.kr = cand_pos(D, p.next, cur, lane);
        d = p.d;
        val = p.tval;
        ++c_fb;
        c_fbu += (uint64_t)(n - t);
      }
      if (lane == 0) mark(vis, x.v);
      len += d;
    } else if (active) {
      x.k = cand_pos(D, cur, start, lane);
      x.kr = cand_pos(D, start, cur, lane);
      len += D.dist[(size_t)cur * D.ldn + start];
    }
    const bool upd = t == n || --left == 0;
    if (left == 0) left = A.lperiod;
    // vmcnt(0): this step's rows have long arrived; without it the loads below
    // would wait, through the registers they reuse, for the store of the word
    __builtin_amdgcn_s_waitcnt(0x0f70);
    if (active && upd) {
      // non-candidate entries of the previous update step's crossing (lanes 0
      // and 1) and of this one (2 and 3; the closing edge's follow below); a
      // compare-and-swap whose result has come back is performed
      const Crossing &c = lane < 2 ? last : x;
      const bool fwd = (lane & 1) == 0;
      const float seen = lane < 2 ? lval : val;
      if (lane < (t < n ? 4 : 0) && c.u >= 0 && (fwd ? c.k : c.kr) < 0 &&
          !map_fixed(seen, al, bl))
        c_retry += cas_apply(wr + (size_t)(fwd ? c.u : c.v) * D.ldn + (fwd ? c.v : c.u),
                             __float_as_uint(seen), al, bl);
      last = x;
      lval = val;
      if (lane == 0) s_word[wv] = pack_crossing(t, x);
    }
    unsigned long long *const set = words + (upds & 1) * set_words;
    if (upd) {
      // every wave has read the block's copy for this step and left its word,
      // which go out in one store
      lds_barrier();
      if ((int)threadIdx.x < apb && (int)(blockIdx.x * apb + threadIdx.x) < m)
        __hip_atomic_store(set + (size_t)kSyncMaxAnts * blockIdx.x + threadIdx.x,
                           (unsigned long long)s_word[threadIdx.x], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    // the next city's rows while the words travel (every ant, every step: no
    // branch, and the byte is widened where it is used, so nothing waits here)
    rec = D.crec[(size_t)x.v * cl + kl];
    rpos = D.rpos[(size_t)x.v * cl + kl];
    pre = prefix_row(D, x.v, lane);
    if (active && t < n) {
      tb = (int)wrlane((uint32_t)x.v, tl, (uint32_t)tb);
      if ((tl == 63 || t == n - 1) && lane <= tl) D.tours[(size_t)ant * n + (t & ~63) + lane] = tb;
    }
    if (upd) {
      uint64_t w = 0;
      if (wv * 64 < m)
        bounded_wait(D, [&]() {
          if (mine) w = __hip_atomic_load(set + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          return !mine || (int)(w >> 46) == t;
        });
      if (mine && (int)(w >> 46) == t) {
        // the map on this block's copy of the crossing's candidate entries,
        // both side by side
        const Crossing c = unpack_crossing(w);
        int e0 = c.k >= 0 ? c.u * cl + c.k : -1, e1 = c.kr >= 0 ? c.v * cl + c.kr : -1;
        uint32_t x0 = smem[max(e0, 0)], x1 = smem[max(e1, 0)];
        while (e0 >= 0 || e1 >= 0) {
          const uint32_t y0 = __float_as_uint(fmaf(al, __uint_as_float(x0), bl));
          const uint32_t y1 = __float_as_uint(fmaf(al, __uint_as_float(x1), bl));
          uint32_t g0 = x0, g1 = x1;
          if (e0 >= 0 && y0 != x0) g0 = atomicCAS(&smem[e0], x0, y0);
          if (e1 >= 0 && y1 != x1) g1 = atomicCAS(&smem[e1], x1, y1);
          if (g0 == x0) e0 = -1;
          if (g1 == x1) e1 = -1;
          x0 = g0;
          x1 = g1;
        }
      }
      lds_barrier();
      ++upds;
    }
    if (t < n) cur = x.v;
  }
  // every block's copy is the final one: each writes its share back
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n * cl; e += gridDim.x * blockDim.x)
    const_cast<uint4 *>(D.crec)[e].w = smem[e];
  if (active) {
    // the closing edge's non-candidate entries, into the buffer last read
    float *const fin = ((upds - 1) & 1) ? D.tau2 : D.tau;
    if (lane < 2 && (lane == 0 ? last.k : last.kr) < 0) {
      float *h = fin + (size_t)(lane == 0 ? last.u : last.v) * D.ldn +
                 (lane == 0 ? last.v : last.u);
      c_retry += cas_apply(h, __float_as_uint(tau_load(h)), al, bl);
    }
    c_retry = (uint32_t)uni((int)(rdlane(c_retry, 0) + rdlane(c_retry, 1) + rdlane(c_retry, 2) +
                                  rdlane(c_retry, 3)));
    if (lane == 0) {
      D.lens[ant] = len;
      add_counters(D, (uint32_t)(n - 1) - c_roul - c_fb, c_roul, c_fb, c_fbu, c_retry);
    }
  }
}

// The grid barrier's words before an iteration in which they are due (see
// barrier_reached): the first one, then every kBarrierClear-th.  (When the handle
// is built their place may still hold the eta^beta table.)
__global__ __launch_bounds__(256) void k_barrier_clear(Dev D, uint32_t it) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < D.nbflags) D.bflags[e] = barrier_epoch(it, 0);
}

// Buffer 1 of the double-buffered synchronous schedules from buffer 0 (dir 0),
// or buffer 0 from buffer 1 (dir 1) when the construction ended in buffer 1.
// words > 0: the candidate entries are not part of it (k_construct_sync_lds);
// dir 0 clears that many words of the place of the exchanged crossings.
__global__ __launch_bounds__(256) void k_sync_buf(Dev D, int dir, int words) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (words > 0) {
    if (dir == 0 && e < (size_t)words) D.ctau[e] = 0.f;
  } else if (e < (size_t)D.n * D.cl) {
    if (dir == 0)
      D.ctau[e] = __uint_as_float(D.crec[e].w);
    else
      const_cast<uint4 *>(D.crec)[e].w = __float_as_uint(D.ctau[e]);
  }
  if (e < (size_t)D.n * D.ldn) {
    if (dir == 0)
      D.tau2[e] = D.tau[e];
    else
      D.tau[e] = D.tau2[e];
  }
}

// ---------------------------------------------------------------------------
// Sequential construction, dense memory (Alg. 1 read literally): step by
// step, and within a step ant by ant, each ant selecting from the pheromone
// after the local updates of the ants before it in the same step.  One block
// of kSeqWaves waves, kSeqGroup ants of a step at a time.
//
// An ant's choice depends on the pheromone only through the row of its
// current city, and an ant's update writes rows cur and next.  So the ants of
// a group all choose from the pheromone as it is (ant i on wave i %
// kSeqWaves); every ant then enters its index at the two rows its choice
// would write (the least index wins; a table in LDS by city, whose slots
// cities share when n is larger than it, which can only add a conflict).  The
// ants before the first whose row an earlier one writes have made exactly the
// sequential choices: they commit (their updates touch disjoint entries).
// The others keep their choice unless a committed ant wrote their row, and
// the entries are made again, without the committed.  Every round commits at
// least the first ant left.  With 64 ants at n = 2392 a step takes two to
// three rounds, of which the first alone has all ants to choose.
//
// Entering, checking and committing take one thread per ant.  One compute
// unit's issue slots bound the first round, the barriers and single choices the
// others.  Rounds of 16 ants, each with its own draws, global reads of the
// current cities and conflict search, took 11.1 us a step at m = 64 and 461 us
// at m = n = 2392; this takes 5.5 and 223.  How many ants make a group
// (`group`, at most kSeqGroup) depends on how often they meet: see seq_group.
// ---------------------------------------------------------------------------
constexpr int kSeqWaves = 16;    // a group is a multiple of it
constexpr int kSeqSlots = kSeqGroup / kSeqWaves;  // per wave
constexpr int kSeqRows = 4096;   // slots of the table of rows (power of two)
constexpr int kSeqCur = 4096;    // current cities in LDS for up to so many ants
// visited bitmaps in LDS when all m of them fit in this many words
constexpr int kSeqLdsWords = 31 * 1024;

// A choice: next city | (k + 1) << 16 | (kr + 1) << 23 | roulette << 30, k the
// position of next in cur's list and kr of cur in next's (-1: none).
__device__ __forceinline__ uint32_t pack_choice(int next, int k, int kr, bool roul) {
  return (uint32_t)next | (uint32_t)(k + 1) << 16 | (uint32_t)(kr + 1) << 23 |
         (roul ? 1u << 30 : 0u);
}

// VIS_LDS: the m visited bitmaps in LDS (dynamic, m * ceil(n/32) words), else
// in global memory.  In this schedule both entries of an edge always hold
// the same value (every map is applied to both), so a committing ant stores
// the map of the value it read to both without reading the second.
template <bool VIS_LDS>
__global__ __launch_bounds__(64 * kSeqWaves) void k_construct_seq_dense(Dev D, Iter A,
                                                                        int group) {
  extern __shared__ uint32_t smem[];
  __shared__ uint32_t s_rows[kSeqRows];   // round (counted down) << 8 | least ant
  __shared__ uint32_t s_choice[kSeqGroup];
  __shared__ float s_val[kSeqGroup];
  __shared__ uint16_t s_now[kSeqGroup];   // the group's current cities
  __shared__ uint8_t s_need[kSeqGroup];
  __shared__ uint16_t s_cur[kSeqCur];
  __shared__ int s_stop;                  // first ant in conflict
  const int tid = threadIdx.x, lane = tid & 63, wv = uni(tid >> 6);
  const int n = D.n, m = D.m, cl = D.cl;
  const int W = (n + 31) >> 5;
  const int kl = lane < cl ? lane : cl - 1;
  const uint64_t clmask = cl >= 64 ? ~0ull : (1ull << cl) - 1;
  uint32_t *const vbase = VIS_LDS ? smem : D.gvis;
  const bool near = m <= kSeqCur;

  for (int r = tid; r < kSeqRows; r += 64 * kSeqWaves) s_rows[r] = kNone;
  for (size_t w = tid; w < (size_t)m * W; w += 64 * kSeqWaves) vbase[w] = 0u;
  __syncthreads();
  for (int a = tid; a < m; a += 64 * kSeqWaves) {
    const uint4 z = philox10(make_uint4(0u, (uint32_t)a, A.it, A.instance), A.key0, A.key1);
    const int start = (int)__umulhi(z.z, (uint32_t)n);
    vbase[(size_t)a * W + (start >> 5)] = 1u << (start & 31);
    D.tours[(size_t)a * n] = start;
    if (near) s_cur[a] = (uint16_t)start;
  }
  __syncthreads();
  uint32_t c_roul = 0, c_fb = 0;  // per thread (commits)
  uint64_t c_fbu = 0;
  uint32_t round = 0xfffffe;
  uint4 draws{};
  uint32_t left = A.lperiod;
  for (int t = 1; t < n; ++t) {
    const bool upd = --left == 0;
    if (upd) left = A.lperiod;
    for (int base = 0; base < m; base += group) {
      const int g = min(group, m - base);
      // draws of this wave's ants: lane l holds ant slot l % kSeqSlots at step
      // (t & ~3) + l / kSeqSlots
      if (m > group || (t & 3) == 0 || t == 1)
        draws = philox10(make_uint4((uint32_t)((t & ~3) + lane / kSeqSlots),
                                    (uint32_t)(base + lane % kSeqSlots * kSeqWaves + wv), A.it,
                                    A.instance),
                         A.key0, A.key1);
      // (one group: its cities are kept up to date where its ants commit)
      if (t == 1 || m > group) {
        if (tid < g) {
          s_now[tid] =
              near ? s_cur[base + tid] : (uint16_t)D.tours[(size_t)(base + tid) * n + t - 1];
          s_need[tid] = 1;
        }
        if (tid == 0) s_stop = g;
        __syncthreads();
      }
      auto choose = [&](int i, int sl, uint4 rec, int8_t rpos) {
        const uint32_t *vis = vbase + (size_t)(base + i) * W;
        const bool unv = !((vis[rec.x >> 5] >> (rec.x & 31)) & 1u);
        const uint64_t umask = __ballot(unv) & clmask;
        uint32_t choice;
        float val;
        if (umask) {
          const float w = unv ? __uint_as_float(rec.w) * __uint_as_float(rec.z) : 0.f;
          const bool roul = (rdlane(draws.x, sl) >> 8) >= A.q0_24;
          int k;
          if (!roul) {
            // Eq. 1: maximum weight, lowest position
            const uint32_t wb = __float_as_uint(w);
            const uint32_t mx = cl <= 32 ? rows_umax_s<32>(wb) : rows_umax_s<64>(wb);
            k = (int)__builtin_ctzll(__ballot(wb == mx) & umask);
          } else {
            // Eq. 2 by roulette, as in pick_candidate
            float P = w;
            for (int off = 1; off < cl; off <<= 1) {
              const float o = __shfl_up(P, off, 64);
              if (lane >= off) P = P + o;
            }
            const float total = __uint_as_float(rdlane(__float_as_uint(P), cl - 1));
            const float r = ((float)(rdlane(draws.y, sl) >> 8) * 0x1p-24f) * total;
            const uint64_t sel = __ballot(P > r) & umask;
            k = sel ? (int)__builtin_ctzll(sel) : 63 - (int)__builtin_clzll(umask);
          }
          choice = pack_choice((int)rdlane(rec.x, k), k, (int)rdlane((uint32_t)(int)rpos, k),
                               roul);
          val = __uint_as_float(rdlane(rec.w, k));
        } else {
          const int cur = uni(s_now[i]);
          const Pick p = fallback_dense<false>(D, vis, cur, lane);
          choice = pack_choice(p.next, -1, upd ? cand_pos(D, p.next, cur, lane) : -1, false);
          val = p.tval;
        }
        if (lane == 0) {
          s_choice[i] = choice;
          s_val[i] = val;
        }
      };
      for (int done = 0; done < g;) {
        // this wave's ants that choose, two at a time with their rows in flight
        // together (need: the wave's slots)
        uint32_t need = (uint32_t)__ballot(lane * kSeqWaves + wv < g &&
                                           lane * kSeqWaves + wv >= done &&
                                           s_need[min(lane * kSeqWaves + wv, kSeqGroup - 1)]);
        while (need) {
          const int sa = __builtin_ctz(need);
          need &= need - 1;
          const int ca = uni(s_now[sa * kSeqWaves + wv]);
          const uint4 ra = D.crec[(size_t)ca * cl + kl];
          const int8_t pa = D.rpos[(size_t)ca * cl + kl];
          if (!need) {
            choose(sa * kSeqWaves + wv, sa + kSeqSlots * (t & 3), ra, pa);
            break;
          }
          const int sb = __builtin_ctz(need);
          need &= need - 1;
          const int cb = uni(s_now[sb * kSeqWaves + wv]);
          const uint4 rb = D.crec[(size_t)cb * cl + kl];
          const int8_t pb = D.rpos[(size_t)cb * cl + kl];
          choose(sa * kSeqWaves + wv, sa + kSeqSlots * (t & 3), ra, pa);
          choose(sb * kSeqWaves + wv, sb + kSeqSlots * (t & 3), rb, pb);
        }
        __syncthreads();
        // one thread per ant of the group from here
        const bool mine = tid >= done && tid < g;
        const int now = mine ? s_now[tid] : 0;
        const uint32_t choice = mine ? s_choice[tid] : 0u;
        const int next = (int)(choice & 0xffffu);
        uint32_t first = kNone;  // the least ant that writes this ant's row
        if (upd) {
          if (mine) {
            const uint32_t key = round << 8 | (uint32_t)tid;
            atomicMin(&s_rows[now & (kSeqRows - 1)], key);
            atomicMin(&s_rows[next & (kSeqRows - 1)], key);
          }
          __syncthreads();
          if (mine) {
            first = s_rows[now & (kSeqRows - 1)] & 255u;
            if ((int)first < tid) atomicMin(&s_stop, tid);
          }
          __syncthreads();
        }
        const int stop = s_stop;
        if (mine && tid < stop) {
          const int k = (int)((choice >> 16) & 127u) - 1, kr = (int)((choice >> 23) & 127u) - 1;
          const int a = base + tid;
          if (upd) {
            const float x = fmaf(A.a_loc, s_val[tid], A.b_loc);
            *home(D, now, next, k) = x;
            *home(D, next, now, kr) = x;
          }
          vbase[(size_t)a * W + (next >> 5)] |= 1u << (next & 31);
          D.tours[(size_t)a * n + t] = next;
          if (near) s_cur[a] = (uint16_t)next;
          s_now[tid] = (uint16_t)next;
          s_need[tid] = 1;
          c_roul += choice >> 30;
          if (k < 0) { ++c_fb; c_fbu += (uint64_t)(n - t); }
        } else if (mine) {
          s_need[tid] = (int)first < stop;
        }
        __syncthreads();
        if (tid == 0) s_stop = g;
        done = stop;
        if (upd && --round == 0) {  // the table's rounds are used up
          for (int r = tid; r < kSeqRows; r += 64 * kSeqWaves) s_rows[r] = kNone;
          round = 0xfffffe;
          __syncthreads();
        }
      }
    }
  }
  // lengths, and closing edges' updates (edges shared by several ants get the
  // map once per ant, in any order)
  uint32_t c_retry = 0;
  for (int a = wv; a < m; a += kSeqWaves) {
    const int32_t *tour = D.tours + (size_t)a * n;
    int64_t len = 0;
#pragma unroll 4
    for (int p = lane; p < n; p += 64)
      len += D.dist[(size_t)tour[p] * D.ldn + tour[p + 1 < n ? p + 1 : 0]];
#pragma unroll
    for (int off = 32; off; off >>= 1) len += __shfl_xor(len, off, 64);
    const int cur = tour[n - 1], start = tour[0];
    const int k1 = cand_pos(D, cur, start, lane);
    const int k2 = cand_pos(D, start, cur, lane);
    float *h = lane == 0 ? home(D, cur, start, k1) : home(D, start, cur, k2);
    if (lane < 2) c_retry += cas_apply(h, __float_as_uint(tau_load(h)), A.a_loc, A.b_loc);
    if (lane == 0) D.lens[a] = len;
  }
  c_roul = wave_sum_u(c_roul);
  c_fb = wave_sum_u(c_fb);
  c_retry = wave_sum_u(c_retry);
#pragma unroll
  for (int off = 32; off; off >>= 1)
    c_fbu += (uint64_t)__shfl_xor((long long)c_fbu, off, 64);
  if (lane == 0) add_counters(D, 0u, c_roul, c_fb, c_fbu, c_retry);
  // every step that was neither was greedy
  if (lane == 0) {
    const unsigned long long other = (unsigned long long)c_roul + c_fb;
    const unsigned long long all = wv == 0 ? (unsigned long long)m * (n - 1) : 0ull;
    atomicAdd(&D.counters[0], all - other);
  }
}

// ---------------------------------------------------------------------------
// Asynchronous construction, dense memory: one launch per iteration, one ant
// per wave, no waiting for the other ants.  Each crossing gets the local
// update of Eq. 3 as a compare-and-swap of the exact map on both directed
// entries of the crossed edge.
//
// The steps of one ant form a dependent chain, so the latency of a step sets
// the iteration time, and the wave waits for its memory operations in issue
// order.  The step is therefore arranged so that nothing slow is issued
// right before the wait for the next record:
//   1. wait for the record of the current city cur (issued at the end of the
//      previous step); check the compare-and-swaps issued one step earlier
//      and repeat any that found the entry changed;
//   2. issue the two compare-and-swaps of the previous move (prev, cur): the
//      forward entry with the pheromone the selection read as its expected
//      value, the reverse entry with the value cur's record holds (or the
//      forward value when prev is not a candidate of cur);
//   3. select the next city (Alg. 2) while those are in flight;
//   4. issue the load of the next city's record.
// ATOMIC = false is the paper's unsynchronised variant (ACS-GPU-Alt,
// Sec. 3.1.2): each entry gets the map of the value the ant read, by a plain
// (not read-modify-write) store, and updates that race with it are lost.
// ---------------------------------------------------------------------------
template <bool ATOMIC>
__device__ __forceinline__ void ant_async_dense(const Dev &D, const Iter &A, int ant,
                                                uint32_t *vis, int lane) {
  uint32_t uleft = A.lperiod;  // steps until the next local update
  const int n = D.n, cl = D.cl, ldn = D.ldn;
  const int W = (n + 31) >> 5;
  const int kl = lane < cl ? lane : cl - 1;
  const float al = A.a_loc, bl = A.b_loc;

  for (int w = lane; w < W; w += 64) vis[w] = 0u;
  uint4 draws = philox_batch(A, ant, 0, lane);
  const int start = (int)__umulhi(rdlane(draws.z, 0), (uint32_t)n);
  if (lane == 0) vis[start >> 5] |= 1u << (start & 31);
  int tb = start;
  uint4 rec = D.crec[(size_t)start * cl + kl];

  int cur = start, prev = -1;
  float *fwd = nullptr;  // home of the forward entry of the previous move
  float fval = 0.f;      // its value as read by the selection
  int64_t len = 0;
  // decisions by kind, 21 bits each: greedy | roulette << 21 | fallback << 42
  uint64_t c_kind = 0;
  uint32_t c_retry = 0;
  uint64_t c_fbu = 0;
  // compare-and-swap in flight on lanes 0 (forward) and 1 (reverse)
  float *pptr = nullptr;
  unsigned int pexp = 0, pret = 0;
  bool pend = false;

  // steps in chunks of 64: a chunk's draws come from one Philox batch and
  // its tour entries leave in one store, so no step tests for either
  for (int t0 = 0; t0 <= n; t0 += 64) {
  if (t0 > 0) draws = philox_batch(A, ant, t0, lane);
  uint32_t clen = 0;  // at most 64 distances below 2^16 each
  const int tend = min(t0 + 64, n + 1);
  for (int t = t0 > 0 ? t0 : 1; t < tend; ++t) {
    // 1. the record of cur is needed now; so are last step's CAS results
    if (pend && pret != pexp) c_retry += 1 + cas_apply(pptr, pret, al, bl);
    pend = false;
    const Cand c = weigh(D, vis, lane, rec);
    // the weights are complete here, before the updates below are issued, so
    // no later wait for this record also waits for those updates
    __asm__ volatile("" ::"v"(c.w), "v"((int)c.unv));
    // 2. updates of the previous move (prev, cur), selected at step t - 1
    if (t > 1 && --uleft == 0) {
      uleft = A.lperiod;
      const uint64_t b = __ballot(lane < cl && rec.x == (uint32_t)prev);
      const int kr = b ? uni((int)__ffsll((unsigned long long)b) - 1) : -1;
      const float rval = kr >= 0 ? __uint_as_float(rdlane(rec.w, kr)) : fval;
      if (ATOMIC) {
        if (lane == 0) {
          pptr = fwd;
          pexp = __float_as_uint(fval);
          pend = true;
        } else if (lane == 1) {
          pptr = home(D, cur, prev, kr);
          pexp = __float_as_uint(rval);
          pend = true;
        }
        if (pend && map_fixed(__uint_as_float(pexp), al, bl)) pend = false;
        if (pend)
          pret = atomicCAS(reinterpret_cast<unsigned int *>(pptr), pexp,
                           __float_as_uint(fmaf(al, __uint_as_float(pexp), bl)));
      } else if (lane < 2 && !map_fixed(lane == 0 ? fval : rval, al, bl)) {
        float *h = lane == 0 ? fwd : home(D, cur, prev, kr);
        __hip_atomic_store(h, fmaf(al, lane == 0 ? fval : rval, bl), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (t == n) break;
    // 3. selection
    const Pick p = select_dense(D, A, vis, cur, lane, rec, c, draw_of(draws, t));
    c_kind += 1ull << (21 * p.kind);
    if (p.kind == 2) c_fbu += (uint64_t)(n - t);
    if (lane == 0) mark(vis, p.next);
    tb = lane == t - t0 ? p.next : tb;
    clen += p.d;
    // 4. record of the next city
    rec = D.crec[(size_t)p.next * cl + kl];
    fwd = home(D, cur, p.next, p.k);
    fval = p.tval;
    prev = cur;
    cur = p.next;
  }
  len += clen;
  // tour entries t0 .. min(t0 + 63, n - 1) of this chunk
  if (t0 < n && lane <= min(63, n - 1 - t0)) D.tours[(size_t)ant * n + t0 + lane] = tb;
  }
  if (pend && pret != pexp) c_retry += 1 + cas_apply(pptr, pret, al, bl);
  // closing edge: both entries, read fresh (once per ant)
  {
    const int k1 = cand_pos(D, cur, start, lane);
    const int k2 = cand_pos(D, start, cur, lane);
    float *h = lane == 0 ? home(D, cur, start, k1) : home(D, start, cur, k2);
    if (lane < 2) {
      if (ATOMIC)
        c_retry += cas_apply(h, __float_as_uint(tau_load(h)), al, bl);
      else
        __hip_atomic_store(h, fmaf(al, tau_load(h), bl), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  len += D.dist[(size_t)cur * ldn + start];
  c_retry = (uint32_t)uni((int)(rdlane(c_retry, 0) + rdlane(c_retry, 1)));
  if (lane == 0) {
    D.lens[ant] = len;
    const uint32_t m21 = (1u << 21) - 1;
    add_counters(D, (uint32_t)c_kind & m21, (uint32_t)(c_kind >> 21) & m21,
                 (uint32_t)(c_kind >> 42) & m21, c_fbu, c_retry);
  }
}

template <bool ATOMIC>
__global__ __launch_bounds__(256) void k_construct_async_dense(Dev D, Iter A) {
  extern __shared__ uint32_t smem[];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int ant = uni(blockIdx.x * (blockDim.x >> 6) + wv);
  if (ant >= D.m) return;  // the whole wave leaves; no block-level sync below
  ant_async_dense<ATOMIC>(D, A, ant, smem + wv * ((D.n + 31) >> 5), lane);
}

// ---------------------------------------------------------------------------
// Local updates handed to an updater wave.  gfx950 counts loads, stores and
// atomics of a wave in one in-order counter, so a wave that waits for its
// next record also waits for every update it issued before that load.  The
// ant wave therefore issues no update: the crossing selected at step t goes
// into lane t % 64 of an entry held in registers, and every kQGroup steps one
// LDS store of those lanes hands the group to the block's updater wave,
// which applies Eq. 3 to both directed entries of each crossed edge.  An
// update thus lands a few steps after its crossing (at most a group plus
// the updater's sleep), where an ant that applied it itself would have
// waited for it.
// Each ant wave owns a ring of kQRing entries indexed by step (single
// producer, single consumer): the entry of step t sits at t % kQRing; the
// ant publishes head = the first step not yet written, the updater tail =
// the first step not yet read.  LDS instructions of one wave take effect in
// issue order, so a published head covers entries already written, and a
// published tail frees entries already read.  Every wait is bounded: on
// exhaustion the error flag (2) is raised and the ant applies its entries
// itself, so every wave still reaches its end.
//
// Entry of the crossing u -> v: {u | v << 16, k, x, kr}: k the position of v
// in u's candidate list (-1 if none), x the pheromone of (u, v) as the ant
// read it, kr the position of u in v's list: -2 = look it up in the reverse
// table (v is the k-th candidate of u), -3 = search v's list (v is not a
// candidate of u), else kr itself (-1: u is not a candidate of v).  Steps
// without an update hold x = kNoEntry in the first word.
// ---------------------------------------------------------------------------
constexpr int kQAnts = 8;     // at most this many ant waves per block
constexpr int kQGroup = 16;   // steps per hand-over (divides 64)
constexpr int kQRing = 256;   // ring entries per ant wave (power of 2, >= 64 + kQGroup)
constexpr uint32_t kQSpin = 1u << 22;
constexpr uint32_t kQIdle = 1u << 20;
constexpr uint32_t kNoEntry = 0xffffffffu;

struct QRing {
  uint4 *ent;      // [ant wave][kQRing]
  uint32_t *head;  // per ant wave: first step not yet written
  uint32_t *tail;  // per ant wave: first step not yet read by the updater
  uint32_t *done;  // ant waves that have written their last entry
};

__device__ __forceinline__ uint32_t lds_ld(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_st(uint32_t *p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Eq. 3 on both directed entries of the crossings held by the lanes of the
// wave (one entry per lane, all lanes active).
// Compare-and-swap mode: one entry of the edge is its canonical home and
// receives every map exactly; the other entry gets the value just written by a
// device-coherent store, for readers at the other endpoint.  The canonical home is a
// candidate slot: the one in the record of the smaller city when each city
// lists the other, else the only one; k_best copies every canonical
// value to its other entry when the construction ends, so both entries
// then hold exactly the result of all the maps.  An edge with both entries
// in the dense matrix (a fallback move between cities that do not list each
// other) gets both compare-and-swaps.  Candidate entries live in ctau
// meanwhile (see k_ctau_in).
// Many ants cross the same edges within a few steps, and a compare-and-swap by
// each of them lets one through per round trip (0.3 us) and sends the others
// round again: 0.35 repeats per step at n = m = 2392, 5.7 at 198, 7 at 198
// cities and 1000 ants, where a popular edge set the construction's time.
// So (COUNT) a crossing is first counted at its home (ccnt): the wave that finds the
// count at 0 owns the entry and writes the map of its own and of all the
// crossings counted meanwhile, until it takes the count back to 0; every other
// wave is done after its one addition.  The maps are the same function, so the
// value after k of them does not depend on whose they are.  The compare-and-swap
// (x, the value the ant read, as the first expected value; another value found is
// the next one expected) then repeats 0.02 to 0.06 times per step.  Iterations of
// n = m = 198: 186 -> 111 us, 198 cities and 1000 ants 560 -> 151, n = m = 1000
// 606 -> 462, 2392 1326 -> 1176; with the count only after a first failed
// compare-and-swap 116, 235, 476, 1213, after the second 130, 360, 519, 1254.
// Taken for a local update at every step by at least n / 2 ants; else the edges
// are too little contended for the count's two extra round trips (n = m = 2392,
// period 16: 1290 us, 1314 with it; 3000 cities and 256 ants 1228, 1257; 4000 and
// 2000 the same with both).  A launch counts everywhere or nowhere.
// Unsynchronised mode (ACS-GPU-Alt, Sec. 3.1.2): each entry is read and its
// map stored back, both device-coherent but not as one atomic operation;
// updates landing in between are lost.  (The value the ant read is several
// steps old by now: storing its map would undo the updates made since.)
// Returns this lane's retries.
template <bool ATOMIC, bool COUNT>
__device__ __forceinline__ uint32_t apply_entries(const Dev &D, const Iter &A, uint4 e,
                                                  int lane) {
  const bool valid = e.x != kNoEntry;
  const int u = (int)(e.x & 0xffffu), v = (int)(e.x >> 16), k = (int)e.y;
  int kr = (int)e.w;
  const float al = A.a_loc, bl = A.b_loc;
  // compare-and-swap mode: the value the ant read is one the edge's entries
  // have held; if the map leaves it unchanged (map_fixed), they hold it now
  // and neither is written.  Tested first, so that such an entry needs
  // neither the reverse position nor the fallback's search.
  const bool fixed = ATOMIC && valid && map_fixed(__uint_as_float(e.z), al, bl);
  // after a fallback move: the whole wave searches v's list, once per entry
  uint64_t need = __ballot(valid && !fixed && kr == -3);
  while (need) {
    const int l = (int)__ffsll((unsigned long long)need) - 1;
    need &= need - 1;
    const int r = cand_pos(D, (int)rdlane((uint32_t)v, l), (int)rdlane((uint32_t)u, l), lane);
    if (lane == l) kr = r;
  }
  if (!valid || fixed) return 0;
  if (kr == -2) kr = (int)D.rpos[(size_t)u * D.cl + k];
  float *pf = qhome(D, u, v, k);
  float *pr = qhome(D, v, u, kr);
  if (ATOMIC) {
    const bool both_dense = k < 0 && kr < 0;
    const bool fwd_canon = k >= 0 && (kr < 0 || u < v);
    float *pc = fwd_canon || both_dense ? pf : pr;
    float *po = fwd_canon || both_dense ? pr : pf;
    if (!COUNT || both_dense) {
      unsigned int seen = e.z, nw;
      uint32_t r = 0;
      while (true) {
        nw = __float_as_uint(fmaf(al, __uint_as_float(seen), bl));
        const unsigned int old = atomicCAS(reinterpret_cast<unsigned int *>(pc), seen, nw);
        if (old == seen) break;
        seen = old;
        ++r;
      }
      // the value the first entry held just before its update is a fresh
      // guess for the second
      if (both_dense) return r + cas_apply(po, seen, al, bl);
      __hip_atomic_store(po, __uint_as_float(nw), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return r;
    }
    // the first wave to count an update of this entry owns it and is its only
    // writer until it has taken the count back to zero
    uint32_t *cnt = D.ccnt + (pc - D.ctau);
    if (atomicAdd(cnt, 1u)) return 0;
    unsigned int seen = e.z;
    uint32_t r = 0, maps = 1;
    while (true) {
      const unsigned int nw = map_times(seen, maps, al, bl);
      const unsigned int old = atomicCAS(reinterpret_cast<unsigned int *>(pc), seen, nw);
      if (old != seen) {
        seen = old;
        ++r;
        continue;
      }
      __hip_atomic_store(po, __uint_as_float(nw), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      maps = atomicSub(cnt, maps) - maps;
      if (maps == 0) return r;
      seen = nw;
    }
  }
  const float xf = tau_load(pf), xr = tau_load(pr);
  if (!map_fixed(xf, al, bl))
    __hip_atomic_store(pf, fmaf(al, xf, bl), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!map_fixed(xr, al, bl))
    __hip_atomic_store(pr, fmaf(al, xr, bl), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return 0;
}

template <bool ATOMIC>
__device__ __forceinline__ uint32_t spm_apply_entries(const Dev &D, const Iter &A, uint4 e,
                                                      uint32_t &hits, uint32_t &misses);

// Hands the entries of steps [g0, g1) (lanes g0 - t0 .. g1 - t0 - 1 of `e`)
// to the updater, or, once the updater has stopped draining, applies them in
// place.  `head` (= g0 on entry), `tail` (last tail seen) and `direct` are
// the wave's own.  SPM: the entries are the selective memory's (see
// spm_apply_entries; hits and misses count its updates).  Returns this
// lane's retries.
template <bool ATOMIC, bool COUNT, bool SPM = false>
__device__ __forceinline__ uint32_t group_push(const Dev &D, const Iter &A, const QRing &q, int w,
                                               uint32_t &head, uint32_t &tail, bool &direct,
                                               int lane, uint4 e, int t0, int g1,
                                               uint32_t &hits, uint32_t &misses) {
  const bool mine = lane + t0 >= (int)head && lane + t0 < g1;
  if (!direct && (uint32_t)g1 - tail > (uint32_t)kQRing) {
    uint32_t spins = 0;
    while (true) {
      tail = (uint32_t)uni((int)lds_ld(q.tail + w));
      if ((uint32_t)g1 - tail <= (uint32_t)kQRing) break;
      __builtin_amdgcn_s_sleep(2);
      if (++spins > (D.wait_limit ? D.wait_limit : kQSpin)) {
        if (lane == 0)
          __hip_atomic_store(D.sync + 1, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        direct = true;
        break;
      }
    }
  }
  if (direct) {
    head = (uint32_t)g1;
    const uint4 own = mine ? e : make_uint4(kNoEntry, 0u, 0u, 0u);
    if (SPM) return spm_apply_entries<ATOMIC>(D, A, own, hits, misses);
    return apply_entries<ATOMIC, COUNT>(D, A, own, lane);
  }
  if (mine) q.ent[(size_t)w * kQRing + ((lane + t0) & (kQRing - 1))] = e;
  head = (uint32_t)g1;
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  if (lane == 0) lds_st(q.head + w, head);
  return 0;
}

// The updater wave: applies the entries of every ant wave of its block until
// all `na` ant waves are done and every entry is applied.  One pass takes
// the pending entries of all rings at once, up to 64 (ring after ring, each
// from its tail), and applies them together, so the updates of different
// rings share their memory round trips.  With nothing pending it sleeps, so
// it takes few issue slots from the ant waves that share its SIMD.
template <bool ATOMIC, bool COUNT, bool SPM = false, int NR = kQAnts>
__device__ __forceinline__ void ring_updater(const Dev &D, const Iter &A, const QRing &q,
                                             int lane, int na) {
  static_assert((kQRing & (kQRing - 1)) == 0 && kQRing >= 64 + kQGroup, "ring size");
  uint32_t tl[NR];  // the updater's own tails (wave-uniform)
#pragma unroll
  for (int w = 0; w < NR; ++w) tl[w] = 0;
  uint32_t retries = 0, idle = 0, hits = 0, misses = 0;
  while (true) {
    // read `done` before the heads: an ant wave publishes its last head
    // before it counts itself done
    const uint32_t done = (uint32_t)uni((int)lds_ld(q.done));
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    uint32_t taken = 0;  // lanes given an entry so far
    uint4 e = make_uint4(kNoEntry, 0u, 0u, 0u);
#pragma unroll
    for (int w = 0; w < NR; ++w) {
      if (w >= na) break;
      const uint32_t h = (uint32_t)uni((int)lds_ld(q.head + w));
      const uint32_t c = min(h - tl[w], 64u - taken);
      if ((uint32_t)lane >= taken && (uint32_t)lane < taken + c)
        e = q.ent[(size_t)w * kQRing + ((tl[w] + (uint32_t)lane - taken) & (kQRing - 1))];
      tl[w] += c;
      taken += c;
    }
    if (taken) {
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
      for (int w = 0; w < NR; ++w)
        if (w < na && lane == 0) lds_st(q.tail + w, tl[w]);
      if (SPM)
        retries += spm_apply_entries<ATOMIC>(D, A, e, hits, misses);
      else
        retries += apply_entries<ATOMIC, COUNT>(D, A, e, lane);
      idle = 0;
      continue;
    }
    if (done == (uint32_t)na) break;
    __builtin_amdgcn_s_sleep(32);
    if (++idle > (D.wait_limit ? D.wait_limit : kQIdle)) {
      if (lane == 0)
        __hip_atomic_store(D.sync + 1, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
  }
  if (retries) atomicAdd(&D.counters[6], (unsigned long long)retries);
  if (SPM) {
    hits = (uint32_t)uni((int)wave_sum_u(hits));
    misses = (uint32_t)uni((int)wave_sum_u(misses));
    if (lane == 0 && (hits | misses)) {
      atomicAdd(&D.counters[3], (unsigned long long)hits);
      atomicAdd(&D.counters[4], (unsigned long long)misses);
    }
  }
}

// ---------------------------------------------------------------------------
// Asynchronous construction, dense memory, local updates through the
// block's updater wave.  The step holds only what Alg. 2 needs: weigh the
// current city's record, choose (Eq. 1 or Eq. 2 over the candidate set, the
// fallback when it is empty), mark, issue the next record's load, and note
// the crossing in the lane of its step; every kQGroup steps the noted
// crossings go to the ring.  Records and their live pheromone (ctau) come by
// buffer loads (the lane's offset fixed, the row's a scalar; a read outside
// the table returns zeros instead of faulting).  HALF: every candidate list
// fits lanes 0..31.  EVERY: every step has a local update (period 1), so
// the per-step test drops out.  Decisions are the same as those of
// ant_async_dense.
// ---------------------------------------------------------------------------
template <bool ATOMIC, bool HALF, bool EVERY = false, bool COUNT = false>
__device__ __forceinline__ void ant_queued(const Dev &D, const Iter &A, int ant, uint32_t *vis,
                                           int lane, const QRing &q, int qw) {
  const int n = D.n, cl = D.cl;
  const int W = (n + 31) >> 5;
  const uint64_t clmask = cl >= 64 ? ~0ull : (1ull << cl) - 1;
  const int dumw = lane % W;  // this lane's word for the visited-bit store
  const int koff = (lane < cl ? lane : cl - 1) * 16;
  const int rowb = cl * 16;  // bytes per record row
  const __amdgpu_buffer_rsrc_t crs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(D.crec), 0, n * rowb, kBufWord3);
  const __amdgpu_buffer_rsrc_t trs =
      __builtin_amdgcn_make_buffer_rsrc(D.ctau, 0, n * cl * 4, kBufWord3);
  // a record's fields and the live pheromone of its slot (the record's own
  // pheromone word is the value of the iteration's start), the latter read
  // device-coherently
  auto load_rec = [&](int city) {
    const auto r = __builtin_amdgcn_raw_buffer_load_b128(crs, koff, city * rowb, 0);
    const uint32_t t =
        __builtin_amdgcn_raw_buffer_load_b32(trs, koff >> 2, city * cl * 4, kCoherent);
    return make_uint4(r[0], r[1], r[2], t);
  };

  for (int w = lane; w < W; w += 64) vis[w] = 0u;
  uint4 draws = philox_batch(A, ant, 0, lane);
  const int start = (int)__umulhi(rdlane(draws.z, 0), (uint32_t)n);
  if (lane == 0) vis[start >> 5] |= 1u << (start & 31);
  uint4 rec = load_rec(start);

  uint32_t qhead = 0, qtail = 0, c_retry = 0, c_roul = 0, c_fb = 0, unused = 0;
  bool qdirect = false;
  uint64_t c_fbu = 0;
  int64_t len = 0;
  int cur = start;
  // steps in chunks of 64: lane l holds step t0 + l's draw, tour entry and
  // crossing, so a chunk's draws come from one Philox batch and its tour
  // entries leave in one store; its crossings leave kQGroup at a time
  for (int t0 = 0; t0 < n; t0 += 64) {
    if (t0 > 0) draws = philox_batch(A, ant, t0, lane);
    const int lt = lane + t0;
    // bit t - t0 of `upd`: step t has a local update (after every
    // lperiod-th selected edge); of `greedy`: step t takes Eq. 1's argmax
    const uint64_t upd = __builtin_amdgcn_ballot_w64(lt % (int)A.lperiod == 0);
    const uint64_t greedy = __builtin_amdgcn_ballot_w64((draws.x >> 8) < A.q0_24);
    // lane t - t0 holds step t's crossing (x = kNoEntry: no update) and
    // tour entry; every crossing is a candidate move (kr = -2) unless the
    // fallback made it
    uint4 e = make_uint4(kNoEntry, 0u, 0u, (uint32_t)-2);
    int tb = start;
    uint32_t clen = 0;  // at most 64 distances below 2^16 each
    const int tend = min(t0 + 64, n);
    for (int g0 = t0 > 0 ? t0 : 1; g0 < tend;) {
      const int g1 = min((g0 & ~(kQGroup - 1)) + kQGroup, tend);
      uint64_t sb = 1ull << (g0 - t0);  // bit t - t0
      for (int t = g0; t < g1; ++t, sb <<= 1) {
        const int tl = t - t0;
        // lanes >= cl repeat candidate cl - 1 (same city, same weight), so
        // they never change a maximum or a prefix sum of positions < cl; the
        // candidate mask leaves them out of every choice
        const uint32_t word = vis[__builtin_amdgcn_ubfe(rec.x, 5, 11)];
        const bool unv = !__builtin_amdgcn_ubfe(word, rec.x, 1);
        const uint64_t umask = __builtin_amdgcn_ballot_w64(unv) & clmask;
        int next, k;
        uint32_t d, tv;
        if (__builtin_expect(umask == 0, 0)) {
          const Pick p = fallback_dense<false>(D, vis, cur, lane);
          next = p.next;
          k = -1;
          d = p.d;
          tv = __float_as_uint(p.tval);
          if (EVERY || (upd & sb)) e.w = wrlane((uint32_t)-3, tl, e.w);
          ++c_fb;
          c_fbu += (uint64_t)(n - t);
        } else {
          // tau * eta^beta >= 0, so its bit pattern orders like the value
          const float w = unv ? __uint_as_float(rec.w) * __uint_as_float(rec.z) : 0.f;
          if (greedy & sb) {
            // Eq. 1: maximum weight, lowest position
            const uint32_t wb = __float_as_uint(w);
            const uint32_t mx = rows_umax_s<HALF ? 32 : 64>(wb);
            k = (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(wb == mx) & umask);
          } else {
            // Eq. 2 by roulette: inclusive Hillis-Steele scan over the
            // positions (offsets 1, 2, 4, ... < cl), r = u * total, first
            // member of the candidate set whose prefix sum exceeds r
            float P = w;
            for (int off = 1; off < cl; off <<= 1) {
              const float o = __shfl_up(P, off, 64);
              if (lane >= off) P = P + o;
            }
            const float total = __uint_as_float(rdlane(__float_as_uint(P), cl - 1));
            const float r = ((float)(rdlane(draws.y, tl) >> 8) * 0x1p-24f) * total;
            const uint64_t sel = __builtin_amdgcn_ballot_w64(P > r) & umask;
            k = sel ? (int)__builtin_ctzll(sel) : 63 - (int)__builtin_clzll(umask);
            ++c_roul;
          }
          next = (int)rdlane(rec.x, k);
          d = rdlane(rec.y, k);
          tv = rdlane(rec.w, k);
        }
        rec = load_rec(next);
        // one lane marks the city (lane k holds it as its candidate)
        if (lane == (k < 0 ? 0 : k))
          __hip_atomic_fetch_or(vis + (next >> 5), 1u << (next & 31), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_WORKGROUP);
        tb = (int)wrlane((uint32_t)next, tl, (uint32_t)tb);
        if (EVERY || (upd & sb)) {
          e.x = wrlane((uint32_t)cur | ((uint32_t)next << 16), tl, e.x);
          e.y = wrlane((uint32_t)k, tl, e.y);
          e.z = wrlane(tv, tl, e.z);
        }
        clen += d;
        cur = next;
      }
      c_retry += group_push<ATOMIC, COUNT>(D, A, q, qw, qhead, qtail, qdirect, lane, e, t0, g1, unused,
                                    unused);
      g0 = g1;
    }
    len += clen;
    if (lane < tend - t0) D.tours[(size_t)ant * n + lt] = tb;
  }
  // closing edge (cur, start), every ant, as step n: both positions
  // searched, the value read fresh
  {
    const int k1 = cand_pos(D, cur, start, lane);
    const int k2 = cand_pos(D, start, cur, lane);
    const uint32_t x = rdlane(__float_as_uint(tau_load(qhome(D, cur, start, k1))), 0);
    const uint4 ce =
        make_uint4((uint32_t)cur | ((uint32_t)start << 16), (uint32_t)k1, x, (uint32_t)k2);
    c_retry += group_push<ATOMIC, COUNT>(D, A, q, qw, qhead, qtail, qdirect, lane, ce, n, n + 1, unused,
                                  unused);
    len += D.dist[(size_t)cur * D.ldn + start];
  }
  c_retry = (uint32_t)uni((int)wave_sum_u(c_retry));
  if (lane == 0) {
    D.lens[ant] = len;
    add_counters(D, (uint32_t)(n - 1) - c_roul - c_fb, c_roul, c_fb, c_fbu, c_retry);
  }
}

// One instance, updates through the block's updater wave: waves 0..na-1 are
// ants blockIdx.x * na + wave, wave na (the last) applies their entries.  The
// host picks na so that every compute unit holds about the same number of
// ants (the slowest unit sets the iteration time).  Dynamic LDS: the rings
// of the na ant waves, then their visited bitmaps.
template <bool ATOMIC, bool HALF, bool EVERY, bool COUNT = false>
__global__ __launch_bounds__(64 * (kQAnts + 1)) void k_construct_async_dense_q(Dev D, Iter A) {
  extern __shared__ uint4 qsm[];
  __shared__ uint32_t qhd[kQAnts], qtl[kQAnts], qdone;
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int na = (int)(blockDim.x >> 6) - 1;
  if (threadIdx.x < kQAnts) {
    qhd[threadIdx.x] = 0;
    qtl[threadIdx.x] = 0;
  }
  if (threadIdx.x == 0) qdone = 0;
  __syncthreads();
  const QRing q{qsm, qhd, qtl, &qdone};
  if (wv == na) {
    ring_updater<ATOMIC, COUNT>(D, A, q, lane, na);
    return;
  }
  uint32_t *vis = reinterpret_cast<uint32_t *>(qsm + (size_t)na * kQRing) +
                  wv * ((D.n + 31) >> 5);
  const int ant = uni(blockIdx.x * na + wv);
  if (ant < D.m) ant_queued<ATOMIC, HALF, EVERY, COUNT>(D, A, ant, vis, lane, q, wv);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  if (lane == 0) atomicAdd(&qdone, 1u);
}

// Many instances in one launch, updates through each block's updater wave:
// block b runs ants bitems[b].y .. bitems[b].y + kBatchQAnts - 1 of
// instance bitems[b].x (one instance per block, so the updater wave works
// with one descriptor), wave kBatchQAnts applies their entries.
constexpr int kBatchQAnts = kBatchQAntsPerBlock;

template <bool ATOMIC, bool HALF>
__global__ __launch_bounds__(64 * (kBatchQAnts + 1)) void k_construct_async_batch_q(
    const Dev *devs, const Iter *iters, const int2 *bitems, int nb, int wmax) {
  extern __shared__ uint4 qsm[];
  __shared__ uint32_t qhd[kBatchQAnts], qtl[kBatchQAnts], qdone;
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  if (threadIdx.x < kBatchQAnts) {
    qhd[threadIdx.x] = 0;
    qtl[threadIdx.x] = 0;
  }
  if (threadIdx.x == 0) qdone = 0;
  __syncthreads();
  const int b = blockIdx.x;  // the grid has exactly nb blocks
  const int2 item = bitems[b];
  const int inst = uni(item.x);
  const Dev D = global_dev(devs[inst]);
  const Iter A = iters[inst];
  const QRing q{qsm, qhd, qtl, &qdone};
  if (wv == kBatchQAnts) {
    ring_updater<ATOMIC, false>(D, A, q, lane, kBatchQAnts);
    return;
  }
  uint32_t *vis = reinterpret_cast<uint32_t *>(qsm + (size_t)kBatchQAnts * kQRing) +
                  wv * wmax;
  const int ant = uni(item.y + wv);
  if (ant < D.m) ant_queued<ATOMIC, HALF>(D, A, ant, vis, lane, q, wv);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  if (lane == 0) atomicAdd(&qdone, 1u);
}

// Many instances in one launch: wave w builds the tour of ant items[w].y of
// instance items[w].x, whose descriptor and iteration state live in device
// memory (so the launch can be replayed from a graph).  The work list is
// ordered by decreasing n, so the longest chains start first.
template <bool ATOMIC>
__global__ __launch_bounds__(256) void k_construct_async_batch(const Dev *devs, const Iter *iters,
                                                               const int2 *items, int nitems,
                                                               int wmax) {
  extern __shared__ uint32_t smem[];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int w = uni(blockIdx.x * (blockDim.x >> 6) + wv);
  if (w >= nitems) return;
  const int2 item = items[w];
  const int inst = uni(item.x);
  const Dev D = global_dev(devs[inst]);
  const Iter A = iters[inst];
  ant_async_dense<ATOMIC>(D, A, uni(item.y), smem + wv * wmax, lane);
}

// ---------------------------------------------------------------------------
// Asynchronous construction with several ants per wave: a group of L lanes
// (L = 32 or 16, L >= cl) carries one ant, so a wave advances 64 / L ants in
// lockstep.  The rule is the same as above, computed group by group: the
// argmax and the roulette scan over candidate positions in the same order
// (so the choice of L never changes a decision), reductions confined to the
// group's rows (DPP within a row of 16, the row-pair swap for L = 32),
// group-local lane reads by ds_bpermute.  All ants of a wave belong to one
// instance and step together (same n); a group whose ant index is past m
// leaves at the start.
// ---------------------------------------------------------------------------
template <int L>
__device__ __forceinline__ uint32_t grp_umax(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
  if (L == 32) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max(v, max((uint32_t)a[0], (uint32_t)a[1]));
  }
  return v;
}

template <int L>
__device__ __forceinline__ uint32_t grp_umin(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
  if (L == 32) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min(v, min((uint32_t)a[0], (uint32_t)a[1]));
  }
  return v;
}

// This group's bits of a wave ballot.
template <int L>
__device__ __forceinline__ uint32_t grp_bits(uint64_t ballot, int base) {
  if (L == 32) return base ? (uint32_t)(ballot >> 32) : (uint32_t)ballot;
  return (uint32_t)(ballot >> base) & 0xffffu;
}

// Value of v on lane k of this group.
__device__ __forceinline__ uint32_t grp_read(uint32_t v, int base, int k) {
  return (uint32_t)__shfl((int)v, base + k, 64);
}

// Many ants per SIMD are in flight, so the instructions of a step set the time
// (256 instances, n in [100, 2000], m = n: 20.8 -> 16.3 ms per
// construction).  The records come by buffer loads (32-bit offsets; pointers read from
// memory are generic to the compiler and become flat accesses, which also
// hold up LDS), an entry's address is computed only where it is updated, the
// chosen lane marks its own city with the bit it has at hand and keeps its
// own sum of distances, and lane masks are scalar.
template <int L, bool ATOMIC>
__device__ __forceinline__ void ants_async_dense(const Dev &D, const Iter &A, int first,
                                                 uint32_t *vis_wave, int lane) {
  const int gi = lane / L, gl = lane % L, base = gi * L;
  const int ant = first + gi;
  if (ant >= D.m) return;  // the whole group leaves
  const int n = D.n, cl = D.cl, ldn = D.ldn;
  const int W = (n + 31) >> 5;
  const int kl = gl < cl ? gl : cl - 1;
  const float al = A.a_loc, bl = A.b_loc;
  uint32_t *vis = vis_wave + gi * W;
  // lanes that hold a candidate, every group
  const uint64_t cand = __ballot(gl < cl);
  const __amdgpu_buffer_rsrc_t crs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(D.crec), 0, n * cl * 16, kBufWord3);
  auto load_rec = [&](int city) {
    const auto r = __builtin_amdgcn_raw_buffer_load_b128(crs, (city * cl + kl) * 16, 0, 0);
    return make_uint4(r[0], r[1], r[2], r[3]);
  };

  for (int w = gl; w < W; w += L) vis[w] = 0u;
  uint4 draws = philox10(make_uint4((uint32_t)gl, (uint32_t)ant, A.it, A.instance), A.key0, A.key1);
  const int start = (int)__umulhi(grp_read(draws.z, base, 0), (uint32_t)n);
  if (gl == 0) vis[start >> 5] |= 1u << (start & 31);
  int tb = start;
  uint4 rec = load_rec(start);

  int cur = start, prev = -1, kprev = -1;  // kprev: position of cur in prev's list
  float fval = 0.f;                        // pheromone of (prev, cur) as read
  uint32_t c_roul = 0, c_fb = 0, c_retry = 0;
  uint64_t c_fbu = 0;
  uint64_t len = 0;                        // the distances this lane's choices added
  // the compare-and-swap in flight; pexp == pret: there is none to repeat.  The
  // empty asm at a step's start keeps pexp a register of its own there.  Seen as a
  // copy of pret, it makes the compiler copy the result of the next one where the
  // paths meet, which waits for it in the step that issued it (two ants, n = 500,
  // 32 lanes: 1.12 us a step instead of 0.79; 1000 cities and 200 ants 1.25 and
  // 1.06).  A flag for "none" waits no more either but costs a batch 9% in
  // instructions (256 instances 17.8 ms instead of 16.3)
  float *pptr = nullptr;
  unsigned int pexp = 0, pret = 0;
  uint32_t uleft = A.lperiod;

  // chunks of L steps: one Philox batch and one tour store per chunk
  for (int t0 = 0; t0 <= n; t0 += L) {
  if (t0 > 0)
    draws = philox10(make_uint4((uint32_t)(t0 + gl), (uint32_t)ant, A.it, A.instance), A.key0,
                     A.key1);
  // the chunk's greedy draws (lane gl: step t0 + gl) as one ballot
  const uint32_t gbits = grp_bits<L>(__ballot((draws.x >> 8) < A.q0_24), base);
  uint32_t clen = 0;
  const int tend = min(t0 + L, n + 1);
  for (int t = t0 > 0 ? t0 : 1; t < tend; ++t) {
    if (ATOMIC) {
      if (pret != pexp) c_retry += 1 + cas_apply(pptr, pret, al, bl);
      pexp = pret;
      __asm__ volatile("" : "+v"(pexp));
    }
    // (lanes past the list repeat its last candidate: they never win, being
    // the highest lanes, and the masks leave them out)
    const uint32_t bit = 1u << (rec.x & 31);
    uint32_t *const vw = vis + (rec.x >> 5);
    const bool unv = (*vw & bit) == 0;
    const float w = unv ? __uint_as_float(rec.w) * __uint_as_float(rec.z) : 0.f;
    __asm__ volatile("" ::"v"(w), "v"((int)unv));
    if (t > 1 && --uleft == 0) {
      uleft = A.lperiod;
      const uint32_t b = grp_bits<L>(__ballot(rec.x == (uint32_t)prev) & cand, base);
      const int kr = b ? __builtin_ctz(b) : -1;
      const float rval = kr >= 0 ? __uint_as_float(grp_read(rec.w, base, kr)) : fval;
      const float seen = gl == 0 ? fval : rval;
      if (gl < 2 && !map_fixed(seen, al, bl)) {
        float *h = gl == 0 ? home(D, prev, cur, kprev) : home(D, cur, prev, kr);
        if (ATOMIC) {
          pptr = h;
          pexp = __float_as_uint(seen);
          pret = atomicCAS(reinterpret_cast<unsigned int *>(h), pexp,
                           __float_as_uint(fmaf(al, seen, bl)));
        } else {
          __hip_atomic_store(h, fmaf(al, seen, bl), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    if (t == n) break;
    const uint32_t umask = grp_bits<L>(__ballot(unv) & cand, base);
    int next, k = -1;
    float tval;
    if (umask) {
      if ((gbits >> (t - t0)) & 1u) {
        const uint32_t mx = grp_umax<L>(__float_as_uint(w));
        k = __builtin_ctz(grp_bits<L>(__ballot(__float_as_uint(w) == mx), base) & umask);
      } else {
        float P = w;
        for (int off = 1; off < cl; off <<= 1) {
          const float o = __shfl_up(P, off, L);
          if (gl >= off) P = P + o;
        }
        const float total = __uint_as_float(grp_read(__float_as_uint(P), base, cl - 1));
        const uint32_t u24 = grp_read(draws.y, base, t - t0) >> 8;
        const float r = ((float)u24 * 0x1p-24f) * total;
        const uint32_t sel = grp_bits<L>(__ballot(P > r), base) & umask;
        k = sel ? __builtin_ctz(sel) : 31 - __builtin_clz(umask);
        ++c_roul;
      }
      next = (int)grp_read(rec.x, base, k);
      tval = __uint_as_float(grp_read(rec.w, base, k));
      const bool won = gl == k;
      __hip_atomic_fetch_or(vw, won ? bit : 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      clen += won ? rec.y : 0u;
    } else {
      // Alg. 2's fallback over every unvisited city, ties -> lowest index;
      // first over the prefix (as in fallback_dense, 128 / L cities per lane)
      const float *trow = D.tau + (size_t)cur * ldn;
      const float *erow = D.etad + (size_t)cur * ldn;
      const uint16_t *drow = D.dist + (size_t)cur * ldn;
      float bv = 0.f, bt = 0.f;
      uint32_t bj = kNone, bd = 0;
      bool found = false;
      if (D.fpre) {
        const uint4 *fr = D.fpre + (size_t)cur * (kFpre / 2);
        const float fb = D.fbound[cur];
        uint4 pe[64 / L];
#pragma unroll
        for (int r = 0; r < 64 / L; ++r) pe[r] = fr[gl + L * r];
#pragma unroll
        for (int r = 0; r < 64 / L; ++r) {
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const uint32_t x = q ? pe[r].z : pe[r].x;
            const uint32_t j = x & 0xffffu;
            const float tq = trow[j];
            const float v = tq * __uint_as_float(q ? pe[r].w : pe[r].y);
            if (!((vis[j >> 5] >> (j & 31)) & 1u) &&
                (bj == kNone || v > bv || (v == bv && j < bj))) {
              bv = v; bj = j; bt = tq; bd = x >> 16;
            }
          }
        }
        found = grp_umax<L>(bj == kNone ? 0u : __float_as_uint(bv)) > __float_as_uint(fb);
        if (!found) { bv = 0.f; bj = kNone; }
      }
#pragma unroll 2
      for (int j0 = 4 * gl; !found && j0 < n; j0 += 4 * L) {
        const float4 tv = *reinterpret_cast<const float4 *>(trow + j0);
        const float4 ev = *reinterpret_cast<const float4 *>(erow + j0);
        const ushort4 dv = *reinterpret_cast<const ushort4 *>(drow + j0);
        const float tq[4] = {tv.x, tv.y, tv.z, tv.w};
        const float eq[4] = {ev.x, ev.y, ev.z, ev.w};
        const uint32_t dq[4] = {dv.x, dv.y, dv.z, dv.w};
        uint32_t bits = (vis[j0 >> 5] >> (j0 & 31)) & 0xfu;
        if (j0 + 4 > n) bits |= (0xfu << (n - j0)) & 0xfu;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float v = tq[q] * eq[q];
          if (!((bits >> q) & 1u) && (bj == kNone || v > bv)) {
            bv = v; bj = (uint32_t)(j0 + q); bt = tq[q]; bd = dq[q];
          }
        }
      }
      const uint32_t mx = grp_umax<L>(bj == kNone ? 0u : __float_as_uint(bv));
      const uint32_t jn = grp_umin<L>((bj != kNone && __float_as_uint(bv) == mx) ? bj : kNone);
      const int owner = __builtin_ctz(grp_bits<L>(__ballot(bj == jn), base));
      next = (int)jn;
      tval = __uint_as_float(grp_read(__float_as_uint(bt), base, owner));
      if (gl == owner) {
        mark(vis, next);
        clen += bd;
      }
      ++c_fb;
      c_fbu += (uint64_t)(n - t);
    }
    tb = gl == t - t0 ? next : tb;
    rec = load_rec(next);
    fval = tval;
    kprev = k;
    prev = cur;
    cur = next;
  }
  len += clen;
  if (t0 < n && gl <= min(L - 1, n - 1 - t0)) D.tours[(size_t)ant * n + t0 + gl] = tb;
  }
  if (ATOMIC && pret != pexp) c_retry += 1 + cas_apply(pptr, pret, al, bl);
  {
    const uint32_t b1 = grp_bits<L>(__ballot(gl < cl && D.crec[(size_t)cur * cl + kl].x ==
                                                         (uint32_t)start), base);
    const uint32_t b2 = grp_bits<L>(__ballot(gl < cl && D.crec[(size_t)start * cl + kl].x ==
                                                         (uint32_t)cur), base);
    const int k1 = b1 ? __builtin_ctz(b1) : -1, k2 = b2 ? __builtin_ctz(b2) : -1;
    float *h = gl == 0 ? home(D, cur, start, k1) : home(D, start, cur, k2);
    if (gl < 2) {
      if (ATOMIC)
        c_retry += cas_apply(h, __float_as_uint(tau_load(h)), al, bl);
      else
        __hip_atomic_store(h, fmaf(al, tau_load(h), bl), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
  }
#pragma unroll
  for (int off = L / 2; off; off >>= 1) len += (uint64_t)__shfl_xor((long long)len, off, L);
  len += D.dist[(size_t)cur * ldn + start];
  c_retry += grp_read(c_retry, base, 1);
  if (gl == 0) {
    D.lens[ant] = (int64_t)len;
    add_counters(D, (uint32_t)(n - 1) - c_roul - c_fb, c_roul, c_fb, c_fbu, c_retry);
  }
}

// Batch of instances, L lanes per ant: wave w runs ants witems[w].y ..
// witems[w].y + 64 / L - 1 of instance witems[w].x.
template <int L, bool ATOMIC>
__global__ __launch_bounds__(256) void k_construct_async_batch_g(const Dev *devs,
                                                                 const Iter *iters,
                                                                 const int2 *witems, int nw,
                                                                 int wmax) {
  extern __shared__ uint32_t smem[];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int w = uni(blockIdx.x * (blockDim.x >> 6) + wv);
  if (w >= nw) return;
  const int2 item = witems[w];
  const int inst = uni(item.x);
  const Dev D = global_dev(devs[inst]);
  const Iter A = iters[inst];
  ants_async_dense<L, ATOMIC>(D, A, uni(item.y), smem + wv * (64 / L) * wmax, lane);
}

// One instance, L lanes per ant.
template <int L, bool ATOMIC>
__global__ __launch_bounds__(256) void k_construct_async_dense_g(Dev D, Iter A) {
  extern __shared__ uint32_t smem[];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int first = uni((blockIdx.x * (blockDim.x >> 6) + wv) * (64 / L));
  if (first >= D.m) return;
  ants_async_dense<L, ATOMIC>(D, A, first, smem + wv * (64 / L) * ((D.n + 31) >> 5), lane);
}

// ---------------------------------------------------------------------------
// Selective pheromone memory (Sec. 3.2, Alg. 3).  The record of city c is s
// pairs {neighbour, pheromone}; a wave holds it with slot i on lane i.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint2 pair_load_coherent(const uint2 *p) {
  const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p),
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}

__device__ __forceinline__ void pair_store_coherent(uint2 *p, uint2 v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p),
                     ((unsigned long long)v.y << 32) | v.x, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long pack(uint2 v) {
  return ((unsigned long long)v.y << 32) | v.x;
}

template <bool COHERENT>
__device__ __forceinline__ uint2 spm_record(const Dev &D, int c, int lane) {
  const int i = lane < D.spm_s ? lane : D.spm_s - 1;
  const uint2 *p = D.spm + (size_t)c * D.spm_s + i;
  return COHERENT ? pair_load_coherent(p) : *p;
}

// Trail of this lane's candidate j from the record pairs on lanes 0..S-1:
// slot I is broadcast over each row of 16 lanes by DPP (row_newbcast), from
// the last slot to the first, so the first slot holding j is the one kept.
template <int I>
__device__ __forceinline__ void spm_trail_rows(uint2 pr, uint32_t j, float &t) {
  if constexpr (I >= 0) {
    const uint32_t node = (uint32_t)__builtin_amdgcn_mov_dpp((int)pr.x, 0x150 + I, 0xF, 0xF, true);
    const uint32_t val = (uint32_t)__builtin_amdgcn_mov_dpp((int)pr.y, 0x150 + I, 0xF, 0xF, true);
    t = j == node ? __uint_as_float(val) : t;
    spm_trail_rows<I - 1>(pr, j, t);
  }
}

// Pheromone of (c, j) for this lane's j: the value of the first slot of c's
// record holding j, else tau0 (every trail not stored is at the minimum).
// S: slots (0: s of them), L: candidate lanes.  With every candidate in lanes
// 0..15 a DPP row broadcast hands each slot to them (no scalar round trip);
// otherwise a lane read per slot.
template <int S, int L>
__device__ __forceinline__ float spm_tau(uint2 pr, int s, uint32_t j, float tau0) {
  float t = tau0;
  if constexpr (L == 16 && S != 0) {
    spm_trail_rows<S - 1>(pr, j, t);
  } else {
#pragma unroll
    for (int i = (S ? S : kMaxSpmS) - 1; i >= 0; --i) {
      if (S == 0 && i >= s) continue;
      const uint32_t node = rdlane(pr.x, i);
      const uint32_t val = rdlane(pr.y, i);
      t = j == node ? __uint_as_float(val) : t;
    }
  }
  return t;
}

template <int S, int L>
__device__ __forceinline__ Cand weigh_spm(const Dev &D, const uint32_t *vis, int lane, uint4 rec,
                                          uint2 pr, float tau0) {
  const uint32_t word = vis[rec.x >> 5];
  Cand c;
  c.unv = (lane < D.cl) & !((word >> (rec.x & 31)) & 1u);
  const float t = spm_tau<S, L>(pr, D.spm_s, rec.x, tau0);
  c.w = c.unv ? t * __uint_as_float(rec.z) : 0.f;
  return c;
}

// One ant's LDS words with the selective memory: the visited bitmap, then the
// unvisited cities of every grid cell as 16-bit counts (D.vw words in all).
// A visit takes its city off its cell's count.  For a candidate the cell comes
// with its record (the last word); for a fallback's choice it follows from
// the coordinates, which are loaded then and used at the ant's next fallback
// (`owed`), the only place that reads the counts.
__device__ __forceinline__ void cells_init(const Dev &D, uint32_t *vis, int lane) {
  const int W = (D.n + 31) >> 5, cells = D.gnx * D.gny;
  for (int w = lane; w < W; w += 64) vis[w] = 0u;
  for (int w = lane; w < D.vw - W; w += 64) {
    const int c = 2 * w;
    const uint32_t lo = c < cells ? (uint32_t)(D.gstart[c + 1] - D.gstart[c]) : 0u;
    const uint32_t hi = c + 1 < cells ? (uint32_t)(D.gstart[c + 2] - D.gstart[c + 1]) : 0u;
    vis[W + w] = lo | hi << 16;
  }
}
__device__ __forceinline__ void cell_take(const Dev &D, uint32_t *vis, uint32_t cell) {
  __hip_atomic_fetch_sub(vis + ((D.n + 31) >> 5) + (cell >> 1), 1u << (16 * (cell & 1)),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Alg. 2's fallback with the selective memory.  Every trail outside cur's
// record holds tau0 and tau0 * eta^beta strictly decreases with d (checked
// when the handle is created), so among the unvisited cities outside the
// record the nearest one by (d, j) has the largest value and the lowest
// index among equals.  The result is the best of that city and the
// unvisited cities of the record, ties -> lowest index: exactly the greedy
// argmax over all unvisited cities.
struct FarList {
  uint32_t e0, e1;  // the first 128 keys of a city's extended list, two per lane
  double2 at;       // its coordinates
};
__device__ __forceinline__ double2 city_at(const Dev &D, int c) {
  return reinterpret_cast<const double2 *>(D.xy)[c];
}
__device__ __forceinline__ FarList far_list(const Dev &D, int cur, int lane) {
  const uint32_t *xr = D.xnn + (size_t)cur * D.xl;
  FarList f;
  f.e0 = lane < D.xl ? xr[lane] : kNone;
  f.e1 = lane + 64 < D.xl ? xr[lane + 64] : kNone;
  f.at = city_at(D, cur);
  return f;
}

// F: far_list of cur.  s = spm_s.
__device__ __forceinline__ Pick fallback_spm(const Dev &D, uint32_t *vis, const FarList &F,
                                             int s, int lane, uint2 pr, float tau0, int unvisited,
                                             double2 &owed) {
  const uint32_t e0 = F.e0, e1 = F.e1;
  const double xc = F.at.x, yc = F.at.y;
  const bool in_rec = lane < s && pr.x != kNone;
  const uint32_t rj = in_rec ? pr.x : 0u;
  const double2 rxy = reinterpret_cast<const double2 *>(D.xy)[rj];
  const bool rec_unv = in_rec && !((vis[rj >> 5] >> (rj & 31)) & 1u);
  if (lane == 0) cell_take(D, vis, (uint32_t)(grid_cy(D, owed.y) * D.gnx + grid_cx(D, owed.x)));
  // hide the record's unvisited cities from the search of the others
  if (rec_unv) atomicOr(&vis[rj >> 5], 1u << (rj & 31));
  // the extended neighbour list is sorted by (d, j), so its first city that
  // is neither visited nor in the record is the nearest such city overall
  uint32_t key = kNone;
  {
    const uint32_t j0 = e0 & 0xffffu, j1 = e1 & 0xffffu;
    const uint64_t ok0 = __ballot(e0 != kNone && !((vis[j0 >> 5] >> (j0 & 31)) & 1u));
    const uint64_t ok1 = __ballot(e1 != kNone && !((vis[j1 >> 5] >> (j1 & 31)) & 1u));
    if (ok0)
      key = rdlane(e0, (int)__ffsll((unsigned long long)ok0) - 1);
    else if (ok1)
      key = rdlane(e1, (int)__ffsll((unsigned long long)ok1) - 1);
  }
  // (when every unvisited city is in the record there is nothing to find)
  const int rec_left = __popcll(__ballot(rec_unv));
  if (key == kNone && unvisited > rec_left) {
    // every listed city is taken: search the grid's cells by their distance
    // from cur, one whole cell (about a wave of cities) at a time, until the
    // nearest cell left is at least d + 1/2 away for the best d found: no
    // city there can reach d, let alone beat it (ties go to the lower index,
    // so cities at the best d are still read).  Cells without unvisited
    // cities are passed over by their counts.
    const uint32_t *count = vis + ((D.n + 31) >> 5);
    // cur relative to the grid; the margin covers fp32 rounding of offsets
    // below 65536
    const float px = (float)(xc - D.gx0), py = (float)(yc - D.gy0), gh = (float)D.gh;
    float bound = INFINITY;  // d + 1/2 for the best key so far
    // one cell per lane (x < 0: none)
    auto search = [&](int x, int y) {
      const int c = x < 0 ? 0 : y * D.gnx + x;
      const int g0 = D.gstart[c], g1 = D.gstart[c + 1];
      uint32_t lb = kNone;
      if (x >= 0 && ((count[c >> 1] >> (16 * (c & 1))) & 0xffffu)) {
        const float x0 = (float)x * gh, y0 = (float)y * gh;
        const float dx = fmaxf(fmaxf(x0 - px, px - (x0 + gh)) - 0.125f, 0.f);
        const float dy = fmaxf(fmaxf(y0 - py, py - (y0 + gh)) - 0.125f, 0.f);
        lb = __float_as_uint(__builtin_amdgcn_sqrtf(dx * dx + dy * dy) * 0.99999f);
      }
      while (true) {
        const uint32_t m = wave_umin_u(lb);
        if (m == kNone || __uint_as_float(m) >= bound) break;
        const int o = uni((int)__ffsll((unsigned long long)__ballot(lb == m)) - 1);
        const int p1 = (int)rdlane((uint32_t)g1, o);
        if (lane == o) lb = kNone;
        uint32_t lkey = kNone;
        for (int p = (int)rdlane((uint32_t)g0, o); p < p1; p += 128) {
          // two cities per lane, their loads together
          const int pa = min(p + lane, p1 - 1), pb = min(p + 64 + lane, p1 - 1);
          const uint32_t ja = D.gcity[pa], jb = D.gcity[pb];
          const double2 qa = D.gxy[pa], qb = D.gxy[pb];
          if (!((vis[ja >> 5] >> (ja & 31)) & 1u))
            lkey = min(lkey, exact_dist(xc, yc, qa.x, qa.y) << 16 | ja);
          if (p + 64 < p1 && !((vis[jb >> 5] >> (jb & 31)) & 1u))
            lkey = min(lkey, exact_dist(xc, yc, qb.x, qb.y) << 16 | jb);
        }
        const uint32_t k = wave_umin_u(lkey);
        if (k < key) {
          key = k;
          bound = (float)(key >> 16) + 0.5f;
        }
      }
    };
    // the 7 x 7 cells around cur's first, then, unless nothing outside them
    // can reach the best found, every other cell
    const int cx = grid_cx(D, xc), cy = grid_cy(D, yc);
    {
      const int x = cx - 3 + lane % 7, y = cy - 3 + lane / 7;
      search(lane < 49 && x >= 0 && y >= 0 && x < D.gnx && y < D.gny ? x : -1, y);
    }
    if (bound > 3.f * gh - 1.f) {
      const int cells = D.gnx * D.gny;
      for (int c0 = 0; c0 < cells; c0 += 64) {
        const int c = c0 + lane, y = c / D.gnx, x = c - y * D.gnx;
        const bool near = abs(x - cx) <= 3 && abs(y - cy) <= 3;
        search(c < cells && !near ? x : -1, y);
      }
    }
  }
  Pick p;
  p.k = -1;
  p.kind = 2;
  const uint64_t any_rec = __ballot(rec_unv);
  if (!any_rec) {  // the off-record candidate alone
    p.next = (int)(key & 0xffffu);
    p.d = key >> 16;
    p.tval = tau0;
    owed = city_at(D, p.next);
    return p;
  }
  if (rec_unv) atomicAnd(&vis[rj >> 5], ~(1u << (rj & 31)));
  // record candidates on lanes < s, the off-record candidate on its own
  const uint32_t rd = rec_unv ? exact_dist(xc, yc, rxy.x, rxy.y) : 0u;
  const bool off = key != kNone;
  const float re = D.eta_tab[rd];
  const float oe = D.eta_tab[off ? key >> 16 : 0u];
  const float rv = rec_unv ? __uint_as_float(pr.y) * re : 0.f;
  const float ov = off ? tau0 * oe : 0.f;
  uint32_t mx = wave_umax_u(rec_unv ? __float_as_uint(rv) : 0u);
  if (off && __float_as_uint(ov) > mx) mx = __float_as_uint(ov);
  const bool rec_win = rec_unv && __float_as_uint(rv) == mx;
  uint32_t jn = wave_umin_u(rec_win ? rj : kNone);
  const bool off_win = off && __float_as_uint(ov) == mx && (key & 0xffffu) < jn;
  if (off_win) {
    jn = key & 0xffffu;
    p.d = key >> 16;
    p.tval = tau0;
  } else {
    const int owner = uni((int)__ffsll((unsigned long long)__ballot(rec_win && rj == jn)) - 1);
    p.d = rdlane(rd, owner);
    p.tval = __uint_as_float(rdlane(pr.y, owner));
  }
  p.next = (int)jn;
  owed = city_at(D, p.next);
  return p;
}

// Alg. 3 on a record held by the wave (slot i on lane i, insert counter
// `tail`): the trail for neighbour nb gets the map x -> fma(a, x, b); a
// missing trail gets the map applied to tau0 in the slot after the most
// recently added one, which overwrites the least recently added trail.
__device__ __forceinline__ void spm_update_wave(uint2 &pr, uint32_t &tail, int s, int lane,
                                                int nb, float a, float b, float tau0,
                                                uint32_t &hits, uint32_t &misses) {
  const uint64_t hit = __ballot(lane < s && pr.x == (uint32_t)nb);
  if (hit) {
    const int i = (int)__ffsll((unsigned long long)hit) - 1;
    if (lane == i) pr.y = __float_as_uint(fmaf(a, __uint_as_float(pr.y), b));
    ++hits;
  } else {
    tail += 1;
    const int slot = (int)(tail % (uint32_t)s);
    if (lane == slot) pr = make_uint2((uint32_t)nb, __float_as_uint(fmaf(a, tau0, b)));
    ++misses;
  }
}

// Synchronous step updates of record r: every registered update of this step
// whose record is r, in increasing update index e = 2 * ant + w (ant
// ascending, the ant's own record before the next city's).  The wave that
// found r's list empty applies it.  When nobody pushed after it (`head` is
// its own update `own`, nearly always), the list is that one update for nb,
// and the record and its insert counter are what the wave loaded before the
// barrier (pr, tail): nothing is written between the barriers before.
// Otherwise up to 64 updates are gathered from the list (in arrival order)
// onto the lanes and applied smallest e first; a longer list is found by
// scanning every registration.  pr and tail return the record's new state.
template <int S>
__device__ __forceinline__ void spm_apply_step(const Dev &D, int r, int head, int own, int nb0,
                                               int ne, float a, float b, float tau0, int lane,
                                               uint2 &pr, uint32_t &tail, uint32_t &hits,
                                               uint32_t &misses) {
  const int s = S ? S : D.spm_s;
  if (head == own) {
    spm_update_wave(pr, tail, s, lane, nb0, a, b, tau0, hits, misses);
  } else {
    int cnt = 0, mine = INT_MAX, e = head;
    while (e >= 0 && cnt <= 64) {
      if (lane == cnt) mine = e;
      ++cnt;
      e = __hip_atomic_load(D.upd_next + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (cnt <= 64) {
      const int nbv = __hip_atomic_load(D.upd_nb + (lane < cnt ? mine : 0), __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
      for (int i = 0; i < cnt; ++i) {
        const int emin = (int)wave_umin_u((uint32_t)mine);
        const int l = uni((int)__ffsll((unsigned long long)__ballot(mine == emin)) - 1);
        if (lane == l) mine = INT_MAX;
        spm_update_wave(pr, tail, s, lane, (int)rdlane((uint32_t)nbv, l), a, b, tau0, hits,
                        misses);
      }
    } else {
      for (int e0 = 0; e0 < ne; e0 += 64) {
        const int ee = e0 + lane;
        int rr = -1, nbv = 0;
        if (ee < ne) {
          rr = __hip_atomic_load(D.upd_rec + ee, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          nbv = __hip_atomic_load(D.upd_nb + ee, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        uint64_t mask = __ballot(rr == r);
        while (mask) {
          const int l = (int)__ffsll((unsigned long long)mask) - 1;
          mask &= mask - 1;
          spm_update_wave(pr, tail, s, lane, (int)rdlane((uint32_t)nbv, l), a, b, tau0, hits,
                          misses);
        }
      }
    }
  }
  if (lane < s) pair_store_coherent(D.spm + (size_t)r * s + lane, pr);
  if (lane == 0) {
    __hip_atomic_store(D.spm_tail + r, tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(D.upd_head + r, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Registers update e (record r, neighbour nb) for this step by pushing it
// onto r's list.  Returns true for the update that found the list empty:
// its wave applies the record's list after the barrier.
__device__ __forceinline__ bool spm_register(const Dev &D, int e, int r, int nb) {
  __hip_atomic_store(D.upd_rec + e, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(D.upd_nb + e, nb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int old = __hip_atomic_exchange(D.upd_head + r, e, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(D.upd_next + e, old, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return old < 0;
}

__device__ __forceinline__ void add_spm_counters(const Dev &D, uint32_t hits, uint32_t misses) {
  atomicAdd(&D.counters[3], (unsigned long long)hits);
  atomicAdd(&D.counters[4], (unsigned long long)misses);
}

// ---------------------------------------------------------------------------
// Synchronous construction with the selective memory.  Per step:
//   SELECT (coherent reads) and registration of the step's 2m updates
//   | barrier | each record's updates applied in (ant, record i then j)
//   order by the wave that leads it | barrier.
// The closing edges are one more such round.
//
// Each phase waits for its slowest ant, so what follows a barrier is kept
// short: the next city's candidates, its record, both insert counters and the
// list a fallback starts from are loaded before the first barrier (records
// change only after it), a wave that has brought the next city's record up to
// date selects from it without reading it again, and the fallback's search is
// bounded by the cells that still hold unvisited cities.  n = 20000, m = 1024:
// 515 -> 215 ms per construction (26 -> 10.8 us per step).
// ---------------------------------------------------------------------------
// S and L as in spm_ant_queued.
template <int S, int L>
__global__ __launch_bounds__(1024) void k_construct_sync_spm(Dev D, Iter A) {
  extern __shared__ uint32_t smem[];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int ant = uni(blockIdx.x * (blockDim.x >> 6) + wv);
  const bool active = ant < D.m;
  const int n = D.n, cl = D.cl;
  const int kl = lane < cl ? lane : cl - 1;
  uint32_t *vis = smem + wv * D.vw;
  const float tau0 = A.tau0;
  auto tail_of = [&](int c) {
    return __hip_atomic_load(D.spm_tail + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };

  const GridBar gbar = grid_join(D, A);
  cells_init(D, vis, lane);
  uint4 draws = philox_batch(A, ant, 0, lane);
  const int start = (int)__umulhi(rdlane(draws.z, 0), (uint32_t)n);
  if (lane == 0) vis[start >> 5] |= 1u << (start & 31);
  int tb = start;
  double2 owed = city_at(D, start);

  int cur = start;
  int64_t len = 0;
  uint32_t c_greedy = 0, c_roul = 0, c_fb = 0, hits = 0, misses = 0;
  uint64_t c_fbu = 0;
  uint32_t bar = 0;
  uint4 rec = D.crec[(size_t)cur * cl + kl];
  uint2 pr = spm_record<true>(D, cur, lane);
  FarList far = far_list(D, cur, lane);
  for (int t = 1; t <= n; ++t) {
    int next = start;
    if ((t & 63) == 0) draws = philox_batch(A, ant, t, lane);
    if (active && t < n) {
      const Cand c = weigh_spm<S, L>(D, vis, lane, rec, pr, tau0);
      Pick p;
      const int k = pick_candidate(A, lane, cl, c, draw_of(draws, t), p.kind);
      if (k >= 0) {
        p.next = (int)rdlane(rec.x, k);
        p.d = rdlane(rec.y, k);
        if (lane == k) cell_take(D, vis, rec.w);
      } else {
        p = fallback_spm(D, vis, far, S ? S : D.spm_s, lane, pr, tau0, n - t, owed);
      }
      c_greedy += p.kind == 0;
      c_roul += p.kind == 1;
      if (p.kind == 2) { ++c_fb; c_fbu += (uint64_t)(n - t); }
      if (lane == 0) mark(vis, p.next);
      tour_put(D, ant, t, lane, p.next, tb);
      len += p.d;
      next = p.next;
    }
    if (active && t == n) len += dist_xy(D, cur, start);
    rec = D.crec[(size_t)next * cl + kl];
    uint2 pn = spm_record<true>(D, next, lane);  // as it was at the step's start
    far = far_list(D, next, lane);
    // t < n: the step's crossing (every lperiod-th step); t == n: the closing edge
    if (t == n || t % A.lperiod == 0) {
      uint32_t tc = tail_of(cur), tn = tail_of(next);
      bool lead = false;
      if (active && lane < 2)
        lead = spm_register(D, 2 * ant + lane, lane == 0 ? cur : next, lane == 0 ? next : cur);
      const uint64_t leads = __ballot(lead);
      grid_barrier_f(D, gbar, barrier_epoch(A.it, ++bar));
      if (leads) {
        const int hv = __hip_atomic_load(D.upd_head + (lane == 0 ? cur : next), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        const int h0 = (int)rdlane((uint32_t)hv, 0), h1 = (int)rdlane((uint32_t)hv, 1);
        if (leads & 1u)
          spm_apply_step<S>(D, cur, h0, 2 * ant, next, 2 * D.m, A.a_loc, A.b_loc, tau0, lane, pr, tc,
                         hits, misses);
        if (leads & 2u)
          spm_apply_step<S>(D, next, h1, 2 * ant + 1, cur, 2 * D.m, A.a_loc, A.b_loc, tau0, lane, pn,
                         tn, hits, misses);
      }
      if (t < n) {
        grid_barrier_f(D, gbar, barrier_epoch(A.it, ++bar));
        if (!(leads & 2u)) pn = spm_record<true>(D, next, lane);
      }
    }
    pr = pn;
    cur = next;
  }
  if (active && lane == 0) {
    D.lens[ant] = len;
    add_counters(D, c_greedy, c_roul, c_fb, c_fbu, 0);
    add_spm_counters(D, hits, misses);
  }
}

// ---------------------------------------------------------------------------
// Asynchronous construction with the selective memory: no barriers; each
// crossing's two record updates are lock-free.  A trail already in the
// record gets the map by a 64-bit compare-and-swap of its {neighbour, value}
// pair (a pair that changed meanwhile is re-examined); a missing trail takes
// the next slot of the record by an atomic increment of its insert counter
// and is written there as one 64-bit store.  Two ants inserting the same
// trail at the same moment can both succeed (a duplicate; reads take the
// first slot).  The updates of a move are issued at the start of the next
// step and checked one step later, like the dense kernel's.
// ---------------------------------------------------------------------------
struct SpmOp {
  uint2 *pair;         // hit: the pair's slot
  uint32_t *tail;      // miss: the record's insert counter
  unsigned long long expect, desired;
  uint32_t ret_lo, ret_hi;
  int nb, rec;
  bool hit, live;
};

__device__ __forceinline__ void spm_async_issue(const Dev &D, SpmOp &op, uint2 pr, int r, int nb,
                                                int lane, int owner, float a, float b,
                                                float tau0, uint32_t &hits, uint32_t &misses) {
  const int s = D.spm_s;
  const uint64_t hm = __ballot(lane < s && pr.x == (uint32_t)nb);
  if (lane != owner) return;
  op.live = true;
  op.nb = nb;
  op.rec = r;
  if (hm) {
    const int i = (int)__ffsll((unsigned long long)hm) - 1;
    const uint32_t v = rdlane(pr.y, i);
    op.hit = true;
    op.pair = D.spm + (size_t)r * s + i;
    op.expect = ((unsigned long long)v << 32) | (uint32_t)nb;
    op.desired = ((unsigned long long)__float_as_uint(fmaf(a, __uint_as_float(v), b)) << 32) |
                 (uint32_t)nb;
    const unsigned long long got = atomicCAS(reinterpret_cast<unsigned long long *>(op.pair),
                                             op.expect, op.desired);
    op.ret_lo = (uint32_t)got;
    op.ret_hi = (uint32_t)(got >> 32);
    ++hits;
  } else {
    op.hit = false;
    op.tail = D.spm_tail + r;
    op.ret_lo = atomicAdd(op.tail, 1u);
    ++misses;
  }
}

// Finishes an issued update: a miss writes its pair into the slot it took;
// a hit whose pair changed is redone against the record's current state.
__device__ __forceinline__ uint32_t spm_async_finish(const Dev &D, SpmOp &op, float a, float b,
                                                     float tau0) {
  if (!op.live) return 0;
  op.live = false;
  const int s = D.spm_s;
  if (!op.hit) {
    const uint32_t slot = (op.ret_lo + 1u) % (uint32_t)s;
    pair_store_coherent(D.spm + (size_t)op.rec * s + slot,
                        make_uint2((uint32_t)op.nb, __float_as_uint(fmaf(a, tau0, b))));
    return 0;
  }
  if ((((unsigned long long)op.ret_hi << 32) | op.ret_lo) == op.expect) return 0;
  // the pair changed: look for the trail again and apply the map
  uint32_t retries = 1;
  while (true) {
    int found = -1;
    uint2 cur_pair = make_uint2(0, 0);
    for (int i = 0; i < s; ++i) {
      const uint2 q = pair_load_coherent(D.spm + (size_t)op.rec * s + i);
      if (found < 0 && q.x == (uint32_t)op.nb) { found = i; cur_pair = q; }
    }
    if (found < 0) {
      const uint32_t t = atomicAdd(D.spm_tail + op.rec, 1u);
      pair_store_coherent(D.spm + (size_t)op.rec * s + (t + 1u) % (uint32_t)s,
                          make_uint2((uint32_t)op.nb, __float_as_uint(fmaf(a, tau0, b))));
      return retries;
    }
    const unsigned long long ex = pack(cur_pair);
    const unsigned long long de =
        ((unsigned long long)__float_as_uint(fmaf(a, __uint_as_float(cur_pair.y), b)) << 32) |
        (uint32_t)op.nb;
    if (atomicCAS(reinterpret_cast<unsigned long long *>(D.spm + (size_t)op.rec * s + found), ex,
                  de) == ex)
      return retries;
    ++retries;
  }
}

// The unsynchronised variant of Alg. 3 (ACS-GPU-Alt): the owner lane writes
// the changed pair of the record the wave read (pr, insert counter tl) and,
// for a new trail, the advanced insert counter, with plain (not
// read-modify-write) device-coherent stores; updates that race with it are
// lost.
__device__ __forceinline__ void spm_racy_issue(const Dev &D, uint2 pr, uint32_t tl, int r, int nb,
                                               int lane, int owner, float a, float b, float tau0,
                                               uint32_t &hits, uint32_t &misses) {
  const int s = D.spm_s;
  const uint64_t hm = __ballot(lane < s && pr.x == (uint32_t)nb);
  if (lane != owner) return;
  if (hm) {
    const int i = (int)__ffsll((unsigned long long)hm) - 1;
    const uint32_t v = rdlane(pr.y, i);
    pair_store_coherent(D.spm + (size_t)r * s + i,
                        make_uint2((uint32_t)nb, __float_as_uint(fmaf(a, __uint_as_float(v), b))));
    ++hits;
  } else {
    const uint32_t slot = (tl + 1u) % (uint32_t)s;
    pair_store_coherent(D.spm + (size_t)r * s + slot,
                        make_uint2((uint32_t)nb, __float_as_uint(fmaf(a, tau0, b))));
    __hip_atomic_store(D.spm_tail + r, tl + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ++misses;
  }
}

// The wave keeps the record of its current city in registers (pr, tl).  Its
// own update of that record (the reverse entry of the move that reached the
// city) is applied to the copy before the copy is read, so an ant always
// sees its own updates, as in Alg. 1; with one ant the result is exactly the
// sequential one.  The memory operations of the update are issued after the
// weights are formed (see the dense kernel for why).
template <bool ATOMIC>
__global__ __launch_bounds__(256) void k_construct_async_spm(Dev D, Iter A) {
  extern __shared__ uint32_t smem[];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int ant = uni(blockIdx.x * (blockDim.x >> 6) + wv);
  if (ant >= D.m) return;
  const int n = D.n, cl = D.cl, s = D.spm_s;
  const int kl = lane < cl ? lane : cl - 1;
  uint32_t *vis = smem + wv * D.vw;
  const float al = A.a_loc, bl = A.b_loc, tau0 = A.tau0;

  cells_init(D, vis, lane);
  uint4 draws = philox_batch(A, ant, 0, lane);
  const int start = (int)__umulhi(rdlane(draws.z, 0), (uint32_t)n);
  if (lane == 0) vis[start >> 5] |= 1u << (start & 31);
  int tb = start;
  double2 owed = city_at(D, start);
  uint4 rec = D.crec[(size_t)start * cl + kl];
  uint2 pr = spm_record<false>(D, start, lane);
  uint32_t tl = D.spm_tail[start];
  uint2 pr_prev = pr;
  uint32_t tl_prev = tl;

  int cur = start, prev = -1;
  int64_t len = 0;
  uint64_t c_kind = 0;  // greedy | roulette << 21 | fallback << 42
  uint32_t c_retry = 0, hits = 0, misses = 0;
  uint64_t c_fbu = 0;
  SpmOp op{};
  op.live = false;
  uint32_t uleft = A.lperiod;

  // chunks of 64 steps: one Philox batch and one tour store per chunk
  for (int t0 = 0; t0 <= n; t0 += 64) {
  if (t0 > 0) draws = philox_batch(A, ant, t0, lane);
  uint32_t clen = 0;
  const int tend = min(t0 + 64, n + 1);
  for (int t = t0 > 0 ? t0 : 1; t < tend; ++t) {
    if (ATOMIC) c_retry += spm_async_finish(D, op, al, bl, tau0);
    bool upd = false;
    if (t > 1 && --uleft == 0) {
      uleft = A.lperiod;
      upd = true;
    }
    // record of cur as it was read, then with this ant's reverse update
    const uint2 pr_read = pr;
    const uint32_t tl_read = tl;
    if (upd) {
      uint32_t h0 = 0, m0 = 0;
      spm_update_wave(pr, tl, s, lane, prev, al, bl, tau0, h0, m0);
    }
    const Cand c = weigh_spm<0, 64>(D, vis, lane, rec, pr, tau0);
    __asm__ volatile("" ::"v"(c.w), "v"((int)c.unv));
    if (upd) {
      // forward entry of the previous move in prev's record (lane 0),
      // reverse entry in cur's record (lane 1)
      if (ATOMIC) {
        spm_async_issue(D, op, pr_prev, prev, cur, lane, 0, al, bl, tau0, hits, misses);
        spm_async_issue(D, op, pr_read, cur, prev, lane, 1, al, bl, tau0, hits, misses);
      } else {
        spm_racy_issue(D, pr_prev, tl_prev, prev, cur, lane, 0, al, bl, tau0, hits, misses);
        spm_racy_issue(D, pr_read, tl_read, cur, prev, lane, 1, al, bl, tau0, hits, misses);
      }
    }
    if (t == n) break;
    Pick p;
    const int k = pick_candidate(A, lane, cl, c, draw_of(draws, t), p.kind);
    if (k >= 0) {
      p.next = (int)rdlane(rec.x, k);
      p.d = rdlane(rec.y, k);
      if (lane == k) cell_take(D, vis, rec.w);
    } else {
      p = fallback_spm(D, vis, far_list(D, cur, lane), s, lane, pr, tau0, n - t, owed);
    }
    c_kind += 1ull << (21 * p.kind);
    if (p.kind == 2) c_fbu += (uint64_t)(n - t);
    if (lane == 0) mark(vis, p.next);
    tb = lane == t - t0 ? p.next : tb;
    clen += p.d;
    rec = D.crec[(size_t)p.next * cl + kl];
    pr_prev = pr;
    tl_prev = tl;
    pr = spm_record<false>(D, p.next, lane);
    tl = D.spm_tail[p.next];
    prev = cur;
    cur = p.next;
  }
  len += clen;
  if (t0 < n && lane <= min(63, n - 1 - t0)) D.tours[(size_t)ant * n + t0 + lane] = tb;
  }
  if (ATOMIC) c_retry += spm_async_finish(D, op, al, bl, tau0);
  // closing edge, read fresh: record cur (neighbour start), record start
  {
    const uint2 q0 = spm_record<true>(D, cur, lane);
    if (ATOMIC) {
      spm_async_issue(D, op, q0, cur, start, lane, 0, al, bl, tau0, hits, misses);
      c_retry += spm_async_finish(D, op, al, bl, tau0);
    } else {
      const uint32_t t0 = __hip_atomic_load(D.spm_tail + cur, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
      spm_racy_issue(D, q0, t0, cur, start, lane, 0, al, bl, tau0, hits, misses);
    }
    const uint2 q1 = spm_record<true>(D, start, lane);
    if (ATOMIC) {
      spm_async_issue(D, op, q1, start, cur, lane, 0, al, bl, tau0, hits, misses);
      c_retry += spm_async_finish(D, op, al, bl, tau0);
    } else {
      const uint32_t t1 = __hip_atomic_load(D.spm_tail + start, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
      spm_racy_issue(D, q1, t1, start, cur, lane, 0, al, bl, tau0, hits, misses);
    }
  }
  len += dist_xy(D, cur, start);
  c_retry = (uint32_t)uni((int)(rdlane(c_retry, 0) + rdlane(c_retry, 1)));
  hits = (uint32_t)uni((int)(rdlane(hits, 0) + rdlane(hits, 1)));
  misses = (uint32_t)uni((int)(rdlane(misses, 0) + rdlane(misses, 1)));
  if (lane == 0) {
    D.lens[ant] = len;
    const uint32_t m21 = (1u << 21) - 1;
    add_counters(D, (uint32_t)c_kind & m21, (uint32_t)(c_kind >> 21) & m21,
                 (uint32_t)(c_kind >> 42) & m21, c_fbu, c_retry);
    add_spm_counters(D, hits, misses);
  }
}

// ---------------------------------------------------------------------------
// Asynchronous construction with the selective memory, updates through the
// block's updater wave (as the dense k_construct_async_dense_q): the ant
// wave issues no update, so its record loads never wait behind an atomic.
// Entry of city r: {r, nbA, nbB, 0}: Alg. 3 on r's record for neighbour nbA
// (the edge that reached r), then for nbB (the edge that left it); kNone
// marks an edge without an update (local-update period).  One entry per
// visited city keeps the two updates of a record in their order, and the
// updates of different entries concern different records of one ant, so an
// ant's updates land in the order Alg. 1 applies them.  The start city's
// entry (its departure, then the closing edge) goes last.
// ---------------------------------------------------------------------------
template <bool ATOMIC>
__device__ __forceinline__ uint32_t spm_apply_entries(const Dev &D, const Iter &A, uint4 e,
                                                      uint32_t &hits, uint32_t &misses) {
  if (e.x == kNoEntry) return 0;
  const int r = (int)e.x, s = D.spm_s;
  uint2 *rec = D.spm + (size_t)r * s;
  const float a = A.a_loc, b = A.b_loc;
  const uint32_t ins = __float_as_uint(fmaf(a, A.tau0, b));  // a new trail: the map of tau0
  uint32_t retries = 0;
  for (int u = 0; u < 2; ++u) {
    const uint32_t nb = u == 0 ? e.y : e.z;
    if (nb == kNone) continue;
    while (true) {
      // the record as it is now; the first slot holding nb is its trail
      int found = -1;
      uint2 cur = make_uint2(0u, 0u);
      for (int i = 0; i < s; ++i) {
        const uint2 x = pair_load_coherent(rec + i);
        if (found < 0 && x.x == nb) {
          found = i;
          cur = x;
        }
      }
      if (found < 0) {
        // miss: the slot after the most recently added one
        uint32_t t;
        if (ATOMIC) {
          t = atomicAdd(D.spm_tail + r, 1u);
        } else {
          t = __hip_atomic_load(D.spm_tail + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(D.spm_tail + r, t + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        pair_store_coherent(rec + (t + 1u) % (uint32_t)s, make_uint2(nb, ins));
        ++misses;
        break;
      }
      const uint2 nw = make_uint2(nb, __float_as_uint(fmaf(a, __uint_as_float(cur.y), b)));
      if (!ATOMIC) {
        pair_store_coherent(rec + found, nw);
        ++hits;
        break;
      }
      if (atomicCAS(reinterpret_cast<unsigned long long *>(rec + found), pack(cur), pack(nw)) ==
          pack(cur)) {
        ++hits;
        break;
      }
      ++retries;  // the pair changed meanwhile: look again
    }
  }
  return retries;
}

// The ant of k_construct_async_spm_q.  Records come by buffer loads: the
// candidates' {j, d, eta^beta} on lanes 0..cl-1, the selective record's
// pairs on lanes 0..s-1 and its insert counter.  Before the record of cur is
// read, the ant applies its own update of the edge that reached cur to its
// copy (Alg. 1 order): only a miss matters there, which replaces the slot
// after the most recently added one by prev (visited, so its trail is never
// read).  S: s when known at compile time (0: D.spm_s).  L: lanes holding
// the candidates (16, 32 or 64).
template <bool ATOMIC, int S, int L>
__device__ __forceinline__ void spm_ant_queued(const Dev &D, const Iter &A, int ant,
                                               uint32_t *vis, int lane, const QRing &q, int qw) {
  const int n = D.n, cl = D.cl, s = S ? S : D.spm_s;
  const uint64_t clmask = cl >= 64 ? ~0ull : (1ull << cl) - 1;
  const int koff = (lane < cl ? lane : cl - 1) * 16;
  const int rowb = cl * 16;
  const int soff = (lane < s ? lane : s - 1) * 8;
  const float tau0 = A.tau0;
  const __amdgpu_buffer_rsrc_t crs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(D.crec), 0, n * rowb, kBufWord3);
  const __amdgpu_buffer_rsrc_t srs =
      __builtin_amdgcn_make_buffer_rsrc(D.spm, 0, n * s * 8, kBufWord3);
  const __amdgpu_buffer_rsrc_t trs =
      __builtin_amdgcn_make_buffer_rsrc(D.spm_tail, 0, n * 4, kBufWord3);
  auto load_rec = [&](int city) {
    const auto r = __builtin_amdgcn_raw_buffer_load_b128(crs, koff, city * rowb, 0);
    return make_uint4(r[0], r[1], r[2], r[3]);
  };
  auto load_pair = [&](int city) {
    const auto r = __builtin_amdgcn_raw_buffer_load_b64(srs, soff, city * s * 8, kCoherent);
    return make_uint2(r[0], r[1]);
  };
  auto load_tail = [&](int city) {
    return __builtin_amdgcn_raw_buffer_load_b32(trs, 0, city * 4, kCoherent);
  };

  cells_init(D, vis, lane);
  uint4 draws = philox_batch(A, ant, 0, lane);
  const int start = (int)__umulhi(rdlane(draws.z, 0), (uint32_t)n);
  if (lane == 0) vis[start >> 5] |= 1u << (start & 31);
  uint4 rec = load_rec(start);
  uint2 pr = load_pair(start);
  uint32_t tlv = load_tail(start);

  uint32_t qhead = 0, qtail = 0, c_retry = 0, hits = 0, misses = 0, c_roul = 0, c_fb = 0;
  bool qdirect = false;
  uint64_t c_fbu = 0;
  int64_t len = 0;
  int cur = start, prev = -1;
  double2 owed = city_at(D, start);
  bool arrived_upd = false;    // the edge that reached cur gets a local update
  uint32_t nb_start = kNone;   // the start city's departure update (applied last)
  const uint32_t lp = A.lperiod;
  for (int t0 = 0; t0 < n; t0 += 64) {
    if (t0 > 0) draws = philox_batch(A, ant, t0, lane);
    const uint64_t upd = __builtin_amdgcn_ballot_w64((uint32_t)(lane + t0) % lp == 0);
    const uint64_t greedy = __builtin_amdgcn_ballot_w64((draws.x >> 8) < A.q0_24);
    // lane t - t0: step t's entry (x = kNoEntry: none) and tour entry
    uint4 e = make_uint4(kNoEntry, 0u, 0u, 0u);
    int tb = start;
    uint32_t clen = 0;
    const int tend = min(t0 + 64, n);
    for (int g0 = t0 > 0 ? t0 : 1; g0 < tend;) {
      const int g1 = min((g0 & ~(kQGroup - 1)) + kQGroup, tend);
      uint64_t sb = 1ull << (g0 - t0);  // bit t - t0
      for (int t = g0; t < g1; ++t, sb <<= 1) {
        const int tl = t - t0;
        if (arrived_upd) {
          const uint64_t hit =
              __builtin_amdgcn_ballot_w64(lane < s && pr.x == (uint32_t)prev);
          if (!hit) {
            const uint32_t tu = (uint32_t)uni((int)tlv) + 1u;
            const int slot = (int)(S ? (tu % (uint32_t)S) : (tu % (uint32_t)s));
            if (lane == slot) pr.x = (uint32_t)prev;
          }
        }
        const float tj = spm_tau<S, L>(pr, s, rec.x, tau0);
        const uint32_t word = vis[__builtin_amdgcn_ubfe(rec.x, 5, 11)];
        const bool unv = !__builtin_amdgcn_ubfe(word, rec.x, 1);
        const uint64_t umask = __builtin_amdgcn_ballot_w64(unv) & clmask;
        int next, k;
        uint32_t d;
        if (__builtin_expect(umask == 0, 0)) {
          const Pick p =
              fallback_spm(D, vis, far_list(D, cur, lane), s, lane, pr, tau0, n - t, owed);
          next = p.next;
          k = -1;
          d = p.d;
          ++c_fb;
          c_fbu += (uint64_t)(n - t);
        } else {
          const float w = unv ? tj * __uint_as_float(rec.z) : 0.f;
          if (greedy & sb) {
            // Eq. 1: maximum weight, lowest position
            const uint32_t wb = __float_as_uint(w);
            const uint32_t mx = rows_umax_s<L>(wb);
            k = (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(wb == mx) & umask);
          } else {
            // Eq. 2 by roulette, as in ant_queued
            float P = w;
            for (int off = 1; off < cl; off <<= 1) {
              const float o = __shfl_up(P, off, 64);
              if (lane >= off) P = P + o;
            }
            const float total = __uint_as_float(rdlane(__float_as_uint(P), cl - 1));
            const float r = ((float)(rdlane(draws.y, tl) >> 8) * 0x1p-24f) * total;
            const uint64_t sel = __builtin_amdgcn_ballot_w64(P > r) & umask;
            k = sel ? (int)__builtin_ctzll(sel) : 63 - (int)__builtin_clzll(umask);
            ++c_roul;
          }
          next = (int)rdlane(rec.x, k);
          d = rdlane(rec.y, k);
        }
        const uint32_t cell = rec.w;
        rec = load_rec(next);
        pr = load_pair(next);
        tlv = load_tail(next);
        if (lane == (k < 0 ? 0 : k)) {
          __hip_atomic_fetch_or(vis + (next >> 5), 1u << (next & 31), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_WORKGROUP);
          if (k >= 0) cell_take(D, vis, cell);
        }
        const bool up = (upd & sb) != 0;
        if (t == 1) {
          nb_start = up ? (uint32_t)next : kNone;
        } else if (arrived_upd || up) {
          e.x = wrlane((uint32_t)cur, tl, e.x);
          e.y = wrlane(arrived_upd ? (uint32_t)prev : kNone, tl, e.y);
          e.z = wrlane(up ? (uint32_t)next : kNone, tl, e.z);
        }
        tb = (int)wrlane((uint32_t)next, tl, (uint32_t)tb);
        clen += d;
        arrived_upd = up;
        prev = cur;
        cur = next;
      }
      c_retry += group_push<ATOMIC, false, true>(D, A, q, qw, qhead, qtail, qdirect, lane, e, t0, g1,
                                          hits, misses);
      g0 = g1;
    }
    len += clen;
    if (lane < tend - t0) D.tours[(size_t)ant * n + t0 + lane] = tb;
  }
  // closing edge (cur, start), always updated: cur's entry, then start's
  {
    const uint4 ce = lane == 0 ? make_uint4((uint32_t)cur, arrived_upd ? (uint32_t)prev : kNone,
                                            (uint32_t)start, 0u)
                               : make_uint4((uint32_t)start, nb_start, (uint32_t)cur, 0u);
    c_retry += group_push<ATOMIC, false, true>(D, A, q, qw, qhead, qtail, qdirect, lane, ce, n, n + 2,
                                        hits, misses);
    len += dist_xy(D, cur, start);
  }
  c_retry = (uint32_t)uni((int)wave_sum_u(c_retry));
  hits = (uint32_t)uni((int)wave_sum_u(hits));
  misses = (uint32_t)uni((int)wave_sum_u(misses));
  if (lane == 0) {
    D.lens[ant] = len;
    add_counters(D, (uint32_t)(n - 1) - c_roul - c_fb, c_roul, c_fb, c_fbu, c_retry);
    if (hits | misses) add_spm_counters(D, hits, misses);
  }
}

// One instance, selective memory, updates through the block's updater wave
// (waves 0..na-1 are ants, wave na applies their entries); LDS as in
// k_construct_async_dense_q.  S and L as in spm_ant_queued (the host picks
// them from s and cl).
template <bool ATOMIC, int S, int L>
__global__ __launch_bounds__(64 * (kQAnts + 1)) void k_construct_async_spm_q(Dev D, Iter A) {
  extern __shared__ uint4 qsm[];
  __shared__ uint32_t qhd[kQAnts], qtl[kQAnts], qdone;
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int na = (int)(blockDim.x >> 6) - 1;
  if (threadIdx.x < kQAnts) {
    qhd[threadIdx.x] = 0;
    qtl[threadIdx.x] = 0;
  }
  if (threadIdx.x == 0) qdone = 0;
  __syncthreads();
  const QRing q{qsm, qhd, qtl, &qdone};
  if (wv == na) {
    ring_updater<ATOMIC, false, true>(D, A, q, lane, na);
    return;
  }
  uint32_t *vis = reinterpret_cast<uint32_t *>(qsm + (size_t)na * kQRing) + wv * D.vw;
  const int ant = uni(blockIdx.x * na + wv);
  if (ant < D.m) spm_ant_queued<ATOMIC, S, L>(D, A, ant, vis, lane, q, wv);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  if (lane == 0) atomicAdd(&qdone, 1u);
}

// ---------------------------------------------------------------------------
// Iteration best, best-so-far and the global update (Alg. 1, Eq. 4), one
// block.  Every directed entry of the best tour is touched exactly once, so
// plain read-modify-writes suffice.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void argmin_len(const Dev &D, int64_t &bl, int &ba) {
  __shared__ int64_t sl[16];
  __shared__ int sa[16];
  bl = INT64_MAX;
  ba = INT_MAX;
  for (int a = threadIdx.x; a < D.m; a += blockDim.x)
    if (D.lens[a] < bl) { bl = D.lens[a]; ba = a; }
#pragma unroll
  for (int off = 32; off; off >>= 1) {
    const int64_t ol = __shfl_xor(bl, off, 64);
    const int oa = __shfl_xor(ba, off, 64);
    if (ol < bl || (ol == bl && oa < ba)) { bl = ol; ba = oa; }
  }
  if ((threadIdx.x & 63) == 0) { sl[threadIdx.x >> 6] = bl; sa[threadIdx.x >> 6] = ba; }
  __syncthreads();
  bl = sl[0];
  ba = sa[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
    if (sl[w] < bl || (sl[w] == bl && sa[w] < ba)) { bl = sl[w]; ba = sa[w]; }
}

// ---------------------------------------------------------------------------
// Local search after the construction (the paper's further research asks
// how a local search heuristic such as 3-opt changes convergence): a
// first-improvement descent over 2-opt and Or-opt moves, each creating an
// edge from the examined city a to one of its candidates, with a FIFO queue
// of cities to examine.  For a popped city the moves are tried in a fixed
// order and the first that shortens the tour is applied:
//   1. 2-opt on a's successor b: candidates c (k ascending) while
//      d(a,c) < d(a,b), e = succ(c): (a,b),(c,e) -> (a,c),(b,e);
//   2. 2-opt on a's predecessor b: while d(a,c) < d(b,a), e = pred(c);
//   3. Or-opt, L = 1, 2, 3: the segment of a and the L - 1 cities after it,
//      p before it, x after it; per candidate c (k ascending): (A) the
//      segment between c and succ(c), a next to c; (B) reversed between
//      pred(c) and c;
//   4. (kind 2) 3-opt, the four reconnections that replace (a,b), (c,d) and
//      (e,f) of a [b..c] [d..e] f by three new edges (see ls_three_opt).
// The cities at the ends of the changed edges are then queued (in the order
// listed per move) unless queued already; at most 50 n moves are applied.
// A 2-opt move reverses the forward path between its two cities when that
// path holds at most half the cities, else the rest of the tour; an Or-opt
// move shifts the shorter of the blocks between the segment's old and new
// places by L positions and writes the segment into the gap.  Tour, positions
// and queue live in LDS as 16-bit indices (n <= kLsMaxN); the queue flags are
// a bitmap.
//
// One block per tour.  A popped city is a chain of LDS and distance loads that
// one wave follows (its lanes evaluate the candidates of a move kind at once
// and the lowest-order improving one is taken, which is the move a sequential
// scan in that order finds), and most pops find nothing.  So the waves of a
// block examine the first cities of the queue at the same time, on the same
// tour; the first in queue order that has a move is applied by all of them,
// it and the cities before it are popped, and those after it are examined
// again on the changed tour: exactly the sequential descent.  A wave gives up
// its search once a wave before it has found a move.  With few tours that
// shortens the descent; with many the repeated examinations cost more than
// they hide, and a tour gets fewer waves.  n = 2392, ms per iteration with the
// 3-opt moves (2-opt and Or-opt alone), one wave per tour as it was, then 1, 2,
// 4, 8 and 16 waves; the host takes the starred:
//   m = 64    16.5 (7.4)   12.9 (7.9)   10.2 (5.8)   7.6 (4.0)   5.9 (3.3)   5.5* (3.4)
//   m = 400   22.2 (9.6)   18.0 (11.1)  14.0 (8.2)   11.3 (6.4)  10.7* (6.4) 17.6 (11.1)
//   m = 800   26.2 (11.3)  19.1 (11.6)  16.0 (8.8)   14.4* (8.0) 21.1 (12.8) 35.2 (22.5)
//   m = 1500  29.6 (12.8)  22.4 (12.8)  19.8* (10.8) 20.9 (11.8) 28.3 (17.3) 56.7 (36.6)
//   m = 2392  36.1 (18.0)  29.6* (15.7) 38.8 (20.9)  35.8 (19.8) 48.4 (28.5) 91.9 (59.2)
// (one wave since without scratch memory: m = 2392 28.7 (15.0)).  The cuts between
// these are by m alone.  At 31 other sizes (n = 6 to 8000, cl = 5 to 64, 1 to 2500
// ants, clustered cities too) the number they give takes 0.23 to 0.83 of the one wave
// as it was with 3-opt moves and 0.26 to 0.93 without, but for n = 2392, 900 ants
// and cl = 64, where it is 0.87 and 0.99.
// ---------------------------------------------------------------------------
struct LsTour {
  uint16_t *t, *pos, *q;
  uint32_t *inq;
  int n;
};

// i in [-n, 2n)
__device__ __forceinline__ int ls_wrap(int i, int n) {
  i = i < 0 ? i + n : i;
  return i >= n ? i - n : i;
}
__device__ __forceinline__ int ls_at(const LsTour &w, int i) { return w.t[ls_wrap(i, w.n)]; }
__device__ __forceinline__ void ls_put(const LsTour &w, int i, int c) {
  i = ls_wrap(i, w.n);
  w.t[i] = (uint16_t)c;
  w.pos[c] = (uint16_t)i;
}
__device__ __forceinline__ int ls_dist(const Dev &D, int u, int v) {
  return (int)D.dist[(size_t)u * D.ldn + v];
}

// What a wave found for its city: the new positions' description and the
// cities to queue, in order.
struct LsMove {
  int kind;    // 1 reversal of positions i .. j, 2 Or-opt, 3 3-opt
  int delta;
  int i, j;    // 1: the shorter side's ends; 2: segment's position and c; 3: pa and boe
  int L;       // 2: segment length; 3: bod
  int side;    // 2: placement; 3: reconnection
  int s0, s1, s2;  // 2: the segment's cities
  int npush, p0, p1, p2, p3, p4, p5;
};

// ONE: the block is one wave, whose LDS operations take effect in order; the
// compiler only has to keep them so.
template <bool ONE>
__device__ __forceinline__ void ls_sync() {
  if (ONE)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  else
    __syncthreads();
}

// the ends of the forward path from city u to city v, or of the rest of the
// tour when that is shorter
__device__ __forceinline__ void ls_shorter(const LsTour &w, int u, int v, int &i, int &j) {
  const int n = w.n;
  i = w.pos[u];
  j = w.pos[v];
  const int len = ls_wrap(j - i, n) + 1;
  if (2 * len > n) {
    const int i2 = ls_wrap(j + 1, n);
    j = ls_wrap(i - 1, n);
    i = i2;
  }
}

// the cities at positions i .. j (forward, j reached from i) in reverse order
__device__ __forceinline__ void ls_reverse_at(const LsTour &w, int i, int j, int tid, int nt) {
  const int len = ls_wrap(j - i, w.n) + 1;
  for (int s = tid; s < len / 2; s += nt) {
    const int a = ls_at(w, i + s), b = ls_at(w, j - s);
    ls_put(w, i + s, b);
    ls_put(w, j - s, a);
  }
}

// block move: positions from .. from + cnt - 1 to from + by .. (by = -L or
// +L), chunks of nt ordered so no chunk reads what an earlier chunk wrote
template <bool ONE>
__device__ __forceinline__ void ls_shift(const LsTour &w, int from, int cnt, int by, int tid,
                                         int nt) {
  const int chunks = (cnt + nt - 1) / nt;
  for (int k = 0; k < chunks; ++k) {
    const int r = (by < 0 ? k : chunks - 1 - k) * nt + tid;
    const int c = r < cnt ? ls_at(w, from + r) : 0;
    ls_sync<ONE>();
    if (r < cnt) ls_put(w, ls_wrap(from + r, w.n) + by, c);
    ls_sync<ONE>();
  }
}

// Or-opt: the L cities at positions i .. i + L - 1 (seg, in order) between
// c and succ(c) (side 0) or reversed between pred(c) and c (side 1)
template <bool ONE>
__device__ __forceinline__ void ls_oropt(const LsTour &w, const LsMove &x, int tid, int nt) {
  const int n = w.n, L = x.L, i = x.i, pc = w.pos[x.j];
  int place;  // where the segment goes
  if (x.side == 0) {
    const int nb = ls_wrap(pc - ls_wrap(i + L, n), n) + 1, nc = n - L - nb;
    if (nb <= nc) {
      ls_shift<ONE>(w, ls_wrap(i + L, n), nb, -L, tid, nt);
      place = ls_wrap(i + nb, n);
    } else {
      place = ls_wrap(pc + 1, n);
      ls_shift<ONE>(w, place, nc, L, tid, nt);
    }
  } else {
    const int nc = ls_wrap(i - 1 - pc, n) + 1, nb = n - L - nc;
    if (nc <= nb) {
      place = pc;
      ls_shift<ONE>(w, pc, nc, L, tid, nt);
    } else {
      ls_shift<ONE>(w, ls_wrap(i + L, n), nb, -L, tid, nt);
      place = ls_wrap(i + nb, n);
    }
  }
  const int k = x.side == 0 ? tid : L - 1 - tid;
  // (values: a choice between the members themselves is one between their
  // addresses, for which the move would have to live in scratch memory)
  const int s0 = x.s0, s1 = x.s1, s2 = x.s2;
  if (tid < L) ls_put(w, place + tid, k == 0 ? s0 : k == 1 ? s1 : s2);
}

// 3-opt for the popped city a at position pa (local search kind 2): with
// b = succ(a), the tour a [B = b..c] [C = d..e] f becomes a C B, a C B',
// a C' B or a B' C' f (reconnections 0 to 3, tried in that order).  The
// first new edge joins a to a candidate x with d(a,x) < d(a,b), x = d, d, e,
// c for the four, in candidate order; the second joins b (c for C B') to one
// of its candidates y, in candidate order, while the partial gain stays
// positive.  The move a sequential scan finds is the lowest (reconnection,
// x, y).  The wave takes one x at a time, two when cl <= 32 (one per half
// wave), with all four reconnections at once (their loads in one round, the
// lanes taking y), keeps the first improving move of the most preferred
// reconnection seen, and stops early once reconnection 0 has one (or a wave
// before it any move: *found < self).
template <class F>
__device__ __forceinline__ bool ls_three_opt(const Dev &D, const LsTour &w, int a, int pa,
                                             uint4 ra, int b, int dab, int lane, const int *found,
                                             int self, F emit) {
  const int n = w.n, cl = D.cl;
  const int per = cl <= 32 ? 2 : 1;  // x at a time
  const int half = per == 2 ? lane >> 5 : 0, y = per == 2 ? lane & 31 : lane;
  const bool cand = y < cl;
  const uint4 rb = D.crec[(size_t)b * cl + (cand ? y : cl - 1)];
  // a's candidates closer than b: a prefix (the lists are sorted by distance)
  const uint64_t far = __ballot(lane >= cl || !((int)ra.y < dab));
  const int nx = far ? (int)__ffsll((unsigned long long)far) - 1 : 64;
  const int yb = (int)rb.x, dyb = (int)rb.y;  // b's candidates
  const int oyb = ls_wrap(w.pos[yb] - pa, n);
  int best = 4, bod = 0, boe = 0, bc = 0, bd = 0, be = 0, bf = 0, bdelta = 0;
  for (int kx = 0; kx < nx && best > 0; kx += per) {
    if (self > 0 &&
        __hip_atomic_load(found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < self)
      return false;
    const int kk = min(kx + half, nx - 1);
    const bool mine = cand && kx + half < nx;
    const int x = __shfl((int)ra.x, kk, 64), dax = __shfl((int)ra.y, kk, 64);
    const int ox = ls_wrap(w.pos[x] - pa, n);
    const int px = ls_at(w, pa + ox - 1), sx = ls_at(w, pa + ox + 1);
    const int g01 = dab - dax + ls_dist(D, px, x);  // x = d: removed (c, d), c = pred(x)
    const int g23 = dab - dax + ls_dist(D, x, sx);  // x = e or c: removed (x, succ(x))
    const uint4 rc = D.crec[(size_t)px * cl + (cand ? y : cl - 1)];  // candidates of c for C B'
    const int yc = (int)rc.x, dyc = (int)rc.y;
    const int oyc = ls_wrap(w.pos[yc] - pa, n);
#pragma unroll
    for (int type = 0; type < 4; ++type) {
      if (type >= best) break;
      int od, oe;
      bool ok;
      if (type == 0) {
        od = ox, oe = oyb;
        ok = mine && dyb < g01 && ox >= 2 && oyb >= ox;
      } else if (type == 1) {
        od = ox, oe = oyc;
        ok = mine && dyc < g01 && ox >= 2 && oyc > ox;
      } else if (type == 2) {
        od = oyb, oe = ox;
        ok = mine && dyb < g23 && ox >= 3 && oyb >= 2 && oyb < ox;
      } else {
        od = ox + 1, oe = oyb;
        ok = mine && dyb < g23 && ox >= 2 && ox <= n - 3 && oyb > ox + 1;
      }
      const int c = ls_at(w, pa + od - 1), d = ls_at(w, pa + od);
      const int e = ls_at(w, pa + oe), f = ls_at(w, pa + oe + 1);
      const int removed = dab + ls_dist(D, c, d) + ls_dist(D, e, f);
      int added;
      if (type == 0) added = ls_dist(D, a, d) + ls_dist(D, e, b) + ls_dist(D, c, f);
      else if (type == 1) added = ls_dist(D, a, d) + ls_dist(D, c, e) + ls_dist(D, b, f);
      else if (type == 2) added = ls_dist(D, a, e) + ls_dist(D, b, d) + ls_dist(D, c, f);
      else added = ls_dist(D, a, c) + ls_dist(D, b, e) + ls_dist(D, d, f);
      const uint64_t imp = __ballot(ok && added - removed < 0);
      if (imp) {
        const int k = (int)__ffsll((unsigned long long)imp) - 1;
        best = type;
        bod = (int)rdlane((uint32_t)od, k), boe = (int)rdlane((uint32_t)oe, k);
        bc = (int)rdlane((uint32_t)c, k), bd = (int)rdlane((uint32_t)d, k);
        be = (int)rdlane((uint32_t)e, k), bf = (int)rdlane((uint32_t)f, k);
        bdelta = (int)rdlane((uint32_t)(added - removed), k);
      }
    }
  }
  if (best == 4) return false;
  emit(LsMove{3, bdelta, pa, boe, bod, best, 0, 0, 0, 6, a, b, bc, bd, be, bf});
  return true;
}

// positions pa + 1 .. pa + oe hold B (od - 1 cities) then C
template <bool ONE>
__device__ __forceinline__ void ls_apply_three(const LsTour &w, const LsMove &x, int tid, int nt) {
  const int n = w.n, p0 = ls_wrap(x.i + 1, n), pe = ls_wrap(x.i + x.j, n);
  const int nb = x.L - 1, nc = x.j - x.L + 1;
  if (x.side == 3) {
    ls_reverse_at(w, p0, ls_wrap(p0 + nb - 1, n), tid, nt);
    ls_reverse_at(w, ls_wrap(p0 + nb, n), pe, tid, nt);
    return;
  }
  ls_reverse_at(w, p0, pe, tid, nt);  // C' B'
  ls_sync<ONE>();
  if (x.side <= 1) ls_reverse_at(w, p0, ls_wrap(p0 + nc - 1, n), tid, nt);  // C
  if (x.side != 1) ls_reverse_at(w, ls_wrap(p0 + nc, n), pe, tid, nt);      // B
}

// The move the descent makes for city a on the tour as it stands, handed to
// `emit` where it is found (a struct carried out of the branches would live in
// scratch memory).  Returns whether there is one.
template <class F>
__device__ __forceinline__ bool ls_examine(const Dev &D, const LsTour &w, int a, int kind,
                                           int lane, const int *found, int self, F emit) {
  const int n = w.n, cl = D.cl;
  const uint4 rec = D.crec[(size_t)a * cl + (lane < cl ? lane : cl - 1)];
  const int c = (int)rec.x, dac = (int)rec.y;
  const bool cand = lane < cl;
  const int pa = uni(w.pos[a]);
  // moves 1 to 3 all read the tour as it stands, so their distances are
  // loaded together (one round of memory latency); the first improving move
  // in the order above is then taken
  const int bs = uni(ls_at(w, pa + 1)), bp = uni(ls_at(w, pa - 1));  // succ, pred of a
  const int pc = w.pos[c];
  const int e = ls_at(w, pc + 1), f = ls_at(w, pc - 1);  // succ, pred of c
  const int dab = ls_dist(D, a, bs), dba = ls_dist(D, bp, a);
  const int dbe = ls_dist(D, bs, e), dce = ls_dist(D, c, e);
  const int dbf = ls_dist(D, bp, f), dfc = ls_dist(D, f, c);
  const int off = ls_wrap(pc - pa, n);
  int sl[3], xl[3], gl[3], dse[3], dfs[3];  // Or-opt, L = 1, 2, 3
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    sl[i] = uni(ls_at(w, pa + i));      // the segment's last city
    xl[i] = uni(ls_at(w, pa + i + 1));  // the city after it
    gl[i] = dba + ls_dist(D, sl[i], xl[i]) - ls_dist(D, bp, xl[i]);
    dse[i] = ls_dist(D, sl[i], e);
    dfs[i] = ls_dist(D, f, sl[i]);
  }
  // 1. 2-opt on the successor
  {
    const int delta = dac + dbe - dab - dce;
    const uint64_t imp = __ballot(cand && dac < dab && c != bs && e != a && delta < 0);
    if (imp) {
      const int k = (int)__ffsll((unsigned long long)imp) - 1;
      const int cc = (int)rdlane((uint32_t)c, k), ee = (int)rdlane((uint32_t)e, k);
      int i, j;
      ls_shorter(w, bs, cc, i, j);
      emit(LsMove{1, (int)rdlane((uint32_t)delta, k), i, j, 0, 0, 0, 0, 0, 4, a, bs, cc, ee, 0, 0});
      return true;
    }
  }
  // 2. 2-opt on the predecessor
  {
    const int delta = dac + dbf - dba - dfc;
    const uint64_t imp = __ballot(cand && dac < dba && c != bp && f != a && delta < 0);
    if (imp) {
      const int k = (int)__ffsll((unsigned long long)imp) - 1;
      const int cc = (int)rdlane((uint32_t)c, k), ee = (int)rdlane((uint32_t)f, k);
      int i, j;
      ls_shorter(w, a, ee, i, j);
      emit(LsMove{1, (int)rdlane((uint32_t)delta, k), i, j, 0, 0, 0, 0, 0, 4, a, bp, cc, ee, 0, 0});
      return true;
    }
  }
  // 3. Or-opt of the segment a .. (L cities)
#pragma unroll
  for (int L = 1; L <= 3; ++L) {
    if (n < L + 3) break;
    const int x = xl[L - 1], g = gl[L - 1];
    const bool out = cand && off >= L;
    const int dA = dac + dse[L - 1] - dce - g;
    const int dB = dfs[L - 1] + dac - dfc - g;
    const uint64_t impA = __ballot(out && c != bp && dA < 0);
    const uint64_t impB = __ballot(out && c != x && dB < 0);
    if (impA | impB) {
      const int k = (int)__ffsll((unsigned long long)(impA | impB)) - 1;
      const int side = ((impA >> k) & 1ull) ? 0 : 1;
      const int cc = (int)rdlane((uint32_t)c, k);
      const int ef = (int)rdlane((uint32_t)(side == 0 ? e : f), k);
      const int delta = (int)rdlane((uint32_t)(side == 0 ? dA : dB), k);
      emit(LsMove{2, delta, pa, cc, L, side, sl[0], sl[1], sl[2], 6, bp, x, a, sl[L - 1],
                  side == 0 ? cc : ef, side == 0 ? ef : cc});
      return true;
    }
  }
  // 4. 3-opt
  return kind >= 2 && n >= 6 &&
         ls_three_opt(D, w, a, pa, rec, bs, dab, lane, found, self, emit);
}

// Pops the first `popped` cities of the queue (its first wave), then queues the
// move's cities that are not queued, each once, in order (push: lane l holds
// the l-th of npush).  Returns how many were added.
__device__ __forceinline__ int ls_requeue(const LsTour &w, int qh, int popped, int left, int push,
                                          int npush, int lane) {
  const int n = w.n;
  if (lane < popped) {
    const int a = w.q[ls_wrap(qh + lane, n)];
    __hip_atomic_fetch_and(w.inq + (a >> 5), ~(1u << (a & 31)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  if (npush == 0) return 0;
  bool need = lane < npush;
#pragma unroll
  for (int u = 0; u < 5; ++u) need = need && !(lane > u && (int)rdlane((uint32_t)push, u) == push);
  need = need && !((w.inq[push >> 5] >> (push & 31)) & 1u);
  const uint64_t add = __ballot(need);
  if (need) {
    const int at = qh + popped + left + __popcll(add & ((1ull << lane) - 1));
    w.q[ls_wrap(ls_wrap(at, n), n)] = (uint16_t)push;
    __hip_atomic_fetch_or(w.inq + (push >> 5), 1u << (push & 31), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  return __popcll(add);
}

template <bool ONE>
__device__ __forceinline__ void ls_apply(const LsTour &w, const LsMove &mv, int tid, int nt) {
  if (mv.kind == 1) ls_reverse_at(w, mv.i, mv.j, tid, nt);
  else if (mv.kind == 2) ls_oropt<ONE>(w, mv, tid, nt);
  else ls_apply_three<ONE>(w, mv, tid, nt);
}

// One block per ant.  Dynamic LDS: t, pos, q (n 16-bit entries each) and the
// queue bitmap.  kind 2 adds the 3-opt move.
constexpr int kLsWaves = 16;
template <bool ONE>
__global__ __launch_bounds__(ONE ? 64 : 64 * kLsWaves) void k_local_search(Dev D, int kind) {
  extern __shared__ uint32_t lsm[];
  __shared__ LsMove s_mv[ONE ? 1 : kLsWaves];
  __shared__ int s_found[2], s_qn;  // first wave with a move (queue_round); queued cities
  const int ant = blockIdx.x, tid = threadIdx.x, nt = ONE ? 64 : blockDim.x, n = D.n;
  const int lane = tid & 63, wv = ONE ? 0 : uni(tid >> 6), nw = nt >> 6;
  const int np2 = (n + 1) & ~1;  // 16-bit arrays padded to whole words
  LsTour w;
  w.t = reinterpret_cast<uint16_t *>(lsm);
  w.pos = w.t + np2;
  w.q = w.pos + np2;
  w.inq = reinterpret_cast<uint32_t *>(w.q + np2);
  w.n = n;
  const int W = (n + 31) >> 5;
  const int32_t *tour = D.tours + (size_t)ant * n;
  for (int p = tid; p < n; p += nt) {
    const int c = tour[p];
    w.t[p] = (uint16_t)c;
    w.pos[c] = (uint16_t)p;
    w.q[p] = (uint16_t)c;
  }
  for (int k = tid; k < W; k += nt) w.inq[k] = k < W - 1 || (n & 31) == 0 ? ~0u
                                                             : (1u << (n & 31)) - 1u;
  if (!ONE && tid < 2) s_found[tid] = kNoWave;
  int qh = 0, qn = n;
  uint32_t round = 0;
  int64_t len = D.lens[ant];
  uint32_t moves = 0;
  const uint32_t cap = 50u * (uint32_t)n;
  ls_sync<ONE>();
  while (qn > 0 && moves < cap) {
    int popped = 1;
    if constexpr (ONE) {
      int push = 0, npush = 0;
      moves += ls_examine(D, w, uni(w.q[qh]), kind, lane, nullptr, 0, [&](const LsMove &mv) {
        push = lane == 0 ? mv.p0 : lane == 1 ? mv.p1 : lane == 2 ? mv.p2 : lane == 3 ? mv.p3
               : lane == 4 ? mv.p4 : mv.p5;
        npush = mv.npush;
        len += mv.delta;
        ls_apply<true>(w, mv, lane, 64);
      });
      qn += ls_requeue(w, qh, 1, qn - 1, push, npush, lane) - 1;
    } else {
      const int heads = min(nw, qn);
      auto examine = [&](int *found) {
        ls_examine(D, w, uni(w.q[ls_wrap(qh + wv, n)]), kind, lane, found, wv,
                   [&](const LsMove &mv) {
                     if (lane == 0) {
                       s_mv[wv] = mv;
                       atomicMin(found, wv);
                     }
                   });
      };
      auto act = [&](int found) {
        const int first = uni(found);
        popped = min(first + 1, heads);
        const LsMove &mv = s_mv[first < heads ? first : 0];
        if (first < heads) {
          ls_apply<false>(w, mv, tid, nt);
          len += mv.delta;
          ++moves;
        }
        if (wv == 0) {
          const int left = qn - popped;
          const int add = ls_requeue(w, qh, popped, left, (&mv.p0)[min(lane, 5)],
                                     first < heads ? mv.npush : 0, lane);
          if (lane == 0) s_qn = left + add;
        }
      };
      queue_round(s_found, round++, wv, heads, [] { __syncthreads(); }, examine, act);
      qn = uni(s_qn);
    }
    qh = ls_wrap(qh + popped, n);
  }
  ls_sync<ONE>();
  int32_t *out = D.tours + (size_t)ant * n;
  for (int p = tid; p < n; p += nt) out[p] = w.t[p];
  if (tid == 0) {
    D.lens[ant] = len;
    if (moves) atomicAdd(&D.counters[7], (unsigned long long)moves);
  }
}

// Block 0: iteration best and best-so-far.  Further blocks, after a construction
// with an updater wave: the records take their pheromone back from ctau
// (`canonical` as in ctau_out_slot).  One launch for both, neither fills the
// chip (4.4 and 4.3 us one after the other, together 4.5).
__global__ __launch_bounds__(1024) void k_best(Dev D, int canonical) {
  if (blockIdx.x > 0) {
    const size_t e = (size_t)(blockIdx.x - 1) * 1024 + threadIdx.x;
    if (e < (size_t)D.n * D.cl) ctau_out_slot(D, e, canonical != 0);
    return;
  }
  __shared__ int s_better;
  int64_t bl;
  int ba;
  argmin_len(D, bl, ba);
  if (threadIdx.x == 0) {
    const int64_t lgb = D.gstate[0];
    s_better = (lgb < 0 || bl < lgb) ? 1 : 0;
    D.gstate[0] = s_better ? bl : lgb;
    D.gstate[1] = bl;
    D.gstate[2] = ba;
  }
  __syncthreads();
  const int n = D.n;
  if (s_better)
    for (int p = threadIdx.x; p < n; p += blockDim.x) D.best[p] = D.tours[(size_t)ba * n + p];
}

// Eq. 4 on the best-so-far tour, dense memory: one wave per tour edge finds
// both candidate positions with one coalesced load of each row; the 2n
// directed entries are distinct, so plain read-modify-writes suffice.
__device__ __forceinline__ void global_edge(const Dev &D, const Iter &A, int p, int lane) {
  const int n = D.n;
  const float ag = A.a_glob;
  const float bg = (float)(A.rho / (double)D.gstate[0]);
  const int u = D.best[p], v = D.best[p + 1 < n ? p + 1 : 0];
  const int ku = cand_pos(D, u, v, lane), kv = cand_pos(D, v, u, lane);
  if (lane < 2) {
    float *h = lane == 0 ? home(D, u, v, ku) : home(D, v, u, kv);
    *h = fmaf(ag, *h, bg);
  }
}

__global__ __launch_bounds__(256) void k_global_dense(Dev D, Iter A) {
  const int p = uni(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (p < D.n) global_edge(D, A, p, threadIdx.x & 63);
}

// Eq. 4 with the selective memory, in the order of the tour: edge p updates
// record u_p then record v_p.  City best[p] is touched by edges p-1 and p
// (edges 0 and n-1 for p = 0), so one wave per tour position applies its
// record's two updates in that order and no record is shared.  The counters
// are added once per block of at most 512 (two atomics per position on the same
// two words took 0.48 ms at n = 20000, now 0.02).
__global__ __launch_bounds__(256) void k_global_spm(Dev D, Iter A) {
  const int lane = threadIdx.x & 63;
  __shared__ uint32_t s_hits, s_misses;
  if (threadIdx.x == 0) s_hits = s_misses = 0u;
  __syncthreads();
  const int n = D.n, s = D.spm_s;
  const int wave = uni(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
  const int waves = gridDim.x * (blockDim.x >> 6);
  const float ag = A.a_glob;
  const float bg = (float)(A.rho / (double)D.gstate[0]);
  uint32_t hits = 0, misses = 0;
  for (int p = wave; p < n; p += waves) {
    const int r = D.best[p];
    const int nb1 = p >= 1 ? D.best[p - 1] : D.best[1];
    const int nb2 = p >= 1 ? D.best[p + 1 < n ? p + 1 : 0] : D.best[n - 1];
    uint2 pr = spm_record<false>(D, r, lane);
    uint32_t tail = D.spm_tail[r];
    spm_update_wave(pr, tail, s, lane, nb1, ag, bg, A.tau0, hits, misses);
    spm_update_wave(pr, tail, s, lane, nb2, ag, bg, A.tau0, hits, misses);
    if (lane < s) D.spm[(size_t)r * s + lane] = pr;
    if (lane == 0) D.spm_tail[r] = tail;
  }
  if (lane == 0) {
    atomicAdd(&s_hits, hits);
    atomicAdd(&s_misses, misses);
  }
  __syncthreads();
  if (threadIdx.x == 0) add_spm_counters(D, s_hits, s_misses);
}

// Batched iteration end: block b handles instance b (iteration best and
// best-so-far), then advances that instance's iteration counter and moves
// its error flag (an exhausted bounded wait) into the batch's flag.
__global__ __launch_bounds__(1024) void k_best_batch(const Dev *devs, Iter *iters,
                                                     uint32_t *flag) {
  __shared__ int s_better;
  const Dev D = devs[blockIdx.x];
  int64_t bl;
  int ba;
  argmin_len(D, bl, ba);
  if (threadIdx.x == 0) {
    const uint32_t f = atomicExch(D.sync + 1, 0u);
    if (f) atomicOr(flag, f);
    const int64_t lgb = D.gstate[0];
    s_better = (lgb < 0 || bl < lgb) ? 1 : 0;
    D.gstate[0] = s_better ? bl : lgb;
    D.gstate[1] = bl;
    D.gstate[2] = ba;
    iters[blockIdx.x].it += 1;
  }
  __syncthreads();
  const int n = D.n;
  if (s_better)
    for (int p = threadIdx.x; p < n; p += blockDim.x) D.best[p] = D.tours[(size_t)ba * n + p];
}

// Batched global update (dense), one wave per tour edge as k_global_dense: grid
// (edges / 4, instances).  (One thread per edge that walks both lists took 121
// us for 256 instances, n up to 2000; this takes 59.)
__global__ __launch_bounds__(256) void k_global_batch(const Dev *devs, const Iter *iters) {
  const Dev D = global_dev(devs[blockIdx.y]);
  const int lane = threadIdx.x & 63;
  const int p = uni(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (p < D.n) global_edge(D, iters[blockIdx.y], p, lane);
}

// Best-so-far exchange between the colonies of a batch that all solve one
// instance (the multi-colony model of the paper's Sec. 2: periodic exchange
// of the best solution found so far along a communication topology).  Every
// colony first offers its best-so-far tour and length (block per colony);
// then every colony takes its source's offer when it is strictly shorter
// than its own: topology 0, the source is the colony with the shortest
// offer (lowest index among equals); topology 1, colony c - 1 (a ring).
// Reading every offer before any colony changes keeps the exchange
// independent of the order the blocks run in.
__global__ __launch_bounds__(256) void k_offer_batch(const Dev *devs, int n, int32_t *offer,
                                                     int64_t *olen) {
  const Dev D = devs[blockIdx.x];
  for (int p = threadIdx.x; p < n; p += blockDim.x) offer[(size_t)blockIdx.x * n + p] = D.best[p];
  if (threadIdx.x == 0) olen[blockIdx.x] = D.gstate[0];
}

__global__ __launch_bounds__(256) void k_accept_batch(const Dev *devs, int count, int n,
                                                      int topology, const int32_t *offer,
                                                      const int64_t *olen) {
  const int c = blockIdx.x;
  int src = (c + count - 1) % count;
  if (topology == 0) {
    src = -1;
    for (int i = 0; i < count; ++i)
      if (olen[i] >= 0 && (src < 0 || olen[i] < olen[src])) src = i;
  }
  if (src < 0 || olen[src] < 0) return;
  const Dev D = devs[c];
  const int64_t own = olen[c];
  if (own >= 0 && olen[src] >= own) return;
  for (int p = threadIdx.x; p < n; p += blockDim.x) D.best[p] = offer[(size_t)src * n + p];
  if (threadIdx.x == 0) D.gstate[0] = olen[src];
}

size_t lds_bytes(const Dev &D, int block) {
  return (size_t)(block / 64) * D.vw * sizeof(uint32_t);
}

constexpr int kAsyncBlock = 256;

}  // namespace

// ---------------------------------------------------------------------------
// Launch wrappers.
// ---------------------------------------------------------------------------
hipError_t launch_dist(const Dev &d, uint32_t *dmax, int r0, int rows, hipStream_t s) {
  dim3 grid((d.ldn + 511) / 512, (rows + 3) / 4);
  hipLaunchKernelGGL(k_dist, grid, dim3(256), 0, s, d, dmax, r0, rows);
  return hipGetLastError();
}

hipError_t launch_dmax(const Dev &d, uint32_t *dmax, hipStream_t s) {
  dim3 grid((d.n + 255) / 256, (d.n + kDmaxRows - 1) / kDmaxRows);
  hipLaunchKernelGGL(k_dmax, grid, dim3(256), 0, s, d, dmax);
  return hipGetLastError();
}

hipError_t launch_grid(const Dev &d, int32_t *cnt, hipStream_t s) {
  const size_t cells = (size_t)d.gnx * d.gny;
  hipError_t e = hipMemsetAsync(cnt, 0, cells * sizeof(int32_t), s);
  if (e != hipSuccess) return e;
  const dim3 g((d.n + 255) / 256);
  hipLaunchKernelGGL(k_grid_count, g, dim3(256), 0, s, d, cnt);
  hipLaunchKernelGGL(k_grid_scan, dim3(1), dim3(1024), 0, s, d, cnt);
  hipLaunchKernelGGL(k_grid_fill, g, dim3(256), 0, s, d, cnt);
  return hipGetLastError();
}

hipError_t launch_near(const Dev &d, int32_t *cand_tmp, const uint32_t *dmax, int r0, int rows,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_near, dim3(rows), dim3(256), 0, s, d, cand_tmp, dmax, r0);
  return hipGetLastError();
}

hipError_t launch_nn_tour(const Dev &d, const int32_t *cand_tmp, uint16_t *near, int64_t *lnn_out,
                          hipStream_t s) {
  // neighbours per city in LDS: 16 serve almost every choice; fewer where n is
  // large (three still serve over half of the choices at n = 20000, one at
  // the largest n = 65535)
  constexpr int kLdsBytes = 144 * 1024;
  const int have = std::min(kNnList, d.xnn ? (int)d.xl : (int)d.cl);
  const int C = std::max(1, std::min(have, kLdsBytes / (2 * d.n)));
  const size_t lds = (size_t)d.n * C * sizeof(uint16_t);
  if (C < have)
    hipLaunchKernelGGL(k_nn_tour<true>, dim3(1), dim3(1024), lds, s, d, cand_tmp, C, near, lnn_out);
  else
    hipLaunchKernelGGL(k_nn_tour<false>, dim3(1), dim3(1024), lds, s, d, cand_tmp, C, near,
                       lnn_out);
  return hipGetLastError();
}

hipError_t launch_crec(const Dev &d, const int32_t *cand_tmp, float tau0, hipStream_t s) {
  const int total = d.n * d.cl;
  hipLaunchKernelGGL(k_crec, dim3((total + 255) / 256), dim3(256), 0, s, d, cand_tmp, tau0);
  return hipGetLastError();
}

hipError_t launch_cand_out(const Dev &d, int32_t *out, hipStream_t s) {
  hipLaunchKernelGGL(k_cand_out, dim3((d.n * d.cl + 255) / 256), dim3(256), 0, s, d, out);
  return hipGetLastError();
}

hipError_t launch_fill(const Dev &d, float tau0, uint32_t dmax, bool eta_falls, hipStream_t s) {
  size_t total = d.tau ? (size_t)d.n * d.ldn : (size_t)d.n;
  if (d.fpre) total = std::max(total, (size_t)d.n * kFpre);
  if (d.spm) total = std::max(total, (size_t)d.n * d.spm_s);
  total = std::max(total, (size_t)8);
  hipLaunchKernelGGL(k_fill, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, d, tau0, dmax,
                     eta_falls ? 1 : 0);
  return hipGetLastError();
}

// Ant waves per block of the kernels with an updater wave: the m ants spread
// evenly over the compute units, two or more blocks per unit, at most
// kQAnts per block.  Dense compare-and-swap updates (`counted`): an updater
// passes over an edge that another one owns, so more of them only shorten the
// entries' wait: at most two ants share one, three above ten ants per unit, where
// the updaters' own waves begin to weigh (m = n, us per iteration with as many as
// the rule allows, with 2, with 3: n = 1500 687, 691, 691; 2000 938, 937, 930;
// 2392 1222, 1143, 1165; 3000 1609, 1533, 1466; 4000 3568, 3461, 3405; 2000
// cities and 8000 ants 2962, 2477, 2255).  Plain stores and the selective memory
// are within noise or slower with fewer.
static hipError_t queued_ants_per_block(int m, bool counted, int *na) {
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return hipErrorInvalidDevice;
  const int per_cu = (m + cus - 1) / cus;
  const int bpc = std::max(2, (per_cu + kQAnts - 1) / kQAnts);
  *na = std::max(1, std::min(kQAnts, (m + cus * bpc - 1) / (cus * bpc)));
  if (counted) *na = std::min(*na, per_cu > 10 ? 3 : 2);
  return hipSuccess;
}

// The selective memory's common shapes get kernels with s = 8 and the
// candidate lanes fixed (the trail lookup unrolls).
static const void *sync_kernel(const Dev &d, int memory) {
  if (d.sync_lds)
    return d.cl <= 32 ? reinterpret_cast<const void *>(&k_construct_sync_lds<true>)
                      : reinterpret_cast<const void *>(&k_construct_sync_lds<false>);
  if (memory == 0) return reinterpret_cast<const void *>(&k_construct_sync_dense);
  if (d.spm_s != 8) return reinterpret_cast<const void *>(&k_construct_sync_spm<0, 64>);
  if (d.cl <= 16) return reinterpret_cast<const void *>(&k_construct_sync_spm<8, 16>);
  if (d.cl <= 32) return reinterpret_cast<const void *>(&k_construct_sync_spm<8, 32>);
  return reinterpret_cast<const void *>(&k_construct_sync_spm<8, 64>);
}

// Dynamic LDS of a block of `ants` ants of that kernel.
static size_t sync_lds_size(const Dev &d, int ants) {
  return (d.sync_lds ? (size_t)d.n * d.cl * sizeof(float) : 0) + lds_bytes(d, 64 * ants);
}

// Whether the construction keeps the candidates' pheromone in ctau.
static bool updater_dense(int mode, int memory, int lanes, int queued) {
  return memory == 0 && lanes == 64 && queued && (mode == 1 || mode == 2);
}

hipError_t launch_construct(const Dev &d, const Iter &it, int mode, int memory, int lanes,
                            int queued, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  // ev0 / ev1 (optional) bracket the construction kernel itself, so that
  // their interval leaves out the bound, buffer and copy kernels beside it
  auto mark = [s](hipEvent_t e) { return e ? hipEventRecord(e, s) : hipSuccess; };
  // the fallback prefix's bound holds where every update maps an entry's own
  // value or a value its edge's other entry held from an equal start; the
  // unsynchronised ants that issue their own updates write f(forward value)
  // into a reverse entry that may differ from it, so they scan whole rows
  const bool queued_dense = updater_dense(mode, memory, lanes, queued);
  const bool far = memory == 0 && d.fpre && (mode != 2 || (lanes == 64 && queued));
  if (far) {
    hipLaunchKernelGGL(k_far_bound, dim3((d.n + 3) / 4), dim3(256), 0, s, d, it,
                       queued_dense ? 1 : 0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (mode == 3) {
    const size_t words = (size_t)d.m * ((d.n + 31) / 32);
    const int group = seq_group(d.n, it.lperiod);
    const hipError_t me = mark(ev0);
    if (me != hipSuccess) return me;
    if (words <= (size_t)kSeqLdsWords)
      hipLaunchKernelGGL(k_construct_seq_dense<true>, dim3(1), dim3(64 * kSeqWaves),
                         words * sizeof(uint32_t), s, d, it, group);
    else
      hipLaunchKernelGGL(k_construct_seq_dense<false>, dim3(1), dim3(64 * kSeqWaves), 0, s, d,
                         it, group);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : mark(ev1);
  }
  if (mode == 0) {
    const bool in_lds = d.sync_lds != 0;
    const int apb = d.sync_apb;
    const int grid = (d.m + apb - 1) / apb;
    Dev dd = d;
    Iter a = it;
    void *args[] = {&dd, &a};
    const void *fn = sync_kernel(d, memory);
    const bool dbuf = memory == 0 && (in_lds || it.lperiod == 1);
    // updates applied to the buffers in turn decide where the last one is
    const bool odd = in_lds ? ((uint32_t)(d.n - 1) / it.lperiod) & 1 : d.n & 1;
    const int words = in_lds ? 4 * kSyncMaxAnts * grid : 0;
    const dim3 gb((unsigned)(((size_t)d.n * d.ldn + 255) / 256));
    if (!in_lds && barrier_clear_due(it.it)) {
      hipLaunchKernelGGL(k_barrier_clear, dim3((d.nbflags + 255) / 256), dim3(256), 0, s, d, it.it);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    if (dbuf) {
      hipLaunchKernelGGL(k_sync_buf, gb, dim3(256), 0, s, d, 0, words);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    const hipError_t me = mark(ev0);
    if (me != hipSuccess) return me;
    hipError_t e = hipLaunchCooperativeKernel(fn, dim3(grid), dim3(64 * apb), args,
                                              sync_lds_size(d, apb), s);
    if (e == hipSuccess) e = mark(ev1);
    if (e != hipSuccess || !dbuf || !odd) return e;
    hipLaunchKernelGGL(k_sync_buf, gb, dim3(256), 0, s, d, 1, words);
    return hipGetLastError();
  }
  const int apb = kAsyncBlock / 64;
  const int grid = (d.m + apb - 1) / apb;
  const size_t lds = lds_bytes(d, kAsyncBlock);
  const bool atomic = mode == 1;
  if (memory == 0 && lanes == 64 && queued) {
    int na = 0;
    const bool every = it.lperiod == 1;
    // crossings counted at their edge (apply_entries): where at least half as
    // many ants as cities update at every step
    const bool counted = atomic && every && 2 * d.m >= d.n;
    const hipError_t qe = queued_ants_per_block(d.m, counted, &na);
    if (qe != hipSuccess) return qe;
    const dim3 gq((d.m + na - 1) / na), bq(64 * (na + 1));
    const size_t lq = (size_t)na * kQRing * sizeof(uint4) +
                      (size_t)na * ((d.n + 31) / 32) * sizeof(uint32_t);
    const bool half = d.cl <= 32;
    const dim3 gc((d.n * d.cl + 255) / 256);
    if (!far) hipLaunchKernelGGL(k_ctau_in, gc, dim3(256), 0, s, d);
    const hipError_t me = mark(ev0);
    if (me != hipSuccess) return me;
#define ACS_DENSE_Q(AT, HF, EV, CT)                                                    \
    if (atomic == AT && half == HF && every == EV && counted == CT)                     \
      hipLaunchKernelGGL((k_construct_async_dense_q<AT, HF, EV, CT>), gq, bq, lq, s, d, it);
    ACS_DENSE_Q(true, true, true, true)
    ACS_DENSE_Q(true, false, true, true)
    ACS_DENSE_Q(true, true, true, false)
    ACS_DENSE_Q(true, true, false, false)
    ACS_DENSE_Q(true, false, true, false)
    ACS_DENSE_Q(true, false, false, false)
    ACS_DENSE_Q(false, true, true, false)
    ACS_DENSE_Q(false, true, false, false)
    ACS_DENSE_Q(false, false, true, false)
    ACS_DENSE_Q(false, false, false, false)
#undef ACS_DENSE_Q
    // (launch_best_global copies ctau back)
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : mark(ev1);
  }
  const hipError_t me = mark(ev0);
  if (me != hipSuccess) return me;
  if (memory == 0 && lanes < 64) {
    const int g = 64 / lanes;
    const dim3 gg((d.m + apb * g - 1) / (apb * g));
    const size_t lg = lds * g;
    Dev dr = d;
    dr.fpre = nullptr;
    if (lanes == 32 && atomic)
      hipLaunchKernelGGL((k_construct_async_dense_g<32, true>), gg, dim3(kAsyncBlock), lg, s, d, it);
    else if (lanes == 32)
      hipLaunchKernelGGL((k_construct_async_dense_g<32, false>), gg, dim3(kAsyncBlock), lg, s, dr, it);
    else if (atomic)
      hipLaunchKernelGGL((k_construct_async_dense_g<16, true>), gg, dim3(kAsyncBlock), lg, s, d, it);
    else
      hipLaunchKernelGGL((k_construct_async_dense_g<16, false>), gg, dim3(kAsyncBlock), lg, s, dr, it);
  } else if (memory == 0) {
    if (atomic) {
      hipLaunchKernelGGL(k_construct_async_dense<true>, dim3(grid), dim3(kAsyncBlock), lds, s, d,
                         it);
    } else {
      Dev dd = d;
      dd.fpre = nullptr;
      hipLaunchKernelGGL(k_construct_async_dense<false>, dim3(grid), dim3(kAsyncBlock), lds, s,
                         dd, it);
    }
  } else if (queued) {
    int na = 0;
    const hipError_t e = queued_ants_per_block(d.m, false, &na);
    if (e != hipSuccess) return e;
    const dim3 gq((d.m + na - 1) / na), bq(64 * (na + 1));
    const size_t lq = (size_t)na * kQRing * sizeof(uint4) +
                      (size_t)na * d.vw * sizeof(uint32_t);
    // the common shapes get kernels with s and the candidate lanes fixed
    const int sk = d.spm_s == 8 ? 8 : 0;
    const int lk = sk == 0 ? 64 : d.cl <= 16 ? 16 : d.cl <= 32 ? 32 : 64;
#define ACS_SPM_Q(AT, SS, LL) \
    if (atomic == AT && sk == SS && lk == LL) \
      hipLaunchKernelGGL((k_construct_async_spm_q<AT, SS, LL>), gq, bq, lq, s, d, it);
    ACS_SPM_Q(true, 8, 16)
    ACS_SPM_Q(true, 8, 32)
    ACS_SPM_Q(true, 8, 64)
    ACS_SPM_Q(true, 0, 64)
    ACS_SPM_Q(false, 8, 16)
    ACS_SPM_Q(false, 8, 32)
    ACS_SPM_Q(false, 8, 64)
    ACS_SPM_Q(false, 0, 64)
#undef ACS_SPM_Q
  } else {
    if (atomic)
      hipLaunchKernelGGL(k_construct_async_spm<true>, dim3(grid), dim3(kAsyncBlock), lds, s, d,
                         it);
    else
      hipLaunchKernelGGL(k_construct_async_spm<false>, dim3(grid), dim3(kAsyncBlock), lds, s, d,
                         it);
  }
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : mark(ev1);
}

int plan_sync(Dev *d, int memory) {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  // blocks of `ants` ants of the kernel chosen by d->sync_lds on the device at once
  auto resident = [&](int ants) {
    int per_cu = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, sync_kernel(*d, memory), 64 * ants, sync_lds_size(*d, ants));
    if (e == hipSuccess) return per_cu * cus;
    (void)hipGetLastError();  // not the last error of the launches that follow
    return 0;
  };
  if (memory == 0 && sync_lds(d->n, d->m, d->cl)) {
    d->sync_lds = 1;
    d->sync_apb = sync_lds_ants_per_block(d->m);
    if (sync_lds_taken(d->n, d->m, d->cl, resident(d->sync_apb))) return 64 * kSyncMaxAnts;
    d->sync_lds = 0;
  }
  d->sync_apb = sync_ants_per_block_on(d->m, resident(sync_ants_per_block(d->m)));
  return resident(kSyncMaxAnts) * kSyncMaxAnts;
}

hipError_t launch_local_search(const Dev &d, int kind, hipStream_t s) {
  const int np2 = (d.n + 1) & ~1;
  const size_t lds = (size_t)3 * np2 * sizeof(uint16_t) + (size_t)((d.n + 31) / 32) * 4;
  // waves per tour (see the kernel)
  const int nw = d.m <= 128 ? 16 : d.m <= 512 ? 8 : d.m <= 1024 ? 4 : d.m <= 1792 ? 2 : 1;
  if (nw == 1)
    hipLaunchKernelGGL(k_local_search<true>, dim3(d.m), dim3(64), lds, s, d, kind);
  else
    hipLaunchKernelGGL(k_local_search<false>, dim3(d.m), dim3(64 * nw), lds, s, d, kind);
  return hipGetLastError();
}

hipError_t launch_best_global(const Dev &d, const Iter &it, int mode, int memory, int lanes,
                              int queued, hipStream_t s) {
  const unsigned out =
      updater_dense(mode, memory, lanes, queued) ? (unsigned)((d.n * d.cl + 1023) / 1024) : 0u;
  hipLaunchKernelGGL(k_best, dim3(1 + out), dim3(1024), 0, s, d, mode == 1 ? 1 : 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (memory == 0)
    hipLaunchKernelGGL(k_global_dense, dim3((d.n + 3) / 4), dim3(256), 0, s, d, it);
  else
    hipLaunchKernelGGL(k_global_spm, dim3(std::min(512, (d.n + 3) / 4)), dim3(256), 0, s, d, it);
  return hipGetLastError();
}

hipError_t launch_exchange_batch(const Dev *devs, int count, int n, int topology,
                                 int32_t *offer, int64_t *olen, hipStream_t s) {
  hipLaunchKernelGGL(k_offer_batch, dim3(count), dim3(256), 0, s, devs, n, offer, olen);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_accept_batch, dim3(count), dim3(256), 0, s, devs, count, n, topology,
                     offer, olen);
  return hipGetLastError();
}

hipError_t launch_batch_iteration(const Dev *devs, Iter *iters, const int2 *items, int nitems,
                                  int count, int nmax, int clmax, int mode, int lanes, int queued,
                                  uint32_t *flag, hipStream_t s) {
  const int apb = kAsyncBlock / 64;
  const int wmax = (nmax + 31) / 32;
  if (mode == 1) {
    // instances without a prefix (and the unsynchronised mode, see
    // launch_construct) have fpre null and scan whole rows
    hipLaunchKernelGGL(k_far_bound_batch, dim3((nmax + 3) / 4, count), dim3(256), 0, s, devs,
                       iters);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (lanes == 64 && queued) {
    const size_t lq = (size_t)kBatchQAnts * kQRing * sizeof(uint4) +
                      (size_t)kBatchQAnts * wmax * sizeof(uint32_t);
    const dim3 gq(nitems), bq(64 * (kBatchQAnts + 1));
    const bool half = clmax <= 32;
    const dim3 gc((nmax * clmax + 255) / 256, count);
    hipLaunchKernelGGL(k_ctau_in_batch, gc, dim3(256), 0, s, devs);
    if (mode == 1 && half)
      hipLaunchKernelGGL((k_construct_async_batch_q<true, true>), gq, bq, lq, s, devs, iters,
                         items, nitems, wmax);
    else if (mode == 1)
      hipLaunchKernelGGL((k_construct_async_batch_q<true, false>), gq, bq, lq, s, devs, iters,
                         items, nitems, wmax);
    else if (half)
      hipLaunchKernelGGL((k_construct_async_batch_q<false, true>), gq, bq, lq, s, devs, iters,
                         items, nitems, wmax);
    else
      hipLaunchKernelGGL((k_construct_async_batch_q<false, false>), gq, bq, lq, s, devs, iters,
                         items, nitems, wmax);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ctau_out_batch, gc, dim3(256), 0, s, devs, mode == 1 ? 1 : 0);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_best_batch, dim3(count), dim3(1024), 0, s, devs, iters, flag);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_global_batch, dim3((nmax + 3) / 4, count), dim3(256), 0, s, devs,
                       iters);
    return hipGetLastError();
  }
  const size_t lds = (size_t)apb * (64 / lanes) * wmax * sizeof(uint32_t);
  const dim3 grid((nitems + apb - 1) / apb), blk(kAsyncBlock);
  const bool atomic = mode == 1;
  if (lanes == 64 && atomic)
    hipLaunchKernelGGL(k_construct_async_batch<true>, grid, blk, lds, s, devs, iters, items,
                       nitems, wmax);
  else if (lanes == 64)
    hipLaunchKernelGGL(k_construct_async_batch<false>, grid, blk, lds, s, devs, iters, items,
                       nitems, wmax);
  else if (lanes == 32 && atomic)
    hipLaunchKernelGGL((k_construct_async_batch_g<32, true>), grid, blk, lds, s, devs, iters,
                       items, nitems, wmax);
  else if (lanes == 32)
    hipLaunchKernelGGL((k_construct_async_batch_g<32, false>), grid, blk, lds, s, devs, iters,
                       items, nitems, wmax);
  else if (atomic)
    hipLaunchKernelGGL((k_construct_async_batch_g<16, true>), grid, blk, lds, s, devs, iters,
                       items, nitems, wmax);
  else
    hipLaunchKernelGGL((k_construct_async_batch_g<16, false>), grid, blk, lds, s, devs, iters,
                       items, nitems, wmax);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_best_batch, dim3(count), dim3(1024), 0, s, devs, iters, flag);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_global_batch, dim3((nmax + 3) / 4, count), dim3(256), 0, s, devs,
                     iters);
  return hipGetLastError();
}

}  // namespace acs
