// Sugarscape-style agents as objects on a square torus (the paper's
// sugarscape application, Sec. 4; its rules are not in the paper, so this is
// a synchronous, deterministic variant).  Agent {sugar, metabolism, vision,
// age, pos, target, world}; the sugar (with occupancy), capacity and request
// grids are plain device arrays.  One step t:
//   regrow (grid kernel): sugar = min(sugar + 1, cap)
//   1 choose  (do-all): best of the own cell and the unoccupied cells up to
//             `vision` away along the four axes: most sugar, then nearest,
//             then lowest index; a move request is the direction and distance
//             of the target, written to the own cell of the request grid
//   2 move    (do-all): the lowest requesting cell index wins the target; a
//             mover looks for lower ones in the cells that can see its target
//   3 eat     (same do-all: an agent touches only the cell it leaves and the
//             one it ends on, which no other agent does): sugar += cell; cell
//             = 0; sugar -= metabolism; age++; die (delete) if sugar <= 0 or
//             age >= max_age
//   4 request (do-all): fertile agents with enough sugar request their
//             lowest-index empty von Neumann neighbour (atomicMin)
//   5 birth   (do-all): the winner creates a child there with half its sugar
//             and traits drawn from hash(seed, stream, t, cell)
// Phases read occupancy only as it was when the phase started and change it
// only where no other agent of the phase looks, so the result does not depend
// on which lane or block runs first.
#include <string.h>

#include <algorithm>
#include <new>

#include "internal.hpp"

namespace dsoar {
namespace {

enum : uint32_t { kAgent = 0 };
enum : uint32_t { kSugar = 0, kMetab = 1, kVision = 2, kAge = 3, kPos = 4, kTarget = 5, kWorld = 6 };
constexpr uint32_t kInf = 0xFFFFFFFFu;
constexpr uint64_t kStreamChildMetab = 10, kStreamChildVision = 11;

// SplitMix64 output finaliser (Steele, Lea, Flood, OOPSLA 2014) and the
// workload hash h(seed, stream, a, b) = mix(mix(mix(seed ^ stream*golden) ^ a) ^ b).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z ^= z >> 30;
  z *= 0xBF58476D1CE4E5B9ull;
  z ^= z >> 27;
  z *= 0x94D049BB133111EBull;
  z ^= z >> 31;
  return z;
}
__device__ __forceinline__ uint64_t hash4(uint64_t seed, uint64_t stream, uint64_t a, uint64_t b) {
  return mix64(mix64(mix64(seed ^ (stream * 0x9E3779B97F4A7C15ull)) ^ a) ^ b);
}
// U{lo..hi}: lo + floor(top32(h) * (hi - lo + 1) / 2^32).
__device__ __forceinline__ int32_t uniform_int(uint64_t h, int32_t lo, int32_t hi) {
  return lo + (int32_t)(((h >> 32) * (uint64_t)(hi - lo + 1)) >> 32);
}

// World table and grids.  Every world lives in its own range [off, off +
// side^2) of the cell arena; pos and target are arena indices.  Each slot has
// its own seed, step index and move count, so a world evolves exactly as it
// would alone.
// A cell's sugar is one byte, its low seven bits the amount and the top bit
// the occupancy (kOccupied), so that a row of the cells an agent looks at is
// one load and the grid of a 2048^2 world (4 MB) stays in an XCD's L2.  Which
// agent stands in a cell is in the agents alone (a grid of handles beside the
// bits cost every move two scattered stores, and only the readout used it).
// Amounts and capacities are 0..kMaxSugar.
constexpr int32_t kOccupied = 0x80;
constexpr int32_t kMaxSugar = 0x7F;
__device__ __forceinline__ int32_t sugar_of(int32_t w) { return w & kMaxSugar; }

struct Grid {
  uint8_t* sugar;     // sugar | kOccupied when an agent stands there
  uint8_t* cap;
  uint8_t* req;       // request of the agent standing there in this step (request_code), 0: none
  uint32_t* breq;     // lowest cell index requesting a birth there or kInf
  uint32_t* w_off;    // per slot
  uint32_t* w_side;
  uint64_t* w_seed;
  uint32_t* w_step;   // index of the step in progress
  uint64_t* w_moves;  // per slot, kMoveShards counters
  uint32_t arena;
  uint32_t max_worlds;
  int32_t max_age, repro_min, fertile_min, fertile_max;
};

constexpr uint32_t kMoveShards = 64;

template <class F, class H>
__device__ __forceinline__ F& af(const H& h, uint32_t self, uint32_t field) {
  return *field_ptr<F>(h, self, kAgent, field);
}

struct Where {
  uint32_t off;
  int32_t side, x, y;
};

__device__ __forceinline__ Where where(const Grid& g, uint32_t wid, uint32_t p) {
  const uint32_t off = g.w_off[wid], side = g.w_side[wid];
  const uint32_t local = p - off;
  return Where{off, (int32_t)side, (int32_t)(local % side), (int32_t)(local / side)};
}

constexpr int32_t kMaxVision = 6;

// Move request k cells along direction d (0 .. 3: x up, x down, y up, y down).
constexpr uint32_t request_code(uint32_t d, uint32_t k) { return 1u + d * kMaxVision + (k - 1u); }

// Byte planes (sugar, capacity, requests) keep a world's rows in groups of
// four, each group column by column (the last group of a side that is not a
// multiple of four has the rows that are left), so a world takes the same
// side^2 bytes as its cells and byte [off, off + side^2) of each plane.  Four
// cells of a column are then a dword and a 128-byte line holds 32 x 4 cells:
// the row and the column that an agent sees are 8 loads from about 5 lines
// (row by row: 13 loads from as many lines, and once the agents of a wavefront
// are scattered over the torus, lines are what the L2s deliver a limited
// number of).
__device__ __forceinline__ uint32_t byte_at(const Where& c, int32_t x, int32_t y) {
  const uint32_t side = (uint32_t)c.side, r = (uint32_t)y & 3u, g = (uint32_t)y - r;
  return c.off + g * side + (uint32_t)x * (g + 4u <= side ? 4u : side & 3u) + r;
}
__device__ __forceinline__ uint32_t byte_here(const Where& c) { return byte_at(c, c.x, c.y); }
// v around the torus, for v at most kMaxVision outside: two selects, and a loop
// that only sides below the vision enter (remainders here made Choose 73 KB of
// code and MoveEat 96, loops alone made worlds of 64^2 13 % slower).
__device__ __forceinline__ int32_t wrapped(int32_t v, int32_t side) {
  v += v < 0 ? side : 0;
  v -= v >= side ? side : 0;
  if (__builtin_expect(side < kMaxVision, 0)) {
    while (v < 0) v += side;
    while (v >= side) v -= side;
  }
  return v;
}

// The cells that an agent at c sees (of a byte plane): col[i] at (x, y + i -
// kMaxVision), row[i] at (x + i - kMaxVision, y), around the torus.
constexpr int32_t kSeen = 2 * kMaxVision + 1;
__device__ __forceinline__ void cross(const uint8_t* plane, const Where& c, uint32_t (&col)[kSeen],
                                      uint32_t (&row)[kSeen]) {
  const int32_t full = c.side & ~3;  // rows in whole groups
  if (c.y >= kMaxVision && c.y + kMaxVision < full) {
    // 13 rows from row y - 6 on lie in the four groups from that row's on.
    const uint32_t y0 = (uint32_t)(c.y - kMaxVision), sh = y0 & 3u;
    const uint8_t* b = plane + c.off + (y0 - sh) * (uint32_t)c.side + 4u * (uint32_t)c.x;
    uint32_t d[4];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) __builtin_memcpy(&d[i], b + i * 4u * (uint32_t)c.side, 4);
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      const uint32_t w = __builtin_amdgcn_alignbyte(i < 3 ? d[i + 1] : 0u, d[i], sh);
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e)
        if (4 * i + e < (uint32_t)kSeen) col[4 * i + e] = (w >> (8 * e)) & 0xFFu;
    }
  } else {
#pragma unroll
    for (int32_t i = 0; i < kSeen; ++i) col[i] = plane[byte_at(c, c.x, wrapped(c.y + i - kMaxVision, c.side))];
  }
  if (c.x >= kMaxVision && c.x + kMaxVision < c.side && c.y < full) {
    const uint32_t r = (uint32_t)c.y & 3u;
    const uint8_t* b = plane + c.off + ((uint32_t)c.y - r) * (uint32_t)c.side + 4u * (uint32_t)(c.x - kMaxVision);
    uint32_t d[kSeen];
    __builtin_memcpy(d, b, sizeof(d));
#pragma unroll
    for (int32_t i = 0; i < kSeen; ++i) row[i] = (d[i] >> (8 * r)) & 0xFFu;
  } else {
#pragma unroll
    for (int32_t i = 0; i < kSeen; ++i) row[i] = plane[byte_at(c, wrapped(c.x + i - kMaxVision, c.side), c.y)];
  }
}

// Index of the cell k steps along direction d (0 .. 3) from c, whose index is p.
__device__ __forceinline__ uint32_t seen_cell(const Where& c, uint32_t p, uint32_t d, int32_t k) {
  const int32_t n = d & 1u ? -k : k;
  return d < 2 ? p + (uint32_t)(wrapped(c.x + n, c.side) - c.x) : p + (uint32_t)((wrapped(c.y + n, c.side) - c.y) * c.side);
}

struct Choose {
  static constexpr uint32_t kKind = 40;
  static constexpr bool kXcdRuns = true;
  using Args = Grid;
  // The best of the cells in sight: most sugar, then nearest, then lowest
  // index.  The order in which the candidates are compared does not matter
  // for that total order.  Bound: scattered lines and addresses; with a load
  // per cell from rows and an atomic minimum per request 82 us for 1.05 M
  // agents, now 50.
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& g) {
    const uint32_t p = af<uint32_t>(h, self, kPos);
    const int32_t vision = af<int32_t>(h, self, kVision);
    const Where c = where(g, af<uint32_t>(h, self, kWorld), p);
    uint32_t col[kSeen], row[kSeen];
    cross(g.sugar, c, col, row);
    uint32_t best = p, best_key = ((uint32_t)sugar_of((int32_t)row[kMaxVision]) << 3) | 7u, code = 0;
#pragma unroll
    for (int32_t k = 1; k <= kMaxVision; ++k)
#pragma unroll
      for (uint32_t d = 0; d < 4; ++d) {
        const uint32_t v = (d < 2 ? row : col)[kMaxVision + (d & 1u ? -k : k)];
        const uint32_t key = (v << 3) | (uint32_t)(7 - k);
        if (k > vision || (v & kOccupied) || key < best_key) continue;
        const uint32_t q = seen_cell(c, p, d, k);
        if (key > best_key || q < best) {
          best = q;
          best_key = key;
          code = request_code(d, (uint32_t)k);
        }
      }
    af<uint32_t>(h, self, kTarget) = best;
    if (best != p) g.req[byte_here(c)] = (uint8_t)code;
    return false;
  }
};

// Move and eat.  The agents that may want cell q stand within kMaxVision of it
// along the axes, and each one's request in its own cell says which cell it
// wants, so a mover reads those 24 cells (8 loads) instead of all requesters
// meeting in an atomic minimum per target, whose 4-byte words cost every mover
// an atomic, a load and a reset beyond the L2.  119 us as two do-alls (Choose
// 82), 84 fused (Choose 68), 90 with the requests (Choose 50).
struct MoveEat {
  static constexpr uint32_t kKind = 42;
  static constexpr bool kXcdRuns = true;
  static constexpr uint32_t kPhases = 2;
  static constexpr uint32_t kMinWaves = 8;
  static constexpr bool kDeletesOnlyThis = true;
  using Args = Grid;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& g) {
    const uint32_t p = af<uint32_t>(h, self, kPos);
    const uint32_t q = af<uint32_t>(h, self, kTarget);
    const uint32_t wid = af<uint32_t>(h, self, kWorld);
    const Where from = where(g, wid, p), to = where(g, wid, q);
    const uint32_t bp = byte_here(from), bq = byte_here(to);
    const int32_t here = g.sugar[bp], there = g.sugar[bq];
    const int32_t had = af<int32_t>(h, self, kSugar), metab = af<int32_t>(h, self, kMetab);
    const int32_t age = af<int32_t>(h, self, kAge) + 1;
    bool moves = q != p;
    if (moves) {
      uint32_t col[kSeen], row[kSeen];
      cross(g.req, to, col, row);
      // A requester k cells from q, whose direction leads to q, wins over this
      // agent from a cell r < p.
#pragma unroll
      for (int32_t k = 1; k <= kMaxVision; ++k)
#pragma unroll
        for (uint32_t d = 0; d < 4; ++d)
          if ((d < 2 ? row : col)[kMaxVision + (d & 1u ? -k : k)] == request_code(d ^ 1u, (uint32_t)k) &&
              seen_cell(to, q, d, k) < p)
            moves = false;
    }
    const uint32_t at_cell = moves ? bq : bp;
    if (moves) g.sugar[bp] = (uint8_t)sugar_of(here);  // distinct cells per mover: q was empty and p occupied
    // Count moves per world: one sharded atomic per world present in the wavefront.
    uint64_t pending = __ballot(moves);
    const uint32_t sh = (blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) & (kMoveShards - 1);
    while (pending) {
      const uint32_t w0 = __builtin_amdgcn_readlane(wid, (uint32_t)__builtin_ctzll(pending));
      const uint64_t mine = __ballot(moves && wid == w0);
      lead_add(g.w_moves + (uint64_t)w0 * kMoveShards + sh, (uint64_t)__popcll(mine));
      pending &= ~mine;
    }
    const int32_t sugar = had + sugar_of(moves ? there : here) - metab;
    if (sugar <= 0 || age >= g.max_age) {
      g.sugar[at_cell] = 0;
      return true;  // delete this; its fields are not written
    }
    g.sugar[at_cell] = kOccupied;  // eaten, still here
    if (moves) af<uint32_t>(h, self, kPos) = q;
    af<int32_t>(h, self, kSugar) = sugar;
    af<int32_t>(h, self, kAge) = age;
    return false;
  }
};

struct Request {
  static constexpr uint32_t kKind = 43;
  static constexpr bool kXcdRuns = true;
  using Args = Grid;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& g) {
    const int32_t sugar = af<int32_t>(h, self, kSugar), age = af<int32_t>(h, self, kAge);
    uint32_t best = kNull;
    if (sugar >= g.repro_min && age >= g.fertile_min && age <= g.fertile_max) {
      const uint32_t p = af<uint32_t>(h, self, kPos);
      const Where c = where(g, af<uint32_t>(h, self, kWorld), p);
      uint32_t occ[4];
#pragma unroll
      for (uint32_t d = 0; d < 4; ++d) {
        const int32_t n = d & 1u ? -1 : 1;
        const int32_t x = d < 2 ? wrapped(c.x + n, c.side) : c.x, y = d < 2 ? c.y : wrapped(c.y + n, c.side);
        occ[d] = g.sugar[byte_at(c, x, y)];
      }
#pragma unroll
      for (uint32_t d = 0; d < 4; ++d) {
        const uint32_t q = seen_cell(c, p, d, 1);
        if (!(occ[d] & kOccupied) && q < best) best = q;
      }
      if (best != kNull) atomicMin(g.breq + best, p);
    }
    af<uint32_t>(h, self, kTarget) = best;
    wave_count(h, kCntMethodAtomics, best != kNull ? 1u : 0u);
    return false;
  }
};

// What a child is made from (inverted words: they are left in LDS, where later
// kernels read search hints): its cell and the cell's byte in the planes, its
// world and its sugar.  The byte's place is found before the request: after it,
// it is two more rounds of loads at the end of the step's longest chain.
struct Child {
  uint32_t not_n, not_b, not_wid, not_give;
};

// The winners' children are queued, so a wavefront's entries share one chain
// of allocation atomics (50 -> 38 us for 1.05 M agents of 2048^2).
struct Birth {
  static constexpr uint32_t kKind = 44;
  static constexpr bool kXcdRuns = true;
  static constexpr uint32_t kMinWaves = 8;
  using Args = Grid;
  using Item = Child;
  static constexpr uint32_t kItemType = kAgent;
  static constexpr uint32_t kItems = 128, kClaimBits = 2;
  struct Found {
    uint32_t claims;  // bit u: object u gives birth
    uint32_t n[2], b[2], wid[2], give[2];
  };
  template <uint32_t N, class H>
  static __device__ __forceinline__ void find(const H& h, uint32_t, const uint32_t (&self)[2], const bool (&lv)[2],
                                              const Args& g, Found& found, bool (&)[2]) {
    uint32_t p[N], asked[N];
    bool asks[N];
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
      found.n[u] = af<uint32_t>(h, self[u], kTarget);
      p[u] = af<uint32_t>(h, self[u], kPos);
      found.wid[u] = af<uint32_t>(h, self[u], kWorld);
      asks[u] = lv[u] && found.n[u] != kNull;
    }
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
      asked[u] = kNull;
      if (!asks[u]) continue;
      asked[u] = __hip_atomic_load(g.breq + found.n[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      found.b[u] = byte_here(where(g, found.wid[u], found.n[u]));
    }
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
      if (!asks[u] || asked[u] != p[u]) continue;
      const int32_t sugar = af<int32_t>(h, self[u], kSugar), give = sugar / 2;
      found.give[u] = (uint32_t)give;
      af<int32_t>(h, self[u], kSugar) = sugar - give;
      __hip_atomic_store(g.breq + found.n[u], kInf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      found.claims |= 1u << u;
    }
  }
  static __device__ __forceinline__ Item item(const Found& f, uint32_t b) {
    return {~(b ? f.n[1] : f.n[0]), ~(b ? f.b[1] : f.b[0]), ~(b ? f.wid[1] : f.wid[0]), ~(b ? f.give[1] : f.give[0])};
  }
  template <class H>
  static __device__ __forceinline__ void make(const H& h, const Args& g, const Item& it, uint32_t o) {
    const uint32_t n = ~it.not_n, b = ~it.not_b, wid = ~it.not_wid;
    const uint64_t seed = g.w_seed[wid];
    const uint32_t t = g.w_step[wid], local = n - g.w_off[wid];
    af<int32_t>(h, o, kSugar) = (int32_t)~it.not_give;
    af<int32_t>(h, o, kMetab) = uniform_int(hash4(seed, kStreamChildMetab, t, local), 1, 4);
    af<int32_t>(h, o, kVision) = uniform_int(hash4(seed, kStreamChildVision, t, local), 1, 6);
    af<int32_t>(h, o, kAge) = 0;
    af<uint32_t>(h, o, kPos) = n;
    af<uint32_t>(h, o, kTarget) = kNull;
    af<uint32_t>(h, o, kWorld) = wid;
    g.sugar[b] = (uint8_t)(g.sugar[b] | kOccupied);
  }
};

struct SugarDeleteWorld {
  static constexpr uint32_t kKind = 45;
  struct Args { uint32_t slot; };
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    return af<uint32_t>(h, self, kWorld) == a.slot;
  }
};

// Regrow every arena cell, 16 per lane, clear its move request, and advance
// every slot's step index (read by the births of this step).  Cells outside resident worlds (and the
// bytes up to the next multiple of 16) are rewritten at admission, so
// regrowing them is harmless.  Bound: the three byte planes' bandwidth (capacities
// of four bytes and one cell per lane took 6.1 us for 2048^2 cells).
__global__ void regrow_kernel(Grid g) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < g.max_worlds) g.w_step[i] += 1;
  uint4* const sv = reinterpret_cast<uint4*>(g.sugar);
  uint4* const rv = reinterpret_cast<uint4*>(g.req);
  const uint4* const cv = reinterpret_cast<const uint4*>(g.cap);
  for (uint32_t c = i; c < (g.arena + 15) / 16; c += gridDim.x * blockDim.x) {
    const uint4 w = sv[c], k = cv[c];
    const uint32_t win[4] = {w.x, w.y, w.z, w.w}, kin[4] = {k.x, k.y, k.z, k.w};
    uint32_t out[4];
#pragma unroll
    for (uint32_t d = 0; d < 4; ++d) {
      const uint32_t grown = (win[d] & 0x7F7F7F7Fu) + 0x01010101u;  // at most 0x80 per byte
      out[d] = win[d] & 0x80808080u;
#pragma unroll
      for (uint32_t e = 0; e < 32; e += 8) {
        const uint32_t a = (grown >> e) & 0xFFu, b = (kin[d] >> e) & 0xFFu;
        out[d] |= (a < b ? a : b) << e;
      }
    }
    sv[c] = make_uint4(out[0], out[1], out[2], out[3]);
    rv[c] = make_uint4(0, 0, 0, 0);
  }
}

__global__ void set_world_kernel(Grid g, uint32_t slot, uint32_t off, uint32_t side, uint64_t seed, uint32_t step0) {
  const uint32_t i = threadIdx.x;
  if (i == 0) {
    g.w_off[slot] = off;
    g.w_side[slot] = side;
    g.w_seed[slot] = seed;
    g.w_step[slot] = step0 - 1;  // the first regrow advances it to step0
  }
  if (i < kMoveShards) g.w_moves[(uint64_t)slot * kMoveShards + i] = 0;
}

// Admission input check: *bad = 1 if any cell's sugar or capacity lies
// outside 0..kMaxSugar (a cell keeps both in seven bits).
__global__ void sugar_zero_kernel(uint32_t* bad) { *bad = 0; }
__global__ void sugar_check_kernel(const int32_t* sugar, const int32_t* cap, uint32_t n, uint32_t* bad) {
  bool out = false;
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x)
    out |= sugar[c] < 0 || sugar[c] > kMaxSugar || cap[c] < 0 || cap[c] > kMaxSugar;
  if (__ballot(out) && is_first_active()) *bad = 1;
}

// Admits a world: a lane takes a column of a group of four rows (the last group
// has the rows that are left), so its plane bytes are a dword, each row's loads
// are coalesced, and one request of a wavefront serves 256 cells (with a cell
// per lane 1010 us for 2048^2 cells with 1.05 M agents, now 850).  Bound: the
// chains of lookups, as the requests crowd into the same active blocks (565 with
// the bounded policy, which would leave more blocks half full).
// Below kAdmitWideMin cells a lane takes one cell: the agents then stand in more
// blocks, whose room the births of the first steps find without a free block.
// Admission and step, us, one row and four (a quarter of the cells occupied):
//   128^2  19 38.4   30 40.7     362^2  42 47.0   34 48.1
//   256^2  32 41.7   29 47.0     430^2  27 53.5   30 50.0
constexpr uint32_t kAdmitWideMin = 1u << 17;
template <uint32_t LG, uint32_t ROWS>
__global__ void sugar_admit_kernel(DevHeapW<LG> h, Grid g, uint32_t slot, uint32_t off, uint32_t side, const int32_t* sugar,
                                   const int32_t* cap, const uint8_t* occ, const int32_t* as, const int32_t* am,
                                   const int32_t* av, const int32_t* aa) {
  const uint32_t i = creation_wg(h) * blockDim.x + threadIdx.x;
  const uint32_t group = i / side, x = i - group * side, y = ROWS * group;
  if (y >= side) return;
  const uint32_t rows = side - y < ROWS ? side - y : ROWS;
  const uint32_t c0 = y * side + x, b = byte_at(Where{off, (int32_t)side, 0, 0}, (int32_t)x, (int32_t)y);
  uint32_t amount = 0, most = 0, here = 0;
#pragma unroll
  for (uint32_t r = 0; r < ROWS; ++r) {
    if (r >= rows) continue;
    const uint32_t c = c0 + r * side;
    amount |= (uint32_t)sugar[c] << (8 * r);  // checked to be 0..kMaxSugar before the launch
    most |= (uint32_t)cap[c] << (8 * r);
    here |= occ[c] ? 1u << r : 0u;
    g.breq[off + c] = kInf;
  }
#pragma unroll
  for (uint32_t r = 0; r < ROWS; ++r) {
    if (r >= rows) continue;
    g.sugar[b + r] = (uint8_t)(amount >> (8 * r));
    g.cap[b + r] = (uint8_t)(most >> (8 * r));
  }
  new_many(h, kAgent, (uint32_t)__popc(here), [&](uint32_t k, uint32_t o) __attribute__((always_inline)) {
    if (o == kNull) return;
    uint32_t m = here;
    for (; k > 0; --k) m &= m - 1u;
    const uint32_t r = (uint32_t)__builtin_ctz(m), c = c0 + r * side;
    af<int32_t>(h, o, kSugar) = as[c];
    af<int32_t>(h, o, kMetab) = am[c];
    af<int32_t>(h, o, kVision) = av[c];
    af<int32_t>(h, o, kAge) = aa[c];
    af<uint32_t>(h, o, kPos) = off + c;
    af<uint32_t>(h, o, kTarget) = kNull;
    af<uint32_t>(h, o, kWorld) = slot;
    g.sugar[b + r] = (uint8_t)((amount >> (8 * r)) | kOccupied);
  });
}

// Readout of one world: which agent stands in a cell is in the agents alone, so
// wavefronts go through the heap's agents, four blocks per unit (a lane takes the
// allocated bits of one unit, so a wavefront sees 64 units per round), and those
// of the world write their fields to its cells.  Beside them, in the same launch,
// the first cell_wgs workgroups write the cells' sugar and occupancy, and zeros
// where no agent stands.  From kReadWideMin cells on (kHandles) the agents write
// their handles only, into the caller's a_sugar, and a second launch takes the
// fields from there, cell by cell: fields stored one by one from many wavefronts
// are part lines.  us per call, with an enumeration, a do-all and a clearing
// kernel, in one launch and in two:
//   64^2 alone           13.6   5.8   7.7     1024^2 alone           29.5  18.2  15.9
//   128^2, one of 256    15.0   5.7   8.2     2048^2 alone           61    56    41
//   384^2, one of 8      14.8   6.8   9.0     512^2, one of 64       22.9  16.9  14.9
// (a call on small worlds cannot take less than 5.7: the launch).
constexpr uint32_t kKindSugarRead = 48;
constexpr uint32_t kReadUnit = 4;
constexpr uint32_t kReadWideMin = 1u << 18;
struct ReadOut {
  uint32_t slot, off, n;
  int32_t* sugar;
  uint8_t* occ;
  int32_t *a_sugar, *a_metab, *a_vision, *a_age;
};

template <uint32_t LG, bool kHandles>
__global__ void __launch_bounds__(256) sugar_read_kernel(DevHeapW<LG> h, Grid g, ReadOut o, uint32_t cell_wgs) {
  if (blockIdx.x < cell_wgs) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= o.n) return;
    const int32_t v = g.sugar[byte_here(where(g, o.slot, o.off + c))];
    o.sugar[c] = sugar_of(v);
    o.occ[c] = (v & kOccupied) ? 1 : 0;
    if (!(v & kOccupied)) o.a_sugar[c] = o.a_metab[c] = o.a_vision[c] = o.a_age[c] = 0;
    return;
  }
  const uint32_t lane = lane_id(), wpb = blockDim.x >> 6, waves = (gridDim.x - cell_wgs) * wpb;
  const uint32_t wave = (blockIdx.x - cell_wgs) * wpb + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Bitmap allocated = allocated_bm(h, kAgent);
  const uint32_t units = (h.num_blocks + kReadUnit - 1) / kReadUnit;
  const uint32_t c = cap_of(h, kAgent), sh = (uint32_t)__builtin_ctz(c), bpw = 64u >> sh;  // blocks per wavefront
  const uint32_t sub = lane >> sh, slot = lane & (c - 1u);
  for (uint64_t u0 = wave; u0 < units; u0 += 64ull * waves) {
    // The first unit's object bitmaps are on their way before its allocated bits are known.
    const uint32_t ahead = (uint32_t)u0 * kReadUnit + lane;
    const uint64_t early = lane < kReadUnit && ahead < h.num_blocks ? meta_load(h.obj_bitmap + ahead) : 0ull;
    const uint64_t mine = u0 + (uint64_t)lane * waves;
    uint32_t have = 0;
    if (mine < units) have = (uint32_t)(meta_load(allocated.group((uint32_t)(mine >> 4))) >> (kReadUnit * (mine & 15u))) & 15u;
    uint64_t todo = __ballot(have != 0);
    while (todo) {
      const uint32_t l = (uint32_t)__builtin_ctzll(todo);
      todo &= todo - 1ull;
      const uint32_t first = ((uint32_t)u0 + l * waves) * kReadUnit, bits = (uint32_t)__builtin_amdgcn_readlane(have, l);
      uint64_t mask = 0;
      if (lane < kReadUnit && ((bits >> lane) & 1u)) mask = l == 0 ? early : meta_load(h.obj_bitmap + first + lane);
      uint32_t self[kReadUnit], world[kReadUnit];
#pragma unroll
      for (uint32_t i = 0; i < kReadUnit; ++i) {
        const uint32_t j = i * bpw + sub;
        const uint64_t m = __shfl(mask, (int)(j & 63u));
        self[i] = make_obj(first + j, slot);
        world[i] = kNull;
        if (j < kReadUnit && ((m >> slot) & 1ull)) world[i] = af<uint32_t>(h, self[i], kWorld);
      }
#pragma unroll
      for (uint32_t i = 0; i < kReadUnit; ++i) {
        if (world[i] != o.slot) continue;
        const uint32_t at = af<uint32_t>(h, self[i], kPos) - o.off;
        if (kHandles) {
          if (at < o.n) o.a_sugar[at] = (int32_t)self[i];
          continue;
        }
        const int32_t sugar = af<int32_t>(h, self[i], kSugar), metab = af<int32_t>(h, self[i], kMetab);
        const int32_t vision = af<int32_t>(h, self[i], kVision), age = af<int32_t>(h, self[i], kAge);
        if (at >= o.n) continue;
        o.a_sugar[at] = sugar;
        o.a_metab[at] = metab;
        o.a_vision[at] = vision;
        o.a_age[at] = age;
      }
    }
  }
}

__global__ void sugar_read_cells_kernel(DevHeap h, Grid g, ReadOut o) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= o.n) return;
  const int32_t v = g.sugar[byte_here(where(g, o.slot, o.off + c))];
  const uint32_t self = (uint32_t)o.a_sugar[c];  // no handle where no agent stands
  const bool here = (v & kOccupied) && (self >> 6) < h.num_blocks && (self & 63u) < cap_of(h, kAgent);
  o.sugar[c] = sugar_of(v);
  o.occ[c] = (v & kOccupied) ? 1 : 0;
  o.a_sugar[c] = here ? af<int32_t>(h, self, kSugar) : 0;
  o.a_metab[c] = here ? af<int32_t>(h, self, kMetab) : 0;
  o.a_vision[c] = here ? af<int32_t>(h, self, kVision) : 0;
  o.a_age[c] = here ? af<int32_t>(h, self, kAge) : 0;
}

bool sugar_heap_ok(const dsoar_heap* h) {
  const dsoar_type_layout& L = h->desc.types[0];
  if (L.num_fields < 7) return false;
  for (uint32_t f = 0; f < 7; ++f)
    if (L.field_bytes[f] != 4) return false;
  return true;
}

}  // namespace
}  // namespace dsoar

using namespace dsoar;

struct dsoar_sugar {
  dsoar_heap* heap;
  Grid g;
  uint32_t* bad_input;  // device word: admission input outside 0..kMaxSugar
  uint64_t default_seed;
  uint32_t* h_off;
  uint32_t* h_side;
  uint8_t* live;
  StepGraphs graphs;
};

namespace {

int sugar_one_step(dsoar_sugar* s, uint32_t flags, hipStream_t st) {
  dsoar_heap* h = s->heap;
  const uint32_t base = flags & DSOAR_DO_PLAIN;
  const uint32_t slots = (s->g.max_worlds + 255) / 256, cells = (s->g.arena + 4095) / 4096;  // workgroups
  const uint32_t grid = std::max(slots, std::min(cells, h->num_cus * 16));
  launch_timed(s->heap, kKindSugarRegrow, regrow_kernel, dim3(grid), dim3(256), st, s->g);
  DSOAR_LAUNCHED(h);
  int rc = launch_doall<Choose>(h, kAgent, s->g, base, st);
  // choose creates and deletes nothing: move and eat reuse the list.
  if (!rc) rc = launch_doall<MoveEat>(h, kAgent, s->g, base | DSOAR_DO_REUSE_ENUM, st);
  // eat deletes: the request phase enumerates again; birth reuses that list.
  if (!rc) rc = launch_doall<Request>(h, kAgent, s->g, base, st);
  if (!rc) rc = launch_doall<Birth>(h, kAgent, s->g, base | DSOAR_DO_REUSE_ENUM, st);
  return rc;
}

size_t plane_bytes(uint64_t cells) { return (size_t)((cells * 4 + 255) / 256 * 256); }
// A plane of one byte per cell, with 16 bytes past the last that a row window
// or a regrowing lane may touch.
size_t byte_plane_bytes(uint64_t cells) { return (size_t)((cells + 16 + 255) / 256 * 256); }

// World table: seeds, offsets, sides, steps; the move counters; one 256-byte
// line for the admission input check.
size_t table_bytes(uint32_t max_worlds) {
  return (size_t)(((uint64_t)max_worlds * (4 + 4 + 8 + 4) + 255) / 256 * 256 +
                  ((uint64_t)max_worlds * kMoveShards * 8 + 255) / 256 * 256 + 256);
}

}  // namespace

extern "C" {

size_t dsoar_sugarpool_bytes(uint32_t max_worlds, uint32_t arena_cells) {
  if (max_worlds == 0 || max_worlds > (1u << 16) || arena_cells == 0 || arena_cells > (1u << 30)) return 0;
  return table_bytes(max_worlds) + 3 * byte_plane_bytes(arena_cells) + plane_bytes(arena_cells);
}

int dsoar_sugarpool_create(dsoar_heap* heap, uint32_t max_worlds, uint32_t arena_cells,
                           const dsoar_sugar_rules* rules, void* dev_mem, size_t dev_bytes, dsoar_sugar** out) {
  if (!out) return DSOAR_ERR_INVALID_ARG;
  *out = nullptr;
  if (!heap_ok(heap) || !sugar_heap_ok(heap) || !rules || !dev_mem || ((uintptr_t)dev_mem & 255u))
    return DSOAR_ERR_INVALID_ARG;
  const size_t need = dsoar_sugarpool_bytes(max_worlds, arena_cells);
  if (need == 0) return DSOAR_ERR_INVALID_ARG;
  if (dev_bytes < need) return DSOAR_ERR_TOO_SMALL;
  dsoar_sugar* s = new (std::nothrow) dsoar_sugar;
  if (!s) return DSOAR_ERR_INVALID_ARG;
  memset(s, 0, sizeof(*s));
  s->heap = heap;
  s->default_seed = rules->seed;
  s->h_off = (uint32_t*)calloc(max_worlds, 4);
  s->h_side = (uint32_t*)calloc(max_worlds, 4);
  s->live = (uint8_t*)calloc(max_worlds, 1);
  if (!s->h_off || !s->h_side || !s->live) {
    free(s->h_off);
    free(s->h_side);
    free(s->live);
    delete s;
    return DSOAR_ERR_INVALID_ARG;
  }
  uint8_t* b = (uint8_t*)dev_mem;
  Grid& g = s->g;
  g.w_seed = (uint64_t*)b;                                   // 8-byte entries first
  g.w_off = (uint32_t*)(b + (uint64_t)max_worlds * 8);
  g.w_side = g.w_off + max_worlds;
  g.w_step = g.w_side + max_worlds;
  g.w_moves = (uint64_t*)(b + ((uint64_t)max_worlds * 20 + 255) / 256 * 256);
  s->bad_input = (uint32_t*)(b + table_bytes(max_worlds) - 256);
  uint8_t* planes = b + table_bytes(max_worlds);
  const uint64_t bytes = byte_plane_bytes(arena_cells);
  g.sugar = planes;
  g.cap = planes + bytes;
  g.req = planes + 2 * bytes;
  g.breq = (uint32_t*)(planes + 3 * bytes);
  g.arena = arena_cells;
  g.max_worlds = max_worlds;
  g.max_age = rules->max_age;
  g.repro_min = rules->repro_min;
  g.fertile_min = rules->fertile_min;
  g.fertile_max = rules->fertile_max;
  *out = s;
  return DSOAR_OK;
}

int dsoar_sugar_admit(dsoar_sugar* s, uint32_t slot, uint32_t cell_offset, uint32_t side, uint64_t seed,
                      uint32_t step0, const int32_t* sugar_dev, const int32_t* cap_dev, const uint8_t* occ_dev,
                      const int32_t* a_sugar_dev, const int32_t* a_metab_dev, const int32_t* a_vision_dev,
                      const int32_t* a_age_dev, void* stream) {
  if (!s || slot >= s->g.max_worlds || s->live[slot] || side == 0 || side > 32768 || !sugar_dev || !cap_dev ||
      !occ_dev || !a_sugar_dev || !a_metab_dev || !a_vision_dev || !a_age_dev)
    return DSOAR_ERR_INVALID_ARG;
  const uint64_t n = (uint64_t)side * side;
  if ((uint64_t)cell_offset + n > s->g.arena) return DSOAR_ERR_INVALID_ARG;
  for (uint32_t k = 0; k < s->g.max_worlds; ++k)
    if (s->live[k] && cell_offset < s->h_off[k] + (uint64_t)s->h_side[k] * s->h_side[k] && s->h_off[k] < cell_offset + n)
      return DSOAR_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  // Sugar and capacities outside the seven bits a cell keeps them in are
  // refused before anything of the pool changes (synchronises the stream).
  hipLaunchKernelGGL(sugar_zero_kernel, dim3(1), dim3(1), 0, st, s->bad_input);
  DSOAR_LAUNCHED(s->heap);
  hipLaunchKernelGGL(sugar_check_kernel, dim3((uint32_t)std::min<uint64_t>((n + 255) / 256, 4096)), dim3(256), 0, st,
                     sugar_dev, cap_dev, (uint32_t)n, s->bad_input);
  DSOAR_LAUNCHED(s->heap);
  uint32_t bad = 0;
  DSOAR_HIP(s->heap, hipMemcpyAsync(&bad, s->bad_input, 4, hipMemcpyDeviceToHost, st));
  DSOAR_HIP(s->heap, hipStreamSynchronize(st));
  if (bad) return DSOAR_ERR_INVALID_ARG;
  hipLaunchKernelGGL(set_world_kernel, dim3(1), dim3(kMoveShards), 0, st, s->g, slot, cell_offset, side, seed, step0);
  DSOAR_LAUNCHED(s->heap);
  const uint32_t rows = n >= kAdmitWideMin ? 4u : 1u;
  const uint64_t columns = (uint64_t)((side + rows - 1) / rows) * side;
  with_width(s->heap, [&](auto w_) {
    constexpr uint32_t kLG = decltype(w_)::value;
    auto go = [&](auto kernel) {
      launch_timed(s->heap, kKindSugarAdmit, kernel, dim3((uint32_t)((columns + 255) / 256)), dim3(256), st,
                   DevHeapW<kLG>(s->heap->dev), s->g, slot, cell_offset, side, sugar_dev, cap_dev, occ_dev, a_sugar_dev,
                   a_metab_dev, a_vision_dev, a_age_dev);
    };
    if (rows == 4) go(sugar_admit_kernel<kLG, 4>);
    else go(sugar_admit_kernel<kLG, 1>);
  });
  DSOAR_LAUNCHED(s->heap);
  s->h_off[slot] = cell_offset;
  s->h_side[slot] = side;
  s->live[slot] = 1;
  return DSOAR_OK;
}

int dsoar_sugar_retire(dsoar_sugar* s, uint32_t slot, void* stream) {
  if (!s || slot >= s->g.max_worlds || !s->live[slot]) return DSOAR_ERR_INVALID_ARG;
  const int rc = launch_doall<SugarDeleteWorld>(s->heap, kAgent, SugarDeleteWorld::Args{slot}, 0, (hipStream_t)stream);
  if (rc) return rc;
  s->live[slot] = 0;
  return DSOAR_OK;
}

int dsoar_sugar_read_world(dsoar_sugar* s, uint32_t slot, int32_t* sugar_dev, uint8_t* occ_dev, int32_t* a_sugar_dev,
                           int32_t* a_metab_dev, int32_t* a_vision_dev, int32_t* a_age_dev, uint64_t* moves,
                           void* stream) {
  if (!s || slot >= s->g.max_worlds || !s->live[slot] || !sugar_dev || !occ_dev || !a_sugar_dev || !a_metab_dev ||
      !a_vision_dev || !a_age_dev)
    return DSOAR_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  const uint32_t n = s->h_side[slot] * s->h_side[slot];
  const ReadOut r{slot, s->h_off[slot], n, sugar_dev, occ_dev, a_sugar_dev, a_metab_dev, a_vision_dev, a_age_dev};
  const bool handles = n >= kReadWideMin;
  const uint32_t cells = (n + 255) / 256, units = (s->heap->dev.num_blocks + kReadUnit - 1) / kReadUnit;
  const uint32_t cell_wgs = handles ? 0u : cells, agent_wgs = std::min((units + 3) / 4, s->heap->num_cus * 8);
  with_width(s->heap, [&](auto w_) {
    constexpr uint32_t kLG = decltype(w_)::value;
    auto go = [&](auto kernel) {
      launch_timed(s->heap, kKindSugarRead, kernel, dim3(cell_wgs + agent_wgs), dim3(256), st, DevHeapW<kLG>(s->heap->dev),
                   s->g, r, cell_wgs);
    };
    if (handles) go(sugar_read_kernel<kLG, true>);
    else go(sugar_read_kernel<kLG, false>);
  });
  if (handles)
    launch_timed(s->heap, kKindSugarRead, sugar_read_cells_kernel, dim3(cells), dim3(256), st, s->heap->dev, s->g, r);
  DSOAR_LAUNCHED(s->heap);
  if (moves) {
    uint64_t m[kMoveShards];
    DSOAR_HIP(s->heap, hipMemcpyAsync(m, s->g.w_moves + (uint64_t)slot * kMoveShards, sizeof(m), hipMemcpyDeviceToHost, st));
    DSOAR_HIP(s->heap, hipStreamSynchronize(st));
    uint64_t t = 0;
    for (uint32_t i = 0; i < kMoveShards; ++i) t += m[i];
    *moves = t;
  }
  return DSOAR_OK;
}

// Single-world interface: a pool of one slot covering the whole arena.
size_t dsoar_sugar_bytes(uint32_t side) {
  if (side < 1 || side > 32768) return 0;
  return dsoar_sugarpool_bytes(1, side * side);
}

int dsoar_sugar_create(dsoar_heap* heap, uint32_t side, const dsoar_sugar_rules* rules, void* dev_mem,
                       size_t dev_bytes, dsoar_sugar** out) {
  if (side < 1 || side > 32768) return DSOAR_ERR_INVALID_ARG;
  return dsoar_sugarpool_create(heap, 1, side * side, rules, dev_mem, dev_bytes, out);
}

int dsoar_sugar_destroy(dsoar_sugar* s) {
  if (!s) return DSOAR_ERR_INVALID_ARG;
  step_graphs_clear(s->graphs);
  free(s->h_off);
  free(s->h_side);
  free(s->live);
  delete s;
  return DSOAR_OK;
}

int dsoar_sugar_init(dsoar_sugar* s, const int32_t* sugar_dev, const int32_t* cap_dev, const uint8_t* occ_dev,
                     const int32_t* a_sugar_dev, const int32_t* a_metab_dev, const int32_t* a_vision_dev,
                     const int32_t* a_age_dev, uint32_t step0, void* stream) {
  if (!s) return DSOAR_ERR_INVALID_ARG;
  uint32_t side = 1;
  while ((uint64_t)side * side < s->g.arena) ++side;
  if ((uint64_t)side * side != s->g.arena) return DSOAR_ERR_INVALID_ARG;
  s->live[0] = 0;  // the heap is reset by the caller: slot 0 starts afresh
  return dsoar_sugar_admit(s, 0, 0, side, s->default_seed, step0, sugar_dev, cap_dev, occ_dev, a_sugar_dev,
                           a_metab_dev, a_vision_dev, a_age_dev, stream);
}

int dsoar_sugar_step(dsoar_sugar* s, uint32_t steps, uint32_t flags, void* stream) {
  if (!s) return DSOAR_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  dsoar_heap* h = s->heap;
  if (flags & DSOAR_GRAPH) {
    if (flags & DSOAR_DO_PLAIN) return DSOAR_ERR_INVALID_ARG;
    return step_graphs_run(h, s->graphs, steps, st, [&](hipStream_t gs) { return sugar_one_step(s, 0, gs); });
  }
  for (uint32_t i = 0; i < steps; ++i) {
    const int rc = sugar_one_step(s, flags, st);
    if (rc) return rc;
  }
  return DSOAR_OK;
}

int dsoar_sugar_read(dsoar_sugar* s, int32_t* sugar_dev, uint8_t* occ_dev, int32_t* a_sugar_dev, int32_t* a_metab_dev,
                     int32_t* a_vision_dev, int32_t* a_age_dev, uint32_t* moves, void* stream) {
  uint64_t m = 0;
  const int rc = dsoar_sugar_read_world(s, 0, sugar_dev, occ_dev, a_sugar_dev, a_metab_dev, a_vision_dev, a_age_dev,
                                        moves ? &m : nullptr, stream);
  if (!rc && moves) *moves = (uint32_t)m;
  return rc;
}

}  // extern "C"
