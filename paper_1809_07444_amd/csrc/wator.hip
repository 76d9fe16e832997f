// Wa-Tor as objects: fish and sharks on a square torus (the paper's "wator"
// application, Fig. 6h; Dewdney's rules, read as a synchronous step).  Fish
// {pos, age, target} and Shark {pos, age, energy, target} objects live in the
// heap; the sea is a plain cell -> kind array (0 empty, 1 fish, 2 shark) and a
// cell -> request array.  One step t:
//   Both lists are enumerated at once; beside them the requests are cleared and
//     t goes up by one (the step index lives on the device, so a captured step
//     replays correctly).
//   FishDecide (do-all Fish): a fish whose cell the sharks took in the step
//     before deletes itself; the others pick, on the sea at the start of the
//     phase, the k-th empty neighbour (up, right, down, left), k = U{0..n-1}
//     from hash(seed, 40, cell, t), and leave the direction in their own cell
//     of the request array.
//   FishMove (same list): the lowest requesting cell wins; the winner moves
//     and, at age >= fish_breed, leaves a new Fish behind (both age 0).
//     Every fish ages by one.
//   SharkDecide (do-all Shark): on the sea after the fish phase, pick a
//     neighbouring fish (k from hash(seed, 41, cell, t)) or, with none and
//     energy above 1, an empty neighbour; request it.
//   SharkMove (same list): the lowest requesting cell wins; a winner that
//     lands on a fish eats it (energy = starve), any other shark loses one
//     unit and deletes itself at 0; breeding as for fish.
// After the last step of a call FishEaten (do-all Fish) deletes the fish whose
// cells the sharks took: nothing between SharkMove and the next FishDecide
// looks at them, so in between the check rides on FishDecide's pass.
#include <string.h>

#include <new>

#include "internal.hpp"

namespace dsoar {
namespace {

enum : uint32_t { kFish = 0, kShark = 1 };
enum : uint32_t { kPos = 0, kAge = 1, kFTarget = 2 };  // Fish fields
enum : uint32_t { kEnergy = 2, kSTarget = 3 };         // Shark fields after pos, age
constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr uint8_t kEmpty = 0, kIsFish = 1, kIsShark = 2;
constexpr uint64_t kStreamFish = 40, kStreamShark = 41;

// SplitMix64 output finaliser (Steele, Lea, Flood, OOPSLA 2014) and the
// workload hash built on it: mix(mix(mix(seed ^ stream * golden) ^ a) ^ b).
__device__ __forceinline__ uint64_t finalise(uint64_t z) {
  z ^= z >> 30;
  z *= 0xBF58476D1CE4E5B9ull;
  z ^= z >> 27;
  z *= 0x94D049BB133111EBull;
  z ^= z >> 31;
  return z;
}
__device__ __forceinline__ uint64_t draw(uint64_t seed, uint64_t stream, uint64_t a, uint64_t b) {
  return finalise(finalise(finalise(seed ^ (stream * 0x9E3779B97F4A7C15ull)) ^ a) ^ b);
}
// U{0..n-1}: floor(top32(h) * n / 2^32).
__device__ __forceinline__ uint32_t pick(uint64_t h, uint32_t n) {
  return (uint32_t)(((h >> 32) * (uint64_t)n) >> 32);
}

struct Sea {
  uint8_t* kind;     // kEmpty, kIsFish or kIsShark
  uint8_t* want;     // this step's requests: 0, kFishWants + d or kSharkWants + d for a move in direction d
  StepClock* clock;  // t: index of the step in progress
  uint32_t side, inverse;
  uint64_t seed;
  int32_t fish_breed, shark_breed, starve;
};
constexpr uint32_t kFishWants = 1, kSharkWants = 5;

// The planes keep the rows in groups of four, each group column by column (the
// last group of a side that is not a multiple of four has the rows that are
// left): a cell and its neighbours are three adjacent dwords and, for the
// outer rows of a group, one byte more, from 1.5 lines instead of three.
// (With an 8-byte word per target, an atomic minimum over the requesters and the
// kinds row by row, a step's FishDecide, FishMove, SharkDecide, SharkMove and
// FishEaten took 52 + 93 + 20 + 41 + 26 us on average over 50 steps of 2048^2,
// 1.75 M fish; now 44 + 80 + 13 + 44 and FishEaten once per call.  The lists in
// runs per XCD do not help: 10.04 ms per 50 steps against 10.07.)
__device__ __forceinline__ uint32_t byte_at(const Sea& a, uint32_t x, uint32_t y) {
  const uint32_t r = y & 3u, g = y - r;
  return g * a.side + x * (g + 4u <= a.side ? 4u : a.side & 3u) + r;
}

// A cell, its place in the planes and its four neighbours' coordinates.
struct Spot {
  uint32_t x, y, up, right, down, left;
};
__device__ __forceinline__ Spot spot(const Sea& a, uint32_t c) {
  Spot p;
  p.y = row_of(c, a.side, a.inverse);
  p.x = c - p.y * a.side;
  p.up = (p.y == 0 ? a.side : p.y) - 1u;
  p.right = p.x + 1u == a.side ? 0u : p.x + 1u;
  p.down = p.y + 1u == a.side ? 0u : p.y + 1u;
  p.left = (p.x == 0 ? a.side : p.x) - 1u;
  return p;
}
// Neighbour d of a cell: up, right, down, left.
__device__ __forceinline__ uint32_t nb(const Sea& a, const Spot& p, uint32_t d) {
  // Values first: a choice among the members would index the struct in scratch.
  const uint32_t x = p.x, y = p.y, up = p.up, right = p.right, down = p.down, left = p.left;
  uint32_t ny = y, nx = x;
  if (d == 0) ny = up;
  if (d == 1) nx = right;
  if (d == 2) ny = down;
  if (d == 3) nx = left;
  return ny * a.side + nx;
}

// The bytes of a cell's four neighbours (v[0..3]: up, right, down, left) and
// its own (v[4]).
__device__ __forceinline__ void around(const uint8_t* plane, const Sea& a, const Spot& p, uint32_t (&v)[5]) {
  const uint32_t r = p.y & 3u;
  if (p.x - 1u < a.side - 2u && (p.y | 3u) < a.side) {
    const uint32_t* d = (const uint32_t*)(plane + (p.y - r) * a.side + 4u * (p.x - 1u));
    const uint32_t left = d[0], mid = d[1], right = d[2];
    uint32_t other = 0;
    if (r == 0 || r == 3) other = plane[byte_at(a, p.x, r == 0 ? p.up : p.down)];
    const uint32_t sh = 8u * r;
    v[0] = r == 0 ? other : (mid >> (sh - 8u)) & 0xFFu;
    v[1] = (right >> sh) & 0xFFu;
    v[2] = r == 3 ? other : (mid >> (sh + 8u)) & 0xFFu;
    v[3] = (left >> sh) & 0xFFu;
    v[4] = (mid >> sh) & 0xFFu;
  } else {
    v[0] = plane[byte_at(a, p.x, p.up)];
    v[1] = plane[byte_at(a, p.right, p.y)];
    v[2] = plane[byte_at(a, p.x, p.down)];
    v[3] = plane[byte_at(a, p.left, p.y)];
    v[4] = plane[byte_at(a, p.x, p.y)];
  }
}

// The k-th direction of a mask of directions.
__device__ __forceinline__ uint32_t nth_direction(uint32_t mask, uint32_t k) {
  for (; k > 0; --k) mask &= mask - 1u;
  return (uint32_t)__builtin_ctz(mask);
}

// The lowest cell that asks for cell q (requests of one kind from `first` on):
// an animal moving in direction d comes from the neighbour opposite to d.
__device__ __forceinline__ uint32_t lowest_asker(const Sea& a, const Spot& q, const uint32_t (&v)[5], uint32_t first) {
  uint32_t best = kNone;
#pragma unroll
  for (uint32_t d = 0; d < 4; ++d) {
    const uint32_t from = (d + 2u) & 3u, c = nb(a, q, from);
    if (v[from] == first + d && c < best) best = c;
  }
  return best;
}

template <class F, class H>
__device__ __forceinline__ F& fish(const H& h, uint32_t self, uint32_t field) {
  return *field_ptr<F>(h, self, kFish, field);
}
template <class F, class H>
__device__ __forceinline__ F& shark(const H& h, uint32_t self, uint32_t field) {
  return *field_ptr<F>(h, self, kShark, field);
}

struct FishDecide {
  static constexpr uint32_t kKind = 70;
  static constexpr bool kPrunes = true;
  using Args = Sea;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    const uint32_t c = fish<uint32_t>(h, self, kPos);
    const Spot p = spot(a, c);
    uint32_t v[5];
    around(a.kind, a, p, v);
    if (v[4] != kIsFish) return true;  // eaten in the step before
    uint32_t empty = 0;
#pragma unroll
    for (uint32_t d = 0; d < 4; ++d) empty |= v[d] == kEmpty ? 1u << d : 0u;
    uint32_t target = kNone;
    if (empty) {
      const uint32_t d = nth_direction(empty, pick(draw(a.seed, kStreamFish, c, a.clock->t), (uint32_t)__popc(empty)));
      target = nb(a, p, d);
      a.want[byte_at(a, p.x, p.y)] = (uint8_t)(kFishWants + d);
    }
    fish<uint32_t>(h, self, kFTarget) = target;
    return false;
  }
};

// What a newborn is made from, inverted: the words are left in LDS, where
// later kernels read search hints, and small ones would send many wavefronts
// to the same groups.
struct Newborn {
  uint32_t not_c;
};

struct FishMove {
  static constexpr uint32_t kKind = 71;
  // Its own visits and, of the fish that FishEaten or FishDecide looks over
  // after the step, those that are not newborn (make counts these).
  static constexpr uint32_t kPhases = 2;
  using Args = Sea;
  using Item = Newborn;
  static constexpr uint32_t kItemType = kFish;
  static constexpr uint32_t kMinWaves = 8;
  static constexpr uint32_t kItems = 256, kClaimBits = 2;
  struct Found {
    uint32_t claims;  // bit u: object u breeds
    uint32_t c[2];
  };
  template <uint32_t N, class H>
  static __device__ __forceinline__ void find(const H& h, uint32_t, const uint32_t (&self)[2], const bool (&lv)[2],
                                              const Args& a, Found& found, bool (&)[2]) {
    uint32_t q[N];
    int32_t age[N];
    bool won[N];
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
      const uint32_t c = fish<uint32_t>(h, self[u], kPos), target = fish<uint32_t>(h, self[u], kFTarget);
      age[u] = fish<int32_t>(h, self[u], kAge) + 1;
      found.c[u] = lv[u] ? c : 0u;
      won[u] = lv[u] && target != kNone;
      q[u] = won[u] ? target : found.c[u];
    }
    Spot to[N];
    uint32_t v[N][5];
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
      to[u] = spot(a, q[u]);
      around(a.want, a, to[u], v[u]);
    }
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
      const uint32_t c = found.c[u];
      won[u] = won[u] && lowest_asker(a, to[u], v[u], kFishWants) == c;
      const bool breed = won[u] && age[u] >= a.fish_breed;
      if (won[u]) {
        a.kind[byte_at(a, to[u].x, to[u].y)] = kIsFish;
        fish<uint32_t>(h, self[u], kPos) = q[u];
        if (!breed) {  // else the newborn keeps the cell
          const uint32_t y = row_of(c, a.side, a.inverse);
          a.kind[byte_at(a, c - y * a.side, y)] = kEmpty;
        }
      }
      if (lv[u]) fish<int32_t>(h, self[u], kAge) = breed ? 0 : age[u];
      if (breed) found.claims |= 1u << u;
    }
  }
  static __device__ __forceinline__ Item item(const Found& f, uint32_t b) { return {~(b ? f.c[1] : f.c[0])}; }
  template <class H>
  static __device__ __forceinline__ void make(const H& h, const Args&, const Item& it, uint32_t o) {
    fish<uint32_t>(h, o, kPos) = ~it.not_c;
    fish<int32_t>(h, o, kAge) = 0;
    fish<uint32_t>(h, o, kFTarget) = kNone;
    lead_add(shard(h) + kCntVisits + kFish, (uint64_t)__popcll(__ballot(true)));
  }
};

struct SharkDecide {
  static constexpr uint32_t kKind = 72;
  using Args = Sea;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    const uint32_t c = shark<uint32_t>(h, self, kPos);
    const bool strong = shark<int32_t>(h, self, kEnergy) > 1;
    const Spot p = spot(a, c);
    uint32_t v[5], fishes = 0, empty = 0;
    around(a.kind, a, p, v);
#pragma unroll
    for (uint32_t d = 0; d < 4; ++d) {
      fishes |= v[d] == kIsFish ? 1u << d : 0u;
      empty |= v[d] == kEmpty ? 1u << d : 0u;
    }
    const uint32_t from = fishes ? fishes : strong ? empty : 0u;
    uint32_t target = kNone;
    if (from) {
      const uint32_t d = nth_direction(from, pick(draw(a.seed, kStreamShark, c, a.clock->t), (uint32_t)__popc(from)));
      target = nb(a, p, d);
      a.want[byte_at(a, p.x, p.y)] = (uint8_t)(kSharkWants + d);
    }
    shark<uint32_t>(h, self, kSTarget) = target;
    return false;
  }
};

struct SharkMove {
  static constexpr uint32_t kKind = 73;
  static constexpr uint32_t kMinWaves = 8;
  static constexpr bool kDeletesOnlyThis = true;
  using Args = Sea;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    const uint32_t c = shark<uint32_t>(h, self, kPos), target = shark<uint32_t>(h, self, kSTarget);
    const int32_t age = shark<int32_t>(h, self, kAge) + 1;
    int32_t energy = shark<int32_t>(h, self, kEnergy) - 1;
    bool won = target != kNone;
    const Spot to = spot(a, won ? target : c);
    const uint32_t there = byte_at(a, to.x, to.y);
    // Only the winner writes its target cell, and no shark targets a shark's
    // cell, so a winner's read sees the sea as the fish phase left it.
    const uint32_t kind = a.kind[there];
    uint32_t v[5];
    around(a.want, a, to, v);
    won = won && lowest_asker(a, to, v, kSharkWants) == c;
    if (won && kind == kIsFish) energy = a.starve;
    const bool starved = energy <= 0;  // a shark that eats never does
    const bool breed = won && !starved && age >= a.shark_breed;
    if (starved || (won && !breed)) {  // else a newborn keeps the cell
      const uint32_t y = row_of(c, a.side, a.inverse);
      a.kind[byte_at(a, c - y * a.side, y)] = kEmpty;
    }
    if (starved) return true;
    if (won) {
      a.kind[there] = kIsShark;
      shark<uint32_t>(h, self, kPos) = target;
    }
    shark<int32_t>(h, self, kEnergy) = energy;
    shark<int32_t>(h, self, kAge) = breed ? 0 : age;
    new_many(h, kShark, breed ? 1u : 0u, [&](uint32_t, uint32_t o) {
      if (o == kNull) return;
      shark<uint32_t>(h, o, kPos) = c;
      shark<int32_t>(h, o, kAge) = 0;
      shark<int32_t>(h, o, kEnergy) = a.starve;
      shark<uint32_t>(h, o, kSTarget) = kNone;
    });
    return false;
  }
};

struct FishEaten {
  static constexpr uint32_t kKind = 74;
  static constexpr bool kDeletesOnlyThis = true;
  static constexpr uint32_t kPhases = 0;  // counted by FishMove
  using Args = Sea;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    const Spot p = spot(a, fish<uint32_t>(h, self, kPos));
    return a.kind[byte_at(a, p.x, p.y)] != kIsFish;
  }
};

struct ReadArgs {
  int32_t* age;
  int32_t* energy;
};

struct FishRead {
  static constexpr uint32_t kKind = 75;
  using Args = ReadArgs;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    a.age[fish<uint32_t>(h, self, kPos)] = fish<int32_t>(h, self, kAge);
    return false;
  }
};

struct SharkRead {
  static constexpr uint32_t kKind = 76;
  using Args = ReadArgs;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    const uint32_t c = shark<uint32_t>(h, self, kPos);
    a.age[c] = shark<int32_t>(h, self, kAge);
    a.energy[c] = shark<int32_t>(h, self, kEnergy);
    return false;
  }
};

// Creates the objects of the initial sea, in cell order, a cell per lane or, from
// kInitWideMin cells on, four of a row, so that one request of a wavefront serves
// 256.  Smaller seas keep the shorter chains, and their animals stand in blocks
// with more room for the first births.  us of the initial sea, and of it and 20
// steps, one cell and four (35 % of the cells taken):
//   64^2   17   787    23   823      724^2   73  1441    61  1570
//   256^2  24   964    30  1001      2048^2 455  5120   324  4867
constexpr uint64_t kInitWideMin = 1u << 19;
template <uint32_t LG, uint32_t CELLS>
__global__ void wator_init_kernel(DevHeapW<LG> h, Sea a, const int32_t* kind, const int32_t* age, const int32_t* energy,
                                  uint32_t step0) {
  const uint32_t n = a.side * a.side;  // at most 2^30
  const uint32_t c0 = (blockIdx.x * blockDim.x + threadIdx.x) * CELLS;
  if (c0 == 0) *a.clock = StepClock{step0 - 1u, 2u};  // the step's enumeration advances it
  uint32_t fishes = 0, sharks = 0;
#pragma unroll
  for (uint32_t i = 0; i < CELLS; ++i) {
    const uint32_t c = c0 + i;
    if (c >= n) continue;
    const int32_t k = kind[c];
    const uint32_t y = row_of(c, a.side, a.inverse);
    a.kind[byte_at(a, c - y * a.side, y)] = (uint8_t)k;
    fishes |= k == kIsFish ? 1u << i : 0u;
    sharks |= k == kIsShark ? 1u << i : 0u;
  }
  new_many(h, kFish, (uint32_t)__popc(fishes), [&](uint32_t i, uint32_t o) __attribute__((always_inline)) {
    if (o == kNull) return;
    const uint32_t c = c0 + nth_direction(fishes, i);
    fish<uint32_t>(h, o, kPos) = c;
    fish<int32_t>(h, o, kAge) = age[c];
    fish<uint32_t>(h, o, kFTarget) = kNone;
  });
  new_many(h, kShark, (uint32_t)__popc(sharks), [&](uint32_t i, uint32_t o) __attribute__((always_inline)) {
    if (o == kNull) return;
    const uint32_t c = c0 + nth_direction(sharks, i);
    shark<uint32_t>(h, o, kPos) = c;
    shark<int32_t>(h, o, kAge) = age[c];
    shark<int32_t>(h, o, kEnergy) = energy[c];
    shark<uint32_t>(h, o, kSTarget) = kNone;
  });
}

// kind out, and zeroed age and energy (the read do-alls fill the occupied cells).
__global__ void wator_read_kernel(Sea a, int32_t* kind, int32_t* age, int32_t* energy) {
  const uint64_t n = (uint64_t)a.side * a.side;
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  const uint32_t y = row_of(c, a.side, a.inverse);
  kind[c] = a.kind[byte_at(a, c - y * a.side, y)];
  age[c] = 0;
  energy[c] = 0;
}

bool wator_heap_ok(const dsoar_heap* h) {
  if (h->desc.num_types < 2) return false;
  const uint32_t want[2] = {3, 4};
  for (uint32_t t = 0; t < 2; ++t) {
    const dsoar_type_layout& L = h->desc.types[t];
    if (L.num_fields < want[t]) return false;
    for (uint32_t f = 0; f < want[t]; ++f)
      if (L.field_bytes[f] != 4) return false;
  }
  return true;
}

}  // namespace
}  // namespace dsoar

using namespace dsoar;

struct dsoar_wator {
  dsoar_heap* heap;
  Sea a;
  StepGraphs graphs;
};

namespace {

size_t round256(uint64_t b) { return (size_t)((b + 255) / 256 * 256); }

int wator_one_step(dsoar_wator* w, uint32_t flags, hipStream_t st) {
  dsoar_heap* h = w->heap;
  const uint32_t reuse = (flags & DSOAR_DO_PLAIN) | DSOAR_DO_REUSE_ENUM;
  // The fish phase neither creates nor deletes sharks, so both lists hold from
  // the start; the newborns of a Move are not visited by it (snapshot
  // semantics).
  const uint64_t n = (uint64_t)w->a.side * w->a.side;
  int rc = launch_enumerate_pair(h, kFish, kShark, st, w->a.clock, (uint4*)w->a.want, (uint32_t)(round256(n) / 16));
  if (!rc) rc = launch_doall<FishDecide>(h, kFish, w->a, reuse, st);
  if (!rc) rc = launch_doall<FishMove>(h, kFish, w->a, reuse, st);
  if (!rc) rc = launch_doall<SharkDecide>(h, kShark, w->a, reuse, st);
  if (!rc) rc = launch_doall<SharkMove>(h, kShark, w->a, reuse, st);
  return rc;
}

}  // namespace

extern "C" {

size_t dsoar_wator_bytes(uint32_t side) {
  const uint64_t n = (uint64_t)side * side;
  if (side == 0 || n > (1ull << 30)) return 0;
  return 256 + round256(n) + round256(n * 8);
}

int dsoar_wator_create(dsoar_heap* heap, uint32_t side, const dsoar_wator_rules* rules, void* dev_mem,
                       size_t dev_bytes, dsoar_wator** out) {
  if (!out) return DSOAR_ERR_INVALID_ARG;
  *out = nullptr;
  if (!heap_ok(heap) || !wator_heap_ok(heap) || !rules || !dev_mem || ((uintptr_t)dev_mem & 255u) ||
      rules->fish_breed < 1 || rules->shark_breed < 1 || rules->starve < 1)
    return DSOAR_ERR_INVALID_ARG;
  const size_t need = dsoar_wator_bytes(side);
  if (need == 0) return DSOAR_ERR_INVALID_ARG;
  if (dev_bytes < need) return DSOAR_ERR_TOO_SMALL;
  dsoar_wator* w = new (std::nothrow) dsoar_wator;
  if (!w) return DSOAR_ERR_INVALID_ARG;
  memset(w, 0, sizeof(*w));
  const uint64_t n = (uint64_t)side * side;
  uint8_t* b = (uint8_t*)dev_mem;
  w->heap = heap;
  w->a.clock = (StepClock*)b;
  w->a.kind = b + 256;
  w->a.want = b + 256 + round256(n);
  w->a.side = side;
  w->a.inverse = inverse_of(side);
  w->a.seed = rules->seed;
  w->a.fish_breed = rules->fish_breed;
  w->a.shark_breed = rules->shark_breed;
  w->a.starve = rules->starve;
  *out = w;
  return DSOAR_OK;
}

int dsoar_wator_destroy(dsoar_wator* w) {
  if (!w) return DSOAR_ERR_INVALID_ARG;
  step_graphs_clear(w->graphs);
  delete w;
  return DSOAR_OK;
}

int dsoar_wator_init(dsoar_wator* w, const int32_t* kind_dev, const int32_t* age_dev, const int32_t* energy_dev,
                     uint32_t step0, void* stream) {
  if (!w || !kind_dev || !age_dev || !energy_dev) return DSOAR_ERR_INVALID_ARG;
  const uint64_t n = (uint64_t)w->a.side * w->a.side;
  with_width(w->heap, [&](auto w_) {
    constexpr uint32_t kLG = decltype(w_)::value;
    const uint32_t cells = n >= kInitWideMin ? 4u : 1u;
    auto go = [&](auto kernel) {
      launch_timed(w->heap, kKindWatorInit, kernel, dim3((uint32_t)((n + 256 * cells - 1) / (256 * cells))), dim3(256),
                   (hipStream_t)stream, DevHeapW<kLG>(w->heap->dev), w->a, kind_dev, age_dev, energy_dev, step0);
    };
    if (cells == 4) go(wator_init_kernel<kLG, 4>);
    else go(wator_init_kernel<kLG, 1>);
  });
  DSOAR_LAUNCHED(w->heap);
  return DSOAR_OK;
}

int dsoar_wator_step(dsoar_wator* w, uint32_t steps, uint32_t flags, void* stream) {
  if (!w) return DSOAR_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  dsoar_heap* h = w->heap;
  if (flags & DSOAR_GRAPH) {
    if (flags & DSOAR_DO_PLAIN) return DSOAR_ERR_INVALID_ARG;
    const int rc = step_graphs_run(h, w->graphs, steps, st, [&](hipStream_t gs) { return wator_one_step(w, 0, gs); });
    if (rc) return rc;
  } else {
    for (uint32_t i = 0; i < steps; ++i) {
      const int rc = wator_one_step(w, flags, st);
      if (rc) return rc;
    }
  }
  return steps ? launch_doall<FishEaten>(h, kFish, w->a, flags & DSOAR_DO_PLAIN, st) : DSOAR_OK;
}

int dsoar_wator_read(dsoar_wator* w, int32_t* kind_dev, int32_t* age_dev, int32_t* energy_dev, void* stream) {
  if (!w || !kind_dev || !age_dev || !energy_dev) return DSOAR_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  const uint64_t n = (uint64_t)w->a.side * w->a.side;
  hipLaunchKernelGGL(wator_read_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, w->a, kind_dev,
                     age_dev, energy_dev);
  DSOAR_LAUNCHED(w->heap);
  const ReadArgs r{age_dev, energy_dev};
  int rc = launch_doall<FishRead>(w->heap, kFish, r, DSOAR_DO_PERSISTENT, st);
  if (!rc) rc = launch_doall<SharkRead>(w->heap, kShark, r, DSOAR_DO_PERSISTENT, st);
  return rc;
}

}  // extern "C"
