// Nagel-Schreckenberg traffic as objects on open single-lane roads (the
// paper's "traffic" application, Fig. 6; the rules are the model's published
// ones).  Car {cell, speed, next speed} objects live in the heap.  One step t is:
//   Decide: on the state at the start of the step, accelerate (v = min(v + 1,
//     vmax)), brake to the empty cells ahead (cells past the road's end count
//     as empty), and dawdle (v -= 1 when v > 0 with probability p_slow, drawn
//     from hash(seed, 32, cell, t)).
//   Move: advance v cells; a car that passes the road's last cell deletes
//     itself.  Moves never collide: a car ends before the old cell of the car
//     ahead.
//   Entry: a car enters an empty first cell at speed 0 with probability p_in,
//     from hash(seed, 33, road, t).
// All three run in one kernel.  The roads are two planes of 16-bit words, one
// per cell: the state that a step reads and the one it writes.  A word holds
// the epoch in which its cell is occupied and the car's speed, so nothing is
// cleared between steps and a cell is empty unless its word carries the
// plane's current epoch; the entry of a road finds from its first two words
// whether the first cell will be empty.  With the roads in one plane of
// handles the phases were three kernels after the enumeration (6.7, 7.6 and
// 10 us at 1024 x 1024 cells, each a few round trips long); one now takes 11.8
// us, bound by the latency of the entries' allocation, and a step 30.5 -> 19.3
// us.  The enumeration advances the clock.
#include <string.h>

#include <new>

#include "internal.hpp"

namespace dsoar {
namespace {

enum : uint32_t { kCar = 0 };
enum : uint32_t { kCellF = 0, kSpeed = 1, kNext = 2 };
constexpr int32_t kMaxSpeed = 8;
constexpr uint64_t kStreamSlow = 32, kStreamIn = 33;

// SplitMix64 output finaliser (Steele, Lea, Flood, OOPSLA 2014) and the
// workload hash built on it: mix(mix(mix(seed ^ stream * golden) ^ a) ^ b).
__device__ __forceinline__ uint64_t splitmix_final(uint64_t z) {
  z ^= z >> 30;
  z *= 0xBF58476D1CE4E5B9ull;
  z ^= z >> 27;
  z *= 0x94D049BB133111EBull;
  z ^= z >> 31;
  return z;
}
__device__ __forceinline__ uint64_t draw(uint64_t seed, uint64_t stream, uint64_t a, uint64_t b) {
  return splitmix_final(splitmix_final(splitmix_final(seed ^ (stream * 0x9E3779B97F4A7C15ull)) ^ a) ^ b);
}

// A road word: epoch << kSpeedBits | speed.  Epochs run from 2 to kEpochs - 1
// and round again (an even number of them: the epoch's low bit names the
// plane); 0 is no epoch.
constexpr uint32_t kSpeedBits = 4;
static_assert(kMaxSpeed < (1 << kSpeedBits) && (kEpochs << kSpeedBits) == 0x10000u, "a word is 16 bits");

struct Road {
  uint16_t* plane[2];
  const StepClock* clock;  // t and the epoch of the state that the step in progress reads
  uint32_t roads, length;
  uint64_t seed;
  int32_t vmax;
  uint32_t p_slow24, p_in24;
};

template <class F, class H>
__device__ __forceinline__ F& car(const H& h, uint32_t self, uint32_t field) {
  return *field_ptr<F>(h, self, kCar, field);
}

__device__ __forceinline__ uint16_t* plane_of(const Road& a, uint32_t epoch) {
  return (epoch & 1u) ? a.plane[1] : a.plane[0];
}

// The speed that the car in cell c (cell i of its road) moves at in step t.
__device__ __forceinline__ int32_t decide(const Road& a, const uint16_t* now, uint32_t epoch, uint32_t t, uint32_t c,
                                          uint32_t i, int32_t v0) {
  int32_t v = v0 + 1 < a.vmax ? v0 + 1 : a.vmax;
  // The cells ahead, all read together; past the road's end they are empty.
  uint32_t ahead[kMaxSpeed];
#pragma unroll
  for (int32_t k = 1; k <= kMaxSpeed; ++k)
    ahead[k - 1] = (k <= v && i + (uint32_t)k < a.length) ? now[c + (uint32_t)k] : 0u;
  int32_t gap = 0;
#pragma unroll
  for (int32_t k = 1; k <= kMaxSpeed; ++k)
    if (gap == k - 1 && k <= v && (ahead[k - 1] >> kSpeedBits) != epoch) gap = k;
  v = v < gap ? v : gap;
  const uint64_t hs = draw(a.seed, kStreamSlow, c, t);
  if (v > 0 && (uint32_t)(hs >> 40) < a.p_slow24) --v;
  return v;
}

// Decide and Move.
struct Drive {
  static constexpr uint32_t kKind = 52;
  static constexpr uint32_t kPhases = 2;
  static constexpr bool kDeletesOnlyThis = true;
  using Args = Road;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    const uint32_t t = a.clock->t, epoch = a.clock->epoch, then = next_epoch(epoch);
    const uint32_t c = car<uint32_t>(h, self, kCellF), i = c % a.length;
    const int32_t v = decide(a, plane_of(a, epoch), epoch, t, c, i, car<int32_t>(h, self, kSpeed));
    if (i + (uint32_t)v >= a.length) return true;  // leaves the road
    plane_of(a, then)[c + (uint32_t)v] = (uint16_t)(then << kSpeedBits | (uint32_t)v);
    car<int32_t>(h, self, kSpeed) = v;
    car<int32_t>(h, self, kNext) = v;
    if (v) car<uint32_t>(h, self, kCellF) = c + (uint32_t)v;
    return false;
  }
};

// A car enters road r if its first cell is empty after the step's moves (no
// car there, or one that moves on) and the road's draw says so.
template <class H>
__device__ __forceinline__ void entry(const H& h, const Road& a, uint32_t r) {
  if (r >= a.roads) return;
  const uint32_t t = a.clock->t, epoch = a.clock->epoch, then = next_epoch(epoch);
  const uint16_t* now = plane_of(a, epoch);
  const uint32_t q = r * a.length, w = now[q];
  const uint64_t hs = draw(a.seed, kStreamIn, r, t);
  bool enter = (uint32_t)(hs >> 40) < a.p_in24;
  if (enter && (w >> kSpeedBits) == epoch)
    enter = decide(a, now, epoch, t, q, 0u, (int32_t)(w & ((1u << kSpeedBits) - 1u))) > 0;
  new_many(h, kCar, enter ? 1u : 0u, [&](uint32_t, uint32_t o) {
    if (o == kNull) return;
    car<uint32_t>(h, o, kCellF) = q;
    car<int32_t>(h, o, kSpeed) = 0;
    car<int32_t>(h, o, kNext) = 0;
    plane_of(a, then)[q] = (uint16_t)(then << kSpeedBits);
  });
}

// Old words would read as occupied when their epoch comes round again: each
// step clears those in one of kSweeps parts of the plane that it reads (and
// nobody writes), so that every part is swept at three epochs or more of a
// round.
constexpr uint32_t kSweeps = 512;
static_assert(kEpochs / 2 >= 3 * kSweeps, "every part swept at several epochs");
__device__ __forceinline__ void sweep(const Road& a, uint64_t me, uint64_t threads) {
  const uint64_t words = ((uint64_t)a.roads * a.length + 1) / 2, part = (words + kSweeps - 1) / kSweeps;
  const uint32_t epoch = a.clock->epoch;
  const uint64_t first = ((epoch >> 1) % kSweeps) * part, end = first + part < words ? first + part : words;
  uint32_t* const p = reinterpret_cast<uint32_t*>(plane_of(a, epoch));
  for (uint64_t j = first + me; j < end; j += threads) {
    const uint32_t w = p[j];
    const uint32_t lo = (w & 0xFFFFu) >> kSpeedBits == epoch ? w & 0xFFFFu : 0u;
    const uint32_t hi = w >> (16 + kSpeedBits) == epoch ? w & 0xFFFF0000u : 0u;
    if ((lo | hi) != w) p[j] = lo | hi;
  }
}

// One step.  The first entry_wgs workgroups take the entries (one road per
// thread: the longest chain of the step, the allocation, starts first), the
// others the cars' do-all; the cars that enter are not in its list.  Either part
// may also be a launch of its own (see traffic_one_step).
template <uint32_t LG>
__global__ void __launch_bounds__(1024)
    traffic_step_kernel(DevHeapW<LG> h, const uint32_t* __restrict__ R, const uint64_t* __restrict__ S,
                        const uint32_t* count_ptr, Road a, uint32_t entry_wgs) {
  if (blockIdx.x < entry_wgs) {
    entry(h, a, blockIdx.x * blockDim.x + threadIdx.x);
  } else {
    const uint32_t wpb = blockDim.x >> 6, skip = entry_wgs * wpb;
    uint32_t visits = 0, freed = 0;
    doall_list<Drive, true>(h, kCar, R, S, bcast32(*count_ptr), grid_wave() - skip, gridDim.x * wpb - skip, a, visits,
                            freed);
    if (visits) lead_add(shard(h) + kCntVisits + kCar, visits * Phases<Drive>::value);
    if (freed) lead_add(shard(h) + kCntFrees + kCar, freed);
  }
  if (gridDim.x != entry_wgs) sweep(a, (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, (uint64_t)gridDim.x * blockDim.x);
}

// Initial state: a car in every cell whose speed is >= 0.  The first step's
// enumeration brings the clock to step0 and epoch 2.
template <uint32_t LG>
__global__ void traffic_init_kernel(DevHeapW<LG> h, Road a, StepClock* clock, const int32_t* vel, uint32_t step0) {
  const uint64_t n = (uint64_t)a.roads * a.length;
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c == 0) {
    clock->t = step0 - 1;
    clock->epoch = 1;
  }
  if (c >= n) return;
  const int32_t v = vel[c];
  a.plane[1][c] = 0;
  bool made = false;
  new_many(h, kCar, v >= 0 ? 1u : 0u, [&](uint32_t, uint32_t o) {
    if (o == kNull) return;
    car<uint32_t>(h, o, kCellF) = c;
    car<int32_t>(h, o, kSpeed) = v;
    car<int32_t>(h, o, kNext) = v;
    made = true;
  });
  a.plane[0][c] = made ? (uint16_t)(2u << kSpeedBits | (uint32_t)(v < 15 ? v : 15)) : (uint16_t)0;
}

__global__ void traffic_read_kernel(Road a, int32_t* vel) {
  const uint64_t n = (uint64_t)a.roads * a.length;
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  const uint32_t state = next_epoch(a.clock->epoch);  // the state that the last step wrote
  const uint32_t w = plane_of(a, state)[c];
  vel[c] = (w >> kSpeedBits) == state ? (int32_t)(w & ((1u << kSpeedBits) - 1u)) : -1;
}

bool traffic_heap_ok(const dsoar_heap* h) {
  if (h->desc.num_types < 1) return false;
  const dsoar_type_layout& L = h->desc.types[kCar];
  if (L.num_fields < 3) return false;
  for (uint32_t f = 0; f < 3; ++f)
    if (L.field_bytes[f] != 4) return false;
  return true;
}

}  // namespace
}  // namespace dsoar

using namespace dsoar;

struct dsoar_traffic {
  dsoar_heap* heap;
  Road a;
  StepClock* clock;
  StepGraphs graphs;
};

namespace {

int traffic_one_step(dsoar_traffic* t, uint32_t flags, hipStream_t st) {
  dsoar_heap* h = t->heap;
  int rc = launch_enumerate(h, kCar, st, t->clock);
  if (rc) return rc;
  const EnumOut& eo = h->enum_out[kCar];
  const uint32_t threads = h->doall_wg_threads;
  uint32_t grid = h->num_cus * h->doall_wgs_per_cu;
  if (flags & DSOAR_DO_PLAIN) {
    uint32_t count = 0;
    rc = read_count(h, kCar, st, &count);
    if (rc) return rc;
    const uint32_t per_wave = 64 / h->dev.capacity[kCar];
    const uint64_t waves = ((uint64_t)count + per_wave - 1) / per_wave;
    grid = (uint32_t)((waves * 64 + threads - 1) / threads);
  }
  if (grid == 0) grid = 1;
  const uint32_t entry_wgs = (t->a.roads + threads - 1) / threads;
  // The entries run beside the cars' do-all only where they never need the slots
  // of the cars that leave in the same step: at most one car stands in a cell and
  // one more enters per road, and no other type holds blocks.  Otherwise they
  // follow it, as a launch of their own (1024 x 1024 cells: 23.4 us per step against
  // 18.2).
  const uint64_t slots = (uint64_t)h->dev.num_blocks * h->dev.capacity[kCar];
  const bool beside = h->desc.num_types == 1 && slots >= (uint64_t)t->a.roads * t->a.length + t->a.roads;
  with_width(h, [&](auto w_) {
    constexpr uint32_t kLG = decltype(w_)::value;
    auto go = [&](uint32_t entries, uint32_t cars) {
      launch_timed(h, Drive::kKind, traffic_step_kernel<kLG>, dim3(entries + cars), dim3(threads), st, DevHeapW<kLG>(h->dev),
                   (const uint32_t*)eo.R, (const uint64_t*)eo.S, (const uint32_t*)&eo.st->count, t->a, entries);
    };
    if (beside) {
      go(entry_wgs, grid);
    } else {
      go(0, grid);
      go(entry_wgs, 0);
    }
  });
  DSOAR_LAUNCHED(h);
  return DSOAR_OK;
}

}  // namespace

extern "C" {

size_t dsoar_traffic_bytes(uint32_t roads, uint32_t length) {
  const uint64_t n = (uint64_t)roads * length;
  if (roads == 0 || length == 0 || n > (1ull << 30)) return 0;
  return (size_t)(256 + (n * 4 + 255) / 256 * 256);
}

int dsoar_traffic_create(dsoar_heap* heap, uint32_t roads, uint32_t length, const dsoar_traffic_rules* rules,
                         void* dev_mem, size_t dev_bytes, dsoar_traffic** out) {
  if (!out) return DSOAR_ERR_INVALID_ARG;
  *out = nullptr;
  if (!heap_ok(heap) || !traffic_heap_ok(heap) || !rules || !dev_mem || ((uintptr_t)dev_mem & 255u) ||
      rules->vmax < 1 || rules->vmax > kMaxSpeed || rules->p_slow24 > (1u << 24) || rules->p_in24 > (1u << 24))
    return DSOAR_ERR_INVALID_ARG;
  const size_t need = dsoar_traffic_bytes(roads, length);
  if (need == 0) return DSOAR_ERR_INVALID_ARG;
  if (dev_bytes < need) return DSOAR_ERR_TOO_SMALL;
  dsoar_traffic* t = new (std::nothrow) dsoar_traffic;
  if (!t) return DSOAR_ERR_INVALID_ARG;
  memset(t, 0, sizeof(*t));
  t->heap = heap;
  uint8_t* b = (uint8_t*)dev_mem;
  t->clock = (StepClock*)b;
  t->a.clock = t->clock;
  // Two planes of an even number of 16-bit words (an odd number of cells
  // leaves at least 4 of the 256-byte rounding's bytes).
  const uint64_t cells = (uint64_t)roads * length;
  t->a.plane[0] = (uint16_t*)(b + 256);
  t->a.plane[1] = t->a.plane[0] + (cells + 1) / 2 * 2;
  t->a.roads = roads;
  t->a.length = length;
  t->a.seed = rules->seed;
  t->a.vmax = rules->vmax;
  t->a.p_slow24 = rules->p_slow24;
  t->a.p_in24 = rules->p_in24;
  *out = t;
  return DSOAR_OK;
}

int dsoar_traffic_destroy(dsoar_traffic* t) {
  if (!t) return DSOAR_ERR_INVALID_ARG;
  step_graphs_clear(t->graphs);
  delete t;
  return DSOAR_OK;
}

int dsoar_traffic_init(dsoar_traffic* t, const int32_t* vel_dev, uint32_t step0, void* stream) {
  if (!t || !vel_dev) return DSOAR_ERR_INVALID_ARG;
  const uint64_t n = (uint64_t)t->a.roads * t->a.length;
  with_width(t->heap, [&](auto w_) {
    constexpr uint32_t kLG = decltype(w_)::value;
    launch_timed(t->heap, kKindTrafficInit, traffic_init_kernel<kLG>, dim3((uint32_t)((n + 255) / 256)), dim3(256), (hipStream_t)stream,
                     DevHeapW<kLG>(t->heap->dev), t->a, t->clock, vel_dev, step0);
  });
  DSOAR_LAUNCHED(t->heap);
  return DSOAR_OK;
}

int dsoar_traffic_step(dsoar_traffic* t, uint32_t steps, uint32_t flags, void* stream) {
  if (!t) return DSOAR_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  dsoar_heap* h = t->heap;
  if (flags & DSOAR_GRAPH) {
    if (flags & DSOAR_DO_PLAIN) return DSOAR_ERR_INVALID_ARG;
    return step_graphs_run(h, t->graphs, steps, st, [&](hipStream_t gs) { return traffic_one_step(t, 0, gs); });
  }
  for (uint32_t i = 0; i < steps; ++i) {
    const int rc = traffic_one_step(t, flags, st);
    if (rc) return rc;
  }
  return DSOAR_OK;
}

int dsoar_traffic_read(dsoar_traffic* t, int32_t* vel_dev, void* stream) {
  if (!t || !vel_dev) return DSOAR_ERR_INVALID_ARG;
  const uint64_t n = (uint64_t)t->a.roads * t->a.length;
  hipLaunchKernelGGL(traffic_read_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                     t->a, vel_dev);
  DSOAR_LAUNCHED(t->heap);
  return DSOAR_OK;
}

}  // extern "C"
