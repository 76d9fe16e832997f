// Merging bodies in the plane as objects (the paper's "collisions"
// application, Fig. 6b).  Body {x, y, vx, vy, ax, ay, m, id} objects live in
// the heap; dense per-id arrays hold what every body reads of every other:
// P[id] = {x, y, m, link} (m = 0 once the body merged away), V[id] = {vx, vy} and
// T[id], the merge decision.  One step is five do-alls over the same
// enumeration (nothing is created, and only the last deletes):
//   Force:  a = sum over all ids j in increasing order of
//           m_j (p_j - p) / (r2 sqrt(r2)), r2 = |p_j - p|^2 + eps2
//           (j = this body and merged bodies add exactly 0)
//   Move:   v += dt a, p += dt v; publish P and V
//   Root:   a root has no live body of lower id within the merge radius
//   Target: a live non-root merges into the lowest-id root within the radius
//   Merge:  a root adds the mass, momentum and mass-weighted position of the
//           bodies merging into it, in increasing id order, and marks their P
//           dead; merged bodies delete themselves
// The merge phases look for the few bodies within the merge radius in a hash
// table of cells (see walk_near), whose chains run through P's link.
// Every float operation is single precision with one rounding (explicit
// fma; correctly rounded division and square root), in the same order as the
// sequential definition, so the results are bit-identical to it.
#include <math.h>
#include <string.h>

#include <new>

#include "internal.hpp"

namespace dsoar {
namespace {

enum : uint32_t { kBody = 0 };
enum : uint32_t { kX = 0, kY = 1, kVX = 2, kVY = 3, kAX = 4, kAY = 5, kM = 6, kId = 7 };
constexpr uint32_t kRoot = 0xFFFFFFFEu, kAlone = 0xFFFFFFFFu;

struct Bodies {
  float4* P;   // id -> {x, y, m, link}: the next body of its bucket (an id's bits, kNoBody: none)
  float2* V;   // id -> {vx, vy}
  uint32_t* T; // id -> kRoot, kAlone or the id of the root it merges into
  uint32_t n;
  float dt, eps2, r2_merge;
  uint32_t* head;      // bucket -> its first body (mask + 1 buckets); null: the merge phases scan
  uint32_t* far_out;   // nonzero: a body lies outside the cells' range, the merge phases scan
  uint32_t mask;
  float inv_cell;
};
constexpr uint32_t kNoBody = 0xFFFFFFFFu;

template <class F, class H>
__device__ __forceinline__ F& fld(const H& h, uint32_t self, uint32_t f) {
  return *field_ptr<F>(h, self, kBody, f);
}

// Entry k of a wavefront-wide chunk: lane k's value, read by every lane.
__device__ __forceinline__ float from_lane(float v, uint32_t k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}
__device__ __forceinline__ uint32_t from_lane(uint32_t v, uint32_t k) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, k);
}

// The per-id arrays are walked in chunks of 64 ids: lane l loads entry j0 + l
// of the next chunk (clamped to the last id, so every load stays in bounds)
// while the wavefront works through the current one.
__device__ __forceinline__ uint32_t chunk_id(uint32_t j0, uint32_t n) {
  const uint32_t j = j0 + lane_id();
  return j < n ? j : n - 1u;
}

// The scale s = m / (r2 sqrt(r2)) of a pair, every operation correctly rounded:
// the general form, for any values.
__device__ __forceinline__ float pair_scale(float r2, float m) { return m / (r2 * __builtin_sqrtf(r2)); }

// The same scale, bit for bit, for 2^-40 <= r2 <= 2^40 and m that passes
// scale_normal_mass, in 13 operations and one reciprocal square root where the general
// form's correctly rounded square root and division expand to about 36: both
// take a residual step from y = rsqrt(r2) (1 ulp).
//  - root: g = r2 y, g + (r2 - g^2) y / 2.
//  - quotient m / b, b = r2 root: 1 / b is y^3 but for 2^-21, one Newton step
//    rounds it, and m / b takes one residual step from m times that.
// No operation leaves the normal range there, so the results scale with the
// exponents of r2 (by pairs) and m, and two binades of r2 times one of m hold
// every case.  Compared over all of them on this part: the 2^24 roots equal the
// general form's, and of the 2^47 quotients all but one, m = 0x1.ccccc4 over
// b = 0x1.fffff6; masses of that mantissa are left to the general form.
constexpr float kScaleLo = 0x1p-40f, kScaleHi = 0x1p40f;
constexpr uint32_t kScaleNot = 0x666662;  // mantissa bits of that m
__device__ __forceinline__ bool scale_normal_mass(float m) {
  return m == 0.0f || (m >= kScaleLo && m <= kScaleHi && (__float_as_uint(m) & 0x7FFFFFu) != kScaleNot);
}
__device__ __forceinline__ float pair_scale_normal(float r2, float m) {
  const float y = __builtin_amdgcn_rsqf(r2);
  const float g = r2 * y;
  const float root = __builtin_fmaf(__builtin_fmaf(-g, g, r2), 0.5f * y, g);
  const float b = r2 * root;
  const float c0 = y * y * y;
  const float c = __builtin_fmaf(__builtin_fmaf(-b, c0, 1.0f), c0, c0);
  const float q = m * c;
  return __builtin_fmaf(__builtin_fmaf(-b, q, m), c, q);
}

// Force: the sum over j is a chain of fma in increasing order of j, which fixes
// the result's bits, but a pair's scale depends on nothing else.  A workgroup
// takes kForceBodies bodies; its first wavefront keeps the chains (lane i the
// x sum of body i, lane i + 32 its y sum), the others compute the scales of
// kForceChunk bodies j at a time into one of two LDS tiles, one tile ahead of
// the chains.  Bound: vector instructions on large sets (about 26 issue slots
// per pair, a reciprocal root counting four), the chains' latency on small
// ones.  With one wavefront per 64 bodies for everything, 4096 bodies kept 64
// of the chip's 1024 SIMDs busy with a chain of about 45 slots per pair: 307 us
// per step; now 37, and 65,536 bodies 4.93 -> 2.76 ms (5.5e10 -> 4.5e11 pairs a
// second and 8.7e11 -> 1.55e12).  Tiles of 64 bodies cost a barrier twice as
// often (4096 bodies 47, 65,536 2.98 ms), tiles of 256 leave room for two
// workgroups per CU (4.4 ms); two makers leave SIMDs idle (65,536: 3.1 ms),
// eight wait for the chains (3.4 ms).
constexpr uint32_t kKindForce = 60;
constexpr uint32_t kForceBodies = 32;
constexpr uint32_t kForceChunk = 128;
constexpr uint32_t kForceMakers = 4;                           // wavefronts computing scales
constexpr uint32_t kForceEach = kForceChunk / kForceMakers;    // bodies j per maker and chunk
constexpr uint32_t kForceThreads = 64 * (kForceMakers + 1);
constexpr uint32_t kForceWgsPerCu = 4;                         // resident: the two tiles take 40 KB of LDS
constexpr uint32_t kForceRow = kForceChunk + 4;                // padded: rows start 4 banks apart
static_assert(kForceEach % 8 == 0 && kForceEach <= 64, "two half-wavefronts, four scales per store");

template <uint32_t LG>
__global__ void __launch_bounds__(kForceThreads)
    force_kernel(DevHeapW<LG> h, const uint32_t* __restrict__ R, const uint64_t* __restrict__ S,
                 const uint32_t* count_ptr, Bodies a) {
  __shared__ float s_scale[2][kForceBodies * kForceRow];
  __shared__ float s_q[2][2][kForceChunk];   // x and y of the chunk's bodies
  __shared__ float4 s_p[2][kForceChunk];
  const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t i = lane & (kForceBodies - 1), half = lane >> 5;
  const uint32_t c = cap_of(h, kBody), sh = (uint32_t)__builtin_ctz(c);
  const uint64_t items = (uint64_t)bcast32(*count_ptr) << sh;  // slots of the listed blocks
  const uint32_t n = a.n, chunks = (n + kForceChunk - 1) / kForceChunk;
  uint32_t visits = 0;
  // The bodies enter the cells' table anew in each step's Move.
  if (a.head) {
    for (uint64_t b = (uint64_t)blockIdx.x * kForceThreads + threadIdx.x; b <= a.mask; b += (uint64_t)gridDim.x * kForceThreads)
      a.head[b] = kNoBody;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.far_out = 0;
  }
  for (uint64_t g = blockIdx.x; g * kForceBodies < items; g += gridDim.x) {
    const uint64_t u = g * kForceBodies + i;
    const uint32_t e = (uint32_t)((u < items ? u : items - 1) >> sh), slot = (uint32_t)u & (c - 1);
    const bool live = u < items && ((S[e] >> slot) & 1ull);
    const uint32_t self = make_obj(R[e], slot);
    // Slots without a body stand at the origin: they take the same path and write nothing.
    const float x = live ? fld<float>(h, self, kX) : 0.0f, y = live ? fld<float>(h, self, kY) : 0.0f;
    if (wave == 0) visits += (uint32_t)__popcll(__ballot(live && half == 0));
    const float own = half ? y : x;  // chains
    float sum = 0.0f;
    // Makers: lane l loads entry l % kForceEach of its wavefront's part, one
    // chunk ahead (clamped to the last id), and computes kForceEach / 2 scales.
    const uint32_t part = wave == 0 ? 0u : (wave - 1) * kForceEach, mine = part + (lane & (kForceEach - 1));
    const bool own_ok = !__ballot(!(__builtin_fabsf(x) <= 0x1p18f && __builtin_fabsf(y) <= 0x1p18f)) &&
                        a.eps2 >= kScaleLo && a.eps2 <= 0x1p38f;
    float4 nxt = a.P[mine < n ? mine : n - 1];
    // Tile k is made while the chains take tile k - 1.
    for (uint32_t k = 0; k <= chunks; ++k) {
      if (wave == 0) {
        const uint32_t t = (k - 1) & 1, j0 = (k - 1) * kForceChunk;
        const float* sc = s_scale[t] + i * kForceRow;
        const float* q = s_q[t][half];
        if (k == 0) {
        } else if (n - j0 >= kForceChunk) {
#pragma unroll 4
          for (uint32_t j = 0; j < kForceChunk; j += 4) {
            const float4 s4 = *reinterpret_cast<const float4*>(sc + j), q4 = *reinterpret_cast<const float4*>(q + j);
            sum = __builtin_fmaf(s4.x, q4.x - own, sum);
            sum = __builtin_fmaf(s4.y, q4.y - own, sum);
            sum = __builtin_fmaf(s4.z, q4.z - own, sum);
            sum = __builtin_fmaf(s4.w, q4.w - own, sum);
          }
        } else {
          for (uint32_t j = 0; j < n - j0; ++j) sum = __builtin_fmaf(sc[j], q[j] - own, sum);
        }
      } else if (k < chunks) {
        const uint32_t t = k & 1, j1 = (k + 1) * kForceChunk + mine;
        const float4 p = nxt;
        nxt = a.P[j1 < n ? j1 : n - 1];
        s_p[t][mine] = p;
        s_q[t][0][mine] = p.x;
        s_q[t][1][mine] = p.y;
        __builtin_amdgcn_wave_barrier();  // this wavefront reads back its own part below
        // With every coordinate within 2^18, r2 lies between eps2 and 2^40.
        const bool ok = own_ok && !__ballot(!(__builtin_fabsf(p.x) <= 0x1p18f && __builtin_fabsf(p.y) <= 0x1p18f &&
                                              scale_normal_mass(p.z)));
        const uint32_t j0 = part + half * (kForceEach / 2);
        const float4* pj = s_p[t] + j0;
        float* out = s_scale[t] + i * kForceRow + j0;
        auto r2_of = [&](const float4& q) {
          const float dx = q.x - x, dy = q.y - y;
          return __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, a.eps2));
        };
        if (ok) {
#pragma unroll
          for (uint32_t j = 0; j < kForceEach / 2; j += 4) {
            const float4 q0 = pj[j], q1 = pj[j + 1], q2 = pj[j + 2], q3 = pj[j + 3];
            *reinterpret_cast<float4*>(out + j) =
                make_float4(pair_scale_normal(r2_of(q0), q0.z), pair_scale_normal(r2_of(q1), q1.z),
                            pair_scale_normal(r2_of(q2), q2.z), pair_scale_normal(r2_of(q3), q3.z));
          }
        } else {
          for (uint32_t j = 0; j < kForceEach / 2; ++j) out[j] = pair_scale(r2_of(pj[j]), pj[j].z);
        }
      }
      __syncthreads();
    }
    if (wave == 0 && live) {
      if (half == 0) fld<float>(h, self, kAX) = sum;
      else fld<float>(h, self, kAY) = sum;
    }
  }
  if (visits) lead_add(shard(h) + kCntVisits + kBody, visits);
}

// Cells of the merge phases: squares of side 4/3 merge radius, hashed into a
// table of at least four buckets per body; a bucket chains its bodies through
// P's link.  Bodies within the radius (by the computed test, whose difference
// is off by at most 2^-23 of itself) lie less than 0.75 (1 + 2^-20) cells
// apart, and a cell coordinate of at most kFarCells is off by at most 2^-4, so
// they lie in the same cell or in neighbouring ones.  A body beyond that range
// (or at a NaN) sets far_out, and the merge phases of that step scan all ids.
constexpr float kFarCells = 0x1p20f;
__device__ __forceinline__ uint32_t bucket(const Bodies& a, int32_t cx, int32_t cy) {
  return hash32((uint32_t)cx * 0x9E3779B1u + (uint32_t)cy) & a.mask;
}
__device__ __forceinline__ bool in_cells(const Bodies& a, float x, float y) {
  return __builtin_fabsf(x * a.inv_cell) <= kFarCells && __builtin_fabsf(y * a.inv_cell) <= kFarCells;
}
__device__ __forceinline__ int32_t cell_of(const Bodies& a, float v) { return (int32_t)floorf(v * a.inv_cell); }

struct BodyMove {
  static constexpr uint32_t kKind = 61;
  using Args = Bodies;
  template <class H>
  static __device__ bool run(const H& h, uint32_t, uint32_t self, const Args& a) {
    const float vx = __builtin_fmaf(a.dt, fld<float>(h, self, kAX), fld<float>(h, self, kVX));
    const float vy = __builtin_fmaf(a.dt, fld<float>(h, self, kAY), fld<float>(h, self, kVY));
    const float x = __builtin_fmaf(a.dt, vx, fld<float>(h, self, kX));
    const float y = __builtin_fmaf(a.dt, vy, fld<float>(h, self, kY));
    fld<float>(h, self, kVX) = vx;
    fld<float>(h, self, kVY) = vy;
    fld<float>(h, self, kX) = x;
    fld<float>(h, self, kY) = y;
    const uint32_t id = fld<uint32_t>(h, self, kId);
    uint32_t link = kNoBody;
    if (a.head) {
      if (in_cells(a, x, y)) link = atomicExch(a.head + bucket(a, cell_of(a, x), cell_of(a, y)), id);
      else *a.far_out = 1;
    }
    a.P[id] = make_float4(x, y, fld<float>(h, self, kM), __uint_as_float(link));
    a.V[id] = make_float2(vx, vy);
    return false;
  }
};

__device__ __forceinline__ bool within(const Bodies& a, float qx, float qy, float x, float y) {
  const float dx = qx - x, dy = qy - y;
  return __builtin_fmaf(dx, dx, dy * dy) < a.r2_merge;
}

// f(j, P[j]) for every body j in the nine cells around (x, y) of each lane with
// `on` (some more than once when cells share a bucket, in no order).  All
// lanes enter.  The nine chains advance together, one round of loads for all
// of them; a lane whose chains are longer than kNearRounds (a crowd: more
// bodies in a bucket than a scan is worth waiting for) gets false and has seen
// only part.
constexpr uint32_t kNearRounds = 16;
template <class F>
__device__ __forceinline__ bool walk_near(const Bodies& a, bool on, float x, float y, F&& f) {
  const int32_t cx = on ? cell_of(a, x) : 0, cy = on ? cell_of(a, y) : 0;
  uint32_t j[9];
#pragma unroll
  for (int32_t c = 0; c < 9; ++c) {
    const uint32_t first = a.head[bucket(a, cx + c % 3 - 1, cy + c / 3 - 1)];
    j[c] = on ? first : kNoBody;
  }
  bool more = true;
  for (uint32_t round = 0; round < kNearRounds && __ballot(more); ++round) {
    float4 q[9];
#pragma unroll
    for (uint32_t c = 0; c < 9; ++c) q[c] = a.P[j[c] < a.n ? j[c] : a.n - 1u];
    more = false;
#pragma unroll
    for (uint32_t c = 0; c < 9; ++c) {
      if (j[c] == kNoBody) continue;
      f(j[c], q[c]);
      j[c] = __float_as_uint(q[c].w);
      more |= j[c] != kNoBody;
    }
  }
  return !more;
}

// Whether this step's merge phases may use the cells.
__device__ __forceinline__ bool have_cells(const Bodies& a) { return a.head && bcast32(*a.far_out) == 0; }

struct BodyRoot {
  static constexpr uint32_t kKind = 62;
  using Args = Bodies;
  static __device__ __forceinline__ float d2(const Args& a, float4 c, uint32_t k, float x, float y) {
    const float dx = from_lane(c.x, k) - x, dy = from_lane(c.y, k) - y;
    return __builtin_fmaf(dx, dx, dy * dy);
  }
  // The scan: the smallest squared distance to a live body of lower id is
  // below r2_merge (a NaN distance is never below it, on either side of this
  // equivalence).  Lanes with nothing to search pass id 0.
  static __device__ bool scan(const Args& a, uint32_t id, float x, float y) {
    const uint32_t n = a.n, lane = lane_id();
    float best = __builtin_inff();
    float4 nxt = a.P[chunk_id(0, n)];
    for (uint32_t j0 = 0; __ballot((j0 < id) & !(best < a.r2_merge)); j0 += 64) {
      const float4 cur = nxt;
      nxt = a.P[chunk_id(j0 + 64, n)];
      uint64_t alive = __ballot((cur.z > 0.0f) & (j0 + lane < n));  // live bodies of this chunk
      if (!__ballot(j0 + 64 > id)) {  // every lane's id lies above the chunk
        if (alive == ~0ull) {
#pragma unroll 8
          for (uint32_t k = 0; k < 64; ++k) best = fminf(best, d2(a, cur, k, x, y));
        } else {
          for (; alive; alive &= alive - 1ull) best = fminf(best, d2(a, cur, (uint32_t)__builtin_ctzll(alive), x, y));
        }
      } else {
        for (; alive; alive &= alive - 1ull) {
          const uint32_t k = (uint32_t)__builtin_ctzll(alive);
          const float d = d2(a, cur, k, x, y);
          if (j0 + k < id) best = fminf(best, d);
        }
      }
    }
    return best < a.r2_merge;
  }
  // Bound: the latency of two or three rounds of loads.  Scanning every lower
  // id took 224 us per step for 4096 bodies and 3.7 ms for 65,536, whose cells
  // hold half a body or fewer; with the cells a whole step takes 70 us and
  // 2.77 ms (before: 311 us and 6.9 ms with this force kernel).
  template <class H>
  static __device__ bool run_wave(const H& h, uint32_t, uint32_t self, bool live, const Args& a) {
    const float x = fld<float>(h, self, kX), y = fld<float>(h, self, kY);
    const uint32_t id = live ? fld<uint32_t>(h, self, kId) : 0u;
    bool near = false, left = live;
    if (have_cells(a)) {
      const bool all = walk_near(a, live, x, y, [&](uint32_t j, const float4& q) {
        near |= j < id && within(a, q.x, q.y, x, y);
      });
      left = live && !all && !near;
    }
    if (__ballot(left)) {
      const bool found = scan(a, left ? id : 0u, x, y);
      near |= left && found;
    }
    if (live) a.T[id] = near ? kAlone : kRoot;
    return false;
  }
};

struct BodyTarget {
  static constexpr uint32_t kKind = 63;
  using Args = Bodies;
  // Few bodies per step are not roots; those that the cells do not serve are
  // searched for by the wavefront in turn, 64 candidate ids at a time (one id
  // per lane).
  template <class H>
  static __device__ bool run_wave(const H& h, uint32_t, uint32_t self, bool live, const Args& a) {
    const uint32_t id = live ? fld<uint32_t>(h, self, kId) : 0u;
    const bool need = live && a.T[id] != kRoot;
    if (!__ballot(need)) return false;
    const float x = fld<float>(h, self, kX), y = fld<float>(h, self, kY);
    const uint32_t n = a.n, lane = lane_id();
    uint32_t found = kAlone;
    bool left = need;
    if (have_cells(a)) {
      // Only roots' entries of T are compared, and they do not change here.
      const bool all = walk_near(a, need, x, y, [&](uint32_t j, const float4& q) {
        if (j < found && within(a, q.x, q.y, x, y) && a.T[j] == kRoot) found = j;
      });
      left = need && !all;
    }
    uint64_t pending = __ballot(left);
    while (pending) {
      const uint32_t i = (uint32_t)__builtin_ctzll(pending);
      pending &= pending - 1ull;
      const float xi = from_lane(x, i), yi = from_lane(y, i);
      uint32_t hit = kAlone;
      uint32_t tn = a.T[chunk_id(0, n)];
      float4 pn = a.P[chunk_id(0, n)];
      for (uint32_t j0 = 0; j0 < n; j0 += 64) {
        const uint32_t tc = tn;
        const float4 pc = pn;
        tn = a.T[chunk_id(j0 + 64, n)];
        pn = a.P[chunk_id(j0 + 64, n)];
        const uint64_t ok = __ballot((j0 + lane < n) & (tc == kRoot) & within(a, pc.x, pc.y, xi, yi));
        if (ok) {  // the lowest such id
          hit = j0 + (uint32_t)__builtin_ctzll(ok);
          break;
        }
      }
      if (lane == i) found = hit;
    }
    if (need && found != kAlone) a.T[id] = found;
    return false;
  }
};

// Merge and removal.  A body that merges is read by its root alone (T names
// it), which marks it dead once it has its values; other roots may pass it in
// a chain, where only its link counts for them.  Up to kScanMerge bodies a scan
// of T is shorter than the walks, of which a root takes one more than it absorbs
// (us, scan and walks: 64 bodies 4.2 and 6.8, 400 5.5 and 8.4, 1000 9.5 and 10.4,
// 1500 12.3 and 9.6, 4096 24 and 11).
constexpr uint32_t kScanMerge = 1024;
struct BodyMerge {
  static constexpr uint32_t kKind = 64;
  static constexpr uint32_t kPhases = 2;
  static constexpr bool kDeletesOnlyThis = true;
  using Args = Bodies;
  template <class H>
  static __device__ bool run_wave(const H& h, uint32_t, uint32_t self, bool live, const Args& a) {
    const uint32_t id = live ? fld<uint32_t>(h, self, kId) : 0u;
    const uint32_t n = a.n, target = live ? a.T[id] : kAlone;
    const bool root = target == kRoot, merges = target < n;
    if (!__ballot(root)) return merges;
    const float m = fld<float>(h, self, kM), x = fld<float>(h, self, kX), y = fld<float>(h, self, kY);
    const float vx = fld<float>(h, self, kVX), vy = fld<float>(h, self, kVY);
    float M = m, px = m * vx, py = m * vy, cx = m * x, cy = m * y;
    bool absorbed = false;
    auto absorb = [&](uint32_t j) {
      const float4 q = a.P[j];
      const float2 w = a.V[j];
      M = M + q.z;
      px = __builtin_fmaf(q.z, w.x, px);
      py = __builtin_fmaf(q.z, w.y, py);
      cx = __builtin_fmaf(q.z, q.x, cx);
      cy = __builtin_fmaf(q.z, q.y, cy);
      a.P[j].z = 0.0f;
      absorbed = true;
    };
    bool left = root;
    if (n > kScanMerge && have_cells(a)) {
      // The bodies merging into this root, in increasing id order: each walk
      // finds the lowest id from `lo` on.
      bool on = root;
      uint32_t lo = 0;
      for (bool first = true; __ballot(on); first = false) {
        uint32_t j1 = kNoBody;
        const bool all = walk_near(a, on, x, y, [&](uint32_t j, const float4& q) {
          if (j >= lo && j < j1 && within(a, q.x, q.y, x, y) && a.T[j] == id) j1 = j;
        });
        if (first) left = on && !all;
        on = on && all && j1 != kNoBody;
        if (on) {
          absorb(j1);
          lo = j1 + 1;
        }
      }
    }
    if (__ballot(left)) {
      uint32_t tn = a.T[chunk_id(0, n)];
      for (uint32_t j0 = 0; j0 < n; j0 += 64) {
        const uint32_t tc = tn, j = chunk_id(j0, n);
        tn = a.T[chunk_id(j0 + 64, n)];
        // Live ids that merge into a root (T of dead ones is an earlier step's).
        uint64_t moving = __ballot(tc < n && j0 + lane_id() < n && a.P[j].z > 0.0f);
        while (moving) {  // in increasing id order
          const uint32_t k = (uint32_t)__builtin_ctzll(moving);
          moving &= moving - 1ull;
          if (left && id == from_lane(tc, k)) absorb(j0 + k);
        }
      }
    }
    if (absorbed) {
      const float nvx = px / M, nvy = py / M;
      const float nx = cx / M, ny = cy / M;
      fld<float>(h, self, kVX) = nvx;
      fld<float>(h, self, kVY) = nvy;
      fld<float>(h, self, kX) = nx;
      fld<float>(h, self, kY) = ny;
      fld<float>(h, self, kM) = M;
      a.P[id].x = nx;  // the link stays: other roots may be walking through it
      a.P[id].y = ny;
      a.P[id].z = M;
      a.V[id] = make_float2(nvx, nvy);
    }
    return merges;
  }
};

// Bodies with m > 0 become objects; every id's P and V entries are set.
template <uint32_t LG>
__global__ void collide_init_kernel(DevHeapW<LG> h, Bodies a, const float* x, const float* y, const float* vx,
                                    const float* vy, const float* m) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  a.P[i] = make_float4(x[i], y[i], m[i] > 0.0f ? m[i] : 0.0f, 0.0f);
  a.V[i] = make_float2(vx[i], vy[i]);
  a.T[i] = kAlone;
  new_many(h, kBody, m[i] > 0.0f ? 1u : 0u, [&](uint32_t, uint32_t o) {
    if (o == kNull) return;
    fld<float>(h, o, kX) = x[i];
    fld<float>(h, o, kY) = y[i];
    fld<float>(h, o, kVX) = vx[i];
    fld<float>(h, o, kVY) = vy[i];
    fld<float>(h, o, kAX) = 0.0f;
    fld<float>(h, o, kAY) = 0.0f;
    fld<float>(h, o, kM) = m[i];
    fld<uint32_t>(h, o, kId) = i;
  });
}

__global__ void collide_read_kernel(Bodies a, float* x, float* y, float* vx, float* vy, float* m) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const float4 p = a.P[i];
  const float2 v = a.V[i];
  x[i] = p.x;
  y[i] = p.y;
  vx[i] = v.x;
  vy[i] = v.y;
  m[i] = p.z;
}

bool collide_heap_ok(const dsoar_heap* h) {
  if (h->desc.num_types < 1) return false;
  const dsoar_type_layout& L = h->desc.types[kBody];
  if (L.num_fields < 8) return false;
  for (uint32_t f = 0; f < 8; ++f)
    if (L.field_bytes[f] != 4) return false;
  return true;
}

}  // namespace
}  // namespace dsoar

using namespace dsoar;

struct dsoar_collide {
  dsoar_heap* heap;
  Bodies a;
  StepGraphs graphs;
};

namespace {

// The do-all of the force over the bodies (see force_kernel): a workgroup per
// kForceBodies slots of the listed blocks.  The list's length is known on the
// device only, so the grid is the most groups it can have, up to what the chip
// holds at once, and loops.
int launch_force(dsoar_heap* h, const Bodies& a, uint32_t flags, hipStream_t st) {
  int rc = launch_enumerate(h, kBody, st);
  if (rc) return rc;
  const EnumOut& eo = h->enum_out[kBody];
  uint64_t blocks = h->dev.num_blocks;
  if (flags & DSOAR_DO_PLAIN) {
    uint32_t count = 0;
    rc = read_count(h, kBody, st, &count);
    if (rc) return rc;
    if (count == 0) return DSOAR_OK;
    blocks = count;
  }
  const uint64_t groups = (blocks * h->dev.capacity[kBody] + kForceBodies - 1) / kForceBodies;
  const uint64_t most = (uint64_t)h->num_cus * kForceWgsPerCu;
  with_width(h, [&](auto w_) {
    constexpr uint32_t kLG = decltype(w_)::value;
    launch_timed(h, kKindForce, force_kernel<kLG>, dim3((uint32_t)(groups < most ? groups : most)), dim3(kForceThreads),
                 st, DevHeapW<kLG>(h->dev), (const uint32_t*)eo.R, (const uint64_t*)eo.S,
                 (const uint32_t*)&eo.st->count, a);
  });
  DSOAR_LAUNCHED(h);
  return DSOAR_OK;
}

int collide_one_step(dsoar_collide* c, uint32_t flags, hipStream_t st) {
  dsoar_heap* h = c->heap;
  const uint32_t base = flags & DSOAR_DO_PLAIN, reuse = base | DSOAR_DO_REUSE_ENUM;
  int rc = launch_force(h, c->a, base, st);
  if (!rc) rc = launch_doall<BodyMove>(h, kBody, c->a, reuse, st);
  // No squared distance is below a merge radius of 0: the bodies then never
  // merge (the paper's nbody application), and the merge phases would change
  // nothing.
  if (!(c->a.r2_merge > 0.0f)) return rc;
  if (!rc) rc = launch_doall<BodyRoot>(h, kBody, c->a, reuse, st);
  if (!rc) rc = launch_doall<BodyTarget>(h, kBody, c->a, reuse, st);
  if (!rc) rc = launch_doall<BodyMerge>(h, kBody, c->a, reuse, st);
  return rc;
}

size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// Buckets of the cells' table: a power of two, four or more per body.
size_t cell_buckets(uint32_t n) {
  size_t b = 64;
  while (b < (size_t)n * 4) b *= 2;
  return b;
}

}  // namespace

extern "C" {

size_t dsoar_collide_bytes(uint32_t n) {
  if (n == 0 || n > (1u << 24)) return 0;
  return align256((size_t)n * 16) + align256((size_t)n * 8) + align256((size_t)n * 4);
}

size_t dsoar_collide_bytes_cells(uint32_t n) {
  const size_t b = dsoar_collide_bytes(n);
  return b ? b + 256 + cell_buckets(n) * 4 : 0;
}

int dsoar_collide_create(dsoar_heap* heap, uint32_t n, const dsoar_collide_params* params, void* dev_mem,
                         size_t dev_bytes, dsoar_collide** out) {
  if (!out) return DSOAR_ERR_INVALID_ARG;
  *out = nullptr;
  if (!heap_ok(heap) || !collide_heap_ok(heap) || !params || !dev_mem || ((uintptr_t)dev_mem & 255u) ||
      !(params->eps2 > 0.0f) || !(params->r2_merge >= 0.0f))
    return DSOAR_ERR_INVALID_ARG;
  const size_t need = dsoar_collide_bytes(n);
  if (need == 0) return DSOAR_ERR_INVALID_ARG;
  if (dev_bytes < need) return DSOAR_ERR_TOO_SMALL;
  dsoar_collide* c = new (std::nothrow) dsoar_collide;
  if (!c) return DSOAR_ERR_INVALID_ARG;
  memset(c, 0, sizeof(*c));
  c->heap = heap;
  uint8_t* b = (uint8_t*)dev_mem;
  c->a.P = (float4*)b;
  c->a.V = (float2*)(b + align256((size_t)n * 16));
  c->a.T = (uint32_t*)(b + align256((size_t)n * 16) + align256((size_t)n * 8));
  c->a.n = n;
  c->a.dt = params->dt;
  c->a.eps2 = params->eps2;
  c->a.r2_merge = params->r2_merge;
  // The cells serve radii whose squares do not run into the ends of the range;
  // a buffer without room for their table keeps the scans.
  if (dev_bytes >= dsoar_collide_bytes_cells(n) && params->r2_merge >= 0x1p-60f &&
      params->r2_merge <= 0x1p60f) {
    c->a.far_out = (uint32_t*)(b + need);
    c->a.head = c->a.far_out + 64;
    c->a.mask = (uint32_t)(cell_buckets(n) - 1);
    c->a.inv_cell = 0.75f / sqrtf(params->r2_merge);
  }
  *out = c;
  return DSOAR_OK;
}

int dsoar_collide_destroy(dsoar_collide* c) {
  if (!c) return DSOAR_ERR_INVALID_ARG;
  step_graphs_clear(c->graphs);
  delete c;
  return DSOAR_OK;
}

int dsoar_collide_init(dsoar_collide* c, const float* x_dev, const float* y_dev, const float* vx_dev,
                       const float* vy_dev, const float* m_dev, void* stream) {
  if (!c || !x_dev || !y_dev || !vx_dev || !vy_dev || !m_dev) return DSOAR_ERR_INVALID_ARG;
  with_width(c->heap, [&](auto w_) {
    constexpr uint32_t kLG = decltype(w_)::value;
    launch_timed(c->heap, kKindCollideInit, collide_init_kernel<kLG>, dim3((uint32_t)(((uint64_t)c->a.n + 255) / 256)), dim3(256), (hipStream_t)stream, DevHeapW<kLG>(c->heap->dev),
                     c->a, x_dev, y_dev, vx_dev, vy_dev, m_dev);
  });
  DSOAR_LAUNCHED(c->heap);
  return DSOAR_OK;
}

int dsoar_collide_step(dsoar_collide* c, uint32_t steps, uint32_t flags, void* stream) {
  if (!c) return DSOAR_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  dsoar_heap* h = c->heap;
  if (flags & DSOAR_GRAPH) {
    if (flags & DSOAR_DO_PLAIN) return DSOAR_ERR_INVALID_ARG;
    return step_graphs_run(h, c->graphs, steps, st, [&](hipStream_t gs) { return collide_one_step(c, 0, gs); });
  }
  for (uint32_t i = 0; i < steps; ++i) {
    const int rc = collide_one_step(c, flags, st);
    if (rc) return rc;
  }
  return DSOAR_OK;
}

int dsoar_collide_read(dsoar_collide* c, float* x_dev, float* y_dev, float* vx_dev, float* vy_dev, float* m_dev,
                       void* stream) {
  if (!c || !x_dev || !y_dev || !vx_dev || !vy_dev || !m_dev) return DSOAR_ERR_INVALID_ARG;
  hipLaunchKernelGGL(collide_read_kernel, dim3((uint32_t)(((uint64_t)c->a.n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, c->a, x_dev,
                     y_dev, vx_dev, vy_dev, m_dev);
  DSOAR_LAUNCHED(c->heap);
  return DSOAR_OK;
}

}  // extern "C"
