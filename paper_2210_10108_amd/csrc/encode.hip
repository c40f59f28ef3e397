// Multiresolution hash encoding of the samples (Sec. III, Instant NGP): the
// gather of every level's 8 vertex features, their trilinear blend, and the
// blend's derivative with respect to the sample position (the table is frozen,
// so the backward pass needs nothing else from it: the MLP backward kernel
// contracts this Jacobian with d loss / d feature, and nothing is re-gathered
// or scattered).
//
// Work split: one group of levels at a time per work item (see k_encode): every
// XCD (own 4 MB L2) works on one group's tables at a time, its home groups
// first.
//
// Hashed levels: two adjacent lanes handle one sample: lane side 0 gathers the
// four vertices at the cell's lower x, side 1 the four at x + 1.  The two x
// neighbours of a vertex nearly always share a cache line: the spatial hash
// (x ^ y' ^ z') of x and x + 1 differs only in the bits that the carry of x + 1
// flips, the lowest bit for even x.  Each gather instruction so touches about
// half as many lines as with one lane per sample, and the gather's cost follows
// the lines: a line that misses the CU's L1 takes 2.25 cycles from L2 at best
// (measured over 1 to 4 MB).  Each lane blends its half; one lane-pair exchange
// completes the sums.  Dense levels take one lane per sample (dense_item).
//
// What bounds it: 4 lines per sample and hashed level, fetched from L2 with about
// 65 of them in flight per CU (tables of 4 MiB; 83 with 16 MiB tables, whose lines
// come from memory, so 65 is no cap of the L1), at half the rate above.  More
// wavefronts do not raise it (4 and 7 blocks per CU are within 1 % of each other
// on large batches).  Then the texture unit (16 cycles for any gather
// instruction, 32 for a 16-byte load) and the vector work beside it.  On
// 39.5 M samples (16 levels, 2^19 entries, fp32) the kernel takes 7.7 ms
// against 8.6 ms with per-lane ray lookups, positions recovered in float and a
// queue per dense level; with every gather in L1 it took 5.0 ms, without
// gathers 4.2 ms.
//
// Features are stored by blocks of 16 samples (a column tile of the MLP
// kernels): block b, lane group g = l % 4, level l / 4 of the group, sample
// s % 16, feature q at ((4 b + g) LPG + l / 4) 32 + (s % 16) 2 + q.  A level's
// share of a block is one cache line, written by one instruction, and a lane of
// the network kernel reads a level's two features with one 8-byte load at a
// constant offset from its tile (rows of one feature each took twice the loads
// and an address each).  The Jacobian d feature /
// d pos of every level (pos = x N_l: bounded by the table's value
// differences, zero along clamped components) is stored in fp16 (rounding
// below 2^-11 of each entry), as one 12-byte record per sample and level: three
// words, (q, a) = (0, 0) (0, 1), then (1, 0) (1, 1), then (0, 2) (1, 2) of
// d feature_q / d pos_a, grouped in blocks of 32 samples: block b, lane group
// g = l % 4, level l / 4 of the group, sample s % 32, at record
// (4 b + g) LPG 32 + (l / 4) 32 + s % 32.  The MLP backward kernel reads each of
// its samples' records of a lane group with one 12-byte load per level, and the
// 32 records of one level and block fill 3 whole cache lines, so no line is
// written from two XCDs.  That kernel applies N_l and 1 / extent in fp32.
#include <algorithm>

#include "pnerf_internal.h"

namespace pnerf {
namespace {

constexpr int kBlock = 256;
constexpr int kFeatBlock = 16 * 8;  // bytes of one level's features of a 16-sample block
constexpr int kJacBlock = 32 * 12;  // bytes of one level's Jacobian records of a 32-sample block
constexpr uint32_t kPrime1 = 2654435761u, kPrime2 = 805459861u;

struct Pos {
  float x[3];        // normalised, clamped position in [0,1]^3 (decides cells)
  float dx[3];       // exact normalised position minus x (0 where clamped)
};

// Sample position p = o + t d and x = (p - min) / extent.  The float chain
// (separately rounded, never fused) decides cells and clamping; x in double,
// along the ray's direction in double, gives dx, what float cannot hold of the
// position, so that interpolation weights are accurate to float precision.
// (The double chain is 21 instructions for the three axes; recovering every
// rounding error of the float chain in float took about 50.)
// clamped: bit a set where component a was clamped.  A sample is clamped only
// when rounding puts it outside the box (or its pose is not finite), so the
// clamps run behind a test of the whole wavefront: 0 <= x <= 1 as unsigned
// bit patterns (negative values, -0 and NaN are all above 1's).
__device__ __forceinline__ Pos sample_pos(const DevField& f, float t, const RayRecord& r,
                                          uint32_t& clamped) {
  Pos ps;
  float o[3], d[3];
  double D[3];
  r.origin(o);
  r.dir(d);
  r.dir64(D);
  const double t64 = (double)t;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float p = __fadd_rn(o[a], __fmul_rn(t, d[a]));
    ps.x[a] = __fmul_rn(__fsub_rn(p, f.mn[a]), f.inv_ext[a]);
    const double x64 = (fma(t64, D[a], (double)o[a]) - f.mn64[a]) * f.inv64[a];
    ps.dx[a] = (float)(x64 - (double)ps.x[a]);
  }
  clamped = 0;
  const uint32_t top = max(max(__float_as_uint(ps.x[0]), __float_as_uint(ps.x[1])),
                           __float_as_uint(ps.x[2]));
  if (__any(top > 0x3F800000u)) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (!(ps.x[a] >= 0.0f)) {  // below the box (or NaN from a non-finite pose)
        ps.x[a] = 0.0f;
        ps.dx[a] = 0.0f;
        clamped |= 1u << a;
      } else if (ps.x[a] > 1.0f) {
        ps.x[a] = 1.0f;
        ps.dx[a] = 0.0f;
        clamped |= 1u << a;
      }
    }
  }
  return ps;
}

// The value held by lane ODD of each lane pair, in both lanes of the pair
// (DPP quad_perm [0,0,2,2] or [1,1,3,3]; all lanes active).
template <int ODD>
__device__ __forceinline__ float from_pair_lane(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), ODD ? 0xF5 : 0xA0, 0xF, 0xF, true));
}

template <int ODD>
__device__ __forceinline__ Pos pos_from_pair_lane(const Pos& p) {
  Pos r;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    r.x[a] = from_pair_lane<ODD>(p.x[a]);
    r.dx[a] = from_pair_lane<ODD>(p.dx[a]);
  }
  return r;
}

// Cell of one level: lower corner, interpolation weights, and the table index
// of corner k (bit 0: x + 1, bit 1: y + 1, bit 2: z + 1).
struct Cell {
  float w[3];
  uint32_t i0[3];
};

// The cell comes from the float product x N (as a reference implementation in
// float decides it); the weights are x N - cell, rounded once, plus N dx, the
// part of the position float cannot hold.
__device__ __forceinline__ void make_cell(int N, const float x[3], const float dx[3], Cell& c) {
  const float Nf = (float)N;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float pos = __fmul_rn(x[a], Nf);
    int ci = (int)pos;
    ci = ci < N - 1 ? ci : N - 1;
    c.i0[a] = (uint32_t)ci;
    c.w[a] = fmaf(Nf, dx[a], fmaf(x[a], Nf, -(float)ci));
  }
}

__device__ __forceinline__ uint32_t corner_index(const DevField& f, int l, const Cell& c, int k) {
  const bool dense = f.dense[l] != 0;
  const uint32_t n1 = f.n1[l];
  const uint32_t sy = dense ? n1 : kPrime1;
  const uint32_t sz = dense ? n1 * n1 : kPrime2;
  const uint32_t xi = c.i0[0] + (k & 1);
  const uint32_t yi = (c.i0[1] + ((k >> 1) & 1)) * sy;
  const uint32_t zi = (c.i0[2] + ((k >> 2) & 1)) * sz;
  const uint32_t h = dense ? (xi + yi + zi) : ((xi ^ yi ^ zi) & (f.T - 1u));
  return (uint32_t)l * f.T + h;
}

template <bool F16>
__device__ __forceinline__ float2 vertex(const DevField& f, uint32_t idx) {
  if (F16) {
    __half2 v = reinterpret_cast<const __half2*>(f.table16)[idx];
    return __half22float2(v);
  }
  return reinterpret_cast<const float2*>(f.table32)[idx];
}

// Feature (2 values) of level l at position x -- blend of the 8 vertices --
// and, when jac != nullptr, its derivative with respect to the level's grid
// coordinate (jac[3 q + a] = d feature_q / d pos_a, pos = x N).
template <bool F16>
__device__ __forceinline__ float2 level_feature(const DevField& f, int l, const float x[3],
                                                const float dx[3], float* jac) {
  Cell c;
  make_cell(f.res[l], x, dx, c);
  float2 v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = vertex<F16>(f, corner_index(f, l, c, k));
  const float wx = c.w[0], wy = c.w[1], wz = c.w[2];
  const float ux = 1.0f - wx, uy = 1.0f - wy, uz = 1.0f - wz;
  float2 r;
  r.x = uz * (uy * (ux * v[0].x + wx * v[1].x) + wy * (ux * v[2].x + wx * v[3].x)) +
        wz * (uy * (ux * v[4].x + wx * v[5].x) + wy * (ux * v[6].x + wx * v[7].x));
  r.y = uz * (uy * (ux * v[0].y + wx * v[1].y) + wy * (ux * v[2].y + wx * v[3].y)) +
        wz * (uy * (ux * v[4].y + wx * v[5].y) + wy * (ux * v[6].y + wx * v[7].y));
  if (jac) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) t[k] = q ? v[k].y : v[k].x;
      jac[3 * q + 0] = uy * uz * (t[1] - t[0]) + wy * uz * (t[3] - t[2]) +
                       uy * wz * (t[5] - t[4]) + wy * wz * (t[7] - t[6]);
      jac[3 * q + 1] = ux * uz * (t[2] - t[0]) + wx * uz * (t[3] - t[1]) +
                       ux * wz * (t[6] - t[4]) + wx * wz * (t[7] - t[5]);
      jac[3 * q + 2] = ux * uy * (t[4] - t[0]) + wx * uy * (t[5] - t[1]) +
                       ux * wy * (t[6] - t[2]) + wx * wy * (t[7] - t[3]);
    }
  }
  return r;
}

// Table entry at byte offset `off` from a level's (uniform) base: an
// instruction with a scalar base and a 32-bit lane offset (T <= 2^24 entries).
template <bool F16>
__device__ __forceinline__ float2 entry(const char* base, uint32_t off) {
  if (F16) return __half22float2(*reinterpret_cast<const __half2*>(base + off));
  return *reinterpret_cast<const float2*>(base + off);
}

// A level as the gather sees it, uniform over a work item (read once per item,
// not once per sample).
struct Level {
  const char* table;
  int res;
  uint32_t mask;  // table entries - 1
};

// Byte offset of a cell's lowest corner in a dense level's table: a 24-bit
// multiply-add per axis (n1^3 <= T <= 2^24, so n1 <= 256 and z n1 + y < 2^16).
// The other corners are the same offset from other scalar bases.
template <bool F16>
__device__ __forceinline__ uint32_t dense_offset(const Level& lv, const Cell& c) {
  const uint32_t n1 = lv.res + 1;
  return (__umul24(__umul24(c.i0[2], n1) + c.i0[1], n1) + c.i0[0]) << (F16 ? 2 : 3);
}

// Byte offsets of the four corners of a lane's half of a cell in a hashed level's
// table (bit 0 of the index: y + 1, bit 1: z + 1).  Bits below T <= 2^24 of y p1
// and z p2 follow from the factors' low 24 bits (y, z <= 2^20), so 24-bit
// multiplies do; the second row is the first plus the prime, and everything is
// kept shifted by the entry size.
template <bool F16>
__device__ __forceinline__ void hashed_offsets(const Level& lv, const Cell& c, int side,
                                               uint32_t off[4]) {
  constexpr int kShift = F16 ? 2 : 3;  // log2 of an entry's bytes
  const uint32_t mask = lv.mask << kShift;
  const uint32_t y0 = __umul24(c.i0[1], kPrime1 & 0xFFFFFFu) << kShift;
  const uint32_t z0 = __umul24(c.i0[2], kPrime2 & 0xFFFFFFu) << kShift;
  const uint32_t y1 = y0 + (kPrime1 << kShift), z1 = z0 + (kPrime2 << kShift);
  const uint32_t x0 = (c.i0[0] + side) << kShift;
  const uint32_t a0 = x0 ^ y0, a1 = x0 ^ y1;
  off[0] = (a0 ^ z0) & mask;
  off[1] = (a1 ^ z0) & mask;
  off[2] = (a0 ^ z1) & mask;
  off[3] = (a1 ^ z1) & mask;
}

// Blend of the four corners over y and z: v[0..1] the two features, and when
// GRAD v[2 + q] and v[4 + q] their derivatives along y and z.
template <bool GRAD>
__device__ __forceinline__ void blend_yz(const float2 e[4], const float wt[3], float v[6]) {
  const float wy = wt[1], wz = wt[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float t[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = q ? e[j].y : e[j].x;
    const float dz0 = t[2] - t[0], dz1 = t[3] - t[1];
    const float a0 = fmaf(wz, dz0, t[0]), a1 = fmaf(wz, dz1, t[1]);
    const float dy = a1 - a0;
    v[q] = fmaf(wy, dy, a0);
    if (GRAD) {
      v[2 + q] = dy;
      v[4 + q] = fmaf(wy, dz1 - dz0, dz0);
    }
  }
}

// Where a level's outputs go, from a uniform sample index `first` (a multiple of
// 32): the level's features and its Jacobian records.  A lane adds a 32-bit byte
// offset (feature_offset, record_offset), so that the stores take a scalar base
// each and no 64-bit addresses per lane.
typedef __attribute__((address_space(1))) char* global_ptr;
struct LevelOut {
  global_ptr feat, jac;
};

__device__ __forceinline__ LevelOut level_out(const DevField& f, const DevWork& w, int l,
                                              int first) {
  const int slot = (l & 3) * f.lpg + (l >> 2);
  LevelOut o;
  o.feat = (global_ptr)w.feat + ((int64_t)(first >> 4) * 4 * f.lpg + slot) * kFeatBlock;
  o.jac = (global_ptr)w.jac + ((int64_t)(first >> 5) * 4 * f.lpg + slot) * kJacBlock;
  // opaque, or the compiler adds the lane's offset to the arrays' bases first
  // and carries 64-bit lane addresses through the whole kernel
  asm("" : "+s"(o.feat), "+s"(o.jac));
  return o;
}

// Byte offset of sample first + i's features from LevelOut::feat, and of its
// record from LevelOut::jac.
__device__ __forceinline__ uint32_t feature_offset(const DevField& f, int i) {
  return (uint32_t)((i >> 4) * 4 * f.lpg * kFeatBlock + (i & 15) * 8);
}

__device__ __forceinline__ uint32_t record_offset(const DevField& f, int i) {
  return (uint32_t)((i >> 5) * 4 * f.lpg * kJacBlock + (i & 31) * 12);
}

template <class T>
__device__ __forceinline__ void stream_out(global_ptr base, uint32_t off, T v) {
  __builtin_nontemporal_store(v, (__attribute__((address_space(1))) T*)(base + off));
}

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// Two floats as fp16, rounded to nearest (one packed convert).
__device__ __forceinline__ uint32_t pack_half2(float lo, float hi) {
  const half2_t h = {(_Float16)lo, (_Float16)hi};
  return __builtin_bit_cast(uint32_t, h);
}

// ------------------------------------------------------------------ forward
// Work items: a run of consecutive samples on a group of levels, taken from
// that group's queue (a counter of the items handed out) by one atomic per
// block.  Hashed groups come first, dense ones last.  Workgroups are dispatched
// round-robin over the XCDs, so block b runs on XCD b % 8: it starts on its
// home queues x, x + 8, ... (x = b % 8), one group at a time, so that each
// XCD's L2 holds one group's tables at a time (a group's tables fit the L2:
// group_levels in api.hip), and once those are drained it takes what is left
// on the other queues in turn.  No XCD idles while another still has work, and
// blocks that find no free slot at launch and start late only take what is
// left.  The next item is claimed before the current one is gathered, hiding
// the atomic's latency.
constexpr int kXcds = 8;
constexpr int kPerWave = 128;                    // hashed: samples per wavefront and item (4 per lane pair)
constexpr int kItem = kBlock / 64 * kPerWave;    // hashed: samples per work item
constexpr int kDenseItem = kBlock;               // dense: samples per work item, one per lane
constexpr int kWaveRays = 64;                    // ray records a wavefront keeps in LDS

__device__ __forceinline__ uint32_t take_item(uint32_t* queue, int q) {
  return __hip_atomic_fetch_add(queue + q * kQueueStride, 1u, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
}

// The next queue for a block with home queue `home`, in the order home + 8, then
// home + 1, home + 2, ... round; -1 when every queue in `drained` is.
__device__ __forceinline__ int next_queue(int home, int n_queue, uint32_t drained) {
  const uint32_t open = ~drained & ((1u << n_queue) - 1u);
  if (open == 0) return -1;
  const uint32_t homes = open & (0x01010101u << (home & 7));  // home, home + 8, ...
  if (homes) return __ffs(homes) - 1;
  const uint32_t later = open >> home >> 1 << home << 1;
  return __ffs(later ? later : open) - 1;
}

__device__ __forceinline__ uint32_t pair_swap_u(uint32_t x) {
  return (uint32_t)__float_as_int(lane_pair_swap(__int_as_float((int)x)));
}

// A lane's part of one sample on one level: feature q (q = lane side) and, when
// GRAD, its Jacobian row as fp16.  With A the half at x, B the half at x + 1 of
// a quantity, the blend is A + wx (B - A): the own side's weight times the own
// half plus the other weight times the half the partner hands over; the
// derivative along x is B - A.
struct Part {
  float feat;
  uint32_t j01, j2;  // d feature_q / d pos_0 and _1; / d pos_2 in the low half
};

template <bool GRAD>
__device__ __forceinline__ Part finish_part(const float2 e[4], const float wt[3], int side) {
  float v[6];
  blend_yz<GRAD>(e, wt, v);
  const float wx = wt[0], ux = 1.0f - wx;
  const float own = side ? wx : ux, other = side ? ux : wx;
  const float keep = side ? v[1] : v[0];
  const float got = lane_pair_swap(side ? v[0] : v[1]);
  Part r{fmaf(other, got, own * keep), 0, 0};
  if (GRAD) {
    float j[3];
    j[0] = side ? keep - got : got - keep;
#pragma unroll
    for (int a = 1; a < 3; ++a) {
      const float jk = side ? v[2 * a + 1] : v[2 * a];
      const float jg = lane_pair_swap(side ? v[2 * a] : v[2 * a + 1]);
      j[a] = fmaf(other, jg, own * jk);
    }
    r.j01 = pack_half2(j[0], j[1]);
    r.j2 = pack_half2(j[2], 0.0f);
  }
  return r;
}

// The record of this lane's ray, for a wavefront whose samples are in ray order
// from ray r0 to ray r1: the rays' records are read once each and handed out
// through LDS, since a record is three 16-byte loads and the texture unit,
// which every load of the kernel passes, takes 32 cycles for each of a
// wavefront's 16-byte loads.  A wavefront with more rays than slots (many rays
// without samples in between) reads one record per lane instead.
__device__ __forceinline__ RayRecord wave_record(const DevWork& w, float4* lds, int lane, int ray,
                                                 int r0, int r1) {
  const bool each = r1 - r0 >= kWaveRays;
  const int n = each ? 64 : r1 - r0 + 1;
  for (int i = lane; i < n; i += 64) {
    const RayRecord r = load_ray(w.rrec, each ? ray : r0 + i);
    lds[3 * i] = r.a;
    lds[3 * i + 1] = r.b;
    lds[3 * i + 2] = r.c;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const RayRecord r = load_ray(lds, each ? lane : ray - r0);
  __builtin_amdgcn_wave_barrier();
  return r;
}

__device__ __forceinline__ Level level_of(const DevField& f, int l) {
  Level lv;
  lv.res = f.res[l];
  lv.mask = f.T - 1u;
  lv.table = f.f16 ? reinterpret_cast<const char*>(f.table16 + 2 * (size_t)l * f.T)
                   : reinterpret_cast<const char*>(f.table32 + 2 * (size_t)l * f.T);
  return lv;
}

// No derivative along a sample's clamped axes (record order: see the top).
__device__ __forceinline__ void clear_clamped(uint32_t r[3], uint32_t clamped) {
  const uint32_t keep = (clamped & 1u ? 0u : 0xFFFFu) | (clamped & 2u ? 0u : 0xFFFF0000u);
  r[0] &= keep;
  r[1] &= keep;
  r[2] = clamped & 4u ? 0u : r[2];
}

// One wavefront's 128 samples from `first` on hashed levels, as four runs of 32:
// the pair of lanes 2 i, 2 i + 1 gathers sample i of every run, so that each
// gather instruction covers consecutive samples and its lanes share lines
// (the L1 holds only 256 lines, eight such instructions' worth: lines shared
// between instructions are often evicted in between).  Side q computes the
// positions of runs 2 k + q, and both lanes take each from the lane that
// computed it.  Samples past the last one (up to the next multiple of 64, which
// the buffers hold) repeat it.  Outputs are streamed out with non-temporal
// stores so that they do not displace the level tables from L2.
template <bool F16, bool GRAD>
__device__ __forceinline__ void hashed_item(const DevField& f, const DevWork& w, float4* lds,
                                            int lane, int first, int S, int q_first, int q_count) {
  const int side = lane & 1;
  const int own = 32 * side + (lane >> 1);  // this lane's sample of step k: first + own + 64 k
  // feature `side` of sample i of runs 2 k and 2 k + 1; the own sample's record
  const uint32_t fo = feature_offset(f, lane >> 1) + 4 * side;
  const uint32_t run = feature_offset(f, 32), jo = record_offset(f, own);
  float t[2];
  int ray[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const uint32_t i = (uint32_t)min(own + 64 * k, S - 1 - first);
    ray[k] = (w.sray + first)[i];
    t[k] = (w.t + first)[i];
  }
  Pos mine[2];
  uint32_t cl[2];  // clamped axes of the samples this lane computed
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    mine[k] = sample_pos(f, t[k], wave_record(w, lds, lane, ray[k],
                                              __builtin_amdgcn_readfirstlane(ray[k]),
                                              __builtin_amdgcn_readlane(ray[k], 63)), cl[k]);
    __builtin_amdgcn_sched_barrier(0);  // one record's registers at a time
  }
  const bool any_clamped = __any((cl[0] | cl[1]) != 0);
  for (int i = 0; i < q_count; ++i) {
    const int l = f.q_level[q_first + i];
    const Level lv = level_of(f, l);
    float wt[2][3];
    float2 e[2][4];
    auto gather = [&](int k) {  // runs 2 k and 2 k + 1
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const Pos ps = j ? pos_from_pair_lane<1>(mine[k]) : pos_from_pair_lane<0>(mine[k]);
        Cell c;
        make_cell(lv.res, ps.x, ps.dx, c);
        uint32_t off[4];
        hashed_offsets<F16>(lv, c, side, off);
#pragma unroll
        for (int q = 0; q < 4; ++q) e[j][q] = entry<F16>(lv.table, off[q]);
#pragma unroll
        for (int a = 0; a < 3; ++a) wt[j][a] = c.w[a];
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    gather(0);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const Part p0 = finish_part<GRAD>(e[0], wt[0], side);
      const Part p1 = finish_part<GRAD>(e[1], wt[1], side);
      // side q completes the record of its own sample (run 2 k + q) and hands
      // the partner its part of the other one: axes 0 and 1 of feature 0, the
      // same of feature 1, axis 2 of both
      uint32_t r[3];
      if (GRAD) {
        const uint32_t k01 = side ? p1.j01 : p0.j01, g01 = pair_swap_u(side ? p0.j01 : p1.j01);
        const uint32_t k2 = side ? p1.j2 : p0.j2, g2 = pair_swap_u(side ? p0.j2 : p1.j2);
        r[0] = side ? g01 : k01;
        r[1] = side ? k01 : g01;
        r[2] = side ? g2 | (k2 << 16) : k2 | (g2 << 16);
        if (any_clamped) clear_clamped(r, cl[k]);
      }
      if (first + 64 * k < S) {
        const LevelOut o = level_out(f, w, l, first + 64 * k);
        stream_out(o.feat, fo, p0.feat);
        stream_out(o.feat, fo + run, p1.feat);
        if (GRAD) {
#pragma unroll
          for (int a = 0; a < 3; ++a) stream_out(o.jac, jo + 4 * a, r[a]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (k == 0) gather(1);
    }
  }
}

// One wavefront's 64 samples from `first` on dense levels, one per lane.
// Consecutive samples of a ray mostly share a dense level's cells, so a
// wavefront's gathers touch few lines however the lanes are split, and the
// vector work sets the time: one lane per sample does the cell and the
// positions once (about 80 instructions a sample and level against 190 over a
// lane pair), and the group's levels share the sample's position.
template <bool F16, bool GRAD>
__device__ __forceinline__ void dense_item(const DevField& f, const DevWork& w, float4* lds,
                                           int lane, int first, int S, int q_first, int q_count) {
  const uint32_t at = (uint32_t)min(lane, S - 1 - first);
  const int ray = (w.sray + first)[at];
  const float t = (w.t + first)[at];
  const uint32_t fo = feature_offset(f, lane), jo = record_offset(f, lane);
  uint32_t clamped;
  const Pos ps = sample_pos(f, t, wave_record(w, lds, lane, ray, __builtin_amdgcn_readfirstlane(ray),
                                              __builtin_amdgcn_readlane(ray, 63)), clamped);
  const bool any_clamped = __any(clamped != 0);
  for (int i = 0; i < q_count; ++i) {
    const int l = f.q_level[q_first + i];
    const Level lv = level_of(f, l);
    Cell c;
    make_cell(lv.res, ps.x, ps.dx, c);
    const uint32_t off = dense_offset<F16>(lv, c);
    const uint32_t n1 = lv.res + 1, r1 = n1 << (F16 ? 2 : 3), r2 = n1 * r1;
    float2 lo[4], hi[4];  // bit 0 of the index: y + 1, bit 1: z + 1
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const char* row = lv.table + (k & 1 ? r1 : 0) + (k & 2 ? r2 : 0);
      lo[k] = entry<F16>(row, off);
      hi[k] = entry<F16>(row + (F16 ? 4 : 8), off);
    }
    float feat[2], j[2][3];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float x[4], dx[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float a = q ? lo[k].y : lo[k].x, b = q ? hi[k].y : hi[k].x;
        dx[k] = b - a;
        x[k] = fmaf(c.w[0], dx[k], a);
      }
      const float dz0 = x[2] - x[0], dz1 = x[3] - x[1];
      const float y0 = fmaf(c.w[2], dz0, x[0]), y1 = fmaf(c.w[2], dz1, x[1]);
      const float dy = y1 - y0;
      feat[q] = fmaf(c.w[1], dy, y0);
      if (GRAD) {
        const float ex0 = fmaf(c.w[2], dx[2] - dx[0], dx[0]), ex1 = fmaf(c.w[2], dx[3] - dx[1], dx[1]);
        j[q][0] = fmaf(c.w[1], ex1 - ex0, ex0);
        j[q][1] = dy;
        j[q][2] = fmaf(c.w[1], dz1 - dz0, dz0);
      }
    }
    const LevelOut o = level_out(f, w, l, first);
    typedef float float2_t __attribute__((ext_vector_type(2)));
    const float2_t both = {feat[0], feat[1]};
    stream_out(o.feat, fo, both);
    if (GRAD) {
      uint32_t r[3] = {pack_half2(j[0][0], j[0][1]), pack_half2(j[1][0], j[1][1]),
                       pack_half2(j[0][2], j[1][2])};
      if (any_clamped) clear_clamped(r, clamped);
#pragma unroll
      for (int a = 0; a < 3; ++a) stream_out(o.jac, jo + 4 * a, r[a]);
    }
  }
}

// Blocks that work on a batch: 4 per CU (kFewPerCu), and all 7 that are resident
// from kManyItems items on.  More blocks cover the gathers' latency better, but
// each finds the queues drained one by one at the end and holds lines of the L1.
// Encode with 4 and with 7 per CU, us, at so many thousand items.  Uniform samples
// of 16 levels: fp32, 2^19 entries: 38 294 308, 146 1182 1192, 391 3081 3053, 791
// 6305 6255 (without gradient 146 1080 1089, 195 1419 1406, 391 2726 2707); fp32,
// 2^21: 156 2696 2713, 416 6815 6816, 843 13935 13871; fp16, 2^19: 22 269 281, 83
// 1021 1051, 446 5481 5535.  Of 8 levels, fp32, 2^19: 23 165 175, 176 1172 1174,
// 234 1498 1494, 475 3129 3072.  Lattice samples, which lie closer together, of 16
// levels: fp32, 2^19: 30 227 244, 81 541 553; fp32, 2^21: 157 2059 2096; fp16,
// 2^19: 23 254 264, 378 4000 3970; a whole call of 5.6 M samples (165) 1880 1859.
constexpr int kFewPerCu = 4, kManyItems = 128 << 10;
__host__ __device__ inline int work_items(const DevField& f, uint32_t samples) {
  // (a batch is below 2^31 samples: at most 2^27 items)
  return (int)((samples + kItem - 1) / kItem) * f.n_hashed_queue +
         (int)((samples + kDenseItem - 1) / kDenseItem) * (f.n_queue - f.n_hashed_queue);
}

template <bool F16, bool GRAD>
__global__ __launch_bounds__(kBlock) void k_encode(DevField f, DevWork w, int n_few) {
  __shared__ int s_q[2];
  __shared__ uint32_t s_item[2];
  __shared__ float4 s_rec[kBlock / 64][3 * kWaveRays];
  const int S = __builtin_amdgcn_readfirstlane(*w.total);
  // the grid is sized for what the batch may hold at most: where it holds less,
  // the blocks past n_few take no item (the others need not wait for S to know)
  int working = 1;
  if ((int)blockIdx.x >= n_few)
    working = __builtin_amdgcn_readfirstlane(work_items(f, S) >= kManyItems);
  const uint32_t n_hashed = (uint32_t)((S + kItem - 1) / kItem);
  const uint32_t n_dense = (uint32_t)((S + kDenseItem - 1) / kDenseItem);
  const int lane = threadIdx.x & 63;
  // uniform values in scalar registers: they make the output and table bases scalar
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int home = (int)(blockIdx.x % kXcds) % f.n_queue;
  uint32_t* known = w.queue + kMaxLevels * kQueueStride;  // bits of drained queues
  uint32_t drained = 0;                                   // thread 0's copy
  int q = home;
  int buf = 0;
  if (working && threadIdx.x == 0) s_item[0] = take_item(w.queue, q);
  __syncthreads();
  uint32_t item = __builtin_amdgcn_readfirstlane(s_item[0]);
  // control flow below is uniform over the block: item and q follow from the
  // same shared words for every thread
  while (working) {
    const bool hashed = q < f.n_hashed_queue;
    const uint32_t n_items = hashed ? n_hashed : n_dense;
    if (item >= n_items) {  // queue q is drained
      buf ^= 1;
      if (threadIdx.x == 0) {
        // The first block past a queue's end tells the others, who then skip it
        // (each trip to a counter is a microsecond, and on a small batch they
        // were most of the kernel).  A stale word costs a trip: every block
        // also notes the queues it found drained, so it ends after n_queue.
        drained |= 1u << q;
        if (item == n_items)
          __hip_atomic_fetch_or(known, 1u << q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        drained |= __hip_atomic_load(known, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int nq = next_queue(home, f.n_queue, drained);
        s_q[buf] = nq;
        if (nq >= 0) s_item[buf] = take_item(w.queue, nq);
      }
      __syncthreads();
      q = __builtin_amdgcn_readfirstlane(s_q[buf]);
      if (q < 0) break;
      item = __builtin_amdgcn_readfirstlane(s_item[buf]);
      continue;
    }
    uint32_t next = 0;
    if (threadIdx.x == 0) next = take_item(w.queue, q);
    const int q_first = f.q_first[q], q_count = f.q_first[q + 1] - q_first;
    if (hashed) {
      const int first = (int)item * kItem + wave * kPerWave;
      if (first < S) hashed_item<F16, GRAD>(f, w, s_rec[wave], lane, first, S, q_first, q_count);
    } else {
      const int first = (int)item * kDenseItem + wave * 64;
      if (first < S) dense_item<F16, GRAD>(f, w, s_rec[wave], lane, first, S, q_first, q_count);
    }
    buf ^= 1;
    if (threadIdx.x == 0) s_item[buf] = next;
    __syncthreads();
    item = __builtin_amdgcn_readfirstlane(s_item[buf]);
  }
}

// ---------------------------------------------------------------- occupancy
// Occupancy grid: bit set iff the density at the cell centre exceeds `thr`.
// One thread per cell (linear index x + R(y + Rz)), plain FMA arithmetic; run
// once at field creation.
template <bool F16>
__global__ __launch_bounds__(kBlock) void k_occupancy(DevField f, uint32_t* bits, int R,
                                                      float thr) {
  __shared__ float s_w1[2 * kMaxLevels * kHidden];
  __shared__ float s_w2[kHidden];
  const int din = 2 * f.L;
  for (int i = threadIdx.x; i < din * kHidden; i += kBlock) s_w1[i] = f.wd1[i];
  if (threadIdx.x < kHidden) s_w2[threadIdx.x] = f.wd2[threadIdx.x * 16];
  __syncthreads();
  const int64_t n = (int64_t)R * R * R;
  const int64_t lin = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  bool occ = false;
  if (lin < n) {
    const int ci[3] = {(int)(lin % R), (int)((lin / R) % R), (int)(lin / ((int64_t)R * R))};
    float x[3];
    const float dx[3] = {0.0f, 0.0f, 0.0f};
    for (int a = 0; a < 3; ++a) {
      float ext = __fsub_rn(f.mx[a], f.mn[a]);
      float cell = __fdiv_rn(ext, (float)R);
      float p = __fadd_rn(f.mn[a], __fmul_rn(__fadd_rn((float)ci[a], 0.5f), cell));
      float xr = __fmul_rn(__fsub_rn(p, f.mn[a]), f.inv_ext[a]);
      x[a] = xr < 0.0f ? 0.0f : (xr > 1.0f ? 1.0f : xr);
    }
    float feat[2 * kMaxLevels];
    for (int l = 0; l < f.L; ++l) {
      float2 v = level_feature<F16>(f, l, x, dx, nullptr);
      feat[2 * l] = v.x;
      feat[2 * l + 1] = v.y;
    }
    float h0 = 0.0f;
    for (int j = 0; j < kHidden; ++j) {
      float a = 0.0f;
      for (int i = 0; i < din; ++i) a += feat[i] * s_w1[i * kHidden + j];
      h0 += (a > 0.0f ? a : 0.0f) * s_w2[j];
    }
    occ = __expf(h0 + f.density_bias) > thr;
  }
  const uint64_t bal = __ballot(occ);
  const int lane = threadIdx.x & 63;
  const int64_t word = (lin - lane) / 32 + (lane == 32 ? 1 : 0);
  const int64_t n_words = (n + 31) / 32;
  if ((lane == 0 || lane == 32) && word < n_words)
    bits[word] = lane == 0 ? (uint32_t)(bal & 0xFFFFFFFFu) : (uint32_t)(bal >> 32);
}

}  // namespace

hipError_t launch_encode(const DevField& f, const DevWork& w, int64_t max_samples, int resident,
                         int n_cu, int with_grad, hipStream_t s) {
  const int items = work_items(f, (uint32_t)max_samples), n_few = kFewPerCu * n_cu;
  const int most = items < kManyItems ? std::min(resident, n_few) : resident;
  const dim3 grid(std::max(1, std::min(most, items)));
  if (f.f16) {
    if (with_grad)
      hipLaunchKernelGGL((k_encode<true, true>), grid, dim3(kBlock), 0, s, f, w, n_few);
    else
      hipLaunchKernelGGL((k_encode<true, false>), grid, dim3(kBlock), 0, s, f, w, n_few);
  } else {
    if (with_grad)
      hipLaunchKernelGGL((k_encode<false, true>), grid, dim3(kBlock), 0, s, f, w, n_few);
    else
      hipLaunchKernelGGL((k_encode<false, false>), grid, dim3(kBlock), 0, s, f, w, n_few);
  }
  return hipGetLastError();
}

int encode_blocks_per_cu(const DevField& f) {
  int n = 0;
  const hipError_t e =
      f.f16 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_encode<true, true>, kBlock, 0)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_encode<false, true>, kBlock, 0);
  return e == hipSuccess && n > 0 ? n : 4;
}

hipError_t launch_occupancy(const DevField& f, uint32_t* bits, int R, float thr, hipStream_t s) {
  const int64_t n = (int64_t)R * R * R;
  const int64_t nb = (n + kBlock - 1) / kBlock;
  if (f.f16)
    hipLaunchKernelGGL(k_occupancy<true>, dim3((unsigned)nb), dim3(kBlock), 0, s, f, bits, R, thr);
  else
    hipLaunchKernelGGL(k_occupancy<false>, dim3((unsigned)nb), dim3(kBlock), 0, s, f, bits, R, thr);
  return hipGetLastError();
}

}  // namespace pnerf
