// Shared device/host definitions of the gfx950 kernels (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace vidax {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kHeadDim = 128;
// Entries (cos, sin) of the per-workgroup rotary table kept in LDS.
constexpr int kRopeTableMax = 4096;
// The attention kernel's table has one extra identity position per axis and
// packs a token's (t, h, w) into one word (w, h in 11-bit fields, t in 10).
constexpr int kAttnTableMax = 4096;
constexpr int kAttnGridHWMax = 1023;
constexpr int kAttnGridTMax = 1023;

// Rotary parameters in the form the kernels consume (derived from
// vidax_rope3d_desc by the host).
struct RopeParams {
  int enabled;
  int gt, gh, gw;      // token grid
  int dt, dh, dw;      // channel widths of the t, h, w blocks
  int pair_mode;       // 0 interleaved, 1 half split
  int keys_prerotated; // attention: keys arrive already rotated
  int inverse;         // standalone rotation: rotate by -angle (the transpose)
  int n_rot;           // gt * gh * gw
  int base1, base2;    // first table entry of the h and w axes
  int n_entries;       // table entries: gt*dt/2 + gh*dh/2 + gw*dw/2
  float log2_theta;
};

// ---------------------------------------------------------------- device ----

__device__ __forceinline__ float bf16lo_to_f32(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16hi_to_f32(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Two fp32 -> packed bf16 pair (lo in bits 0-15), round to nearest even:
// one v_cvt_pk_bf16_f32 on gfx950.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Fills the (cos, sin) table: entry base_a + pos * (d_a / 2) + j of axis a,
// frequency theta^(-2j/d_a).  A thread keeps one channel pair (its frequency is
// formed once, no division per entry) and takes every (nthreads / 64)-th position.
__device__ __forceinline__ void build_rope_table(const RopeParams& r, float2* tab, int tid, int nthreads) {
  const int pi = tid & 63, ht = r.dt >> 1, hh = r.dh >> 1;
  int j, half, n, base;
  if (pi < ht) { j = pi; half = ht; n = r.gt; base = 0; }
  else if (pi < ht + hh) { j = pi - ht; half = hh; n = r.gh; base = r.base1; }
  else { j = pi - ht - hh; half = r.dw >> 1; n = r.gw; base = r.base2; }
  const float omega = exp2f(-((float)(2 * j) / (float)(2 * half)) * r.log2_theta);
  for (int pos = tid >> 6; pos < n; pos += nthreads >> 6) {
    float s, c;
    sincosf((float)pos * omega, &s, &c);
    tab[base + pos * half + j] = make_float2(c, s);
  }
}

// Table entry of channel pair `pi` (interleaved numbering, pi in [0, 64)) at
// coordinates (t, h, w): base of the pair's axis + pos * (d_a/2) + j.
struct PairSlot {
  int axis;   // 0, 1, 2
  int base;   // base_a + j
  int stride; // d_a / 2
};

__host__ __device__ inline PairSlot pair_slot(const RopeParams& r, int pi) {
  PairSlot s;
  int ht = r.dt >> 1, hh = r.dh >> 1;
  if (pi < ht) {
    s.axis = 0; s.base = pi; s.stride = ht;
  } else if (pi < ht + hh) {
    s.axis = 1; s.base = r.base1 + (pi - ht); s.stride = hh;
  } else {
    s.axis = 2; s.base = r.base2 + (pi - ht - hh); s.stride = r.dw >> 1;
  }
  return s;
}

// f(0), ..., f(N - 1) with compile-time arguments.
template <int N, typename F, int... I>
__device__ __forceinline__ void for_slots_of(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void for_slots(F&& f) {
  for_slots_of<N>(f, std::make_integer_sequence<int, N>());
}

// Between LDS writes of a wave's lanes and reads of them by its other lanes (or
// the reverse): the compiler moves no LDS access across.  No instruction: a
// wave's LDS accesses are carried out in order.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// End of a slot of a hand-scheduled block: no instruction moves across it.
#define SLOT() __builtin_amdgcn_sched_barrier(0)

// Logical tile of workgroup i of n (n / B per batch, batch after batch).
// Workgroups are dispatched round-robin over the 8 XCDs; each XCD gets a
// contiguous range of positions, so that the tiles of one (b, h) share that
// XCD's L2.  The positions run over the eighths of every batch in turn (eighth
// 0 of batch 0, of batch 1, ..., eighth 1 of batch 0, ...), so that each XCD
// gets about an eighth of every batch: batches of different valid lengths then
// load the XCDs evenly (with batch after batch, the XCDs holding the longer
// batches finished last).  One batch: position = logical tile.
__device__ __forceinline__ int balanced_tile(int i, int n, int B) {
  const int per = n >> 3, rem = n & 7, xcd = i & 7, kk = i >> 3;
  const int pos = xcd < rem ? xcd * (per + 1) + kk : rem * (per + 1) + (xcd - rem) * per + kk;
  const int N = n / B;  // tiles per batch: eighth c holds p + (c < r) of them
  const int p = N >> 3, r = N & 7;
  const int big = B * r * (p + 1);  // positions in the eighths of size p + 1
  const int c = pos < big ? pos / (B * (p + 1)) : r + (pos - big) / (B * p);
  const int sc = c < r ? p + 1 : p;
  const int cs = c * p + (c < r ? c : r);  // start of eighth c within a batch
  const int rm = pos - B * cs;
  return (rm / sc) * N + cs + rm % sc;
}

}  // namespace vidax
