// Arguments, rotary table and tile layout shared by the forward attention
// kernels that stream 64-key tiles (attn_fwd.hip, attn_fwd_split.hip).
#pragma once

#include "attn_tile.hpp"

namespace vidax {
namespace tile {

constexpr int D = kHeadDim;
constexpr int BN = 64;  // keys per tile
struct AttnArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* o;
  float* lse;
  const int32_t* kv_valid_len;
  int B, H, Lq, Lk;
  int nqt;      // query tiles per (b, h)
  int nwg;      // total workgroups
  float qmul;   // scale * log2(e): the rotated query is multiplied by it before rounding to bf16
  float c2;     // unrotated query: |scale| * log2(e) (1 when scale == 0), applied in the exponent
  float qsign;  // unrotated query: +1, -1 or 0 (scale == 0) applied to the query
  RopeParams rp;
  // attention rotary table: axis a holds (G_a + 1) positions x d_a/2 pairs
  int tbase1, tbase2, tentries;
  uint32_t pos_step;  // packed (t, h, w) increment of BN tokens
  uint32_t pos_sent;  // packed identity position (gt, gh, gw)
};

// Rotates one interleaved bf16 pair (x0 low, x1 high) by (cos, sin) in fp32.
__device__ __forceinline__ uint32_t rotate_pair(uint32_t x, float2 cs) {
  const float x0 = bf16lo_to_f32(x), x1 = bf16hi_to_f32(x);
  return pack_bf16x2(fmaf(x0, cs.x, -x1 * cs.y), fmaf(x0, cs.y, x1 * cs.x));
}

// Table entry e of the attention kernel (see AttnArgs): position G_a of each
// axis is the identity.
__device__ __forceinline__ float2 attn_table_entry(const AttnArgs& a, int e) {
  const RopeParams& r = a.rp;
  int f, half, da, g;
  if (e < a.tbase1) { f = e; half = r.dt >> 1; da = r.dt; g = r.gt; }
  else if (e < a.tbase2) { f = e - a.tbase1; half = r.dh >> 1; da = r.dh; g = r.gh; }
  else { f = e - a.tbase2; half = r.dw >> 1; da = r.dw; g = r.gw; }
  const int pos = f / half;
  const int j = f - pos * half;
  float c = 1.f, s = 0.f;
  if (pos < g) {
    const float omega = exp2f(-((float)(2 * j) / (float)da) * r.log2_theta);
    sincosf((float)pos * omega, &s, &c);
  }
  return make_float2(c, s);
}

// Per channel pair: byte offset of its first table entry, byte stride per
// position, and which coordinate of the packed (t << 22 | h << 11 | w)
// position selects the row.  The w and h fields have one spare bit so a
// BN-token step plus carry never overflows them.
struct PairIdx {
  int base, stride, shift;
};
constexpr int kEntryBytes = 8;

__device__ __forceinline__ PairIdx pair_idx(const AttnArgs& a, int pi) {
  const RopeParams& r = a.rp;
  const int ht = r.dt >> 1, hh = r.dh >> 1;
  PairIdx p;
  if (pi < ht) { p.base = pi; p.stride = ht; p.shift = 22; }
  else if (pi < ht + hh) { p.base = a.tbase1 + pi - ht; p.stride = hh; p.shift = 11; }
  else { p.base = a.tbase2 + pi - ht - hh; p.stride = r.dw >> 1; p.shift = 0; }
  p.base *= kEntryBytes;
  p.stride *= kEntryBytes;
  return p;
}

// Table entry of pair p at packed position pos (24-bit multiply-add).
__device__ __forceinline__ float2 table_entry(const float2* tab, const PairIdx& p, uint32_t pos) {
  // the t field is the top 10 bits, so an 11-bit extract at offset 22 is exact
  const uint32_t off = __umul24(__builtin_amdgcn_ubfe(pos, p.shift, 11), (uint32_t)p.stride) + (uint32_t)p.base;
  return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(tab) + off);
}

__device__ __forceinline__ uint32_t packed_pos(const AttnArgs& a, int n) {
  if (n >= a.rp.n_rot) return a.pos_sent;
  const int t = n / (a.rp.gh * a.rp.gw);
  const int rem = n - t * a.rp.gh * a.rp.gw;
  const int h = rem / a.rp.gw;
  return ((uint32_t)t << 22) | ((uint32_t)h << 11) | (uint32_t)(rem - h * a.rp.gw);
}

// K and V tiles sit in LDS in MFMA operand order: 16 blocks of 1 KB, each
// holding exactly what one wave reads for one matrix instruction, lane by lane.
//   K block 2 st + blk: lane l's 16 bytes = key row 32 blk + (l & 31),
//     d = 16 st + 8 (l >> 5) .. + 7 (A operand of S^T = K Q^T, d-step st).
//   V block 4 ks + mb, half r (512 bytes): lane l's 8 bytes = key row
//     16 ks + 8 r + 4 (l >> 5) + ((l & 15) >> 2), d = 32 mb + 16 ((l >> 4) & 1)
//     + 4 (l & 3) .. + 3 (what the transposing read of lane l fetches for the
//     V^T operand of d block mb, keys 16 ks .. 16 ks + 15).
// Every operand read is one contiguous, bank-conflict-free 1 KB (K) or 512 B
// (V) access at an offset that is a constant of the instruction, and each
// block is filled by one direct 1 KB global -> LDS copy.
constexpr int TILE = BN * D;  // elements per K or V tile
constexpr int BLK = 512;      // elements per operand block

}  // namespace tile

// Launcher of attn_fwd_split.hip (a.nqt, a.nwg: its 128-row query tiles).
constexpr int kSplitRows = 128;
hipError_t launch_attn_fwd_split(const tile::AttnArgs& a, hipStream_t stream);
}  // namespace vidax
