// Flash-attention forward for launches that leave compute units idle with
// 256-row query tiles: the dense kernel's formulation (attn_fwd.hip: matrix-core
// layout, softmax, rotary table) with 128 query rows a workgroup, twice the
// workgroups.  Its 8 waves are two groups of 4 that take alternate tiles of 32
// keys for the same queries; group 1 hands its output, reference and sum to
// group 0 through LDS at the end (an online-softmax merge).
//
// What bounds such a launch is the latency of a workgroup's serial chain: one
// step per 64 keys (32 a group), each a quarter of the dense kernel's products
// per wave.  K and V have four tile buffers, so that a copy has three steps to
// land (the dense kernel's two give it one, enough where every compute unit is
// at work and a step is longer than a copy's latency).
// No instance spills: a spilled register's store or reload waits behind the copies
// just issued, at the start and end of a chain that is little else (54, 35 and 17
// spilled registers cost 13, 10 and 5 % at 12 x 512).
// At 12 heads x 1560 x 1560 (rotated queries): 42.2 -> 35.0 us; 8 heads x 4000 x
// 4000: 86.5 -> 72.0; keys rotated here too, 59.9 -> 44.3 and 125.6 -> 89.0 (see
// the rule at use_split).
//
// LDS: K and V tiles 8 x 16 KB (rotating keys: 4), rotary table <= 32 KB; query
// and output staging in the K and V buffers.
#include <type_traits>

#include "attn_args.hpp"
#include "launch.hpp"

namespace vidax {
namespace {

using namespace tile;

constexpr int S = 2;            // key groups of a workgroup
constexpr int BM = kSplitRows;  // query rows of a workgroup
constexpr int NW = 8;
constexpr int NT = NW * 64;
constexpr int WQ = NW / S;         // waves (32 query rows each) of a key group
constexpr int BNG = 32;            // keys of a group's tile
constexpr int BN_STEP = S * BNG;   // keys of a step
constexpr int TILE = BNG * D;      // elements of a group's K or V tile

// A barrier without a fence's wait for the copies in flight; the clobber keeps
// the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ROPE: rotate the queries (and build the table); ROPE_K: also rotate the keys
// while staging them (false when the caller passes pre-rotated keys).
// HALF: half-split pairs (queries only; ROPE_K is then false).
template <bool ROPE, bool ROPE_K, bool HALF>
__global__ __launch_bounds__(NT) void attn_fwd_split_kernel(AttnArgs a) {
  constexpr int NBUF = ROPE_K ? 2 : 4;  // tile buffers (rotated keys pass through registers)
  // K and V buffers (a tile of every group), each its own LDS object so that
  // the compiler can tell the direct copies into one buffer from the operand
  // reads of another (and does not wait for the copies before those reads).
  __shared__ __attribute__((aligned(16))) uint16_t K0[S * TILE], K1[S * TILE], V0[S * TILE], V1[S * TILE];
  __shared__ __attribute__((aligned(16))) uint16_t K2[NBUF == 4 ? S * TILE : 1], K3[NBUF == 4 ? S * TILE : 1];
  __shared__ __attribute__((aligned(16))) uint16_t V2[NBUF == 4 ? S * TILE : 1], V3[NBUF == 4 ? S * TILE : 1];
  // buffer of tile i (i mod NBUF at compile time)
  auto kbuf = [&](int i) __attribute__((always_inline)) -> uint16_t* {
    if constexpr (NBUF == 4)
      if (i & 2) return i & 1 ? K3 : K2;
    return i & 1 ? K1 : K0;
  };
  auto vbuf = [&](int i) __attribute__((always_inline)) -> uint16_t* {
    if constexpr (NBUF == 4)
      if (i & 2) return i & 1 ? V3 : V2;
    return i & 1 ? V1 : V0;
  };
  __shared__ float2 tab[ROPE ? kAttnTableMax : 1];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / WQ, wq = wave % WQ;  // key group, 32-row block of queries
  const int l32 = lane & 31;
  const int hi = lane >> 5;
  const int tok = a.H * D;     // elements between consecutive tokens
  const int rbytes = tok * 2;  // bytes between consecutive tokens

  // ---- the workgroup's query tile: tile lid % nqt of (b, h) = (lid / nqt / H,
  // lid / nqt % H).  The query tiles of one (b, h) are consecutive (the K/V
  // stream of that head is then shared in an XCD's L2).
  const int lid = balanced_tile(blockIdx.x, a.nwg, a.B);
  const int qt = lid % a.nqt, bh = lid / a.nqt, h = bh % a.H, b = bh / a.H;
  int lvb = a.Lk;
  if (a.kv_valid_len) lvb = min(max(a.kv_valid_len[b], 0), a.Lk);
  const int lv = __builtin_amdgcn_readfirstlane(lvb);  // uniform: keeps buffer descriptors in SGPRs
  const uint16_t* const kbh = a.k + (size_t)b * a.Lk * tok + (size_t)h * D;
  const uint16_t* const vbh = a.v + (size_t)b * a.Lk * tok + (size_t)h * D;
  const int row0 = qt * BM + wq * 32;  // the wave's first query row
  const int qrow = row0 + l32;
  const bool qlive = qrow < a.Lq;
  const bool live = grp * BNG < lv;  // the wave's key group has keys (uniform)
  const int nsteps = (lv + BN_STEP - 1) / BN_STEP;

  // Query rows come in and output rows go out whole: each 16-lane group of a
  // wave moves one 256-byte row (coalesced), and the wave's 8 KB staging area
  // in LDS (32 rows x 16 chunks of 16 bytes, chunk c of row r at slot
  // stage_slot(c, r)) converts between that layout and the operand layout in
  // which a lane holds one query.  It borrows the K/V buffers (free before
  // the first copies and after the last tile).
  uint16_t* const stage = (wave < 2 ? K0 : wave < 4 ? K1 : wave < 6 ? V0 : V1) + (wave & 1) * 32 * D;

  // The wave's 32 query rows into its staging area: copy i brings
  // rows 4 i .. 4 i + 3, lane l the chunk that belongs in slot l & 15 of row
  // 4 i + (l >> 4).  Rows past Lq read as zero.  Exactly 8 copies a wave.
  auto dma_q = [&]() __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.q + (size_t)b * a.Lq * tok + (size_t)h * D), (short)0, a.Lq * rbytes,
        kBufferFlags);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = 4 * i + (lane >> 4);
      const int off = row0 + r < a.Lq ? (row0 + r) * rbytes + stage_slot(lane & 15, r) * 16 : 0x7ffffff0;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rq, (lds_ptr)(stage + 4 * i * D), 16, off, 0, 0, 0);
    }
  };

  // raw[s] = chunk 2 s + hi of the lane's own query row l32, from the staging area
  auto read_q = [&](uint4 raw[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 8; ++s)
      raw[s] = *reinterpret_cast<const uint4*>(stage + l32 * D + stage_slot(2 * s + hi, l32) * 8);
  };

  // ---- Q: lane holds query qrow, d-chunks 2s + hi (s = 0..7) as MFMA B operands
  bf16x8 qreg[8];
  // Half-split pairs (keys then come rotated by vidax_rope3d): pair j of the
  // block of axis a (offset o_a, width d_a) is channels o_a + j and
  // o_a + j + d_a / 2, which different lanes read out.  So the staged query
  // row is rotated and scaled in place first, the two lanes of a row taking
  // 32 pairs each (one rounding, as in the interleaved path), and make_q then
  // takes the values as they are.
  auto rotate_staged_half_split = [&]() __attribute__((always_inline)) {
    const RopeParams& r = a.rp;
    const uint32_t qpos = packed_pos(a, qlive ? qrow : r.n_rot);
    const float qm = a.qmul;
    uint16_t* const row = stage + l32 * D;
    const int ht = r.dt >> 1, hh = r.dh >> 1;
#pragma unroll 1
    for (int pi = 32 * hi; pi < 32 * hi + 32; ++pi) {
      int o, hl, j;
      if (pi < ht) { o = 0; hl = ht; j = pi; }
      else if (pi < ht + hh) { o = r.dt; hl = hh; j = pi - ht; }
      else { o = r.dt + r.dh; hl = r.dw >> 1; j = pi - ht - hh; }
      const int c0 = o + j, c1 = c0 + hl;
      uint16_t* const p0 = row + stage_slot(c0 >> 3, l32) * 8 + (c0 & 7);
      uint16_t* const p1 = row + stage_slot(c1 >> 3, l32) * 8 + (c1 & 7);
      const float x0 = __uint_as_float((uint32_t)*p0 << 16), x1 = __uint_as_float((uint32_t)*p1 << 16);
      const float2 cs = table_entry(tab, pair_idx(a, pi), qpos);
      const uint32_t y = pack_bf16x2(fmaf(x0, cs.x, -x1 * cs.y) * qm, fmaf(x0, cs.y, x1 * cs.x) * qm);
      *p0 = (uint16_t)(y & 0xffffu);
      *p1 = (uint16_t)(y >> 16);
    }
  };
  auto make_q = [&](const uint4 raw[8]) __attribute__((always_inline)) {
    const uint32_t qpos = ROPE ? packed_pos(a, qlive ? qrow : a.rp.n_rot) : 0u;
    const float qm = a.qmul;
    const uint32_t sgn = a.qsign < 0.f ? 0x80008000u : 0u;
    const uint32_t keep = a.qsign == 0.f ? 0u : 0xffffffffu;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int c = 2 * s + hi;
      uint32_t wq[4] = {raw[s].x, raw[s].y, raw[s].z, raw[s].w};
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        if (ROPE) {  // rotated and scaled in fp32, rounded once
          if (!HALF) {  // (half-split rows were rotated in the staging area)
            const float x0 = bf16lo_to_f32(wq[p]), x1 = bf16hi_to_f32(wq[p]);
            const float2 cs = table_entry(tab, pair_idx(a, 4 * c + p), qpos);
            wq[p] = pack_bf16x2(fmaf(x0, cs.x, -x1 * cs.y) * qm, fmaf(x0, cs.y, x1 * cs.x) * qm);
          }
        } else {  // exact: sign only
          wq[p] = (wq[p] ^ sgn) & keep;
        }
      }
      qreg[s] = __builtin_bit_cast(bf16x8, make_uint4(wq[0], wq[1], wq[2], wq[3]));
    }
  };

  // ---- staging: wave wq of a group fills K blocks 2 wq, 2 wq + 1 and V blocks
  // 2 wq, 2 wq + 1 of every tile of the group.  Byte offsets from the tile's first row of what
  // lane `lane` copies:
  const int kr0 = l32;          // K row kr0,
  const int kc = 4 * wq + hi;  // 16-byte chunks kc and kc + 2
  const int kg0 = kr0 * rbytes + kc * 16;
  const int kg1 = kg0 + 32;
  int vg0, vg1;
  {
    const int vrow = 8 * hi + 4 * ((lane >> 4) & 1) + ((lane & 7) >> 1);
    const int vd = 16 * ((lane >> 3) & 1) + 8 * (lane & 1);
    const int b0 = 2 * wq, b1 = 2 * wq + 1;  // blocks (ks, mb) = (b >> 2, b & 3)
    vg0 = (vrow + 16 * (b0 >> 2)) * rbytes + 2 * (vd + 32 * (b0 & 3));
    vg1 = (vrow + 16 * (b1 >> 2)) * rbytes + 2 * (vd + 32 * (b1 & 3));
  }

  // rotary state of the fused path: the thread owns chunks kc and kc + 2 of K row kr0
  PairIdx kpi[2][4];
  uint32_t kpos = 0u;
  if (ROPE_K) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < 4; ++p) kpi[c][p] = pair_idx(a, 4 * (kc + 2 * c) + p);
    const int n = grp * BNG + kr0;
    const int t = n / (a.rp.gh * a.rp.gw);
    const int rem = n - t * a.rp.gh * a.rp.gw;
    const int hh = rem / a.rp.gw;
    kpos = ((uint32_t)t << 22) | ((uint32_t)hh << 11) | (uint32_t)(rem - hh * a.rp.gw);
  }

  // Buffer resource of the group's tile of step j: its records end at the last
  // valid key, so rows at or beyond lv read as zero (and land in LDS as zero);
  // tiles past the end read all zeros and are never used.
  auto tile_rsrc = [&](const uint16_t* base, int j) __attribute__((always_inline)) {
    const int tile = S * j + grp;
    const int rows = min(max(lv - tile * BNG, 0), BNG);
    const int nbytes = __builtin_amdgcn_readfirstlane(rows * rbytes);  // uniform
    return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (size_t)tile * BNG * tok), (short)0, nbytes, kBufferFlags);
  };

  // Direct global -> LDS copy of the wave's two operand blocks of step j's tile (16
  // bytes a lane, landing at the block base + 16 * lane).
  auto dma_tile = [&](const uint16_t* base, int j, uint16_t* buf, int g0, int g1) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(base, j);
    uint16_t* const dst = buf + grp * TILE + 2 * wq * BLK;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)dst, 16, g0, 0, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(dst + BLK), 16, g1, 0, 0, 0);
  };

  // fused path: the thread's two K chunks through registers
  auto load_k = [&](int j, uint4 reg[2]) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(kbh, j);
    const int g[2] = {kg0, kg1};
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rs, g[r], 0, 0);
      reg[r] = make_uint4(x[0], x[1], x[2], x[3]);
    }
  };

  // Coefficients for the two K chunks of step j's tile; advances the row's packed
  // coordinates by one step's tokens.  A row at or past the rotated prefix takes
  // the identity position.
  auto fetch_coef = [&](int j, float2 cs[2][4]) __attribute__((always_inline)) {
    const uint32_t pos = (S * j + grp) * BNG + kr0 < a.rp.n_rot ? kpos : a.pos_sent;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < 4; ++p) cs[c][p] = table_entry(tab, kpi[c][p], pos);
    // mixed-radix step; past the grid the t field may wrap, but those rows use pos_sent
    uint32_t np = kpos + a.pos_step;
    if ((np & 2047u) >= (uint32_t)a.rp.gw) np += (1u << 11) - (uint32_t)a.rp.gw;
    if (((np >> 11) & 2047u) >= (uint32_t)a.rp.gh) np += (1u << 22) - ((uint32_t)a.rp.gh << 11);
    kpos = np;
  };

  auto store_k = [&](uint16_t* buf, const uint4 reg[2], const float2 cs[2][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      uint4 kv = reg[r];
      kv.x = rotate_pair(kv.x, cs[r][0]);
      kv.y = rotate_pair(kv.y, cs[r][1]);
      kv.z = rotate_pair(kv.z, cs[r][2]);
      kv.w = rotate_pair(kv.w, cs[r][3]);
      *reinterpret_cast<uint4*>(buf + grp * TILE + (2 * wq + r) * BLK + lane * 8) = kv;
    }
  };

  // per-lane LDS element offsets of the MFMA operands (operand order, above)
  const int koff = grp * TILE + lane * 8;
  const int voff = grp * TILE + lane * 4;

  float mref = -INFINITY;  // reference max (log2 units), identical in both lane halves
  auto qk = [&](const uint16_t* kb, f32x16& s) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < 8; ++st)
      s = mfma32(*reinterpret_cast<const bf16x8*>(kb + st * BLK + koff), qreg[st], st == 0 ? f32x16{} : s);
  };

  f32x16 oacc[4];
  float sum0 = INFINITY;   // start of the row sums: +inf until the first reset forces it
  float lsum = 0.f;        // this lane half's partial sum of p
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) oacc[mb] = f32x16{};

  // p = exp2(s c2 - mref) for the 32 keys of one key block as two bf16 MFMA
  // operands (16 keys each); returns tsum plus this lane's sum of p.  A rotated
  // query is scaled into log2 units (c2 = 1).  (The dense kernel starts the
  // score accumulators of rotated queries at -mref instead; here the 16
  // registers of that start are what would spill.)
  const float c2 = ROPE ? 1.f : a.c2;
  auto softmax_p = [&](const f32x16& s, bf16x8 pop[2], float tsum) __attribute__((always_inline)) {
    const float nm = -mref;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      uint32_t pw[4];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[8 * ks + e], c2, nm));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[8 * ks + e + 1], c2, nm));
        pw[e >> 1] = pack_bf16x2(p0, p1);
        tsum = dot2(pw[e >> 1], kOnesBf16x2, tsum);
      }
      pop[ks] = __builtin_bit_cast(bf16x8, make_uint4(pw[0], pw[1], pw[2], pw[3]));
    }
    return tsum;
  };

  // Probabilities of one key block.  The first block (its sum starts at
  // +inf) and a block whose row sum of p leaves [0, 2^64) reset the
  // reference to the running max, rescaling the output and the sum.
  auto softmax_blk = [&](const f32x16& s, bf16x8 pop[2]) __attribute__((always_inline)) {
    float tsum = softmax_p(s, pop, sum0);
    if (__builtin_amdgcn_ballot_w64(!(tsum < kSumLimit)) != 0) {
      sum0 = 0.f;
      float m = fmaxf(s[0], s[1]);
#pragma unroll
      for (int i = 2; i < 16; ++i) m = fmaxf(m, s[i]);
      const float mnew = fmaxf(mref, wave_half_max(m) * c2);
      const float alpha = __builtin_amdgcn_exp2f(mref - mnew);
      lsum *= alpha;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[mb][i] *= alpha;
      mref = mnew;
      tsum = softmax_p(s, pop, 0.f);
    }
    lsum += tsum;
  };

  // O^T += V^T P^T over the tile's 32 keys
  auto pv = [&](const uint16_t* vb, const bf16x8 pop[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        const i16x4 lo = lds_read_tr16(vb + (4 * ks + mb) * BLK + voff);
        const i16x4 hi4 = lds_read_tr16(vb + (4 * ks + mb) * BLK + BLK / 2 + voff);
        const bf16x8 vop = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
        oacc[mb] = mfma32(vop, pop[ks], oacc[mb]);
      }
    }
  };
  auto softmax_pv = [&](const f32x16& s, const uint16_t* vb) __attribute__((always_inline)) {
    bf16x8 pop[2];
    softmax_blk(s, pop);
    pv(vb, pop);
  };

  // The first NBUF K tiles and NBUF - 1 V tiles into their buffers, in the
  // order in which they are needed.
  auto first_copies = [&]() __attribute__((always_inline)) {
    if (ROPE_K) {
      uint4 k0[2], k1[2];
      float2 cs0[2][4], cs1[2][4];
      load_k(0, k0);
      load_k(1, k1);
      fetch_coef(0, cs0);
      fetch_coef(1, cs1);
      store_k(K0, k0, cs0);
      store_k(K1, k1, cs1);
      dma_tile(vbh, 0, V0, vg0, vg1);
    } else {
#pragma unroll
      for (int i = 0; i < NBUF; ++i) {
        dma_tile(kbh, i, kbuf(i), kg0, kg1);
        if (i + 1 < NBUF) dma_tile(vbh, i, vbuf(i), vg0, vg1);
      }
    }
  };
  // K_{j+2} and V_{j+1} (and all before them) have landed, as far as this wave
  // copied them; four buffers: the copies of the last two steps (2 x 4) may be
  // in flight.  LDS stores (rotated keys) are done.
  auto copies_landed = [&]() __attribute__((always_inline)) {
    if constexpr (NBUF == 2) __builtin_amdgcn_s_waitcnt(0);
    else __builtin_amdgcn_s_waitcnt(wait_vm(8));
  };
  // the step's barrier: with copies in flight, one without the fence's wait
  // for them (what the waves share otherwise, they share through the barrier
  // of the merge)
  auto step_barrier = [&]() __attribute__((always_inline)) {
    if constexpr (NBUF == 2) __syncthreads();
    else {
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);  // operand reads of the freed buffers are done
      lds_barrier();
    }
  };

  f32x16 sa, sb;

  // Step j (R = j mod NBUF): scores of tile j + 1, softmax and PV of tile j,
  // while K_{j+NBUF} and V_{j+NBUF-1} stream into the buffers that tiles j and
  // j - 1 have freed.  The buffers are chosen at compile time.
  // LAST (rotated keys): the last tile but one, no K tile to rotate behind it.
  auto step_of = [&](auto phase, auto last, int j, f32x16& scur, f32x16& snext) __attribute__((always_inline)) {
    constexpr int R = decltype(phase)::value;
    constexpr bool LOAD_K = ROPE_K && !decltype(last)::value;
    uint16_t* const kfree = kbuf(R);               // held K_j
    uint16_t* const knext = kbuf(R + 1);           // holds K_{j+1}
    uint16_t* const vcur = vbuf(R);                // holds V_j
    uint16_t* const vfree = vbuf(R + NBUF - 1);    // held V_{j-1}
    uint4 kn[2];
    float2 cs[2][4];
    if (LOAD_K) {
      load_k(j + 2, kn);
      fetch_coef(j + 2, cs);
    } else if (!ROPE_K) {
      dma_tile(kbh, j + NBUF, kfree, kg0, kg1);
    }
    dma_tile(vbh, j + NBUF - 1, vfree, vg0, vg1);
    if (live) {
      qk(knext, snext);
      softmax_pv(scur, vcur);
    }
    if (LOAD_K) store_k(kfree, kn, cs);
    copies_landed();
    step_barrier();
  };
  auto step = [&](auto phase, int j, f32x16& scur, f32x16& snext) __attribute__((always_inline)) {
    step_of(phase, std::false_type(), j, scur, snext);
  };

  // the tile whose first copies have landed (and been published): scores of
  // tile 0, the pipelined steps, and the last tile's softmax and PV
  auto run_tile = [&]() __attribute__((always_inline)) {
    if (live) qk(K0, sa);
    // step 0 refills K0: every wave must be done reading K_0 first
    step_barrier();
    using r0 = std::integral_constant<int, 0>;
    using r1 = std::integral_constant<int, 1>;
    using r2 = std::integral_constant<int, 2>;
    using r3 = std::integral_constant<int, 3>;
    int j = 0;
    if constexpr (NBUF == 4) {
      for (; j + 4 < nsteps; j += 4) {
        step(r0(), j, sa, sb);
        step(r1(), j + 1, sb, sa);
        step(r2(), j + 2, sa, sb);
        step(r3(), j + 3, sb, sa);
      }
    } else {
      for (; j + 2 < nsteps; j += 2) {
        step(r0(), j, sa, sb);
        step(r1(), j + 1, sb, sa);
      }
    }
    // the last tile's softmax and PV
    auto finish = [&](f32x16& s, const uint16_t* vb) __attribute__((always_inline)) {
      if (!live) return;
      const int rem = lv - (S * j + grp) * BNG;  // valid keys of the last tile (none: p = 0)
      if (rem < BNG) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + 4 * hi + (i & 3) >= rem) s[i] = -INFINITY;
      }
      softmax_pv(s, vb);
    };
    // (a copy of the end for each place where the steps can stop: a choice of
    // the score registers at run time would put them into memory)
    if (j + 1 >= nsteps) return finish(sa, vbuf(0));
    step_of(r0(), std::integral_constant<bool, ROPE_K>(), j, sa, sb);
    if (NBUF == 2 || j + 2 >= nsteps) {
      ++j;
      return finish(sb, vbuf(1));
    }
    ++j;
    step(r1(), j, sb, sa);
    if (++j + 1 >= nsteps) return finish(sa, vbuf(2));
    step(r2(), j, sa, sb);
    ++j;
    finish(sb, vbuf(3));
  };

  // ---- output: O = O^T / l (zero when no key is valid), LSE = m + ln l,
  // through the staging area.  Buffer stores: rows past Lq address past the
  // records and are dropped.
  auto store_o = [&](uint16_t* stage, float l, bool empty) __attribute__((always_inline)) {
    const float inv = empty ? 0.f : 1.0f / l;
    // formed here: shared with dma_q, the rows' offsets would be held (in
    // scratch) through the whole kernel
    int l16 = lane >> 4;
    asm("" : "+v"(l16));
    // the lane's row l32, d = 32 mb + 8 g + 4 hi .. + 3: half hi of chunk 4 mb + g
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        u32x2 pk;
        pk[0] = pack_bf16x2(oacc[mb][4 * g + 0] * inv, oacc[mb][4 * g + 1] * inv);
        pk[1] = pack_bf16x2(oacc[mb][4 * g + 2] * inv, oacc[mb][4 * g + 3] * inv);
        *reinterpret_cast<u32x2*>(stage + l32 * D + stage_slot(4 * mb + g, l32) * 8 + 4 * hi) = pk;
      }
    wave_lds_fence();
    // whole rows out: slot lane & 15 of row 4 i + (lane >> 4) holds chunk stage_slot(lane & 15, row)
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.o + (size_t)b * a.Lq * tok + (size_t)h * D), (short)0, a.Lq * rbytes, kBufferFlags);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = 4 * i + l16;
      const u32x4 v = *reinterpret_cast<const u32x4*>(stage + r * D + (lane & 15) * 8);
      const int grow = row0 + r;
      const int off = grow < a.Lq ? grow * rbytes + stage_slot(lane & 15, r) * 16 : 0x7ffffff0;
      __builtin_amdgcn_raw_buffer_store_b128(v, ro, off, 0, 0);
    }
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.lse ? a.lse + ((size_t)b * a.H + h) * a.Lq : a.lse), (short)0, a.lse ? a.Lq * 4 : 0,
        kBufferFlags);
    const float lse = empty ? -INFINITY : (mref + __log2f(l)) * 0.69314718055994531f;
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(lse), rl, qlive && hi == 0 ? qrow * 4 : 0x7ffffff0, 0, 0);
  };

  if (lv == 0) {  // no valid key: O = 0, LSE = -inf
    if (grp == 0) store_o(stage, 0.f, true);
    return;
  }
  dma_q();  // into the K/V buffers, which are free until the first copies
  if (ROPE) {
    for (int e = tid; e < a.tentries; e += NT) tab[e] = attn_table_entry(a, e);
    __syncthreads();
  }
  __builtin_amdgcn_s_waitcnt(0);  // this wave's query rows have landed
  {
    if (HALF) {
      rotate_staged_half_split();
      wave_lds_fence();
    }
    uint4 raw[8];
    read_q(raw);
    make_q(raw);
  }
  __syncthreads();  // every wave has its queries out of the K/V buffers
  first_copies();
  copies_landed();  // K_0, K_1 and V_0, as far as this wave copied them
  step_barrier();
  run_tile();
  __builtin_amdgcn_s_waitcnt(0);  // the copies past the last tile: the buffers are used again
  __syncthreads();  // every wave is done with the last V tile
  float l = wave_half_sum(lsum);
  {
    // Group 1 hands its output (16 KB a wave, one buffer each), reference and
    // sum to group 0.
    uint16_t* const buf = wq == 0 ? K0 : wq == 1 ? K1 : wq == 2 ? (NBUF == 4 ? K2 : V0) : (NBUF == 4 ? K3 : V1);
    float* const part = reinterpret_cast<float*>(buf) + lane * 4;
    float* const ml = (NBUF == 4 ? reinterpret_cast<float*>(V0) : reinterpret_cast<float*>(tab)) + wq * 64 + l32;
    if (grp == 1) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<float4*>(part + (4 * mb + g) * 256) =
              make_float4(oacc[mb][4 * g], oacc[mb][4 * g + 1], oacc[mb][4 * g + 2], oacc[mb][4 * g + 3]);
      if (hi == 0) {
        ml[0] = mref;
        ml[32] = l;
      }
    }
    __syncthreads();
    if (grp == 1) return;
    // group 0 always has keys, so its reference is finite; a group 1 without
    // any has reference -inf and factor 0
    const float mx = fmaxf(mref, ml[0]);
    const float f0 = __builtin_amdgcn_exp2f(mref - mx), f1 = __builtin_amdgcn_exp2f(ml[0] - mx);
    l = fmaf(l, f0, ml[32] * f1);
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 v = *reinterpret_cast<const float4*>(part + (4 * mb + g) * 256);
        oacc[mb][4 * g] = fmaf(v.x, f1, oacc[mb][4 * g] * f0);
        oacc[mb][4 * g + 1] = fmaf(v.y, f1, oacc[mb][4 * g + 1] * f0);
        oacc[mb][4 * g + 2] = fmaf(v.z, f1, oacc[mb][4 * g + 2] * f0);
        oacc[mb][4 * g + 3] = fmaf(v.w, f1, oacc[mb][4 * g + 3] * f0);
      }
    mref = mx;
    wave_lds_fence();  // the wave's part is read before its lanes write over it
    store_o(buf, l, false);  // staged in the area that only this wave reads
  }
}

}  // namespace

hipError_t launch_attn_fwd_split(const AttnArgs& a, hipStream_t stream) {
  const RopeParams& rp = a.rp;
  const unsigned g = (unsigned)a.nwg;
  if (rp.enabled && !rp.keys_prerotated) return launch_kernel(attn_fwd_split_kernel<true, true, false>, g, (unsigned)NT, stream, a);
  if (rp.enabled && rp.pair_mode != 0) return launch_kernel(attn_fwd_split_kernel<true, false, true>, g, (unsigned)NT, stream, a);
  if (rp.enabled) return launch_kernel(attn_fwd_split_kernel<true, false, false>, g, (unsigned)NT, stream, a);
  return launch_kernel(attn_fwd_split_kernel<false, false, false>, g, (unsigned)NT, stream, a);
}

}  // namespace vidax
