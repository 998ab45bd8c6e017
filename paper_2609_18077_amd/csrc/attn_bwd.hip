// Attention backward for gfx950: the gradient of o = softmax(scale q k^T) v
// (non-causal, per-batch valid-key prefix) for a given dO, from the forward's
// output O and natural-log sum-exp.  bf16 in/out, fp32 accumulation, head
// dim 128.  With P = exp(scale q k^T - lse):
//
//   D_i = <dO_i, O_i>            dq kernel, from the own rows' dO (loaded
//                                  anyway) and O; written for the dkdv kernel
//   dQ  = scale dS K             dq kernel: one query tile per workgroup,
//                                  streaming K and V tiles
//   dV  = P^T dO, dK = scale dS^T Q   dkdv kernel: one key tile per
//                                  workgroup, streaming Q and dO tiles
//   dS  = P * (dO V^T - D)
//
// Both matrix kernels stream tiles of 64 rows straight from global memory
// into LDS (buffer loads with the LDS flag), two buffers per tensor, one
// barrier per tile, and keep the tiles as 256-byte rows with XOR-permuted
// 16-byte chunks (the row layout at the dq kernel), which every operand read
// -- 16-byte row reads and the transposing ds_read_b64_tr_b16 -- hits without
// bank conflicts.  The dq kernel follows the forward kernel's formulation:
// a wave's 32 own queries (q and dO) stay in registers as the B operand of
// v_mfma_f32_32x32x16_bf16, the K and V rows are the A operand, S^T and dP^T
// land in accumulators whose lanes each hold one query, and dS^T, converted
// to bf16 in place, is the B operand of dQ^T += K^T dS^T with K^T from the
// transposing read of the same K tile, in the matching key order.  The dkdv
// kernel is its mirror image: 32 own keys per wave, Q and dO streamed, both
// key gradients from one pass over the queries.  Workgroups are ordered so
// that every XCD gets its share of every batch (balanced_tile): with batch
// after batch, the XCDs of the longer batches finished last.
#include <mutex>
#include <type_traits>

#include "launch.hpp"

namespace vidax {
namespace {

constexpr int D = kHeadDim;
constexpr int BN = 64;        // rows per streamed tile
constexpr int NW = 8;         // waves of a dkdv workgroup
constexpr int NT = NW * 64;   // its threads
constexpr int kBufferFlags = 0x00020000;  // raw buffer, 32-bit data format
constexpr float kLog2e = 1.4426950408889634f;

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

struct BwdArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const uint16_t* o;
  const uint16_t* dout;
  const float* lse;
  float* delta;
  uint16_t* dq;
  uint16_t* dk;
  uint16_t* dv;
  const int32_t* kv_valid_len;
  int B, H, Lq, Lk;
  float scale;
  float c;    // scale * log2(e)
  int ntile;  // own-row tiles per (b, h) of the launched kernel
  int nwg;    // workgroups of the launched kernel
  // key-side kernels: the query stream is cut into qsplit runs of qper
  // 64-row tiles, one workgroup each; with qsplit > 1 each writes its fp32
  // partial dK or dV to part ([qsplit][B][Lk][H][d], dV after dK) and the
  // reduce kernel sums them
  int qsplit, qper;
  float* part;
  int kper;  // keys per workgroup of the dkdv kernel (kBwdKeys or half of it)
};

[[maybe_unused]] __device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ i16x4 lds_read_tr16(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p));
}

// Sum over lanes l and l ^ 32.
__device__ __forceinline__ float half_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Lv of batch b (uniform).
__device__ __forceinline__ int valid_keys(const BwdArgs& a, int b) {
  int lv = a.Lk;
  if (a.kv_valid_len) lv = min(max(a.kv_valid_len[b], 0), a.Lk);
  return __builtin_amdgcn_readfirstlane(lv);
}

// Buffer resource of 64-row tile `tile` of rows [0, limit): later rows read
// as zero (and land in LDS as zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const uint16_t* base, int tile, int limit, int tok) {
  const int rows = min(max(limit - tile * BN, 0), BN);
  const int nbytes = __builtin_amdgcn_readfirstlane(rows * tok * 2);
  return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (size_t)tile * BN * tok), (short)0, nbytes, kBufferFlags);
}

// B operand of the wave's own row: chunks 2 s + hi (s = 0..7) of the row at
// p (zero when !live).
__device__ __forceinline__ void own_operand(const uint16_t* p, bool live, int hi, bf16x8 op[8]) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    uint4 x = make_uint4(0, 0, 0, 0);
    if (live) x = *reinterpret_cast<const uint4*>(p + (2 * s + hi) * 8);
    op[s] = __builtin_bit_cast(bf16x8, x);
  }
}

// Rows 16 k2 .. + 15 of a 32 x 32 fp32 accumulator (tile rows x own rows) ->
// a bf16 B operand, in the accumulator's row order.
__device__ __forceinline__ bf16x8 pack8(const f32x16& x, int k2) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 8; e += 2) w[e >> 1] = pack_bf16x2(x[8 * k2 + e], x[8 * k2 + e + 1]);
  return __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
}

// Tile row (0..63) of register i of accumulator blk for lane half hi.
[[maybe_unused]] __device__ __forceinline__ int acc_row(int blk, int i, int hi) { return 32 * blk + 8 * (i >> 2) + 4 * hi + (i & 3); }

// ---- dQ: one tile of 32 NWQ queries of one (b, h) per workgroup of NWQ
// waves: 8 for long key sequences, 4 for short ones (two workgroups then
// share a CU, so that one's start and end overlap the other's products --
// with few key tiles per workgroup those dominate).  K and V tiles of 64 keys
// in the swizzled row layout (see below), double-buffered:
//   S^T = K Q^T, dP^T = V dO^T (A: key rows, one 16-byte read), P^T =
//   exp2(S^T c - lse log2 e), dS^T = P^T (dP^T - D), dQ^T += K^T dS^T (A: the
//   transposing read of the same K tile: 4 keys x 16 d per 16-lane group, in
//   the key order of the dS^T operand taken from the accumulator).
constexpr int STILE = BN * D;  // elements of a swizzled tile
// key tiles at or below which the dq workgroups have 4 waves instead of 8
constexpr int kDqShortTiles = 16;

// Tiles of 64 rows sit in LDS as 256-byte rows whose 16-byte chunks are
// permuted: chunk c of row r at position c ^ swz(r), swz(r) = 4 (r mod 4) +
// (r / 4) mod 4.  Any 4 consecutive rows then put a 64-byte span into 4
// different quarters of the banks (the transposing reads), and the 16 rows of
// a row read's phase put one chunk into 16 different places: no bank
// conflicts.  Copy j of a tile fills rows 4 j .. 4 j + 3: lane l writes
// position l & 15 of row 4 j + (l >> 4), fetching its chunk (l & 15) ^
// swz(row) (each row read whole, 256 contiguous bytes).
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// Per-lane LDS element offsets of the operands in a swizzled tile, one register
// each (the step's constants enter by XOR):
//   row operand st, tile row l32 (+ 32 blk), d = 16 st + 8 hi: chunk 2 st + hi
//     of the row at row ^ (16 st);
//   transposed operand mb (reads h = 0, 1 of a 16-row step), row 8 h + 4 hi +
//     (w >> 2), d = 32 mb + 16 (g & 1) + 4 (w & 3) for lane l = 16 g + w: at
//     (tr ^ (32 mb) ^ (16 h)) + 8 h rows.
struct TileOffsets {
  int row, tr;
};
__device__ __forceinline__ TileOffsets tile_offsets(int lane) {
  const int l32 = lane & 31, hi = lane >> 5, g = lane >> 4, w = lane & 15, r = 4 * hi + (w >> 2);
  TileOffsets o;
  o.row = l32 * D + 8 * (hi ^ swz(l32));
  o.tr = r * D + 8 * ((2 * (g & 1) + ((w >> 1) & 1)) ^ swz(r)) + 4 * (w & 1);
  return o;
}
// x, as a value of iteration t: what is computed from it stays in the loop
// (hoisted, every buffer's addresses would live in registers of their own
// instead of in the reads' immediate offsets).
__device__ __forceinline__ int in_loop(int x, int t) {
  asm("" : "+v"(x) : "s"(t));
  return x;
}
__device__ __forceinline__ bf16x8 read_row(const uint16_t* tile, int row, int st) {
  return *reinterpret_cast<const bf16x8*>(tile + (row ^ (16 * st)));
}
__device__ __forceinline__ bf16x8 read_tr(const uint16_t* rows16, int tr, int mb) {
  const i16x4 lo = lds_read_tr16(rows16 + (tr ^ (32 * mb)));
  const i16x4 up = lds_read_tr16(rows16 + (tr ^ (32 * mb) ^ 16) + 8 * D);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int NWQ>
__device__ __forceinline__ void dq_body(const BwdArgs& a) {
  constexpr int BWQ = NWQ * 32;       // queries per workgroup
  constexpr int NCOPY = 16 / NWQ;     // copies per wave of a tile (16 of 4 rows)
  __shared__ __attribute__((aligned(16))) uint16_t K0[STILE], K1[STILE], V0[STILE], V1[STILE];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lid = balanced_tile(blockIdx.x, a.nwg, a.B);
  const int qt = lid % a.ntile, bh = lid / a.ntile, h = bh % a.H, b = bh / a.H;
  const int tok = a.H * D, rbytes = tok * 2;
  const int lv = valid_keys(a, b);
  const int qrow = qt * BWQ + wave * 32 + l32;
  const bool qlive = qrow < a.Lq;
  const size_t lrow = ((size_t)b * a.H + h) * a.Lq + (qlive ? qrow : 0);
  // The wave's 32 rows come in and go out whole (16 lanes a 256-byte row),
  // through 8 KB staging areas in the tile buffers, free before the first
  // copies and after the last tile: one per wave, or with 4 waves two (q and
  // dO at once).  Per-lane 16-byte pieces of 32 rows would fetch every line
  // several times: at short key sequences these rows are most of the traffic
  // (2 x 40 heads x 32760 x 512: backward 1696 -> 1602 us).
  constexpr int AREAS = 8 / NWQ;
  const int wa = AREAS * wave;
  uint16_t* const area = (wa < 2 ? K0 : wa < 4 ? K1 : wa < 6 ? V0 : V1) + (wa & 1) * 32 * D;
  const int row0 = qt * BWQ + wave * 32;
  const size_t off0 = ((size_t)b * a.Lq + row0) * tok + (size_t)h * D;  // first row (may lie past Lq: no records then)
  auto rows_rsrc = [&](const uint16_t* base) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc(
        (void*)(base + off0), (short)0, __builtin_amdgcn_readfirstlane(min(max(a.Lq - row0, 0), 32) * rbytes), kBufferFlags);
  };
  // rows 4 i .. 4 i + 3: byte offset of what the lane moves (position lane & 15 of row 4 i + (lane >> 4))
  auto row_off = [&](int i) __attribute__((always_inline)) {
    const int r = 4 * i + (lane >> 4);
    return r * rbytes + ((lane & 15) ^ swz(r)) * 16;
  };
  auto rows_in = [&](const uint16_t* base, uint16_t* dst) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = rows_rsrc(base);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(dst + 4 * i * D), 16, row_off(i), 0, 0, 0);
  };
  const TileOffsets off = tile_offsets(lane);
  auto own_rows = [&](const uint16_t* src, bf16x8 op[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 8; ++s) op[s] = read_row(src, off.row, s);
  };
  // dQ = acc * mul, row l32, d = 32 mb + 8 g + 4 hi .. + 3: half hi of chunk 4 mb + g
  auto rows_out = [&](const f32x16 acc[4], float mul) __attribute__((always_inline)) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 pk;
        pk.x = pack_bf16x2(acc[mb][4 * g + 0] * mul, acc[mb][4 * g + 1] * mul);
        pk.y = pack_bf16x2(acc[mb][4 * g + 2] * mul, acc[mb][4 * g + 3] * mul);
        *reinterpret_cast<uint2*>(area + l32 * D + ((4 * mb + g) ^ swz(l32)) * 8 + 4 * hi) = pk;
      }
    wave_lds_fence();
    const __amdgpu_buffer_rsrc_t rs = rows_rsrc(a.dq);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(area + (4 * i + (lane >> 4)) * D + (lane & 15) * 8);
      __builtin_amdgcn_raw_buffer_store_b128(v, rs, row_off(i), 0, 0);  // rows past Lq: past the records, dropped
    }
  };
  bf16x8 dop[8], qop[8], oop[8];
  rows_in(a.dout, area);
  if (AREAS == 2) rows_in(a.q, area + 32 * D);
  own_operand(a.o + ((size_t)b * a.Lq + (qlive ? qrow : 0)) * tok + (size_t)h * D, qlive, hi, oop);
  const float lse2 = qlive ? a.lse[lrow] * kLog2e : INFINITY;  // dead rows: P = 0
  __builtin_amdgcn_s_waitcnt(0);  // this wave's rows have landed
  own_rows(area, dop);
  if (AREAS == 2) {
    own_rows(area + 32 * D, qop);
  } else {
    __builtin_amdgcn_s_waitcnt(0);  // dO is out of the area
    rows_in(a.q, area);
  }
  // D of the own row: this lane half's 64 products <dO, O>, then the other
  // half's; stored for the dkdv kernel (every row, also without valid keys)
  float dl;
  {
    // packed bf16 pair products, two fp32 chains
    float sum[2] = {0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const uint4 x = __builtin_bit_cast(uint4, dop[s]), y = __builtin_bit_cast(uint4, oop[s]);
      const uint32_t xw[4] = {x.x, x.y, x.z, x.w}, yw[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
      for (int p = 0; p < 4; ++p)
        sum[p & 1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, xw[p]), __builtin_bit_cast(bf16x2, yw[p]),
                                                     sum[p & 1], false);
    }
    dl = half_sum(sum[0] + sum[1]);
    if (qlive && hi == 0) a.delta[lrow] = dl;
  }
  if (AREAS == 1) {
    __builtin_amdgcn_s_waitcnt(0);
    own_rows(area, qop);
  }
  f32x16 acc[4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) acc[mb] = f32x16{};
  __builtin_amdgcn_s_waitcnt(0);  // the rows are out of the staging areas
  __syncthreads();
  if (lv == 0) {  // no valid key: dQ = 0
    rows_out(acc, 0.f);
    return;
  }

  const uint16_t* kbh = a.k + (size_t)b * a.Lk * tok + (size_t)h * D;
  const uint16_t* vbh = a.v + (size_t)b * a.Lk * tok + (size_t)h * D;
  const int ntiles = (lv + BN - 1) / BN;
  // the wave's copies NCOPY wave .. + NCOPY - 1 of a tile: byte offsets from its first row
  int cg[NCOPY];
#pragma unroll
  for (int u = 0; u < NCOPY; ++u) {
    const int row = 4 * (NCOPY * wave + u) + (lane >> 4);
    cg[u] = row * rbytes + ((lane & 15) ^ swz(row)) * 16;
  }
  auto copies = [&](int j, uint16_t* kb, uint16_t* vb) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rk = tile_rsrc(kbh, j, lv, tok);
    const __amdgpu_buffer_rsrc_t rv = tile_rsrc(vbh, j, lv, tok);
#pragma unroll
    for (int u = 0; u < NCOPY; ++u) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_ptr)(kb + (NCOPY * wave + u) * 512), 16, cg[u], 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_ptr)(vb + (NCOPY * wave + u) * 512), 16, cg[u], 0, 0, 0);
    }
  };
  copies(0, K0, V0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // One tile, hand-scheduled: one slot per product, each slot also issuing the
  // operand reads of the product three slots later and its share of the vector
  // work.  S of block 0, dP of block 0 beside its exponentials, S of block 1
  // beside dS of block 0, dP of block 1 beside its exponentials, dQ of block 0
  // beside dS of block 1, dQ of block 1: no product waits for the vector work
  // before it.  At 32760 x 32760 x 12 heads: 8.16 -> 7.60 ms, matrix cores busy 80 %
  // of the cycles, at the clock (1.6 GHz of 2.4) that the board's power limit
  // leaves.  TAIL: the last tile, whose keys past Lv get P = 0.
  auto step = [&](auto par, auto tl, int j) __attribute__((always_inline)) {
    constexpr int P = decltype(par)::value;
    constexpr bool TAIL = decltype(tl)::value;
    const uint16_t* kt = P ? K1 : K0;
    const uint16_t* vt = P ? V1 : V0;
    if (!TAIL) copies(j + 1, P ? K0 : K1, P ? V0 : V1);
    const int orow = in_loop(off.row, j), otr = in_loop(off.tr, j);
    // operand reads in the order of their products: S0, dP0, S1, dP1, dQ0, dQ1
    bf16x8 op[48];
    auto read_op = [&](auto N) __attribute__((always_inline)) {
      constexpr int n = decltype(N)::value;
      if constexpr (n < 48) {
        constexpr int blk = n < 32 ? n >> 4 : (n - 32) >> 3;
        if constexpr (n >= 32) op[n] = read_tr(kt + (32 * blk + 16 * ((n >> 2) & 1)) * D, otr, n & 3);
        else op[n] = read_row((n & 8 ? vt : kt) + 32 * blk * D, orow, n & 7);
      }
    };
    f32x16 sc[2], dp[2];
    bf16x8 ds[2][2];
    const int left = lv - j * BN - 4 * hi;  // TAIL: valid keys of the tile, from this lane half's first
    auto exps = [&](int blk, int i0) __attribute__((always_inline)) {  // P of elements i0, i0 + 1
#pragma unroll
      for (int i = i0; i < i0 + 2; ++i) {
        const float x = fmaf(sc[blk][i], a.c, -lse2);
        sc[blk][i] = __builtin_amdgcn_exp2f(TAIL && acc_row(blk, i, 0) >= left ? -INFINITY : x);
      }
    };
    auto mul4 = [&](int blk, int i0) __attribute__((always_inline)) {  // dS of elements i0 .. i0 + 3
#pragma unroll
      for (int i = i0; i < i0 + 4; ++i) dp[blk][i] *= sc[blk][i];
    };
    for_slots<3>(read_op);
    SLOT();
    for_slots<48>([&](auto N) __attribute__((always_inline)) {
      constexpr int n = decltype(N)::value, blk = n < 32 ? n >> 4 : (n - 32) >> 3, u = n & 7;
      if constexpr (n >= 32) acc[u & 3] = mfma32(op[n], ds[blk][u >> 2], acc[u & 3]);
      else if constexpr (n & 8) {
        if constexpr (u == 0)
#pragma unroll
          for (int i = 0; i < 16; ++i) dp[blk][i] = -dl;
        dp[blk] = mfma32(op[n], dop[u], dp[blk]);
      }
      else sc[blk] = mfma32(op[n], qop[u], u == 0 ? f32x16{} : sc[blk]);
      read_op(std::integral_constant<int, n + 3>());
      // vector work of block 0 from its second dP slot on (10), of block 1 from 26 on:
      // eight slots of exponentials, four of products, the packs
      for_slots<2>([&](auto V) __attribute__((always_inline)) {
        constexpr int vb = decltype(V)::value, r = n - (vb ? 26 : 10);
        if constexpr (r >= 0 && r < 8) exps(vb, 2 * r);
        if constexpr (r >= 8 && r < 12) mul4(vb, 4 * (r - 8));
        if constexpr (r == 10) ds[vb][0] = pack8(dp[vb], 0);
        if constexpr (r == 12) ds[vb][1] = pack8(dp[vb], 1);
      });
      SLOT();
    });
    if (!TAIL) {
      __builtin_amdgcn_s_waitcnt(0);  // this wave's copies have landed
      __syncthreads();
    }
  };
  using even = std::integral_constant<int, 0>;
  using odd = std::integral_constant<int, 1>;
  using full = std::false_type;
  using last = std::true_type;
  int j = 0;
  for (; j + 2 < ntiles; j += 2) {
    step(even(), full(), j);
    step(odd(), full(), j + 1);
  }
  if (j + 1 < ntiles) {
    step(even(), full(), j);
    step(odd(), last(), j + 1);
  } else {
    step(even(), last(), j);
  }
  __syncthreads();  // every wave is done with the last tile
  rows_out(acc, a.scale);
}

// 4 waves (128 queries) a workgroup where the key sequence is short, 8
// waves (256 queries) otherwise.
__global__ __launch_bounds__(256, 2) void bwd_dq4_kernel(BwdArgs a) { dq_body<4>(a); }
__global__ __launch_bounds__(512) void bwd_dq8_kernel(BwdArgs a) { dq_body<8>(a); }

// ---- dK and dV together: one tile of 256 keys of one (b, h) per workgroup,
// 32 keys per wave, one workgroup per CU.  The mirror image of the dq kernel:
// the own rows are keys, the streamed tiles Q and dO.  Per 64-query tile and
// 32-query block:
//   S = Q K^T, dP - D = dO V^T - D  (A: Q / dO rows, one 16-byte read; the
//     dP accumulators start at -D, so the subtraction costs no vector work)
//   P = exp2(S c - lse log2 e), dS = P (dP - D)   (lane: key column, 16 queries)
//   dV^T += dO^T P, dK^T += Q^T dS  (A: the transposing read of the same
//     tiles, B: P / dS from the accumulator, in the same query order)
// Bound: LDS reads against the matrix cores.  With 32 keys a wave, each 8 KB
// of streamed operands feed a 32 x 32 x 128 product (with 16 keys a wave half
// of that: 13.7 -> 11.2 ms at 32760 x 32760 x 12 heads).  The two accumulators take
// 128 registers and v 32; k does not fit beside them without spills, so each
// wave keeps it in LDS in operand order (8 KB, one conflict-free 1 KB read
// per product).  A key column past the valid length needs no mask: nothing of
// it reaches another column, and the column is written as zero.
// A workgroup with at most 128 valid keys gives each of its 32-key groups to
// two waves, which take alternate query blocks and add up at the end (short
// texts would leave more than half of the waves idle).  So does every workgroup
// of a launch with 128 keys a workgroup (kper; the rule is at attn_bwd_split):
// half the chain per workgroup where that takes no more rounds.
constexpr int BK = kBwdKeys;  // keys per workgroup
constexpr int KOWN = 32 * D;  // elements of one wave's own keys in LDS

__global__ __launch_bounds__(NT) void bwd_dkdv_kernel(BwdArgs a) {
  // the tiles' larger alignment puts them below 64 KB of LDS, where one
  // address register a lane reaches all four through the reads' 16-bit offset
  __shared__ __attribute__((aligned(1024))) uint16_t Qk0[STILE], Qk1[STILE], Ok0[STILE], Ok1[STILE];
  __shared__ __attribute__((aligned(16))) uint16_t KB[NW * KOWN];
  __shared__ __attribute__((aligned(16))) float Lt[2][BN], Dt[2][BN];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lid = balanced_tile(blockIdx.x, a.nwg, a.B);
  const int kt = lid % a.ntile, sbh = lid / a.ntile, sp = sbh % a.qsplit, bh = sbh / a.qsplit;
  const int h = bh % a.H, b = bh / a.H;
  const int tok = a.H * D, rbytes = tok * 2;
  const int lv = valid_keys(a, b);
  const int key0 = kt * a.kper;
  const int nvalid = lv - key0;  // valid keys from the workgroup's first on (may be past its own, or negative)
  const int t0 = sp * a.qper;
  const int t1 = min(t0 + a.qper, (a.Lq + BN - 1) / BN);
  f32x16 dk[4], dv[4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) dk[mb] = dv[mb] = f32x16{};
  // With runs: the fp32 partials of key row `row` (lane holds it), d = 32 mb +
  // 8 g + 4 hi .. + 3: the accumulators where `row` is a valid key, zero otherwise
  auto partials_out = [&](int row) __attribute__((always_inline)) {
    if (row >= a.Lk) return;
    const size_t rowoff = ((size_t)b * a.Lk + row) * tok + (size_t)h * D, n = (size_t)a.B * a.Lk * tok;
    float* pk = a.part + (size_t)sp * n + rowoff;
    float* pv = a.part + (size_t)(a.qsplit + sp) * n + rowoff;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
        if (row < lv) {
          x = make_float4(dk[mb][4 * g], dk[mb][4 * g + 1], dk[mb][4 * g + 2], dk[mb][4 * g + 3]);
          y = make_float4(dv[mb][4 * g], dv[mb][4 * g + 1], dv[mb][4 * g + 2], dv[mb][4 * g + 3]);
        }
        *reinterpret_cast<float4*>(pk + 32 * mb + 8 * g + 4 * hi) = x;
        *reinterpret_cast<float4*>(pv + 32 * mb + 8 * g + 4 * hi) = y;
      }
  };
  // Otherwise the gradient rows leave whole (16 lanes a 256-byte row), through
  // an LDS area of the wave's own: stored from the accumulators, 8 bytes of 64
  // rows an instruction, they made short query streams 5 to 30 % slower (64
  // queries x 300 keys x 130 heads, whole backward: 45.4 -> 33.6 us).
  // buffer over 32 key rows from `row` on (none past Lk) of dk or dv, and what the lane
  // moves of rows 4 i .. 4 i + 3 (position lane & 15 of row 4 i + (lane >> 4))
  auto rows_rsrc = [&](uint16_t* base, int row) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc(
        (void*)(base + ((size_t)b * a.Lk + row) * tok + (size_t)h * D), (short)0,
        __builtin_amdgcn_readfirstlane(min(max(a.Lk - row, 0), 32) * rbytes), kBufferFlags);
  };
  auto row_off = [&](int i) __attribute__((always_inline)) {
    const int r = 4 * i + (lane >> 4);
    return r * rbytes + ((lane & 15) ^ swz(r)) * 16;
  };
  // zeros to the 32 rows from `row` on
  auto zero_rows = [&](int row) __attribute__((always_inline)) {
    if (a.qsplit > 1) return partials_out(row + l32);
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      __builtin_amdgcn_raw_buffer_store_b128(z, rows_rsrc(a.dk, row), row_off(i), 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(z, rows_rsrc(a.dv, row), row_off(i), 0, 0);
    }
  };
  // acc * mul (zero past the valid keys) to the 32 rows from `row` on, whole rows, through area
  auto rows_out = [&](uint16_t* dst, int row, const f32x16 acc[4], float mul, uint16_t* area) __attribute__((always_inline)) {
    const bool keep = row + l32 < lv;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 pk = make_uint2(0u, 0u);
        if (keep) {
          pk.x = pack_bf16x2(acc[mb][4 * g + 0] * mul, acc[mb][4 * g + 1] * mul);
          pk.y = pack_bf16x2(acc[mb][4 * g + 2] * mul, acc[mb][4 * g + 3] * mul);
        }
        *reinterpret_cast<uint2*>(area + l32 * D + ((4 * mb + g) ^ swz(l32)) * 8 + 4 * hi) = pk;
      }
    wave_lds_fence();
    const __amdgpu_buffer_rsrc_t rs = rows_rsrc(dst, row);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const u32x4 x = *reinterpret_cast<const u32x4*>(area + (4 * i + (lane >> 4)) * D + (lane & 15) * 8);
      __builtin_amdgcn_raw_buffer_store_b128(x, rs, row_off(i), 0, 0);
    }
    wave_lds_fence();
  };
  if (nvalid <= 0 || t0 >= t1) {  // no valid key (zero gradient) or no query in this run
    if (wave * 32 < a.kper) zero_rows(key0 + wave * 32);
    return;
  }
  const bool paired = nvalid <= BK / 2 || a.kper < BK;  // uniform: two waves per 32-key group
  const int kg = paired ? wave & 3 : wave, part = wave >> 2;
  const int krow = key0 + kg * 32 + l32;
  const bool wlive = kg * 32 < nvalid;  // uniform
  const bool klive = krow < a.Lk;
  // own k and v as B operands: lane holds key krow, chunk 2 st + hi; k goes to LDS
  uint16_t* const kb = KB + wave * KOWN + lane * 8;
  bf16x8 vop[8];
  {
    const size_t rowoff = ((size_t)b * a.Lk + (klive ? krow : 0)) * tok + (size_t)h * D;
    bf16x8 kop[8];
    own_operand(a.k + rowoff, klive, hi, kop);
    own_operand(a.v + rowoff, klive, hi, vop);
#pragma unroll
    for (int st = 0; st < 8; ++st) *reinterpret_cast<bf16x8*>(kb + st * 512) = kop[st];
  }

  const uint16_t* qbh = a.q + (size_t)b * a.Lq * tok + (size_t)h * D;
  const uint16_t* obh = a.dout + (size_t)b * a.Lq * tok + (size_t)h * D;
  const float* lseb = a.lse + ((size_t)b * a.H + h) * a.Lq;
  const float* delb = a.delta + ((size_t)b * a.H + h) * a.Lq;
  // the wave's copies 2 wave, 2 wave + 1 of a tile: byte offsets from its first row
  int cg[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int row = 4 * (2 * wave + u) + (lane >> 4);
    cg[u] = row * rbytes + ((lane & 15) ^ swz(row)) * 16;
  }
  auto copy_tile = [&](__amdgpu_buffer_rsrc_t rs, uint16_t* buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(buf + (2 * wave + u) * 512), 16, cg[u], 0, 0, 0);
  };
  float lrow = INFINITY, drow = 0.f;
  auto copies = [&](int t, uint16_t* qk, uint16_t* ok) __attribute__((always_inline)) {
    copy_tile(tile_rsrc(qbh, t, a.Lq, tok), qk);
    copy_tile(tile_rsrc(obh, t, a.Lq, tok), ok);
    if (tid < BN) {
      const int r = t * BN + tid;
      lrow = r < a.Lq ? lseb[r] : INFINITY;  // rows past Lq: P = 0
      drow = r < a.Lq ? delb[r] : 0.f;
    }
  };
  auto put_rows = [&](int buf) __attribute__((always_inline)) {
    if (tid < BN) {
      Lt[buf][tid] = -lrow * kLog2e;
      Dt[buf][tid] = -drow;
    }
  };
  copies(t0, Qk0, Ok0);
  put_rows(0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const TileOffsets off = tile_offsets(lane);
  auto step = [&](auto par, int t) __attribute__((always_inline)) {
    constexpr int P = decltype(par)::value;
    const uint16_t* qt = P ? Qk1 : Qk0;
    const uint16_t* ot = P ? Ok1 : Ok0;
    if (t + 1 < t1) copies(t + 1, P ? Qk0 : Qk1, P ? Ok0 : Ok1);
    const int orow = in_loop(off.row, t), otr = in_loop(off.tr, t);
    if (wlive) {
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) {
        if (paired && blk != part) continue;  // uniform
        // Hand-scheduled: one slot per product, each slot also issuing the
        // operand reads of the product three slots later and its share of
        // the vector work, so that a wave waits neither for LDS nor for its
        // exponentials (left to the compiler, every score product waited for
        // a read issued just before it).  At 32760 x 32760 x 12 heads: 11.2 ->
        // 10.3 ms, matrix cores busy 77 % of the cycles.
        const uint16_t* qb = qt + 32 * blk * D;
        const uint16_t* ob = ot + 32 * blk * D;
        f32x16 s = f32x16{}, dp;
        bf16x8 qa[8], ka[8], oa[8], ta[8], tb[8], pb[2], db[2];
        float4 nl[4];
        auto exps = [&](int i) __attribute__((always_inline)) {  // P of elements i, i + 1
          const float4 l4 = nl[i >> 2];
          s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], a.c, (i & 2) ? l4.z : l4.x));
          s[i + 1] = __builtin_amdgcn_exp2f(fmaf(s[i + 1], a.c, (i & 2) ? l4.w : l4.y));
        };
        auto read_qk = [&](int st) __attribute__((always_inline)) {
          qa[st] = read_row(qb, orow, st);
          ka[st] = *reinterpret_cast<const bf16x8*>(kb + st * 512);
        };
#pragma unroll
        for (int st = 0; st < 3; ++st) read_qk(st);
        SLOT();
#pragma unroll
        for (int st = 0; st < 8; ++st) {  // S
          s = mfma32(qa[st], ka[st], s);
          if (st + 3 < 8) read_qk(st + 3);
          else oa[st - 5] = read_row(ob, orow, st - 5);
          if (st >= 1 && st < 5) {
            const float4 d4 = *reinterpret_cast<const float4*>(&Dt[P][32 * blk + 8 * (st - 1) + 4 * hi]);
            dp[4 * st - 4] = d4.x; dp[4 * st - 3] = d4.y; dp[4 * st - 2] = d4.z; dp[4 * st - 1] = d4.w;
          }
          SLOT();
        }
#pragma unroll
        for (int st = 0; st < 8; ++st) {  // dP - D; P of elements 0 .. 11
          dp = mfma32(oa[st], vop[st], dp);
          if (st + 3 < 8) oa[st + 3] = read_row(ob, orow, st + 3);
          else ta[st - 5] = read_tr(ob, otr, st - 5);
          if (st < 4) nl[st] = *reinterpret_cast<const float4*>(&Lt[P][32 * blk + 8 * st + 4 * hi]);
          if (st >= 2) exps(2 * (st - 2));
          if (st == 6) pb[0] = pack8(s, 0);
          SLOT();
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {  // dV; the rest of P, then dS
          const int mb = u & 3;
          dv[mb] = mfma32(ta[u], pb[u >> 2], dv[mb]);
          if (u + 3 < 8) ta[u + 3] = read_tr(ob + 16 * ((u + 3) >> 2) * D, otr, (u + 3) & 3);
          else tb[u - 5] = read_tr(qb, otr, u - 5);
          if (u < 2) exps(12 + 2 * u);
          if (u == 2) pb[1] = pack8(s, 1);
          if (u >= 3 && u < 7) {
#pragma unroll
            for (int i = 4 * (u - 3); i < 4 * (u - 3) + 4; ++i) dp[i] *= s[i];
          }
          if (u == 5) db[0] = pack8(dp, 0);
          if (u == 7) db[1] = pack8(dp, 1);
          SLOT();
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {  // dK
          const int mb = u & 3;
          dk[mb] = mfma32(tb[u], db[u >> 2], dk[mb]);
          if (u + 3 < 8) tb[u + 3] = read_tr(qb + 16 * ((u + 3) >> 2) * D, otr, (u + 3) & 3);
          SLOT();
        }
      }
    }
    if (t + 1 < t1) put_rows(1 - P);
    __builtin_amdgcn_s_waitcnt(0);  // this wave's copies have landed
    __syncthreads();
  };
  using even = std::integral_constant<int, 0>;
  using odd = std::integral_constant<int, 1>;
  int t = t0;
  for (; t + 1 < t1; t += 2) {
    step(even(), t);
    step(odd(), t + 1);
  }
  if (t < t1) step(even(), t);
  if (paired) {
    // waves 4..7 hand their sums to waves 0..3 through the buffers (all free
    // after the last step's barrier): dK in the own-key area, dV in the tiles
    float* const xk = reinterpret_cast<float*>(KB) + kg * 4096 + lane * 4;
    float* const xv = reinterpret_cast<float*>(kg == 0 ? Qk0 : kg == 1 ? Qk1 : kg == 2 ? Ok0 : Ok1) + lane * 4;
    if (part == 1) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          *reinterpret_cast<float4*>(xk + (4 * mb + g) * 256) =
              make_float4(dk[mb][4 * g], dk[mb][4 * g + 1], dk[mb][4 * g + 2], dk[mb][4 * g + 3]);
          *reinterpret_cast<float4*>(xv + (4 * mb + g) * 256) =
              make_float4(dv[mb][4 * g], dv[mb][4 * g + 1], dv[mb][4 * g + 2], dv[mb][4 * g + 3]);
        }
    }
    __syncthreads();
    if (part == 1) {
      if (a.kper == BK) zero_rows(key0 + kg * 32 + BK / 2);  // the upper half of the tile holds no valid key: zero
      return;
    }
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 x = *reinterpret_cast<const float4*>(xk + (4 * mb + g) * 256);
        const float4 y = *reinterpret_cast<const float4*>(xv + (4 * mb + g) * 256);
        dk[mb][4 * g] += x.x; dk[mb][4 * g + 1] += x.y; dk[mb][4 * g + 2] += x.z; dk[mb][4 * g + 3] += x.w;
        dv[mb][4 * g] += y.x; dv[mb][4 * g + 1] += y.y; dv[mb][4 * g + 2] += y.z; dv[mb][4 * g + 3] += y.w;
      }
  }
  if (a.qsplit > 1) return partials_out(krow);
  uint16_t* const area = KB + (paired ? 2 : 1) * kg * KOWN;  // read by this wave alone
  rows_out(a.dk, key0 + kg * 32, dk, a.scale, area);
  rows_out(a.dv, key0 + kg * 32, dv, 1.f, area);
}

// ---- dK = scale * sum of the partials, dV = sum of the partials (qsplit >
// 1): 8 consecutive d values of one (b, key, h) row per thread.
__global__ __launch_bounds__(256) void bwd_reduce_kernel(BwdArgs a) {
  const size_t n = (size_t)a.B * a.Lk * a.H * D;  // elements per gradient
  const size_t groups = n / 8;
  for (size_t g = (size_t)blockIdx.x * 256 + threadIdx.x; g < 2 * groups; g += (size_t)gridDim.x * 256) {
    const bool isk = g < groups;
    const size_t e = (isk ? g : g - groups) * 8;
    const float* src = a.part + (isk ? 0 : (size_t)a.qsplit * n) + e;
    float4 x0 = make_float4(0.f, 0.f, 0.f, 0.f), x1 = x0;
    for (int sp = 0; sp < a.qsplit; ++sp) {
      const float4 u = *reinterpret_cast<const float4*>(src + (size_t)sp * n);
      const float4 v = *reinterpret_cast<const float4*>(src + (size_t)sp * n + 4);
      x0.x += u.x; x0.y += u.y; x0.z += u.z; x0.w += u.w;
      x1.x += v.x; x1.y += v.y; x1.z += v.z; x1.w += v.w;
    }
    const float mul = isk ? a.scale : 1.f;
    uint4 o;
    o.x = pack_bf16x2(x0.x * mul, x0.y * mul);
    o.y = pack_bf16x2(x0.z * mul, x0.w * mul);
    o.z = pack_bf16x2(x1.x * mul, x1.y * mul);
    o.w = pack_bf16x2(x1.z * mul, x1.w * mul);
    *reinterpret_cast<uint4*>((isk ? a.dk : a.dv) + e) = o;
  }
}

}  // namespace

// Compute units of the current device (queried once per device).
int device_cu_count() {
  static std::mutex mu;
  static int counts[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  std::lock_guard<std::mutex> lock(mu);
  if (counts[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    counts[dev] = n;
  }
  return counts[dev];
}

hipError_t launch_attn_bwd(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* o,
                           const uint16_t* dout, const float* lse, float* ws, size_t ws_floats, uint16_t* dq,
                           uint16_t* dk, uint16_t* dv, int B, int H, int Lq, int Lk, float scale,
                           const int32_t* kv_valid_len, hipStream_t stream) {
  BwdArgs a;
  a.q = q; a.k = k; a.v = v; a.o = o; a.dout = dout; a.lse = lse; a.delta = ws;
  a.dq = dq; a.dk = dk; a.dv = dv; a.kv_valid_len = kv_valid_len;
  a.B = B; a.H = H; a.Lq = Lq; a.Lk = Lk;
  a.scale = scale;
  a.c = scale * kLog2e;
  const BwdSplit sp = attn_bwd_split(B, H, Lq, Lk, device_cu_count(), ws_floats, kv_valid_len != nullptr);
  a.qsplit = sp.qsplit;
  a.qper = sp.qper;
  a.part = sp.qsplit > 1 ? ws + sp.part_offset : nullptr;
  a.kper = sp.kper;
  hipError_t e = hipSuccess;
  if (Lq > 0) {
    const bool short_keys = (Lk + BN - 1) / BN <= kDqShortTiles;
    const int nwq = short_keys ? 4 : 8;
    a.ntile = (Lq + 32 * nwq - 1) / (32 * nwq);
    a.nwg = a.ntile * B * H;
    e = short_keys ? launch_kernel(bwd_dq4_kernel, (unsigned)a.nwg, 256u, stream, a)
                   : launch_kernel(bwd_dq8_kernel, (unsigned)a.nwg, 512u, stream, a);
    if (e != hipSuccess) return e;
  }
  if (Lk > 0) {
    a.ntile = (Lk + a.kper - 1) / a.kper;
    a.nwg = a.ntile * B * H * a.qsplit;
    e = launch_kernel(bwd_dkdv_kernel, (unsigned)a.nwg, (unsigned)NT, stream, a);
    if (e != hipSuccess) return e;
    if (a.qsplit > 1) {
      const size_t groups = 2 * (size_t)B * Lk * H * D / 8;
      size_t g = (groups + 255) / 256;
      if (g > 16384) g = 16384;
      e = launch_kernel(bwd_reduce_kernel, (unsigned)g, 256u, stream, a);
    }
  }
  return e;
}

// ---- allocation-free backward ------------------------------------------
//
// D of the allocation-free entry point lives in this fixed array instead of a
// caller workspace: kNoAllocRows fp32 values (16 MiB), one copy per GPU the
// library runs on, held until the process ends.  In host code `scratch` is
// only a stand-in for the symbol; its device address (different on every
// GPU) is looked up once per device and only that address is handed to the
// kernels.  Calls that overlap on one GPU share the array and race; the dq
// kernel writes every value the dkdv kernel then reads, so nothing is
// cleared.
static __device__ __align__(256) float scratch[kNoAllocRows];

constexpr int kMaxDevices = 64;

// Device address of `scratch` on the current device (looked up on the first
// call made with that device current).
static hipError_t scratch_address(float** out) {
  static std::mutex mu;
  static float* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    addr[dev] = static_cast<float*>(ptr);
  }
  *out = addr[dev];
  return hipSuccess;
}

hipError_t launch_attn_bwd_noalloc(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* o,
                                   const uint16_t* dout, const float* lse, uint16_t* dq, uint16_t* dk, uint16_t* dv,
                                   int B, int H, int Lq, int Lk, float scale, const int32_t* kv_valid_len,
                                   hipStream_t stream) {
  if ((long)B * H * Lq > kNoAllocRows) return hipErrorInvalidValue;  // the entry point rejects this first
  float* delta = nullptr;
  const hipError_t e = scratch_address(&delta);
  if (e != hipSuccess) return e;
  // D only (the array holds no room for split partials): unsplit
  return launch_attn_bwd(q, k, v, o, dout, lse, delta, (size_t)B * H * Lq, dq, dk, dv, B, H, Lq, Lk, scale,
                         kv_valid_len, stream);
}

}  // namespace vidax
