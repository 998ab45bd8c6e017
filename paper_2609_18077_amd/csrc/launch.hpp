// Launchers of the gfx950 kernels (not part of the C ABI), implemented in the
// .hip files and called by the C ABI layer after validation.  Kept apart
// from the kernels' shared definitions so that a new entry point changes no
// file a kernel is built from.
#pragma once

#include "common.hpp"

// All pointers are device pointers; sizes already validated.
namespace vidax {

// Enqueues kernel(arg) on `stream` and returns the status of this launch
// alone (an error left behind by an earlier, unrelated HIP call is not
// reported as this launch's failure, as hipGetLastError would).
template <typename A>
inline hipError_t launch_kernel(void (*kernel)(A), dim3 grid, unsigned block, hipStream_t stream, A arg) {
  void* args[] = {&arg};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3(block), args, 0, stream);
}

// Work split of the per-token kernels (rotation, norm): workgroups of 16
// tokens, gx x gy x gz of them.  Workgroup (x, y, z) takes heads x * rows ..
// + rows - 1 of batches z * nb .. + nb - 1 for every gy-th group of tokens.
// Every share of a token's rows forms the token's angles anew.  Up to 320 groups
// (about a workgroup per compute unit) the launch is one workgroup's chain over
// its rows, four at a time: shares of four rows as far as 1024 workgroups, or of
// eight as far as 2048, where they halve that chain.  Past that a compute unit
// has another workgroup beside one that waits: equal shares of 12 rows or of 8,
// as far as 2560 workgroups (unequal ones leave units idle: 7800 tokens x 40
// heads 26.5 us unshared, 25.8 in shares of 8, 28.9 in shares of 12, 12, 12 and
// 4).  Half-split norm: 4680 x 12 11.4 us unshared and 10.3 in three shares, but
// 7800 x 12 12.8 and 13.5 in two; 7800 x 24 20.1 and 18.7.
constexpr int kTokenGroup = 16;
struct TokenSplit {
  int rows, nb;
  int gx, gy, gz;
};
inline TokenSplit token_split(int B, int L, int H) {
  const int64_t groups = ((int64_t)L + kTokenGroup - 1) / kTokenGroup;
  TokenSplit s{H, B, 1, (int)(groups < 1024 ? groups : 1024), 1};
  if (groups >= 1024) return s;  // the workgroups walk the tokens
  const int64_t all = (int64_t)B * H;
  auto cut = [&](int gx, int gz) {  // about gx x gz shares, the heads in multiples of four
    TokenSplit c = s;
    c.rows = gx > 1 ? (H + gx * 4 - 1) / (gx * 4) * 4 : H;
    c.nb = (B + gz - 1) / gz;
    c.gx = (H + c.rows - 1) / c.rows;
    c.gz = (B + c.nb - 1) / c.nb;
    return c;
  };
  if (groups > 320) {
    const int gx = H < 24 ? 1 : H % 12 == 0 ? H / 12 : H % 8 == 0 ? H / 8 : 1;
    int nb = 1;  // of every batch, or of as many at a time as the limits ask for
    while (nb < B && (B % nb != 0 || (int64_t)nb * H < 12 || groups * gx * (B / nb) > 2560)) ++nb;
    return groups * gx * (B / nb) <= 2560 ? cut(gx, B / nb) : s;
  }
  const int64_t fours = groups <= 128 ? (all + 3) / 4 : all / 4;  // up to 128: the last one may be smaller
  const int64_t fine = 1024 / groups < fours ? 1024 / groups : fours;
  const int64_t coarse = 2048 / groups < all / 8 ? 2048 / groups : all / 8;
  const int parts = (int)(fine > coarse ? fine : coarse);
  if (parts < 2) return s;
  const TokenSplit c = parts > B ? cut((groups <= 128 ? parts + B - 1 : parts) / B, B) : cut(1, parts);
  auto chain = [](const TokenSplit& t) { return ((int64_t)t.rows * t.nb + 3) / 4; };
  return 2 * chain(c) <= chain(s) ? c : s;
}
hipError_t launch_rope3d(const uint16_t* x, uint16_t* y, int B, int L, int H, const RopeParams& rp,
                         hipStream_t stream);
// Compute units of the current device (queried once per device).
int device_cu_count();

// Shape of the backward's key-side launch: workgroups of kper = kBwdKeys keys
// of one (b, h), or of half as many (two waves a 32-key group), one workgroup
// per compute unit, that stream the queries in 64-row tiles; with full
// workgroups the tiles may be cut into qsplit runs of qper tiles (at least 2
// tiles a run, at most 32 runs), whose fp32 partial dK and dV a further launch
// adds up.  Chosen is the least time in units of one tile's:
//   unsplit   rounds x (tiles + 2.6), half workgroups rounds x (0.55 tiles +
//             2.8), fitted to 150 shapes of 64 to 500 queries x 256 to 640 keys
//             x 70 to 400 heads.  300 x 300: 130 heads, 2 rounds of either,
//             61.8 (full) and 53.6 us; 200 heads, 2 and 3 rounds, 73.0 and
//             75.8.  Where batches have lengths of their own, half workgroups
//             only if that takes no more rounds: the full ones past a batch's
//             end cost nothing (2 x 12 heads x 3000, lengths 1000 and 3000:
//             2 and 3 rounds, 285 and 303 us);
//   runs      rounds x (tiles a run + 2) + 3 for the extra launch + the bytes
//             of the partials, written and read: 16 bytes a gradient value and
//             run, 14 MB in a tile's time.
// Runs are considered where full workgroups number less than twice the compute
// units and there are more than 8 query tiles (up to 8, unsplit was faster by
// 3 to 22 %), as far as the partials stay within kBwdPartFloats and the whole
// within max_floats.  The line is 384 MiB because larger partials won nothing:
// 3 heads x 39167 took five runs and 601 MB for 6569 us, against 6508 unsplit;
// 2 x 2 heads x 28000 four runs and 459 MB for 4431, against 4381.  Half of it
// was slower: 3 heads x 23058, two runs and 142 MB 3037 us, five runs and 354
// MB 2901.  The partials follow D in the workspace, from a
// 256-byte aligned offset; `floats` is the workspace the choice needs (B * H * Lq
// when qsplit is 1).
constexpr int kBwdKeys = 256;
constexpr size_t kBwdPartFloats = (size_t)96 << 20;
struct BwdSplit {
  int kper, qsplit, qper;
  size_t part_offset, floats;
};

inline BwdSplit attn_bwd_split(int B, int H, int Lq, int Lk, int cus, size_t max_floats, bool lengths) {
  constexpr int kRows = 64;
  BwdSplit r;
  const size_t rows = (size_t)B * H * Lq;
  const int qtiles = (Lq + kRows - 1) / kRows;
  auto workgroups = [&](int keys) { return (int64_t)((Lk + keys - 1) / keys) * B * H; };
  auto rounds = [&](int64_t wgs) { return (wgs + cus - 1) / cus; };
  const int64_t nkv = workgroups(kBwdKeys), r_full = rounds(nkv), r_half = rounds(workgroups(kBwdKeys / 2));
  const double full = r_full * (qtiles + 2.6), half = r_half * (0.55 * qtiles + 2.8);
  r.kper = half < full && (!lengths || r_half <= r_full) ? kBwdKeys / 2 : kBwdKeys;
  r.qsplit = 1;
  r.part_offset = (rows + 63) / 64 * 64;
  if (nkv > 0 && nkv < 2 * (int64_t)cus && qtiles > 8) {
    const size_t run = 2 * (size_t)B * Lk * H * kHeadDim;  // partial values of a run
    double best = half < full ? half : full;
    for (int s = 2; s <= 32 && s <= qtiles / 2; ++s) {
      if (s * run > kBwdPartFloats || r.part_offset + s * run > max_floats) break;
      const double cost = rounds(nkv * s) * ((qtiles + s - 1) / s + 2) + 3 + s * (run * 8 / 14e6);
      if (cost < best) {
        best = cost;
        r.kper = kBwdKeys;
        r.qsplit = s;
      }
    }
  }
  r.qper = (qtiles + r.qsplit - 1) / r.qsplit;
  r.floats = r.qsplit > 1 ? r.part_offset + 2 * (size_t)r.qsplit * B * Lk * H * kHeadDim : rows;
  return r;
}
// ws: D in its first B * H * Lq values; the split needs ws_floats >=
// attn_bwd_workspace_floats(...), fewer run unsplit.
hipError_t launch_attn_bwd(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* o,
                           const uint16_t* dout, const float* lse, float* ws, size_t ws_floats, uint16_t* dq,
                           uint16_t* dk, uint16_t* dv, int B, int H, int Lq, int Lk, float scale,
                           const int32_t* kv_valid_len, hipStream_t stream);
// The backward with D in the library's fixed device array (allocation-free
// entry point); B * H * Lq must not exceed kNoAllocRows.
constexpr long kNoAllocRows = 4194304;
hipError_t launch_attn_bwd_noalloc(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* o,
                                   const uint16_t* dout, const float* lse, uint16_t* dq, uint16_t* dk, uint16_t* dv,
                                   int B, int H, int Lq, int Lk, float scale, const int32_t* kv_valid_len,
                                   hipStream_t stream);
hipError_t launch_qk_norm(const uint16_t* x, uint16_t* y, const float* gain, float eps, int B, int L, int H,
                          const RopeParams& rp, hipStream_t stream);
hipError_t launch_attn_naive(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* o,
                             float* lse, int B, int H, int Lq, int Lk, float scale,
                             const int32_t* kv_valid_len, const RopeParams& rp, hipStream_t stream);
bool attn_rope_supported(const RopeParams& rp);
hipError_t launch_na3d_fwd(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* o, float* lse, int B,
                           int H, int T, int Hp, int Wp, int kt, int kh, int kw, int shift, float scale,
                           hipStream_t stream);
hipError_t launch_attn_fwd(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* o,
                           float* lse, int B, int H, int Lq, int Lk, float scale,
                           const int32_t* kv_valid_len, const RopeParams& rp, hipStream_t stream);
// Short unrotated key sequences (text cross-attention): one persistent
// workgroup per CU (`cus` compute units).
hipError_t launch_xattn_fwd(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* o, float* lse,
                            int B, int H, int Lq, int Lk, float scale, const int32_t* kv_valid_len, int cus,
                            hipStream_t stream);
hipError_t launch_qkv_proj(const uint16_t* x, const uint16_t* w, const float* bias, const float* gain_q,
                           const float* gain_k, float eps, uint16_t* q, uint16_t* k, uint16_t* v, int B, int L, int H,
                           int C, const RopeParams& rp, hipStream_t stream);
}  // namespace vidax
