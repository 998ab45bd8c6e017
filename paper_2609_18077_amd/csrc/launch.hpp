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
inline hipError_t launch_kernel(void (*kernel)(A), unsigned grid, unsigned block, hipStream_t stream, A arg) {
  void* args[] = {&arg};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3(grid), dim3(block), args, 0, stream);
}

// Work split of the per-token kernels (rotation, norm): workgroups of 16
// tokens.  With at least 1024 of them (4 per compute unit) the workgroups walk
// the tokens and take all B * H rows of a token; with fewer, the rows are cut
// into `parts` of `rows` (multiples of four, the loads in flight) so that about
// 2048 workgroups exist.
constexpr int kTokenGroup = 16;
struct TokenSplit {
  int parts, rows, grid;
};
inline TokenSplit token_split(int B, int L, int H) {
  const int64_t groups = ((int64_t)L + kTokenGroup - 1) / kTokenGroup, rows = (int64_t)B * H;
  TokenSplit s{1, (int)rows, 1024};
  if (groups < 1024) {
    int64_t parts = (2048 + groups - 1) / groups;
    const int64_t most = (rows + 3) / 4;
    if (parts > most) parts = most;
    const int64_t per = (rows + parts * 4 - 1) / (parts * 4) * 4;
    parts = (rows + per - 1) / per;
    s = TokenSplit{(int)parts, (int)per, (int)(groups * parts)};
  }
  return s;
}
hipError_t launch_rope3d(const uint16_t* x, uint16_t* y, int B, int L, int H, const RopeParams& rp,
                         hipStream_t stream);
// Compute units of the current device (queried once per device).
int device_cu_count();

// Query-stream split of the backward's key-side kernel.  Its workgroups own
// kBwdKeys keys of one (b, h), one workgroup per compute unit, and stream
// every query in 64-row tiles; where there are fewer of them than twice the
// compute units and more than 8 query tiles, the tiles may be cut into qsplit
// runs of qper tiles (at least 2 tiles a run, at most 32 runs; up to 8
// tiles, 128-key workgroups without a split were faster by 3 to 22%).  Chosen: the least time in
// units of one tile's (about 3.6 us): rounds x (tiles a run + 2 for a workgroup's
// start and end), and for a split 3 for the extra launch and the bytes of the
// fp32 partials (written and read: 16 bytes a gradient value and run, about
// 14 MB in a tile's time).  The partial dK and dV of the runs follow D in the
// workspace, from a 256-byte aligned offset; `floats` is the workspace size
// this needs (B * H * Lq when qsplit is 1).
constexpr int kBwdKeys = 256;
struct BwdSplit {
  int qsplit, qper;
  size_t part_offset, floats;
};

inline BwdSplit attn_bwd_split(int B, int H, int Lq, int Lk, int cus) {
  constexpr int kRows = 64;
  BwdSplit r;
  const size_t rows = (size_t)B * H * Lq;
  const int qtiles = (Lq + kRows - 1) / kRows;
  const int64_t nkv = (int64_t)((Lk + kBwdKeys - 1) / kBwdKeys) * B * H;
  r.qsplit = 1;
  if (nkv > 0 && nkv < 2 * (int64_t)cus && qtiles > 8) {
    const double part = (double)B * Lk * H * kHeadDim * 16 / 14e6;
    double best = 0;
    for (int s = 1; s <= 32 && (s == 1 || s <= qtiles / 2); ++s) {
      const double rounds = (double)((nkv * s + cus - 1) / cus);
      const double cost = rounds * ((qtiles + s - 1) / s + 2) + (s > 1 ? 3 + s * part : 0);
      if (s == 1 || cost < best) {
        best = cost;
        r.qsplit = s;
      }
    }
  }
  r.qper = (qtiles + r.qsplit - 1) / r.qsplit;
  r.part_offset = (rows + 63) / 64 * 64;
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
