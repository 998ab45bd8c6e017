// Standalone 3D rotary embedding, bf16 [B, L, H, 128] -> bf16 (HBM-bound),
// and its transpose (every pair rotated by minus its angle).
//
// A token's 16 channel chunks (16 B each) are handled by 16 consecutive lanes;
// a lane forms the (cos, sin) of its chunk's channels in registers (no table,
// no barrier) and applies them to the same chunk of the token's rows, one for
// every batch and head, four rows' loads in flight at a time, so every global
// access is a 16-byte, row-contiguous load or store.  Long sequences:
// workgroups walk the tokens with a grid stride and take all rows of a token,
// so the angle work is amortised.  Short ones: the rows of a token are shared
// out over several workgroups (token_split), because the launch is then as long
// as one workgroup's chain of loads and stores.  Few rows a token: a workgroup
// is little more than its start, so its part of the work comes from a
// three-dimensional grid (from one index, with five divisions: 16384 tokens x 4
// heads 7.2 -> 6.4 us).
// Half-split pairs: a channel's partner lies d_a / 2 channels away, usually in
// another lane's chunk, so the row's values pass through an LDS buffer written
// and read by the row's 16 lanes (one wave's: a fence for the compiler, no
// barrier), and a lane forms the angles of its 8 channels instead of 4 pairs
// (an LDS table per workgroup and two barriers a row before: 8200 x 24 heads
// 27.2 -> 19.8 us, 1560 x 12 12.0 -> 6.1; interleaved pairs 18.1 -> 17.5 and
// 5.1 -> 4.7 us).
#include "launch.hpp"

namespace vidax {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kTokensPerPass = kTokenGroup;
static_assert(kTokensPerPass * 16 == kThreads, "16 lanes a token");

struct Rope3dArgs {
  const uint16_t* x;
  uint16_t* y;
  int B, L, H;
  TokenSplit sp;
  RopeParams rp;
};

__device__ __forceinline__ int pos_of_axis(int axis, int t, int h, int w) {
  return axis == 0 ? t : (axis == 1 ? h : w);
}

// HALF: half-split pairs.
template <bool HALF>
__global__ __launch_bounds__(kThreads) void rope3d_kernel(Rope3dArgs a) {
  constexpr int NA = HALF ? 8 : 4;  // angles per lane: its channels or its pairs
  __shared__ __attribute__((aligned(16))) uint16_t rows[HALF ? 4 * kTokensPerPass * kHeadDim : 8];
  const RopeParams& rp = a.rp;
  const int c = threadIdx.x & 15;
  // the workgroup's heads and batches
  const int h0 = blockIdx.x * a.sp.rows, h1 = min(h0 + a.sp.rows, a.H);
  const int b0 = blockIdx.z * a.sp.nb, b1 = min(b0 + a.sp.nb, a.B);
  const size_t tok_stride = (size_t)a.H * kHeadDim;      // elements between tokens
  const size_t batch_stride = (size_t)a.L * tok_stride;  // elements between batches
  // per angle: axis and frequency; half split also: whether the channel is the
  // first of its pair, and its partner
  int axis[NA], part[NA];
  bool lead[NA];
  float omega[NA];
#pragma unroll
  for (int e = 0; e < NA; ++e) {
    int j, da;
    if (HALF) {
      const int ch = 8 * c + e;
      int o;
      if (ch < rp.dt) { o = 0; da = rp.dt; axis[e] = 0; }
      else if (ch < rp.dt + rp.dh) { o = rp.dt; da = rp.dh; axis[e] = 1; }
      else { o = rp.dt + rp.dh; da = rp.dw; axis[e] = 2; }
      const int hl = da >> 1;
      lead[e] = ch - o < hl;
      j = lead[e] ? ch - o : ch - o - hl;
      part[e] = lead[e] ? ch + hl : ch - hl;
    } else {
      const PairSlot slot = pair_slot(rp, 4 * c + e);
      axis[e] = slot.axis;
      j = slot.base - (slot.axis == 0 ? 0 : (slot.axis == 1 ? rp.base1 : rp.base2));
      da = 2 * slot.stride;
    }
    omega[e] = exp2f(-((float)(2 * j) / (float)da) * rp.log2_theta);
  }

  for (int n = blockIdx.y * kTokensPerPass + (threadIdx.x >> 4); n < a.L; n += gridDim.y * kTokensPerPass) {
    const size_t row_n = (size_t)n * tok_stride + c * 8;  // the lane's chunk of the token's first row
    u32x4 v[4];
    // A lane reads and writes only its own chunks, after the
    // loads of its row, so in-place calls stay race free.
    const bool rot = n < rp.n_rot;
    float cs[NA], sn[NA];
    if (rot) {
      const int t = n / (rp.gh * rp.gw);
      const int r = n - t * rp.gh * rp.gw;
      const int h = r / rp.gw;
      const int w = r - h * rp.gw;
#pragma unroll
      for (int e = 0; e < NA; ++e) {
        float sv, cv;
        sincosf((float)pos_of_axis(axis[e], t, h, w) * omega[e], &sv, &cv);
        cs[e] = cv;
        sn[e] = rp.inverse ? -sv : sv;
      }
    }
    // row u of the four: rotate (or copy) its chunk
    auto put = [&](int u, uint16_t* out) __attribute__((always_inline)) {
      if (!rot) {
        if (a.x != a.y) *reinterpret_cast<u32x4*>(out) = v[u];
        return;
      }
      const uint32_t wv[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
      uint32_t o[4];
      if (HALF) {
        uint16_t* const row = rows + (4 * (threadIdx.x >> 4) + u) * kHeadDim;
        *reinterpret_cast<u32x4*>(row + 8 * c) = v[u];
        wave_lds_fence();
        float y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = e & 1 ? bf16hi_to_f32(wv[e >> 1]) : bf16lo_to_f32(wv[e >> 1]);
          const float xp = __uint_as_float((uint32_t)row[part[e]] << 16);
          y[e] = lead[e] ? fmaf(x, cs[e], -xp * sn[e]) : fmaf(xp, sn[e], x * cs[e]);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) o[p] = pack_bf16x2(y[2 * p], y[2 * p + 1]);
        wave_lds_fence();
      } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const float x0 = bf16lo_to_f32(wv[p]);
          const float x1 = bf16hi_to_f32(wv[p]);
          o[p] = pack_bf16x2(fmaf(x0, cs[p], -x1 * sn[p]), fmaf(x0, sn[p], x1 * cs[p]));
        }
      }
      *reinterpret_cast<uint4*>(out) = make_uint4(o[0], o[1], o[2], o[3]);
    };
    // four rows' loads in flight; the heads of a batch, then the next batch's
    int left = (b1 - b0) * (h1 - h0), h = h0;
    size_t row0 = b0 * batch_stride + row_n;
    size_t off[4];
    auto load = [&](int u) __attribute__((always_inline)) {
      off[u] = row0 + (size_t)h * kHeadDim;
      if (++h == h1) {  // uniform
        h = h0;
        row0 += batch_stride;
      }
      v[u] = *reinterpret_cast<const u32x4*>(a.x + off[u]);
    };
    for (; left >= 4; left -= 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) load(u);
#pragma unroll
      for (int u = 0; u < 4; ++u) put(u, a.y + off[u]);
    }
    if (left > 0) {
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (u < left) load(u);
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (u < left) put(u, a.y + off[u]);
    }
  }
}

}  // namespace

hipError_t launch_rope3d(const uint16_t* x, uint16_t* y, int B, int L, int H, const RopeParams& rp,
                         hipStream_t stream) {
  const Rope3dArgs a{x, y, B, L, H, token_split(B, L, H), rp};
  return launch_kernel(rp.pair_mode ? rope3d_kernel<true> : rope3d_kernel<false>, dim3(a.sp.gx, a.sp.gy, a.sp.gz),
                       (unsigned)kThreads, stream, a);
}

}  // namespace vidax
