// Forward kernel of 3D Deformable Slide Attention (MegaSlide-DiT, Section 5.2, Eq. (1)).
//
// A query's P points have 8 P corner rows of K and of V, and the rate at which a compute unit takes
// row requests bounds a kernel that loads them all.  A wave goes one of two ways, by the spread
// of its points (compact_wave):
//  * slots_tile: four neighbouring queries of a wave read each distinct voxel of their points
//    once (dsa3d_slots.h), logits first, then one softmax, then the weighted sum of V;
//  * gather_tile: an L-lane group owns one query row, loads the 8 K and 8 V rows of each point
//    (16-byte buffer loads, zeros outside the grid) and folds the point into an online softmax.
// Measured, gather against slots where the points are compact (U[-8, 8] offsets always gather):
// 64x68x120, 24 heads x 128, 3x3x3, offsets N(0, 1): 48.2 -> 24.7 ms; 16x34x60, 24 x 128, 3x7x7:
// 14.1 -> 6.7 ms; 64x34x60, 16 x 64, 3x3x3, U[-2, 2]: 4.07 -> 3.87 ms; 2 x 9x33x47, 6 x 64 fp32:
// 0.55 -> 0.40 ms.  Nothing per point is written to memory; the output row and its LSE are stored
// once.
//
// Memory order: tiles are handed out in pencils (tile_order.h): each XCD walks one pencil of
// about 12 x 12 tokens of a (batch, head) frame by frame, so the K/V rows its in-flight
// queries reach stay in its L2.
#include "dsa3d_slots.h"

namespace dsa3d {
namespace {

using namespace dev;

// Per-point coordinate work shared across the L lanes of a row: in each chunk of L points,
// lane `sub` of a row computes point chunk + sub once and leaves its corner indices, weights
// and cell in its LDS slot (80 bytes), and the row's lanes read each point from there (one
// broadcast read per 16 bytes) instead of every lane repeating the same arithmetic.  Against
// fetching them from the owner's registers with ds_bpermute this keeps 14 fewer registers
// live in the point loop (138) and measured 1% faster; four waves per SIMD (128 registers,
// a few spilled outside the loop) did not pay.
//
// PW (the predicted-weights variant): the logit of a point is given (`logits`, one fp32 per
// (row, point)) instead of scale <q, k_p>, so neither q nor the K corners are read.
template <int D, bool BF16, bool PW, bool SLOTS>
__device__ inline __attribute__((always_inline)) void gather_tile(
    const Geometry& g, const PencilOrder& po, const PencilTile& tl, const void* __restrict__ q,
    const void* __restrict__ k, const void* __restrict__ v, const float* __restrict__ logits,
    const float* __restrict__ offsets, void* __restrict__ out, float* __restrict__ lse, int4* pts) {
  using LY = Layout<D, BF16>;
  constexpr int L = LY::kLanes;
  constexpr int VEC = LY::kVec;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane / L, sub = lane % L;
  const int lane_off = sub * 16;
  const char* qb = static_cast<const char*>(q);
  const char* kb = static_cast<const char*>(k);
  const char* vb = static_cast<const char*>(v);
  const int HW = g.H * g.W;
  const int rt = (g.kt - 1) / 2, rh = (g.kh - 1) / 2, rw = (g.kw - 1) / 2;
  const int khw = g.kh * g.kw;
  // The point each lane formed for the current chunk, read back by its row's lanes: corner
  // indices, weights, and for the global-load path its window flag and cell.  A row's lanes
  // are in one wave, whose LDS accesses complete in order: no barrier.
  int4* const mine_at = pts + slot_of<L, 5>(lane);

  const int b = tl.group / g.by_heads, m = tl.group - b * g.heads;
  const int t = tl.frame;
  const RowWindow win = make_window<LY::kRowBytes>(g, k, v, b, m, t);
  int i, j;
  const bool active = query_token<SLOTS, LY::kGroups>(po, g, tl, wave, grp, i, j);
  if (!active) {  // an idle row computes on a valid token and stores nothing
    i = min(i, g.H - 1);
    j = min(j, g.W - 1);
  }
  const int n = t * HW + i * g.W + j;
  const int64_t row = ((int64_t)b * g.N + n) * g.heads + m;

  uint4 qr = make_uint4(0u, 0u, 0u, 0u);
  if constexpr (!PW) qr = load16(qb, row * LY::kRowBytes + lane_off);
  const float* off = offsets + row * g.P * 3;
  float o[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) o[e] = 0.0f;
  float mx = -INFINITY, l = 0.0f;

  for (int p0 = 0; p0 < g.P; p0 += L) {
    // this lane's point of the chunk
    const int pm = min(p0 + sub, g.P - 1);
    const int it = pm / g.by_khw, rp = pm - it * khw, ih = rp / g.by_kw, iw = rp - ih * g.kw;
    {
      Point mine;
      make_point(g, win, t, i, j, it - rt, ih - rh, iw - rw, off[3 * pm], off[3 * pm + 1],
                 off[3 * pm + 2], mine);
      mine_at[0] = make_int4(mine.vidx[0], mine.vidx[1], mine.vidx[2], mine.vidx[3]);
      mine_at[1] = make_int4(mine.vidx[4], mine.vidx[5], mine.vidx[6], mine.vidx[7]);
      mine_at[2] = make_int4(__float_as_int(mine.w[0]), __float_as_int(mine.w[1]),
                             __float_as_int(mine.w[2]), __float_as_int(mine.w[3]));
      mine_at[3] = make_int4(__float_as_int(mine.w[4]), __float_as_int(mine.w[5]),
                             __float_as_int(mine.w[6]), __float_as_int(mine.w[7]));
      mine_at[4] = make_int4((int)mine.slow, mine.cx, mine.cy, mine.cz);
    }
    float mylog2 = 0.0f;  // PW: this lane's point's logit, base 2
    if constexpr (PW) mylog2 = logits[row * g.P + pm] * kLog2e;
    const int nk = min(L, g.P - p0);
    for (int kk = 0; kk < nk; ++kk) {
      const int src = (grp * L + kk) << 2;
      const int4* at = pts + slot_of<L, 5>(grp * L) + kk * 5;
      const int4 i0 = at[0], i1 = at[1], w0 = at[2], w1 = at[3];
      Point pt;
      pt.vidx[0] = i0.x; pt.vidx[1] = i0.y; pt.vidx[2] = i0.z; pt.vidx[3] = i0.w;
      pt.vidx[4] = i1.x; pt.vidx[5] = i1.y; pt.vidx[6] = i1.z; pt.vidx[7] = i1.w;
      pt.w[0] = __int_as_float(w0.x); pt.w[1] = __int_as_float(w0.y);
      pt.w[2] = __int_as_float(w0.z); pt.w[3] = __int_as_float(w0.w);
      pt.w[4] = __int_as_float(w1.x); pt.w[5] = __int_as_float(w1.y);
      pt.w[6] = __int_as_float(w1.z); pt.w[7] = __int_as_float(w1.w);
      uint4 vr[8];
      float s2;
      if constexpr (PW) {
        load_stashed_corners<LY::kRowBytes, false>(g, win, kb, vb, b, m, lane_off, at + 4,
                                                   pt.vidx, nullptr, vr);
        s2 = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(mylog2)));
      } else {
        uint4 kr[8];
        load_stashed_corners<LY::kRowBytes, true>(g, win, kb, vb, b, m, lane_off, at + 4,
                                                  pt.vidx, kr, vr);
        float sp = 0.0f;
#pragma unroll
        for (int c = 0; c < 8; ++c) sp = fmaf(pt.w[c], chunk_dot<BF16>(qr, kr[c]), sp);
        s2 = group_sum<L>(sp) * g.scale_log2;
      }
      // One exponential per point: a new maximum rescales the running sums by
      // 2^(old max - new max) and enters with weight exactly 1; otherwise the point enters
      // with 2^(s - max).  (A first finite logit takes the first branch: 2^-inf = 0.)  A
      // given logit of -inf enters with weight 0 even while the maximum is still -inf,
      // where s - max would be NaN.
      const bool up = s2 > mx;
      float ex = exp2f(up ? mx - s2 : s2 - mx);
      if constexpr (PW) ex = s2 == -INFINITY ? 0.0f : ex;
      const float corr = up ? ex : 1.0f;
      const float e = up ? 1.0f : ex;
      l = fmaf(l, corr, e);
      mx = up ? s2 : mx;
#pragma unroll
      for (int x = 0; x < VEC; ++x) o[x] *= corr;
#pragma unroll
      for (int c = 0; c < 8; ++c) chunk_axpy<BF16>(o, e * pt.w[c], vr[c]);
    }
  }
  if (active) {
    const float inv = 1.0f / l;
    char* ob = static_cast<char*>(out) + row * LY::kRowBytes + lane_off;
    if constexpr (BF16) {
      uint4 wv;
      wv.x = bf16_bits(o[0] * inv) | (bf16_bits(o[1] * inv) << 16);
      wv.y = bf16_bits(o[2] * inv) | (bf16_bits(o[3] * inv) << 16);
      wv.z = bf16_bits(o[4] * inv) | (bf16_bits(o[5] * inv) << 16);
      wv.w = bf16_bits(o[6] * inv) | (bf16_bits(o[7] * inv) << 16);
      *reinterpret_cast<uint4*>(ob) = wv;
    } else {
      *reinterpret_cast<float4*>(ob) = make_float4(o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
    }
    if (lse != nullptr && sub == 0) lse[row] = (mx + log2f(l)) * kLn2;
  }
}

// The same for waves whose points lie close together, reading each voxel of four neighbouring
// queries once (dsa3d_slots.h).  A chunk of points (all of them up to 32, or 80) has its logits
// complete before its softmax, so one maximum is taken per chunk and only rows of several chunks
// rescale.
template <int D, bool BF16, bool PW, int R, bool WHOLE>
__device__ inline __attribute__((always_inline)) void slots_tile(
    const Geometry& g, const PencilOrder& po, const PencilTile& tl, const void* __restrict__ q,
    const void* __restrict__ k, const void* __restrict__ v, const float* __restrict__ logits,
    const float* __restrict__ offsets, void* __restrict__ out, float* __restrict__ lse,
    SlotLds& lds) {
  using LY = Layout<D, BF16>;
  using U = SlotSum<D, BF16>;
  constexpr int L = kSlotLanes;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qi = lane / L, lp = lane % L;
  float* const val = lds.val[qi];
  const int HW = g.H * g.W;

  for (int e0 = kSlotQueries * wave; e0 < tile_tokens(po);
       e0 += kWavesPerBlock * kSlotQueries) {
    int i, j;
    const bool active = slot_token(po, g, tl, e0 + qi, i, j);
    if (__builtin_amdgcn_ballot_w64(active) == 0) continue;
    i = min(i, g.H - 1);  // an idle query computes on a valid token and stores nothing
    j = min(j, g.W - 1);
    const int b = tl.group / g.by_heads, m = tl.group - b * g.heads;
    const int t = tl.frame;
    const SlotWindow win = slot_window<LY::kRowBytes>(g, b, m, t);
    const int64_t row = ((int64_t)b * g.N + (t * HW + i * g.W + j)) * g.heads + m;
    const float* off = offsets + row * g.P * 3;
    int64_t qrow[kSlotQueries];
#pragma unroll
    for (int w = 0; w < kSlotQueries; ++w)
      qrow[w] = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(row >> 32), w * L)
                           << 32) |
                          (uint32_t)__builtin_amdgcn_readlane((int)row, w * L));
    float mx = -INFINITY, l = 0.0f;  // of this lane's query
    float o[U::kVec];                // of this lane's query, channels kVec (lane % kLanes) ..
#pragma unroll
    for (int x = 0; x < U::kVec; ++x) o[x] = 0.0f;

    for (int c0 = 0; c0 < g.P;) {
      // equal chunks, as few as the rounds allow
      const int left = g.P - c0, chunks = (left + R * L - 1) / (R * L);
      int npts = (left + chunks - 1) / chunks;
      SlotPoint pt[R];
      float s[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        s[r] = -INFINITY;
        if (r * L >= npts) break;
        const int p = c0 + min(r * L + lp, npts - 1);
        pt[r].set(g, t, i, j, p, off + 3 * p);
        if constexpr (PW) s[r] = logits[row * g.P + p] * kLog2e;
      }
      bool global;
      int n;
      npts = number_slots<R, WHOLE>(g, win, (uint32_t)g.heads * LY::kRowBytes, lds, pt, npts, n, global);
      if constexpr (!PW) {
        const SlotRows rows = slot_rows<LY::kRowBytes>(g, k, win, b, m, global);
        auto combine = [&] {
          bool nan = false;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            if (r * L >= npts) break;
            float w[8], d[8];
            pt[r].weights(w);
            pt[r].read(val, d);
            s[r] = 0.0f;
#pragma unroll
            for (int c = 0; c < 8; ++c) s[r] = fmaf(w[c], d[c], s[r]);
            nan = nan || s[r] != s[r];
            s[r] *= g.scale_log2;
          }
          return nan;
        };
        row_dots<D, BF16>(rows, lds, q, qrow, n);
        if (dots_again<BF16>(combine())) {
          row_dots<D, BF16, true>(rows, lds, q, qrow, n);
          combine();
        }
      }
      float mc = mx;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r * L >= npts) break;
        if (r * L + lp >= npts) s[r] = -INFINITY;
        mc = fmaxf(mc, s[r]);
      }
      mc = lane_maxf<L>(mc);
      const float corr = mx == mc ? 1.0f : exp2f(mx - mc);  // the first chunk: 0 (or of zeros)
      mx = mc;
      float lc = 0.0f;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r * L >= npts) break;
        // a logit of -inf has weight 0 also while the maximum is -inf, where s - max is NaN; the
        // maximum has weight 1 also where it is +inf
        const float e = s[r] == -INFINITY ? 0.0f : s[r] == mx ? 1.0f : exp2f(s[r] - mx);
        s[r] = r * L + lp < npts ? e : 0.0f;
        lc += s[r];
      }
      lc = group_sum<L>(lc);
      l = fmaf(l, corr, lc);
      sum_coefs<R, BF16>(lds, pt, s, npts, n);
      float sum[U::kVec];
      row_sums<D, BF16>(slot_rows<LY::kRowBytes>(g, v, win, b, m, global), lds, n, sum);
#pragma unroll
      for (int x = 0; x < U::kVec; ++x) o[x] = fmaf(o[x], corr, sum[x]);
      c0 += npts;
    }
    if (!active) continue;
    const float inv = 1.0f / l;
    if (lp < U::kLanes) {
      char* ob = static_cast<char*>(out) + row * LY::kRowBytes + 16 * lp;
      if constexpr (BF16) {
        uint4 wv;
        wv.x = bf16_bits(o[0] * inv) | (bf16_bits(o[1] * inv) << 16);
        wv.y = bf16_bits(o[2] * inv) | (bf16_bits(o[3] * inv) << 16);
        wv.z = bf16_bits(o[4] * inv) | (bf16_bits(o[5] * inv) << 16);
        wv.w = bf16_bits(o[6] * inv) | (bf16_bits(o[7] * inv) << 16);
        *reinterpret_cast<uint4*>(ob) = wv;
      } else {
        *reinterpret_cast<float4*>(ob) =
            make_float4(o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
      }
    }
    if (lse != nullptr && lp == 0) lse[row] = (mx + log2f(l)) * kLn2;
  }
}

// A wave goes one way or the other by the spread of its points (R = 0: every one gathers).  Three
// waves per SIMD either way, and the same LDS.
template <int D, bool BF16, bool PW, int R, bool WHOLE>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(R > 0 ? 3 : 1))) void
fwd_kernel(Geometry g, const void* __restrict__ q, const void* __restrict__ k,
           const void* __restrict__ v, const float* __restrict__ logits,
           const float* __restrict__ offsets, void* __restrict__ out, float* __restrict__ lse,
           PencilOrder po, int64_t vt0) {
  constexpr size_t kLds = wave_lds<Layout<D, BF16>::kLanes, 5, (R > 0)>();
  __shared__ __attribute__((aligned(16))) char block_lds[kWavesPerBlock * kLds];
  char* const lds = block_lds + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * kLds;
  PencilTile tl;
  if (!pencil_tile(po, vt0 + blockIdx.x, tl)) return;  // no pencil left on this XCD
  if constexpr (R > 0) {
    if (compact_wave<(R > 2 ? 4 : 2)>(g, po, tl, offsets, forward_box(D, BF16, g.P))) {
      slots_tile<D, BF16, PW, R, WHOLE>(g, po, tl, q, k, v, logits, offsets, out, lse,
                                        *reinterpret_cast<SlotLds*>(lds));
      return;
    }
  }
  gather_tile<D, BF16, PW, (R > 0)>(g, po, tl, q, k, v, logits, offsets, out, lse,
                                    reinterpret_cast<int4*>(lds));
}

// ---------------------------------------------------------------------------- launch

template <int D, bool BF16>
hipError_t fwd_dispatch(const Geometry& g, const void* q, const void* k, const void* v,
                        const float* logits, const float* off, void* out, float* lse,
                        hipStream_t s) {
  const bool pw = logits != nullptr;
#define DSA3D_FWD(PW, R, WHOLE) \
  reinterpret_cast<const void*>(&fwd_kernel<D, BF16, PW, R, WHOLE>)
#define DSA3D_FWD_OF(R, WHOLE) (pw ? DSA3D_FWD(true, R, WHOLE) : DSA3D_FWD(false, R, WHOLE))
  const int rounds = forward_rounds(D, BF16, (int64_t)g.B * g.N * g.heads, g.P, pw);
  const PencilOrder po = query_order<D, BF16>(g, rounds > 0, true);
  const bool whole = g.win_frames == g.T;
  const void* kern = DSA3D_FWD_OF(0, false);
  if constexpr (slot_rows_ok(D, BF16)) {
    if (rounds == 2) {
      if constexpr (pw_two_rounds_ok(D, BF16))
        kern = whole ? DSA3D_FWD_OF(2, true) : DSA3D_FWD_OF(2, false);
      else
        kern = whole ? DSA3D_FWD(false, 2, true) : DSA3D_FWD(false, 2, false);
    }
    if (rounds == 5) kern = whole ? DSA3D_FWD_OF(5, true) : DSA3D_FWD_OF(5, false);
  }
#undef DSA3D_FWD_OF
#undef DSA3D_FWD
  return launch_tiles(po.vtiles, [&](int64_t vt0, int blocks) {
    void* args[] = {(void*)&g,   (void*)&q,   (void*)&k,   (void*)&v,  (void*)&logits,
                    (void*)&off, (void*)&out, (void*)&lse, (void*)&po, (void*)&vt0};
    return hipLaunchKernel(kern, dim3(blocks), dim3(kBlockThreads), args, 0, s);
  });
}

}  // namespace

hipError_t launch_forward(const Geometry& g, bool bf16, const void* q, const void* k,
                          const void* v, const float* logits, const float* offsets, void* out,
                          float* lse, hipStream_t stream) {
#define DSA3D_FWD(DIM, BF) fwd_dispatch<DIM, BF>(g, q, k, v, logits, offsets, out, lse, stream)
  switch (g.D) {
    case 32: return bf16 ? DSA3D_FWD(32, true) : DSA3D_FWD(32, false);
    case 64: return bf16 ? DSA3D_FWD(64, true) : DSA3D_FWD(64, false);
    case 128: return bf16 ? DSA3D_FWD(128, true) : DSA3D_FWD(128, false);
    default: return hipErrorInvalidValue;
  }
#undef DSA3D_FWD
}

}  // namespace dsa3d
