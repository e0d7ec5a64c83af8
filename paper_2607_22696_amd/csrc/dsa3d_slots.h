// Distinct-voxel slots: how the query-owned kernels read a corner row once for four queries.
//
// The P sampling points of a query have 8 P trilinear corners, but its points share most of their
// voxels, and so do neighbouring queries: with offsets of about one token the 4 x 216 corners of
// four neighbours under a 3x3x3 kernel are 267 distinct voxels, and the 4 x 1176 of a 3x7x7 kernel
// 792.  What bounds a kernel that loads every corner is the rate at which a compute unit takes
// row requests, so here a wave first gives every distinct voxel of its four queries a slot and
// then sweeps the slots: a sweep forms each slot row's dot product with the four queries' vectors
// (row_dots), the points combine their eight values from LDS, and a sweep for weighted sums
// (row_sums) reads each row once with each query's summed coefficient of all corners on it.
//
// A wave holds four neighbours along x, 16 lanes each, one point per lane and round.  Slots come
// from a bitmap of the wave's box of voxels (32 along x in a word, 16 x 16 words): every point sets
// the two bits of its four corner pairs, a scan over the words' bit counts numbers the set bits,
// and the slot of a pair's lower x corner is the number of bits below it (its upper corner has the
// next slot).  Points that leave the box, or need more slots than there are, are taken a round at
// a time with slot = 8 lane + corner and the same sweeps: always correct, but slow, so waves
// whose points spread far are left to the code that loads every corner (compact_wave).
//
// The sweeps use the matrix cores for bf16 rows:
//  * row_dots: lane l reads 16 bytes of the row of slot l / 4, so that four neighbouring lanes
//    read 64 contiguous bytes (with the 16 slots on neighbouring lanes a load takes four times
//    as long).  As the A of v_mfma_f32_16x16x32_bf16 that lane is row l % 16 = 4 (slot % 4) +
//    chunk and K group slot / 4; column n = 4 a + c of B holds the vector's chunk c in K group a
//    and zeros elsewhere, so result (4 s + c, 4 a + c) is what chunk c of slot 4 a + s adds.
//    An infinity or a NaN meets the zeros of the other groups, so a wave that sees a NaN takes
//    its products again on the vector ALU, row by row.
//  * row_sums: the slots are the products' K.  A row is read whole by D / 8 lanes; after eight
//    loads a lane holds 8 channels of 8 slots, and byte permutes pair them into the B operand of
//    one product per channel.  A holds the slots' fp32 coefficients as three bf16 parts (8 bits
//    each, exact), one part of one query per row, so that one product takes them all.
// fp32 rows take the vector ALU: products and sums in fp32.
//
// Coefficients are summed per slot and query in LDS as 32-bit integers with a block exponent: a
// first round of integer maxima finds the largest magnitude that a corner adds to the slot, and
// the corners are then added at 2^-25 (up to 32 points; 2^-23 up to 80) of its power of two.  The
// sum cannot overflow, since a point adds to a slot once, and what is rounded off a corner is at
// most the rounding of an fp32 sum of that slot, however small the slot's coefficients are beside
// the query's others.  (An LDS float add takes 194 cycles of a compute unit per instruction and
// an integer add 11, with addresses as they come here.  One scale per query, without the maxima,
// takes 23.2 instead of 24.6 ms at 64x68x120, 24 heads x 128, 3x3x3, and 199 instead of 230 us at
// 16x32x32, 8 x 64, but a coefficient then keeps only the bits above 2^-31 of the query's sum.)
#pragma once

#include "dsa3d_device.h"
#include "slot_rules.h"

namespace dsa3d {
namespace dev {

typedef __bf16 slot_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float slot_f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kSlotBoxX = 32, kSlotBoxY = 16, kSlotBoxZ = 16;
constexpr int kSlotWords = kSlotBoxY * kSlotBoxZ;  // four per lane
static_assert(kSlotWords == 256, "four words per lane");

// Up to R rounds of points are numbered together, in 640 slots (a round of 64 lanes on its own
// needs 512): LDS holds three workgroups on a compute unit, as many as the registers allow.
constexpr int kSlotCap = 640;

// A wave's slots: the voxel of each, and per query its dot product or coefficient.  The bitmap
// (bits and the number of slots before a word) is needed only until the slots are numbered.
struct SlotLds {
  __attribute__((aligned(16))) uint32_t list[kSlotCap];
  union {
    __attribute__((aligned(16))) uint2 words[kSlotWords];
    // 16 words of padding: the four queries' values of a slot lie on different banks
    __attribute__((aligned(16))) float val[kSlotQueries][kSlotCap + 16];
  };
};

// Lanes of one wave exchange data through LDS, whose accesses a wave makes in order: only the
// compiler has to keep them so.
__device__ inline __attribute__((always_inline)) void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lane, as a value that the compiler takes for another one at each call: what depends on the
// lane is then formed where it is used and not kept in registers around the loops over tokens and
// chunks (at head_dim 64 those values cost the backward 60 spilled registers).
__device__ inline __attribute__((always_inline)) int lane_id() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  __builtin_assume(l >= 0 && l < 64);
  return l;
}

// ---------------------------------------------------------------------------- lane reductions

template <int CTRL>
__device__ inline __attribute__((always_inline)) int dpp_movi(int x) {
  return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
}

// op over the N (16 or 64) lanes of a query or of the wave; every lane gets the result.
template <int N, class Op>
__device__ inline __attribute__((always_inline)) int lane_reduce(int x, Op op) {
  x = op(x, dpp_movi<0xB1>(x));   // lane ^ 1
  x = op(x, dpp_movi<0x4E>(x));   // lane ^ 2
  x = op(x, dpp_movi<0x141>(x));  // the other quad of 8
  x = op(x, dpp_movi<0x140>(x));  // the other half of 16
  if constexpr (N == 64) {
    const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
    x = op((int)r[0], (int)r[1]);
    const auto s = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
    x = op((int)s[0], (int)s[1]);
  }
  return x;
}
template <int N>
__device__ inline __attribute__((always_inline)) int lane_min(int x) {
  return lane_reduce<N>(x, [](int a, int b) { return a < b ? a : b; });
}
template <int N>
__device__ inline __attribute__((always_inline)) float lane_maxf(float x) {
  return __int_as_float(lane_reduce<N>(__float_as_int(x), [](int a, int b) {
    return __float_as_int(fmaxf(__int_as_float(a), __int_as_float(b)));
  }));
}
// Inclusive scan over the wave.
__device__ inline __attribute__((always_inline)) uint32_t lane_scan(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
  return (uint32_t)x;
}

// ---------------------------------------------------------------------------- tiles

// Tokens of a tile.
DSA3D_TILE_FN int tile_tokens(const PencilOrder& o) { return o.run * o.cell; }

// Token e of a tile (four neighbours to a wave of the slots): of a cell of four tokens along x, or
// in raster order of the pencil's rectangle.  False if it is past the pencil or the grid.
__device__ inline __attribute__((always_inline)) bool slot_token(const PencilOrder& po,
                                                                 const Geometry& g,
                                                                 const PencilTile& tl, int e,
                                                                 int& i, int& j) {
  if (po.cell == 1) return pencil_cell(po, tl, e, i, j);
  int cell;
  const bool in = pencil_cell(po, tl, e / kSlotQueries, i, cell);
  j = cell * kSlotQueries + e % kSlotQueries;
  return in && j < g.W;
}

// ---------------------------------------------------------------------------- rows

// Byte offset of a voxel outside the grid: beyond every buffer (a window ends below it), and
// adding a row's bytes to it does not wrap.
constexpr uint32_t kNoVoxel = 0xfffff000u;

struct SlotWindow {
  int t0, frames;  // window [t0, t0 + frames); frames == 0: no window
  int64_t base;    // byte offset of head m's row of its first token
  uint32_t bytes;  // from there to the end of the window
};

template <int ROW_BYTES>
__device__ inline __attribute__((always_inline)) SlotWindow slot_window(const Geometry& g, int b,
                                                                       int m, int t) {
  SlotWindow w;
  w.frames = g.win_frames;
  w.t0 = w.frames > 0 ? min(max(t - (w.frames - 1) / 2, 0), g.T - w.frames) : 0;
  w.base = (((int64_t)b * g.T + w.t0) * g.H * g.W * g.heads + m) * ROW_BYTES;
  const uint64_t span = (uint64_t)w.frames * g.H * g.W * g.heads * ROW_BYTES;
  w.bytes = w.frames > 0 ? (uint32_t)(span - (uint32_t)m * ROW_BYTES) : 0u;
  return w;
}

// Rows of one (batch item, head): a raw buffer over the window of frames around the tile when
// every corner of the wave lies in it (an entry is the byte offset of the voxel's row), else the
// batch item's tokens through global loads (an entry is the token).
struct SlotRows {
  __amdgpu_buffer_rsrc_t rsrc;
  const char* base;  // head m's row of the batch item's first token
  uint32_t tok_bytes;
  bool global;       // wave-uniform
};

template <int ROW_BYTES>
__device__ inline __attribute__((always_inline)) SlotRows slot_rows(const Geometry& g,
                                                                    const void* x,
                                                                    const SlotWindow& w, int b,
                                                                    int m, bool global) {
  SlotRows r;
  r.rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(static_cast<const char*>(x) + w.base),
                                             (short)0, (int)w.bytes, kBufferFlags);
  r.base = static_cast<const char*>(x) + ((int64_t)b * g.N * g.heads + m) * ROW_BYTES;
  r.tok_bytes = (uint32_t)g.heads * ROW_BYTES;
  r.global = global;
  return r;
}

// 16 bytes at `off` of the row of list entry e (zeros for a voxel outside the grid).
template <bool GLOBAL>
__device__ inline __attribute__((always_inline)) uint4 slot_load(const SlotRows& r, uint32_t e,
                                                                 uint32_t off) {
  if constexpr (GLOBAL) {
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (e != kNoVoxel)
      x = *reinterpret_cast<const uint4*>(r.base + (uint64_t)e * r.tok_bytes + off);
    return x;
  } else {
    return __builtin_bit_cast(
        uint4, __builtin_amdgcn_raw_buffer_load_b128(r.rsrc, (int)(e + off), 0, 0));
  }
}

// ---------------------------------------------------------------------------- points

// One sampling point of a lane: cell, fractions and the slots of its four corner pairs.
struct SlotPoint {
  int x, y, z;
  float fx, fy, fz;
  uint32_t s01, s23;  // slots of the lower x corners of pairs e = 2 cz + cy, 16 bits each

  __device__ inline __attribute__((always_inline)) void set(const Geometry& g, int t, int i, int j,
                                                            int p, const float* off) {
    const int it = p / g.by_khw, r = p - it * (g.kh * g.kw), ih = r / g.by_kw, iw = r - ih * g.kw;
    axis((float)(j + iw - (g.kw - 1) / 2), off[0], g.W, x, fx);
    axis((float)(i + ih - (g.kh - 1) / 2), off[1], g.H, y, fy);
    axis((float)(t + it - (g.kt - 1) / 2), off[2], g.T, z, fz);
  }
  __device__ inline __attribute__((always_inline)) int slot(int e) const {
    const uint32_t s = e < 2 ? s01 : s23;
    return (int)(e & 1 ? s >> 16 : s & 0xffffu);
  }
  // weights of the corners c = 4 cz + 2 cy + cx, times f
  __device__ inline __attribute__((always_inline)) void weights(float (&w)[8],
                                                                float f = 1.0f) const {
    const float ax[2] = {f * (1.0f - fx), f * fx}, ay[2] = {1.0f - fy, fy}, az[2] = {1.0f - fz, fz};
#pragma unroll
    for (int c = 0; c < 8; ++c) w[c] = ax[c & 1] * (ay[(c >> 1) & 1] * az[c >> 2]);
  }
  // the point's eight values of its query's `val`
  __device__ inline __attribute__((always_inline)) void read(const float* val,
                                                             float (&v)[8]) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* p = val + slot(e);
      v[2 * e] = p[0];
      v[2 * e + 1] = p[1];
    }
  }
};

// Whether a wave's queries (every fourth four of the tile's tokens) are worth numbering: the points
// of each, with their corners, span at most `limit` voxels.  All points up to 16 SAMPLES, else so
// many of them, evenly spread.  Each wave decides for itself, so that a calm token beside wide ones
// sends none of those to the rounds without shared slots: with offsets N(0, 0.5) at every second
// token and U[-8, 8] at the others, 16x34x60, 24 heads x 128 bf16, 3x3x3, a step takes 9.3 ms (9.3
// loading every corner), and took 13.3 where the first token of a workgroup decided for all of them.
template <int SAMPLES>
__device__ inline __attribute__((always_inline)) bool compact_wave(const Geometry& g,
                                                                   const PencilOrder& po,
                                                                   const PencilTile& tl,
                                                                   const float* offsets,
                                                                   int limit) {
  constexpr int kPoints = SAMPLES * kSlotLanes;
  const int lane = threadIdx.x & 63, lp = lane % kSlotLanes;
  const int b = tl.group / g.by_heads, m = tl.group - b * g.heads;
  bool wide = false;
  for (int e0 = kSlotQueries * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
       e0 < tile_tokens(po); e0 += kWavesPerBlock * kSlotQueries) {
    int i, j;
    slot_token(po, g, tl, e0 + lane / kSlotLanes, i, j);
    i = min(i, g.H - 1);  // an idle query: the valid token that stands in for it
    j = min(j, g.W - 1);
    const int64_t row = ((int64_t)b * g.N + ((tl.frame * g.H + i) * g.W + j)) * g.heads + m;
    const float* off = offsets + row * g.P * 3;
    SlotPoint pt[SAMPLES];
#pragma unroll
    for (int u = 0; u < SAMPLES; ++u) {
      const int s = lp + u * kSlotLanes;
      const int p = g.P > kPoints ? s * g.P / kPoints : min(s, g.P - 1);
      pt[u].set(g, tl.frame, i, j, p, off + 3 * p);
    }
    int x0 = pt[0].x, x1 = x0, y0 = pt[0].y, y1 = y0, z0 = pt[0].z, z1 = z0;
#pragma unroll
    for (int u = 1; u < SAMPLES; ++u) {
      x0 = min(x0, pt[u].x);
      x1 = max(x1, pt[u].x);
      y0 = min(y0, pt[u].y);
      y1 = max(y1, pt[u].y);
      z0 = min(z0, pt[u].z);
      z1 = max(z1, pt[u].z);
    }
    // extents with the upper corners, each at most 257 so that the product stays in range
    const int ex = min(-lane_min<kSlotLanes>(-x1) - lane_min<kSlotLanes>(x0), 255) + 2;
    const int ey = min(-lane_min<kSlotLanes>(-y1) - lane_min<kSlotLanes>(y0), 255) + 2;
    const int ez = min(-lane_min<kSlotLanes>(-z1) - lane_min<kSlotLanes>(z0), 255) + 2;
    wide = wide || ex * ey * ez > limit;
  }
  return __builtin_amdgcn_ballot_w64(wide) == 0;
}

// WHOLE: the window spans all frames, so no corner can lie outside it.
//
// Numbers the slots of a wave's queries for rounds of points (npts per query) and writes the
// voxel list.  In: pt[r], the lane's point of round r (lanes past the end repeat a point of the
// range).  Returns the number of points taken per query: npts, or half of the rounds as often as it
// takes for their voxels to fit the slots, or one round without sharing when they leave the box;
// n: the slot count; `global`: the list holds tokens.
template <int R, bool WHOLE>
__device__ inline __attribute__((always_inline)) int number_slots(const Geometry& g,
                                                                  const SlotWindow& win,
                                                                  uint32_t tok_bytes,
                                                                  SlotLds& lds,
                                                                  SlotPoint (&pt)[R], int npts,
                                                                  int& n, bool& global) {
  constexpr int L = kSlotLanes;
  const int lane = lane_id();
  // the box starts at the smallest cell
  int x0 = pt[0].x, y0 = pt[0].y, z0 = pt[0].z;
#pragma unroll
  for (int r = 1; r < R; ++r) {
    if (r * L >= npts) break;
    x0 = min(x0, pt[r].x);
    y0 = min(y0, pt[r].y);
    z0 = min(z0, pt[r].z);
  }
  x0 = __builtin_amdgcn_readfirstlane(lane_min<64>(x0));
  y0 = __builtin_amdgcn_readfirstlane(lane_min<64>(y0));
  z0 = __builtin_amdgcn_readfirstlane(lane_min<64>(z0));
  bool out = false, slow = !WHOLE && win.frames == 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r * L >= npts) break;
    out = out || pt[r].x - x0 > kSlotBoxX - 2 || pt[r].y - y0 > kSlotBoxY - 2 ||
          pt[r].z - z0 > kSlotBoxZ - 2;
#pragma unroll
    for (int c = 0; c < 2 && !WHOLE; ++c)
      slow = slow || ((unsigned)(pt[r].z + c) < (unsigned)g.T &&
                      (unsigned)(pt[r].z + c - win.t0) >= (unsigned)win.frames);
  }
  const bool fits = __builtin_amdgcn_ballot_w64(out) == 0;
  global = !WHOLE && __builtin_amdgcn_ballot_w64(slow) != 0;
  n = 0;
  wave_sync();
  uint4* const w4 = reinterpret_cast<uint4*>(lds.words) + 2 * lane;
  while (fits) {
    w4[0] = make_uint4(0u, 0u, 0u, 0u);
    w4[1] = make_uint4(0u, 0u, 0u, 0u);
    wave_sync();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r * L >= npts) break;
      const uint32_t bits = 3u << (pt[r].x - x0);
      const int at = (pt[r].z - z0) * kSlotBoxY + pt[r].y - y0;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        __hip_atomic_fetch_or(&lds.words[at + (e & 1) + (e >> 1) * kSlotBoxY].x, bits,
                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    wave_sync();
    uint4 a = w4[0], b = w4[1];
    const uint32_t n0 = __popc(a.x), n1 = n0 + __popc(a.z), n2 = n1 + __popc(b.x),
                   n3 = n2 + __popc(b.z);
    const uint32_t incl = lane_scan(n3), s = incl - n3;
    n = __builtin_amdgcn_readlane((int)incl, 63);
    if (n > kSlotCap) {  // at least two rounds: one round has at most 512 corners
      npts = (npts + 2 * L - 1) / (2 * L) * L;
      wave_sync();
      continue;
    }
    a.y = s;
    a.w = s + n0;
    b.y = s + n1;
    b.w = s + n2;
    w4[0] = a;
    w4[1] = b;
    wave_sync();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r * L >= npts) break;
      const uint32_t below = (1u << (pt[r].x - x0)) - 1u;
      const int at = (pt[r].z - z0) * kSlotBoxY + pt[r].y - y0;
      uint32_t s4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint2 w = lds.words[at + (e & 1) + (e >> 1) * kSlotBoxY];
        s4[e] = w.y + __popc(w.x & below);
      }
      pt[r].s01 = s4[0] | (s4[1] << 16);
      pt[r].s23 = s4[2] | (s4[3] << 16);
    }
    break;
  }
  if (!fits) {
    npts = min(npts, L);
    n = 64 * 8;
    pt[0].s01 = (uint32_t)(8 * lane) * 0x10001u + 0x20000u;
    pt[0].s23 = pt[0].s01 + 0x40004u;
  }
  // the list: corners on one voxel write the same entry
  const int HW = g.H * g.W;
  const uint32_t step = global ? 1u : tok_bytes;
  const uint32_t dy = (uint32_t)g.W * step, dz = (uint32_t)HW * step;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r * L >= npts) break;
    const int x = pt[r].x, y = pt[r].y, z = pt[r].z;
    // modulo 2^32: only the sums of corners inside the grid are used, and those are exact
    const uint32_t org = (uint32_t)(z - (global ? 0 : win.t0)) * dz + (uint32_t)y * dy +
                         (uint32_t)x * step;
    const bool okx[2] = {(unsigned)x < (unsigned)g.W, (unsigned)(x + 1) < (unsigned)g.W};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = (unsigned)(y + (e & 1)) < (unsigned)g.H &&
                      (unsigned)(z + (e >> 1)) < (unsigned)g.T;
      const uint32_t o = org + ((e & 1) ? dy : 0u) + ((e >> 1) ? dz : 0u);
      uint32_t* p = lds.list + pt[r].slot(e);
      p[0] = ok && okx[0] ? o : kNoVoxel;
      p[1] = ok && okx[1] ? o + step : kNoVoxel;
    }
  }
  wave_sync();
  if (n + lane < ((n + 63) & ~63)) lds.list[n + lane] = kNoVoxel;  // the sweeps' last batch
  wave_sync();
  return npts;
}

// ---------------------------------------------------------------------------- dot products

// The four queries' bf16 vectors as the B operand of each 32-channel block.
template <int D>
struct SlotVecs {
  static constexpr int kParts = D / 32;
  uint4 f[kSlotQueries][kParts];
  __device__ inline __attribute__((always_inline)) void load(const char* x,
                                                             const int64_t (&row)[kSlotQueries]) {
    const int lane = lane_id();
    const bool mine = (lane >> 4) == ((lane >> 2) & 3);
#pragma unroll
    for (int w = 0; w < kSlotQueries; ++w)
#pragma unroll
      for (int k = 0; k < kParts; ++k) {
        f[w][k] = make_uint4(0u, 0u, 0u, 0u);
        if (mine)
          f[w][k] = *reinterpret_cast<const uint4*>(x + row[w] * (2 * D) + 64 * k + 16 * (lane & 3));
      }
  }
};

// val[w][s] = <vector of query w, row of slot s> for n slots on the vector ALU, U loads in flight:
// a row's lanes hold 16 bytes of it each, vec[w] the same 16 bytes of query w's vector.
template <int D, bool BF16, bool GLOBAL, int U>
__device__ inline __attribute__((always_inline)) void row_dots_valu(
    const SlotRows& rows, SlotLds& lds, const uint4 (&vec)[kSlotQueries], int n) {
  constexpr int L = D * (BF16 ? 2 : 4) / 16, SPL = 64 / L;
  const int lane = lane_id(), sub = lane % L, grp = lane / L;
  for (int base = 0; base < n; base += U * SPL) {
    uint4 a[U];
#pragma unroll
    for (int i = 0; i < U; ++i)
      a[i] = slot_load<GLOBAL>(rows, lds.list[base + i * SPL + grp], 16u * sub);
#pragma unroll
    for (int w = 0; w < kSlotQueries; ++w) {
      float keep = 0.0f;
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const float s = group_sum<L>(chunk_dot<BF16>(vec[w], a[i]));
        keep = sub == i ? s : keep;
      }
      if (sub < U) lds.val[w][base + sub * SPL + grp] = keep;
    }
  }
}

// The same on the matrix cores (bf16 rows).  A row with an infinity or a NaN meets the zeros of B
// and makes the products of three other slots NaN.
template <int D, bool GLOBAL>
__device__ inline __attribute__((always_inline)) void row_dots_mfma(const SlotRows& rows,
                                                                    SlotLds& lds,
                                                                    const SlotVecs<D>& vec,
                                                                    int n) {
  const int lane = lane_id();
  constexpr int KS = D / 32;
  const uint32_t off = 16u * (lane & 3);
  float* const out = &lds.val[lane & 3][(lane & 12) + (lane >> 4)];
  for (int base = 0; base < n; base += 32) {
    uint4 a[2][KS];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t e = lds.list[base + 16 * h + (lane >> 2)];  // past the end: no voxel
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) a[h][ks] = slot_load<GLOBAL>(rows, e, off + 64u * ks);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float s[kSlotQueries];
#pragma unroll
      for (int w = 0; w < kSlotQueries; ++w) {
        slot_f32x4_t c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(slot_bf16x8_t, a[h][ks]),
              __builtin_bit_cast(slot_bf16x8_t, vec.f[w][ks]), c, 0, 0, 0);
        // lane l: results (4 (l / 16) + i, l % 16); chunk l % 4 of slot 4 ((l / 4) % 4) + l / 16
        const float lo = lane & 1 ? c[1] : c[0], hi = lane & 1 ? c[3] : c[2];
        s[w] = lane & 2 ? hi : lo;
      }
      // the sum over the four lanes of a slot, query l % 4's in lane l
      const float u0 = (lane & 1 ? s[1] : s[0]) + dpp_mov<0xB1>(lane & 1 ? s[0] : s[1]);
      const float u1 = (lane & 1 ? s[3] : s[2]) + dpp_mov<0xB1>(lane & 1 ? s[2] : s[3]);
      out[base + 16 * h] = (lane & 2 ? u1 : u0) + dpp_mov<0x4E>(lane & 2 ? u0 : u1);
    }
  }
}

// val[w][s] = <row qrow[w] of x, row of slot s> for n slots.  APART: row by row, so that a row with an
// infinity or a NaN reaches its own slot only; for a wave whose points saw a NaN (dots_again).
template <int D, bool BF16, bool GLOBAL, bool APART>
__device__ inline __attribute__((always_inline)) void row_dots_of(
    const SlotRows& rows, SlotLds& lds, const char* x, const int64_t (&qrow)[kSlotQueries], int n) {
  if constexpr (BF16 && !APART) {
    SlotVecs<D> vec;
    vec.load(x, qrow);
    row_dots_mfma<D, GLOBAL>(rows, lds, vec, n);
  } else {
    constexpr int kRowBytes = D * (BF16 ? 2 : 4);
    uint4 own[kSlotQueries];
#pragma unroll
    for (int w = 0; w < kSlotQueries; ++w)
      own[w] = *reinterpret_cast<const uint4*>(x + qrow[w] * kRowBytes +
                                               16 * (lane_id() % (kRowBytes / 16)));
    row_dots_valu<D, BF16, GLOBAL, BF16 ? 2 : 8>(rows, lds, own, n);
  }
}

template <int D, bool BF16, bool APART = false>
__device__ inline __attribute__((always_inline)) void row_dots(const SlotRows& rows, SlotLds& lds,
                                                               const void* x,
                                                               const int64_t (&qrow)[kSlotQueries],
                                                               int n) {
  wave_sync();
  if (!rows.global)
    row_dots_of<D, BF16, false, APART>(rows, lds, static_cast<const char*>(x), qrow, n);
  else
    row_dots_of<D, BF16, true, APART>(rows, lds, static_cast<const char*>(x), qrow, n);
  wave_sync();
}

// Whether the products have to be formed again row by row: some point of the wave combined them to
// NaN.
template <bool BF16>
__device__ inline __attribute__((always_inline)) bool dots_again(bool nan) {
  return BF16 && __builtin_amdgcn_ballot_w64(nan) != 0;
}

// ---------------------------------------------------------------------------- weighted sums

// Lanes that read a row of row_sums (16 bytes each) and the channels a lane ends up with: lane l
// gets channels kVec (l % kLanes) .. of a query's sum.
template <int D, bool BF16>
struct SlotSum {
  static constexpr int kLanes = D * (BF16 ? 2 : 4) / 16;
  static constexpr int kVec = BF16 ? 8 : 4;
  static constexpr int kPer = 64 / kLanes;  // rows per load
  static constexpr int kBatch = 8 * kPer;   // slots of eight loads: load i takes slots 8 k + i
};

// val[query][s] = the sum over the query's corners on slot s of c[r] * (the corner's weight), for
// rounds of npts points per query; 0 for a slot that the query does not touch, a zero with other bits
// where it does and the sum is zero: -0 for the vector ALU, for the matrix cores a denormal number
// below 2^-141, none of whose bits are in their parts.  Needs finite c; the exponents take the
// place of the list, which waits in registers.
template <int R, bool BF16>
__device__ inline __attribute__((always_inline)) void sum_coefs(SlotLds& lds,
                                                                const SlotPoint (&pt)[R],
                                                                const float (&c)[R], int npts,
                                                                int n) {
  constexpr int L = kSlotLanes;
  constexpr int kBits = R <= 2 ? 25 : 23;  // npts 2^(kBits + 1) < 2^31
  static_assert(R * L <= 1 << (30 - kBits), "the sums fit 31 bits");
  const int lane = lane_id(), lp = lane % L;
  uint32_t* const val = reinterpret_cast<uint32_t*>(lds.val[lane / L]);
  uint8_t* const expo = reinterpret_cast<uint8_t*>(lds.list) + (lane / L) * kSlotCap;
  uint4* const l4 = reinterpret_cast<uint4*>(lds.list) + lane;
  static_assert(kSlotCap == 640, "two and a half 16-byte words per lane");
  wave_sync();
  const uint4 list0 = l4[0], list1 = l4[64], list2 = lane < 32 ? l4[128] : list0;
  for (int base = 0; base < n; base += 64)
    *reinterpret_cast<uint4*>(val + base + 4 * lp) = make_uint4(0u, 0u, 0u, 0u);
  wave_sync();
  // the largest of the slot's magnitudes, exponent + 1 in the top byte (0: untouched)
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r * L >= npts) break;
    if (r * L + lp >= npts) continue;
    float w[8];
    pt[r].weights(w, c[r]);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      __hip_atomic_fetch_max(val + pt[r].slot(e >> 1) + (e & 1),
                             (__float_as_uint(w[e]) << 1) + (1u << 24), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  wave_sync();
  for (int base = 0; base < n; base += 64) {
    const int s = base + 4 * lp;
    const uint4 m = *reinterpret_cast<const uint4*>(val + s);
    const uint32_t lo = __builtin_amdgcn_perm(m.y, m.x, 0x0c0c0703u);
    const uint32_t hi = __builtin_amdgcn_perm(m.w, m.z, 0x07030c0cu);
    *reinterpret_cast<uint32_t*>(expo + s) = lo | hi;
    *reinterpret_cast<uint4*>(val + s) = make_uint4(0u, 0u, 0u, 0u);
  }
  wave_sync();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r * L >= npts) break;
    if (r * L + lp >= npts) continue;
    float w[8];
    pt[r].weights(w, c[r]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int s = pt[r].slot(e);
      uint16_t b;  // of both slots of the pair, at any address
      __builtin_memcpy(&b, expo + s, 2);
#pragma unroll
      for (int cx = 0; cx < 2; ++cx) {
        const int bits = kBits + 128 - (int)(cx ? b >> 8 : b & 0xff);
        __hip_atomic_fetch_add(reinterpret_cast<int*>(val) + s + cx,
                               __float2int_rn(ldexpf(w[2 * e + cx], bits)), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WAVEFRONT);
      }
    }
  }
  wave_sync();
  for (int base = 0; base < n; base += 64) {
    const int s = base + 4 * lp;
    const uint32_t b = *reinterpret_cast<const uint32_t*>(expo + s);
    const int4 x = *reinterpret_cast<const int4*>(val + s);
    auto coef = [](int x, uint32_t b) {
      const float f = ldexpf((float)x, (int)b - 128 - kBits);
      const float zero = BF16 ? __uint_as_float(b) : b != 0u ? -0.0f : 0.0f;
      return x != 0 ? f : zero;
    };
    *reinterpret_cast<float4*>(val + s) = make_float4(coef(x.x, b & 255u), coef(x.y, (b >> 8) & 255u),
                                                      coef(x.z, (b >> 16) & 255u), coef(x.w, b >> 24));
  }
  wave_sync();
  l4[0] = list0;
  l4[64] = list1;
  if (lane < 32) l4[128] = list2;
  wave_sync();
}

// The part that lane l keeps of per-lane sums of the four queries: query l / 16, summed over the
// lanes that hold the same channels.
template <int LANES>
__device__ inline __attribute__((always_inline)) float keep_sum(const float (&q)[kSlotQueries]) {
  float s[kSlotQueries];
#pragma unroll
  for (int w = 0; w < kSlotQueries; ++w)
    s[w] = LANES == 8 ? q[w] + dpp_mov<0x128>(q[w]) : q[w];  // row_ror:8
  // each swap hands one half (one row) of the first over for one of the second
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(s[0]), __float_as_uint(s[2]),
                                                  false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s[1]), __float_as_uint(s[3]),
                                                  false, false);
  const float s02 = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const float s13 = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(s02), __float_as_uint(s13), false,
                                                  false);
  return __uint_as_float(c[0]) + __uint_as_float(c[1]);
}

// sum[x] = sum over n slots of val[query][s] * row s in fp32 on the vector ALU.  SAFE: a row that a
// query does not touch is not multiplied for it.
template <int D, bool BF16, bool GLOBAL, bool SAFE>
__device__ inline __attribute__((always_inline)) void row_sums_valu(
    const SlotRows& rows, const SlotLds& lds, int n, float (&sum)[SlotSum<D, BF16>::kVec]) {
  using U = SlotSum<D, BF16>;
  const int lane = lane_id(), sub = lane % U::kLanes, grp = lane / U::kLanes;
  float part[kSlotQueries][U::kVec];
#pragma unroll
  for (int w = 0; w < kSlotQueries; ++w)
#pragma unroll
    for (int x = 0; x < U::kVec; ++x) part[w][x] = 0.0f;
  for (int base = 0; base < n; base += U::kBatch) {
    const int at = base + 8 * grp;
    uint4 a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = slot_load<GLOBAL>(rows, lds.list[at + i], 16u * sub);
#pragma unroll
    for (int w = 0; w < kSlotQueries; ++w) {
      const float4* c4 = reinterpret_cast<const float4*>(&lds.val[w][at]);
      const float4 ca = c4[0], cb = c4[1];
      const float c[8] = {ca.x, ca.y, ca.z, ca.w, cb.x, cb.y, cb.z, cb.w};
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if constexpr (SAFE) {  // a sum of zero counts: 0 * infinity
          const uint32_t u = __float_as_uint(c[i]);
          if (u != 0u) chunk_axpy<BF16>(part[w], u < 256u ? 0.0f : c[i], a[i]);
        } else {
          chunk_axpy<BF16>(part[w], c[i], a[i]);
        }
    }
  }
#pragma unroll
  for (int x = 0; x < U::kVec; ++x) {
    const float q[kSlotQueries] = {part[0][x], part[1][x], part[2][x], part[3][x]};
    sum[x] = keep_sum<U::kLanes>(q);
  }
}

// The same on the matrix cores (bf16 rows).  Lane l reads the row of slot base + 8 (l / kLanes) +
// i; as the products' B its column is l % 16 and its K group l / 16, so a 16-lane group holds
// SETS = 16 / kLanes sets of rows side by side.  A's row 4 s + p holds part p (the upper, middle and
// lower 8 bits; p = 3 is not used) of the coefficients of set s % SETS for query SETS (s / SETS) + t
// in product t; result element p of lane group G is then part p's share of the sum of set
// G % SETS, meant for the columns of that set.
template <int D, bool GLOBAL>
__device__ inline __attribute__((always_inline)) void row_sums_mfma(const SlotRows& rows,
                                                                    const SlotLds& lds, int n,
                                                                    float (&sum)[8]) {
  using U = SlotSum<D, true>;
  constexpr int SETS = 16 / U::kLanes;
  static_assert(SETS == 1 || SETS == 2, "head_dim 64 or 128");
  const int lane = lane_id(), sub = lane % U::kLanes, grp = lane / U::kLanes;
  const int a_s = (lane >> 2) & 3, a_set = a_s % SETS, a_q = a_s / SETS * SETS;
  const uint32_t m1 = (lane & 3) >= 1 ? 0xffff0000u : 0u, m2 = (lane & 3) >= 2 ? 0xffff0000u : 0u;
  slot_f32x4_t acc[SETS][8];
#pragma unroll
  for (int t = 0; t < SETS; ++t)
#pragma unroll
    for (int x = 0; x < 8; ++x) acc[t][x] = slot_f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  for (int base = 0; base < n; base += U::kBatch) {
    uint32_t e[8];
    {
      const uint4* l4 = reinterpret_cast<const uint4*>(lds.list + base + 8 * grp);
      const uint4 ea = l4[0], eb = l4[1];
      e[0] = ea.x; e[1] = ea.y; e[2] = ea.z; e[3] = ea.w;
      e[4] = eb.x; e[5] = eb.y; e[6] = eb.z; e[7] = eb.w;
    }
    uint4 r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = slot_load<GLOBAL>(rows, e[i], 16u * sub);
    slot_bf16x8_t a[SETS];
#pragma unroll
    for (int t = 0; t < SETS; ++t) {
      const float4* c4 = reinterpret_cast<const float4*>(
          &lds.val[a_q + t][base + 8 * ((lane >> 4) * SETS + a_set)]);
      const float4 ca = c4[0], cb = c4[1];
      const float c[8] = {ca.x, ca.y, ca.z, ca.w, cb.x, cb.y, cb.z, cb.w};
      uint32_t u[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {  // less the parts above this lane's; its part is the upper half
        const float mid = c[i] - __uint_as_float(__float_as_uint(c[i]) & m1);
        u[i] = __float_as_uint(mid - __uint_as_float(__float_as_uint(mid) & m2));
      }
      a[t] = __builtin_bit_cast(
          slot_bf16x8_t, make_uint4(__builtin_amdgcn_perm(u[1], u[0], 0x07060302u),
                                    __builtin_amdgcn_perm(u[3], u[2], 0x07060302u),
                                    __builtin_amdgcn_perm(u[5], u[4], 0x07060302u),
                                    __builtin_amdgcn_perm(u[7], u[6], 0x07060302u)));
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      uint32_t lo[4], hi[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint4 ra = r[2 * i], rb = r[2 * i + 1];
        const uint32_t ua = w == 0 ? ra.x : w == 1 ? ra.y : w == 2 ? ra.z : ra.w;
        const uint32_t ub = w == 0 ? rb.x : w == 1 ? rb.y : w == 2 ? rb.z : rb.w;
        lo[i] = __builtin_amdgcn_perm(ub, ua, 0x05040100u);
        hi[i] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
      }
      const slot_bf16x8_t bl =
          __builtin_bit_cast(slot_bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
      const slot_bf16x8_t bh =
          __builtin_bit_cast(slot_bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
#pragma unroll
      for (int t = 0; t < SETS; ++t) {
        acc[t][2 * w] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], bl, acc[t][2 * w], 0, 0, 0);
        acc[t][2 * w + 1] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], bh, acc[t][2 * w + 1], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    float s[SETS];
#pragma unroll
    for (int t = 0; t < SETS; ++t) {
      s[t] = acc[t][x][0] + (acc[t][x][1] + acc[t][x][2]);
      if constexpr (SETS == 2) {
        // lane groups 2 h and 2 h + 1 hold sets 0 and 1 of query 2 h + t: the sum of the two
        s[t] = (lane & 15) / U::kLanes == ((lane >> 4) & 1) ? s[t] : 0.0f;
        s[t] += dpp_mov<0x128>(s[t]);  // row_ror:8
        const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[t]),
                                                        __float_as_uint(s[t]), false, false);
        s[t] = __uint_as_float(h[0]) + __uint_as_float(h[1]);
      }
    }
    sum[x] = SETS == 2 && (lane & 16) ? s[SETS - 1] : s[0];
  }
}

// sum[x]: channel kVec (l % kLanes) + x of the sum over n slots of coefficient * row for query
// l / 16.  An infinite or NaN row value meets the zero coefficients of the queries that do not
// sample it, and on the matrix cores the zero parts of those that do, and gives NaN; a wave that
// sees a NaN takes its sums again over the rows that each query samples.
template <int D, bool BF16, bool GLOBAL>
__device__ inline __attribute__((always_inline)) void row_sums_of(
    const SlotRows& rows, const SlotLds& lds, int n, float (&sum)[SlotSum<D, BF16>::kVec]) {
  if constexpr (BF16)
    row_sums_mfma<D, GLOBAL>(rows, lds, n, sum);
  else
    row_sums_valu<D, false, GLOBAL, false>(rows, lds, n, sum);
  bool nan = false;
#pragma unroll
  for (int x = 0; x < SlotSum<D, BF16>::kVec; ++x) nan = nan || sum[x] != sum[x];
  if (__builtin_amdgcn_ballot_w64(nan) != 0)
    row_sums_valu<D, BF16, GLOBAL, true>(rows, lds, n, sum);
}

template <int D, bool BF16>
__device__ inline __attribute__((always_inline)) void row_sums(
    const SlotRows& rows, const SlotLds& lds, int n, float (&sum)[SlotSum<D, BF16>::kVec]) {
  wave_sync();
  if (!rows.global)
    row_sums_of<D, BF16, false>(rows, lds, n, sum);
  else
    row_sums_of<D, BF16, true>(rows, lds, n, sum);
  wave_sync();
}

// ---------------------------------------------------------------------------- launch shape

// Pencil order of the query-owned kernels.  A tile is a workgroup's rows with a row on kLanes lanes;
// pencils are about 12 x 12 tokens: at 64x68x120, 24 heads x 128, 3x5x5, offsets U[-8, 8], the
// forward took 159 / 162 / 197 ms with pencils of about 12 x 12 / 16 x 16 / 24 x 24 tokens.
// Where tiles may be taken by slots, cells are four tokens along x, which keeps a wave's queries
// in one grid row, unless the grid's width would leave more than 1 in 32 of them empty (43x16x18:
// 10% of the gathering kernels' lanes).
// With slots, a grid whose tiles would leave compute units idle gets smaller ones, down to four
// tokens, of which a workgroup's other waves have nothing (4x8x8 tokens, 2 heads x 32, fp32: 17.6
// -> 10.6 us).
constexpr int kFillTiles = 512;  // two workgroups per compute unit
// Pencils taken in raster order stay narrow: a wave at the turn of a row spans their width, and with
// the points' reach it has to fit the 32 bits of a word.
constexpr int kRasterCols = 13;

template <int D, bool BF16>
inline PencilOrder query_order(const Geometry& g, bool slots, bool fill = false) {
  constexpr int Q = kSlotQueries;
  int run = Layout<D, BF16>::kRowsPerBlock;
  if (!slots) return plan_pencils(g.B * g.heads, g.T, g.H, g.W, run, 12, 12);
  const int64_t tokens = (int64_t)g.B * g.heads * g.N;
  while (fill && run > Q && tokens < (int64_t)run * kFillTiles) run /= 2;
  const int cols = (g.W + Q - 1) / Q;
  if (32 * (cols * Q - g.W) > g.W)
    return plan_pencils(g.B * g.heads, g.T, g.H, g.W, run, 12, 12, kRasterCols);
  PencilOrder o = plan_pencils(g.B * g.heads, g.T, g.H, cols, run / Q, 12, 12 / Q);
  o.cell = Q;
  return o;
}

// Token of row group `grp` of a gathering wave; false if it is past the tile, the pencil or the grid.
// SLOTS: the tokens that the wave would take by slots, four and four.
template <bool SLOTS, int GROUPS>
__device__ inline __attribute__((always_inline)) bool query_token(const PencilOrder& po,
                                                                  const Geometry& g,
                                                                  const PencilTile& tl, int wave,
                                                                  int grp, int& i, int& j) {
  if constexpr (SLOTS) {
    constexpr int Q = kSlotQueries;
    static_assert(GROUPS % Q == 0, "whole fours");
    const int e = Q * wave + grp % Q + grp / Q * (kWavesPerBlock * Q);
    return slot_token(po, g, tl, e, i, j) && e < tile_tokens(po);
  }
  return pencil_cell(po, tl, wave * GROUPS + grp, i, j);
}

// LDS of one wave of a kernel that keeps N 16-byte words per lane and, with SLOTS, may take its tokens
// by slots instead.
template <int L, int N, bool SLOTS>
constexpr size_t wave_lds() {
  constexpr size_t pts = slot_words<L, N>() * sizeof(int4);
  return SLOTS && sizeof(SlotLds) > pts ? sizeof(SlotLds) : pts;
}

// Launches one workgroup per virtual tile, at most kMaxBlocks (a multiple of 8, which keeps a tile
// on its XCD) at a time: launch(first tile, workgroups).  The kernels hold no loop over tiles, as
// one makes the compiler keep everything that does not depend on the tile in registers.
template <class Launch>
hipError_t launch_tiles(int64_t vtiles, Launch launch) {
  hipError_t e = hipSuccess;
  for (int64_t vt0 = 0; vt0 < vtiles && e == hipSuccess; vt0 += kMaxBlocks)
    e = launch(vt0, grid_blocks(vtiles - vt0));
  return e;
}

}  // namespace dev
}  // namespace dsa3d
