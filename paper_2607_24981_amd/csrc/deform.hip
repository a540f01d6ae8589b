// deform.hip -- multi-scale deformable sampling core with integer weights
// (Sec. 3.1.1: the sampled value is the nearest grid point instead of a
// bilinear blend; Sec. 3.3.2: the sampling weights are Constrained Shiftmax
// of the L*P logits of each (image, query, head)).
//
// A group of lanes serves one (image, query, head); a lane owns four channels,
// so the head slice of one sample (head_dim bytes) is read by the group as
// consecutive 32-bit words.  The group kernel divides the L*P samples among its
// lanes, which exchange their words and weights through LDS; the general
// kernel, for what that one does not hold (launch_deform), has head_dim/4 lanes
// a group and makes every weight in every lane.
//
// Sampling locations are Q8 pixels of each level.  A reference point (x, y)
// lands at floor(x W / 2^8) and the offset adds Q8 pixels.  A reference box
// (cx, cy, w, h) takes the offset in units of the box, location = c +
// (off / 2^8) / P * size / 2, floored once in Q8 pixels:
// X = floor((cx 2^9 P + off_x w) W / (2^17 P)).
#include "ilw_internal.h"

namespace ilw {
namespace {

constexpr uint32_t NXCD_D = 8;

// This workgroup's place in the output.  Workgroup i runs on XCD i % 8, and
// each XCD has its own L2: consecutive (image, query, head) groups go to one
// XCD, so that it gathers from few images' value maps and not from all of
// them (8 images, 300 queries, 8 heads, 80^2 / 40^2 / 20^2 maps, bilinear:
// 14.3 -> 10.1 us).
__device__ __forceinline__ uint32_t xcd_block() {
  const uint32_t per = gridDim.x / NXCD_D, rem = gridDim.x % NXCD_D, xcd = blockIdx.x % NXCD_D;
  return xcd * per + min(xcd, rem) + blockIdx.x / NXCD_D;
}

// floor(n / d) for d > 0
__device__ __forceinline__ int64_t floor_div_pos(int64_t n, int64_t d) {
  const int64_t q = n / d;
  return (n % d != 0 && n < 0) ? q - 1 : q;
}

// Output requantization of a bilinear sum, scaled by 2^16 (the corner
// weights): sat8(floor((acc mult + 2^(shift + 15)) / 2^(shift + 16))) for
// |acc| <= 64 127 2^16 127 < 2^36.  With acc = 2^16 hi + lo the quotient is
// floor((hi mult + floor((lo mult + 2^(shift + 15)) / 2^16)) / 2^shift): every
// term stays below 2^62 where acc mult takes 67 bits.
__device__ __forceinline__ int32_t rq_bilinear(int64_t acc, int32_t mult, int32_t shift) {
  const int64_t lo = (int64_t)(uint32_t)(acc & 0xffff) * mult + ((int64_t)1 << (shift + 15));
  return sat8(((acc >> 16) * mult + (lo >> 16)) >> shift);
}

__global__ __launch_bounds__(256) void deform_kernel(DeformArgs a) {
  __shared__ int32_t elut[256];
  elut[threadIdx.x] = shift_exp(-(int32_t)threadIdx.x, a.I0, a.k_inter);
  __syncthreads();

  const int32_t G = a.Dh >> 2;  // lanes per (b, q, h)
  const int64_t gid = (int64_t)xcd_block() * 256 + threadIdx.x;
  const int64_t grp = gid / G;
  const int32_t cl = (int32_t)(gid % G);
  if (grp >= (int64_t)a.B * a.Q * a.H) return;
  const int32_t h = (int32_t)(grp % a.H);
  const int64_t bq = grp / a.H;
  const int32_t b = (int32_t)(bq / a.Q);
  const int32_t LP = a.L * a.P;

  // Constrained Shiftmax over the L*P logits of this (b, q, h)
  const int8_t* lg = a.logits + grp * LP;
  int32_t m = -128;
  for (int32_t i = 0; i < LP; ++i) m = max(m, (int32_t)lg[i]);
  uint64_t sum = 0;
  for (int32_t i = 0; i < LP; ++i) sum += (uint32_t)elut[m - lg[i]];
  const int32_t sd = a.s_d >= 0 ? a.s_d : calibrate_shift(sum, a.m_p);
  const uint32_t F = shiftmax_factor(sum, sd);
  // e F < 2^30 2^31: a shift of 61 or more leaves 0, as does 63, so the cap
  // keeps the 64-bit shift defined (s_d reaches 36 with m_p = 31)
  const int32_t sh = min(32 - a.k_out + sd, 63);
  const uint64_t cap = (1u << (a.k_out - 1)) - 1;

  const bool box = a.ref_dims == 4;
  const int32_t* r = a.ref + bq * a.ref_dims;
  const int64_t rx = r[0], ry = r[1];
  const int64_t bw = box ? r[2] : 0, bh = box ? r[3] : 0;
  // box locations divide by 2^17 P: a shift when P is a power of two
  const int32_t pshift = (a.P & (a.P - 1)) == 0 ? 17 + __builtin_ctz(a.P) : -1;
  const int64_t den = (int64_t)131072 * a.P;
  const int64_t cxs = rx * 512 * a.P, cys = ry * 512 * a.P;
  auto box_loc = [&](int64_t num) {
    return pshift >= 0 ? num >> pshift : floor_div_pos(num, den);
  };
  const int16_t* off = a.offs + grp * LP * 2;
  const int8_t* off8 = a.offs8 + grp * LP * 2;
  auto offset = [&](int32_t k) {  // offset word k of this (b, q, h)
    return a.offs8 ? (int64_t)off8[k] << a.off_shift : (int64_t)off[k];
  };
  const int64_t head_stride = (int64_t)a.H * a.Dh;
  const int8_t* vbase = a.value + (int64_t)b * a.S * head_stride + (int64_t)h * a.Dh + cl * 4;

  // The samples go in chunks whose gathers are all issued before any is
  // used: addresses of samples outside the map are clamped onto the base
  // row (a valid address) and their weights are 0.
  int32_t acc[4] = {0, 0, 0, 0};
  int64_t accw[4] = {0, 0, 0, 0};
  int32_t l = 0, p = 0;  // level and point of sample i0
  constexpr int CH = 8;
  for (int32_t i0 = 0; i0 < LP; i0 += CH) {
    uint32_t v[CH][4];
    int64_t wt[CH][4];
    int32_t ll = l, pp = p;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int32_t i = i0 + u;
      const bool live = i < LP;
      const int32_t Hl = a.hw[ll][0], Wl = a.hw[ll][1];
      const int8_t* vl = vbase + (int64_t)a.start[ll] * head_stride;
      const int32_t ic = live ? i : LP - 1;
      const uint64_t pw = ((uint64_t)(uint32_t)elut[m - lg[ic]] * F) >> sh;
      const int32_t wgt = live ? (int32_t)(pw > cap ? cap : pw) : 0;
      const int64_t ox = offset(2 * ic), oy = offset(2 * ic + 1);
      const int64_t X = box ? box_loc((cxs + ox * bw) * Wl) : ((rx * Wl) >> 8) + ox;
      const int64_t Y = box ? box_loc((cys + oy * bh) * Hl) : ((ry * Hl) >> 8) + oy;
      if (a.mode == 0) {
        const int64_t ix = X >> 8, iy = Y >> 8;  // floor
        const bool in = ix >= 0 && ix < Wl && iy >= 0 && iy < Hl;
        v[u][0] = *(const uint32_t*)(in ? vl + (iy * Wl + ix) * head_stride : vbase);
        wt[u][0] = in ? wgt : 0;
      } else {
        const int64_t Xc = X - 128, Yc = Y - 128;  // half-pixel grid
        const int64_t x0 = Xc >> 8, y0 = Yc >> 8;
        const int32_t fx = (int32_t)(Xc & 255), fy = (int32_t)(Yc & 255);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int dx = c & 1, dy = c >> 1;
          const int64_t xi = x0 + dx, yi = y0 + dy;
          const bool in = xi >= 0 && xi < Wl && yi >= 0 && yi < Hl;
          const int32_t wc = (dx ? fx : 256 - fx) * (dy ? fy : 256 - fy);
          v[u][c] = *(const uint32_t*)(in ? vl + (yi * Wl + xi) * head_stride : vbase);
          wt[u][c] = in ? (int64_t)wgt * wc : 0;
        }
      }
      if (++pp == a.P) {
        pp = 0;
        ll = min(ll + 1, a.L - 1);
      }
    }
    l = ll;
    p = pp;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      if (a.mode == 0) {
        const int32_t w0 = (int32_t)wt[u][0];
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] += w0 * (int32_t)(int8_t)(v[u][0] >> (8 * c));
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int c = 0; c < 4; ++c) accw[c] += wt[u][k] * (int32_t)(int8_t)(v[u][k] >> (8 * c));
      }
    }
  }
  uint32_t packed = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int32_t r = a.mode == 0 ? rq(acc[c], a.out_mult, a.out_shift)
                                  : rq_bilinear(accw[c], a.out_mult, a.out_shift);
    packed |= (uint32_t)(r & 0xff) << (8 * c);
  }
  *(uint32_t*)(a.out + grp * a.Dh + cl * 4) = packed;
}

// Lanes per group for a head of `words` 4-channel words: the next power of
// two, at least 4.
__host__ __device__ __forceinline__ int32_t group_lanes(int32_t words) {
  int32_t g = 4;
  while (g < words) g <<= 1;
  return g;
}

// The same sampler without the per-lane redundancy, on groups of
// G = group_lanes(head_dim) lanes that align with waves: lane k of a group
// owns samples k, k + G, ..., computes their Shiftmax weights and the value
// words they read, the group combines the row maximum and the exponential sum
// with XOR shuffles, and each sample's (words, weights) reach the G lanes of
// its group through LDS.  J = ceil(L*P / G) samples per lane; MODE 0 nearest,
// 1 bilinear.  The first head_dim / 4 lanes of a group sum and store.
//
// A decoder's call has a few waves per SIMD, so a wave's own chain of
// latencies and instructions is the time: everything the lanes read of their
// own samples is loaded before the table's barrier, and the gathers of one
// chunk of samples are in flight while the chunk before is summed.  A word
// offset is computed once, by the owner: made by every lane of the group, with
// a shuffle per corner, it cost as much as the products (8 x 300 queries, 8
// heads, 12 samples, boxes, bilinear: 15.8 -> 14.3 us; 3 x 794 queries, 12
// heads, 15 samples, nearest: 9.5 -> 7.9 us).
template <int MODE, int J>
__global__ __launch_bounds__(256) void deform_group_kernel(DeformArgs a) {
  constexpr int NC = MODE == 0 ? 1 : 4;  // value words per sample
  constexpr int CH = 4;                  // samples per chunk of gathers
  // per sample of a group, its value words and weights; a group's slots are
  // followed by an empty one, so that the groups' reads of one sample lie on
  // different banks
  struct __attribute__((aligned(4 * NC))) Words { uint32_t w[NC]; };
  struct __attribute__((aligned(4 * NC))) Weights { int32_t w[NC]; };
  __shared__ Words swords[256 * J + 64];
  __shared__ Weights sweights[256 * J + 64];
  __shared__ int32_t elut[256];

  const int32_t words = a.Dh >> 2, G = group_lanes(words), gs = __builtin_ctz(G);
  const int32_t cl = threadIdx.x & (G - 1);
  const uint32_t ngrp = (uint32_t)a.B * a.Q * a.H;  // below 2^31: the host's rule
  const int64_t grp0 = ((int64_t)xcd_block() * 256 + threadIdx.x) >> gs;
  const bool live = grp0 < (int64_t)ngrp;
  const uint32_t grp = live ? (uint32_t)grp0 : ngrp - 1;  // idle lanes still join the shuffles
  const uint32_t bq = grp / (uint32_t)a.H, h = grp - bq * (uint32_t)a.H;
  const int32_t LP = a.L * a.P;
  const int32_t slot0 = (int32_t)(threadIdx.x >> gs) * (J * G + 1);

  // what this lane's samples read, before the table's barrier
  const int8_t* lg = a.logits + (int64_t)grp * LP;
  const int16_t* off = a.offs + (int64_t)grp * LP * 2;
  const int8_t* off8 = a.offs8 + (int64_t)grp * LP * 2;
  const bool box = a.ref_dims == 4;
  const int32_t* r = a.ref + (int64_t)bq * a.ref_dims;
  int32_t lgv[J], ox[J], oy[J], Hl[J], Wl[J], st[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int32_t i = cl + j * G, ic = i < LP ? i : 0;
    const int32_t l = (int32_t)((uint32_t)ic / (uint32_t)a.P);
    lgv[j] = i < LP ? (int32_t)lg[ic] : -128;
    ox[j] = a.offs8 ? (int32_t)off8[2 * ic] : (int32_t)off[2 * ic];
    oy[j] = a.offs8 ? (int32_t)off8[2 * ic + 1] : (int32_t)off[2 * ic + 1];
    Hl[j] = a.hw[l][0];
    Wl[j] = a.hw[l][1];
    st[j] = a.start[l];
  }
  const int64_t rx = r[0], ry = r[1];
  const int64_t bw = box ? r[2] : 0, bh = box ? r[3] : 0;
  elut[threadIdx.x] = shift_exp(-(int32_t)threadIdx.x, a.I0, a.k_inter);
  lds_sync();

  // Constrained Shiftmax over the group's L*P logits
  int32_t m = -128;
#pragma unroll
  for (int j = 0; j < J; ++j) m = max(m, lgv[j]);
  for (int o = 1; o < G; o <<= 1) m = max(m, __shfl_xor(m, o, 64));
  uint64_t sum = 0;
#pragma unroll
  for (int j = 0; j < J; ++j)
    if (cl + j * G < LP) sum += (uint32_t)elut[m - lgv[j]];
  for (int o = 1; o < G; o <<= 1) {
    const uint32_t lo = __shfl_xor((uint32_t)sum, o, 64);
    const uint32_t hi = __shfl_xor((uint32_t)(sum >> 32), o, 64);
    sum += ((uint64_t)hi << 32) | lo;
  }
  const int32_t sd = a.s_d >= 0 ? a.s_d : calibrate_shift(sum, a.m_p);
  const uint32_t F = shiftmax_factor(sum, sd);
  // e F < 2^30 2^31: a shift of 61 or more leaves 0, as does 63, so the cap
  // keeps the 64-bit shift defined (s_d reaches 36 with m_p = 31)
  const int32_t sh = min(32 - a.k_out + sd, 63);
  const uint64_t cap = (1u << (a.k_out - 1)) - 1;

  const int32_t pshift = (a.P & (a.P - 1)) == 0 ? 17 + __builtin_ctz(a.P) : -1;
  const int64_t den = (int64_t)131072 * a.P;
  const int64_t cxs = rx * 512 * a.P, cys = ry * 512 * a.P;
  auto box_loc = [&](int64_t num) {
    return pshift >= 0 ? num >> pshift : floor_div_pos(num, den);
  };
  const uint32_t row_words = (uint32_t)a.H * (uint32_t)words;

  // the lane's own samples (off the map: word 0 with weight 0)
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const uint64_t pw = ((uint64_t)(uint32_t)elut[m - lgv[j]] * F) >> sh;
    const int32_t wgt = cl + j * G < LP ? (int32_t)(pw > cap ? cap : pw) : 0;
    const int64_t dx0 = a.offs8 ? (int64_t)ox[j] << a.off_shift : (int64_t)ox[j];
    const int64_t dy0 = a.offs8 ? (int64_t)oy[j] << a.off_shift : (int64_t)oy[j];
    const int64_t X = box ? box_loc((cxs + dx0 * bw) * Wl[j]) : ((rx * Wl[j]) >> 8) + dx0;
    const int64_t Y = box ? box_loc((cys + dy0 * bh) * Hl[j]) : ((ry * Hl[j]) >> 8) + dy0;
    Words ws;
    Weights wt;
    if (MODE == 0) {
      const int64_t ix = X >> 8, iy = Y >> 8;  // floor
      const bool in = ix >= 0 && ix < Wl[j] && iy >= 0 && iy < Hl[j];
      ws.w[0] = in ? ((uint32_t)st[j] + (uint32_t)iy * (uint32_t)Wl[j] + (uint32_t)ix) * row_words : 0;
      wt.w[0] = in ? wgt : 0;
    } else {
      const int64_t Xc = X - 128, Yc = Y - 128;  // half-pixel grid
      const int64_t x0 = Xc >> 8, y0 = Yc >> 8;
      const int32_t fx = (int32_t)(Xc & 255), fy = (int32_t)(Yc & 255);
      const uint32_t row0 = (uint32_t)st[j] + (uint32_t)y0 * (uint32_t)Wl[j] + (uint32_t)x0;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int dx = c & 1, dy = c >> 1;
        const bool in = x0 >= -dx && x0 < Wl[j] - dx && y0 >= -dy && y0 < Hl[j] - dy;
        ws.w[c] = in ? (row0 + (dy ? (uint32_t)Wl[j] : 0) + dx) * row_words : 0;
        wt.w[c] = in ? wgt * (dx ? fx : 256 - fx) * (dy ? fy : 256 - fy) : 0;
      }
    }
    swords[slot0 + cl + j * G] = ws;
    sweights[slot0 + cl + j * G] = wt;
  }
  // a group lies in one wave: its own stores, in order
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  // every sample of the group; slots past L*P hold weight 0
  const uint32_t* vbase = (const uint32_t*)a.value +
                          (int64_t)(bq / (uint32_t)a.Q) * a.S * row_words + h * (uint32_t)words +
                          min(cl, words - 1);
  int32_t acc[4] = {0, 0, 0, 0};
  int64_t accw[4] = {0, 0, 0, 0};
  auto fetch = [&](uint32_t(&v)[CH][NC], int i0) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const Words ws = swords[slot0 + i0 + u];
#pragma unroll
      for (int c = 0; c < NC; ++c) v[u][c] = vbase[ws.w[c]];
    }
  };
  auto use = [&](const uint32_t(&v)[CH][NC], int i0) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const Weights wt = sweights[slot0 + i0 + u];
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int32_t x = (int32_t)(int8_t)(v[u][c] >> (8 * q));
          if (MODE == 0) acc[q] += wt.w[c] * x;
          else accw[q] += (int64_t)wt.w[c] * x;
        }
    }
  };
  uint32_t va[CH][NC], vb[CH][NC];
  fetch(va, 0);
  for (int i0 = 0; i0 < LP; i0 += 2 * CH) {
    const bool second = i0 + CH < LP;
    if (second) fetch(vb, i0 + CH);
    use(va, i0);
    if (i0 + 2 * CH < LP) fetch(va, i0 + 2 * CH);
    if (second) use(vb, i0 + CH);
  }
  if (!live || cl >= words) return;
  uint32_t packed = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int32_t rv = MODE == 0 ? rq(acc[c], a.out_mult, a.out_shift)
                                 : rq_bilinear(accw[c], a.out_mult, a.out_shift);
    packed |= (uint32_t)(rv & 0xff) << (8 * c);
  }
  ((uint32_t*)a.out)[(int64_t)grp * words + cl] = packed;
}

template <int MODE>
hipError_t launch_group(const DeformArgs& a, int32_t J, dim3 grid, hipStream_t s) {
  switch (J) {
    case 1: hipLaunchKernelGGL((deform_group_kernel<MODE, 1>), grid, dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((deform_group_kernel<MODE, 2>), grid, dim3(256), 0, s, a); break;
    case 3: hipLaunchKernelGGL((deform_group_kernel<MODE, 3>), grid, dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((deform_group_kernel<MODE, 4>), grid, dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_deform(const DeformArgs& a, hipStream_t s) {
  const int64_t groups = (int64_t)a.B * a.Q * a.H;
  if (groups == 0) return hipSuccess;
  const int32_t words = a.Dh / 4, G = group_lanes(words), LP = a.L * a.P, J = (LP + G - 1) / G;
  // The group kernel up to 4 samples a lane, where a launch holds its threads
  // (fewer than 2^32 in whole workgroups) and an image's word offsets are
  // 32-bit.  It is the faster one also with idle lanes: 48 channels per head on
  // 16 lanes, 8 x 300 queries, 8 heads, 12 samples: nearest 7.6 us (the general
  // kernel 25.8), boxes and bilinear 13.1 (44.3).
  if (J <= 4 && groups * G <= (int64_t)UINT32_MAX - 255 &&
      (int64_t)a.S * a.H * words <= UINT32_MAX) {
    const dim3 grid((unsigned)((groups * G + 255) / 256));
    return a.mode == 0 ? launch_group<0>(a, J, grid, s) : launch_group<1>(a, J, grid, s);
  }
  const dim3 grid((unsigned)((groups * words + 255) / 256)), block(256);
  hipLaunchKernelGGL(deform_kernel, grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace ilw
