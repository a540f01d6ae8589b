// attention.hip -- fused integer attention for one (image, window, head,
// block of query rows) per workgroup:
//
//   S = Q K^T (MFMA int8) -> per-tensor dyadic -> int8 scores
//   P = Constrained Shiftmax of every score row (Alg. 2)
//   O = P V   (MFMA int8) -> per-tensor dyadic -> int8 output (token order)
//
// Constrained Shiftmax needs the exact row maximum before any exponential
// (ShiftExp of x - max cannot be rescaled bit-exactly when the maximum
// changes), so every score of a row is held until the maximum is known.  The
// scores, then their exponentials, stay in registers from the first matmul to
// the second: the waves of a workgroup split the keys of its R query rows in
// blocks of 16, and a lane holds 4 consecutive keys of one row per block.
// Those are also 4 bytes of the P V product's B operand once the key order of
// the contraction is permuted, which V's layout does (blocks of 16 keys, see
// QkvLayout), so neither scores nor probabilities pass through LDS.  Only the
// row maxima, the row sums and the waves' partial P V sums cross waves.
//
// Because the scores are int8, max - score takes the values 0..254 and
// ShiftExp is one 256-entry table; S_sum >> s_d is exactly the
// quotient-remainder denominator of Alg. 2.
//
// Bound: VALU instructions.  gfx950 issues the 64-bit multiply-add, the
// permutes and the medians at one rate, 4 cycles per wave, so their number is
// what counts: by the counters 12.1 per 64 scores of 1600-key rows (7 of them
// requantize, address the table, sum, multiply and pack) at 60 to 70% VALU
// busy, 14.7 on 400-key windows, where score rows in LDS took 11.9 at 55 to 65%
// and 19.8; the two matmuls take an eighth of the time beside them.  Against
// 32-row blocks whose scores and probabilities went through LDS, on 1600-key
// rows (2400 workgroups) 64.4 -> 59.0 us, 1200 workgroups 36.7 -> 30.5 us,
// 400-key windows (4992 workgroups) 40.8 -> 34.8 us.
#include "ilw_internal.h"

namespace ilw {
namespace {

constexpr int kXcds = 8;  // accelerator complex dies, each with its own L2

// Copies of the ShiftExp table: lane l reads copy l % kCopies, entry d at word
// kCopies d + l % kCopies, so that few lanes of a lookup meet on an LDS bank
// (with one copy a lookup of spread scores takes 5.5 LDS cycles; 32 copies
// against 16 are 1% faster on the medium encoder, and free: the P V sums need
// the bytes later).
constexpr int kCopies = 32;
constexpr int kRow = kCopies * 4;  // bytes per table entry

// Slots of 16 keys whose exponentials a wave keeps in registers, of nb; the
// scores of the others are kept as bytes and looked up twice (for the sum, and
// again for P), which keeps the kernel within the 128 registers of four waves
// per SIMD up to 13 slots.  14 to 16 (rows past 1664 keys) still spill 2 to 24
// registers in the score phase, with fewer slots kept as well.
constexpr int full_slots(int nb) { return nb <= 10 ? nb : nb <= 12 ? 10 : nb <= 14 ? 9 : 8; }

// The scores are kept complemented, n = ~q = -q - 1 in [-128, 126]: the row
// maximum of q is the row minimum of n, and max - q = n - min.
//   ~floor((acc m + r) / 2^s) = floor((-acc m - r - 1) / 2^s),
// so with nm = -m and c = -2^(s-1) - 1 the complement costs nothing.
// |acc| <= 2^20 for a 64-channel head, |m| < 2^31 and s in [22, 54]
// (launch_attention) keep the 64-bit sum exact and the result inside int32.
// From 32 on the shift is one of the sum's high word, below it is the low word
// of the 64-bit shift: one instruction each.
template <bool HIGH>
__device__ __forceinline__ int32_t score(int32_t acc, int32_t nm, int64_t c, int32_t s) {
  const int64_t p = (int64_t)acc * nm + c;
  const int32_t v = HIGH ? (int32_t)(p >> 32) >> (s - 32)
                         : (int32_t)__builtin_amdgcn_alignbit((uint32_t)(p >> 32), (uint32_t)p, s);
  return min(max(v, ~kQmax), ~kQmin);
}

// Either, for one more instruction: with k = max(32 - s, 0), acc, c and the
// shift are scaled by 2^k first, |acc| 2^k <= 2^30.
__device__ __forceinline__ int32_t score_any(int32_t acc, int32_t k, int32_t nm, int64_t ck,
                                             int32_t s32) {
  const int32_t v =
      (int32_t)(((int64_t)(int32_t)((uint32_t)acc << k) * nm + ck) >> 32) >> s32;
  return min(max(v, ~kQmax), ~kQmin);
}

// Ends a step of an unrolled loop: neither loads nor arithmetic move across,
// which keeps a step's temporaries from being live in its neighbours.  The
// running values listed are computed by then.
__device__ __forceinline__ void step_end() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
template <typename T, typename... More>
__device__ __forceinline__ void step_end(T& v, More&... more) {
  asm volatile("" : "+v"(v));
  step_end(more...);
}

// Bytes 0 of a, b, c, d packed into one word.
__device__ __forceinline__ uint32_t pack_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);
  const uint32_t hi = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
  return lo | (hi << 16);
}

// How P = min(floor(e F / 2^sh), cap) is made, from what the host can show for
// every row (p_form, launch_slots):
//   P_MUL    the high word of one multiply; 32-bit sums over a wave's keys of a row
//   P_SHIFT  that and a 32-bit shift; 32-bit sums over a lane's keys of a row
//   P_ANY    64-bit products and sums, clamped
// 8 images of 6 heads of 1600 keys take 58.0, 62.1 and 67.2 us (one general
// instance for the last two, which spilled 28 registers, 71.0 us).
enum PForm { P_MUL, P_SHIFT, P_ANY };

template <PForm P>
struct SumType {
  typedef uint32_t lane;
  typedef uint64_t row;
};
template <>
struct SumType<P_MUL> {
  typedef uint32_t lane, row;
};
template <>
struct SumType<P_ANY> {
  typedef uint64_t lane, row;
};

// R query rows (16 or 32) per workgroup of NW waves; wave w takes the 16-key
// blocks w, w + NW, ... : NB slots, of which only the last can be missing or
// partial (NB = ceil(blocks / NW)).  HIGH: how P_MUL and P_SHIFT shift the
// scores (P_ANY, for parameters that no calibration gives, takes any shift).
template <int R, int NW, int NB, PForm P, bool HIGH>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4)))
void attention_kernel(AttnArgs a, uint32_t nrb, uint32_t ntiles) {
  constexpr int NF = R / 16;                      // query fragments of 16 rows
  constexpr int NBF = full_slots(NB);             // slots held as exponentials
  constexpr int NPK = NB - NBF;                   // slots held as bytes
  // The table's copies; once the exponentials are looked up the same bytes
  // hold the partial P V sums [wave][channel group][fragment][lane].
  constexpr int PARTS = NW * 4 * NF * 64;  // 16-byte words
  constexpr int TAB = 256 * kRow;
  __shared__ __attribute__((aligned(1024))) int8_t sbuf[PARTS * 16 > TAB ? PARTS * 16 : TAB];
  __shared__ __attribute__((aligned(16))) int32_t pmin[R][NW];
  typedef typename SumType<P>::lane LaneSum;
  typedef typename SumType<P>::row Sum;
  __shared__ __attribute__((aligned(16))) Sum psum[R][NW];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int32_t Tw = a.Tw;
  // Workgroups go to the 8 XCDs round-robin; XCD x takes the contiguous
  // tiles x * per + min(x, rem) + ..., so the row blocks of one (window,
  // head) share one XCD's L2 for their keys and values.
  const uint32_t bid = blockIdx.x;
  const uint32_t per = ntiles / kXcds, rem = ntiles % kXcds, xcd = bid % kXcds;
  const uint32_t tile = xcd * per + min(xcd, rem) + bid / kXcds;
  const uint32_t slice = tile / nrb;  // (image * nW + window) * H + head
  const int32_t i0 = (int32_t)(tile - slice * nrb) * R;
  const int8_t* __restrict__ Q = a.q + (int64_t)slice * Tw * 64;
  const int8_t* __restrict__ K = a.k + (int64_t)slice * Tw * 64;
  const int8_t* __restrict__ V = a.vt + (int64_t)slice * 64 * a.Twp;

  const int32_t nkb = (Tw + 15) >> 4;
  // slot j: block wave + j NW; the last slot may be missing in this wave
  // (uniform bases and one 32-bit lane offset each, so the addresses take no
  // vector arithmetic)
  const uint32_t krow = (lane & 15) * 64 + (lane >> 4) * 16;
  auto kload = [&](int j) {
    if (j < NB - 1) return *(const v4i*)(K + (wave + j * NW) * 1024 + krow);
    // keys past the window repeat the last one: they never change the maximum
    const uint32_t key = min((wave + j * NW) * 16 + (lane & 15), Tw - 1);
    return *(const v4i*)(K + (key * 64 + (lane >> 4) * 16));
  };

  // Query fragments (MFMA B operand: columns = query rows).  Rows past the
  // window are clamped to a valid row; their results are never stored.
  // Past the head dimension (32-dim heads) the query fragment is zero, so
  // the unused key bytes there contribute nothing.
  const v4i zero = {0, 0, 0, 0};
  v4i qf[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const uint32_t r = min(i0 + f * 16 + (lane & 15), Tw - 1);
    qf[f] = *(const v4i*)(Q + (r * 64 + (lane >> 4) * 16));
  }
  constexpr int RING = NB < 4 ? NB : 4;  // key fragments in flight
  v4i kr[RING];
#pragma unroll
  for (int j = 0; j < RING; ++j) kr[j] = kload(j);
  if ((lane >> 4) * 16 >= a.hd) {
#pragma unroll
    for (int f = 0; f < NF; ++f) qf[f] = zero;
  }

  // ShiftExp(-d) for d = 0..254 (entry 255, never a valid max - score, is 0),
  // kCopies times; a thread starts its entry's 16-byte stores at another chunk
  // than its neighbours
#pragma unroll
  for (int d = tid; d < 256; d += 64 * NW) {
    const uint32_t z = min((uint32_t)(d + ((d + 1) >> 1) - ((d + 15) >> 4)),
                           (uint32_t)(a.k_inter * a.I0));
    const uint32_t n = __umulhi(z, a.inv_I0);  // floor(z / I0), or z for I0 = 1
    const uint32_t q = a.I0 == 1 ? z : n;
    const uint32_t fr = z - q * (uint32_t)a.I0;
    const int32_t e = d < 255 ? (a.I0 - (int32_t)((fr + 1) >> 1)) << (a.k_inter - (int32_t)q) : 0;
    const v4i e4 = {e, e, e, e};
#pragma unroll
    for (int c = 0; c < kCopies / 4; ++c)
      *(v4i*)(sbuf + d * kRow + ((c + d) % (kCopies / 4)) * 16) = e4;
  }

  // ---- phase 1: scores.  The key fragment is the A operand, so a lane holds
  // 4 consecutive keys of row lane % 16 of each fragment.  The products of
  // the next slot are issued before the current one is requantized.
  int32_t sc[NBF][NF][4];  // complemented scores, then exponentials
  uint32_t pk[NPK > 0 ? NPK : 1][NF];  // packed slots: complemented scores + 128, as bytes
  int32_t mn[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) mn[f] = ~kQmin;
  {
    const int32_t nm = -a.score_mult, ss = a.score_shift;
    const int64_t c = -((int64_t)1 << (ss - 1)) - 1;
    const int32_t k = max(32 - ss, 0), s32 = max(ss - 32, 0);
    const int64_t ck = c * ((int64_t)1 << k);
    v4i pr[2][NF];  // products, alternating
    auto products = [&](int j) {
#pragma unroll
      for (int f = 0; f < NF; ++f)
        pr[j & 1][f] = __builtin_amdgcn_mfma_i32_16x16x64_i8(kr[j % RING], qf[f], zero, 0, 0, 0);
      if (j + RING < NB) kr[j % RING] = kload(j + RING);
    };
    auto emit = [&](int j) {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        int32_t n[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          n[r] = P == P_ANY ? score_any(pr[j & 1][f][r], k, nm, ck, s32)
                            : score<HIGH>(pr[j & 1][f][r], nm, c, ss);
        mn[f] = min(min(mn[f], n[0]), n[1]);
        mn[f] = min(min(mn[f], n[2]), n[3]);
        if (j < NBF) {
#pragma unroll
          for (int r = 0; r < 4; ++r) sc[j < NBF ? j : 0][f][r] = n[r];
        } else {
          pk[j < NBF ? 0 : j - NBF][f] =
              pack_bytes((uint32_t)n[0], (uint32_t)n[1], (uint32_t)n[2], (uint32_t)n[3]) ^
              0x80808080u;
        }
      }
    };
    products(0);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j + 1 < NB) products(j + 1);
      emit(j);
      step_end(mn[0], mn[NF - 1]);
    }
  }
  // row minima: combine the 4 lanes sharing a row, then the waves
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    mn[f] = min(mn[f], __shfl_xor(mn[f], 16, 64));
    mn[f] = min(mn[f], __shfl_xor(mn[f], 32, 64));
    if (lane < 16) pmin[f * 16 + lane][wave] = mn[f];
  }
  lds_sync();  // also publishes the table

  // ---- phase 2: exponentials and their sums
  int32_t base[NF];  // table address of score 0's exponential in this lane's copy
  // the exponential of key r of the last slot: keys past the window have none
  auto masked = [&](int r, int32_t e) {
    return (wave + (NB - 1) * NW) * 16 + (lane >> 4) * 4 + r < Tw ? e : 0;
  };
  auto packed_exp = [&](int j, int f, int32_t(&e)[4]) {
    // (opaque, so that the second lookup unpacks again instead of keeping the
    // first one's four addresses)
    asm volatile("" : "+v"(pk[j - NBF][f]));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      e[r] = *(const int32_t*)(sbuf + (base[f] - 128 * kRow +
                                       (int32_t)((pk[j - NBF][f] >> (8 * r)) & 255) * kRow));
      if (j == NB - 1) e[r] = masked(r, e[r]);
    }
  };
  {
    LaneSum sum[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      int32_t m = pmin[f * 16 + (lane & 15)][0];
#pragma unroll
      for (int w = 1; w < NW; ++w) m = min(m, pmin[f * 16 + (lane & 15)][w]);
      base[f] = (lane & (kCopies - 1)) * 4 - m * kRow;
      sum[f] = 0;
    }
    auto lookup = [&](int j, int f) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        sc[j][f][r] = *(const int32_t*)(sbuf + (base[f] + sc[j][f][r] * kRow));
    };
    auto add = [&](const int32_t(&e)[4], int f) {  // 4 values below 2^30 each
      sum[f] += (uint32_t)e[0] + (uint32_t)e[1] + (uint32_t)e[2] + (uint32_t)e[3];
    };
    // two fragments' lookups in flight
    lookup(0, 0);
#pragma unroll
    for (int u = 0; u < NBF * NF; ++u) {
      const int j = u / NF, f = u % NF;
      if (u + 1 < NBF * NF) lookup((u + 1) / NF, (u + 1) % NF);
      if (j == NB - 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[j][f][r] = masked(r, sc[j][f][r]);
      }
      add(sc[j][f], f);
      step_end(sum[f]);
    }
#pragma unroll
    for (int j = NBF; j < NB; ++j)
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        int32_t e[4];
        packed_exp(j, f, e);
        add(e, f);
        step_end(sum[f]);
      }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      Sum t = sum[f];
#pragma unroll
      for (int o = 16; o < 64; o <<= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)t, o, 64);
        // (32-bit lane sums have no high word yet at the first exchange)
        const uint32_t hi = sizeof(Sum) == 8 && (sizeof(LaneSum) == 8 || o > 16)
                                ? __shfl_xor((uint32_t)((uint64_t)t >> 32), o, 64)
                                : 0;
        t += (Sum)(((uint64_t)hi << 32) | lo);
      }
      if (lane < 16) psum[f * 16 + lane][wave] = t;
    }
  }
  lds_sync();

  // each row's normalization factor: lane l does row l % R, once per wave
  uint32_t F;
  int32_t sh;
  {
    const int row = lane & (R - 1);
    uint64_t s = psum[row][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += psum[row][w];
    const int32_t sd = a.s_d >= 0 ? a.s_d : calibrate_shift(s, a.m_p);
    uint64_t sr = s >> sd;
    sr = sr < 1 ? 1 : (sr > 0x7fffffffull ? 0x7fffffffull : sr);
    F = div_2p31m1((uint32_t)sr);
    // e F < 2^30 2^31: a shift of 61 or more leaves 0, as does 63, so
    // the cap keeps the 64-bit shift defined (large m_p gives s_d up to 41)
    sh = min(32 - a.k_out + sd, 63);
  }
  // With sh < 32 and F < 2^sh, Fs = F 2^(32-sh) fits in 32 bits and
  // floor(e F / 2^sh) is the high word of e Fs; from sh = 32 on it is the high
  // word of e F shifted by the rest.  P_ANY: the quotient is below 2^k_out <=
  // 2^8 whatever the parameters (e F < 2^(32 + s_d) when S_sum >> s_d fits S_R;
  // smaller when S_R is clamped), so the 16-bit clamp-and-pack holds it.
  const uint32_t pcap = (1u << (a.k_out - 1)) - 1;

  // ---- phase 3: P and O = P V.  V is the A operand (rows = channels), P the
  // B operand (columns = query rows): a lane's bytes 4 u .. 4 u + 3 are the 4
  // keys of slot 4 st + u it holds, in both operands.  The waves' partial
  // sums are added through LDS.
  const uint32_t vrow = lane * 4;  // channel lane % 16, keys 4 (lane / 16) ..
  auto vload = [&](int j, int g) {  // of channel group g
    const int32_t kb = j < NB - 1 ? wave + j * NW : min(wave + j * NW, nkb - 1);
    return *(const int32_t*)(V + (kb * 1024 + g * 256) + vrow);
  };
  constexpr int NG = (NB + 3) / 4;  // P V steps of 4 slots (64 keys)
  v4i vf[2][4];
  auto vload_step = [&](int st) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        vf[st & 1][g][u] = st * 4 + u < NB ? vload(st * 4 + u, g) : 0;
  };
  // Every slot is packed before the first product: the words take a quarter
  // of the exponentials' registers, which makes room for the sums.
  v4i pw[NG][NF];
  auto pack_all = [&](auto word) {
#pragma unroll
    for (int j = 0; j < NG * 4; ++j) {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        if (j < NBF)
          pw[j / 4][f][j % 4] = (int32_t)word(sc[j < NBF ? j : 0][f], f);
        else if (j < NB) {
          int32_t e[4];
          packed_exp(j, f, e);
          pw[j / 4][f][j % 4] = (int32_t)word(e, f);
        } else {
          pw[j / 4][f][j % 4] = 0;
        }
        step_end(pw[j / 4][f]);
      }
      if (j == (NBF - 1) / 2) vload_step(0);
    }
  };
  if (P != P_ANY) {
    const uint32_t Fs = F << (sh < 32 ? 32 - sh : 0);
    uint32_t Fr[NF], tr[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      Fr[f] = __shfl(Fs, f * 16 + (lane & 15), 64);
      tr[f] = P == P_SHIFT ? (uint32_t)__shfl(max(sh - 32, 0), f * 16 + (lane & 15), 64) : 0;
    }
    pack_all([&](const int32_t(&e)[4], int f) {
      return pack_bytes(__umulhi((uint32_t)e[0], Fr[f]) >> tr[f],
                        __umulhi((uint32_t)e[1], Fr[f]) >> tr[f],
                        __umulhi((uint32_t)e[2], Fr[f]) >> tr[f],
                        __umulhi((uint32_t)e[3], Fr[f]) >> tr[f]);
    });
  } else {
    const u16x2 pcap2 = {(unsigned short)pcap, (unsigned short)pcap};
    uint32_t Fr[NF];
    int32_t hr[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      Fr[f] = __shfl(F, f * 16 + (lane & 15), 64);
      hr[f] = __shfl(sh, f * 16 + (lane & 15), 64);
    }
    pack_all([&](const int32_t(&e)[4], int f) {
      uint32_t p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = (uint32_t)(((uint64_t)(uint32_t)e[r] * Fr[f]) >> hr[f]);
      return pack_min_bytes(p[0], p[1], p[2], p[3], pcap2);
    });
  }
  if (NPK > 0) lds_sync();  // the table is no longer read
  v4i o[4][NF];
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int f = 0; f < NF; ++f) o[g][f] = zero;
#pragma unroll
  for (int st = 0; st < NG; ++st) {
    if (st + 1 < NG) vload_step(st + 1);
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int f = 0; f < NF; ++f)
        o[g][f] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf[st & 1][g], pw[st][f], o[g][f], 0, 0, 0);
    step_end();
  }
  v4i* part = (v4i*)sbuf;
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int f = 0; f < NF; ++f) part[((wave * 4 + g) * NF + f) * 64 + lane] = o[g][f];
  lds_sync();

  const uint32_t bw = slice / (uint32_t)a.H;  // image * nW + window
  const int32_t h = (int32_t)(slice - bw * (uint32_t)a.H);
  const int32_t b_img = (int32_t)(bw / (uint32_t)a.nW), w = (int32_t)(bw - (uint32_t)b_img * a.nW);
  const int32_t wy = w / a.nwx, wx = w - wy * a.nwx;
  int8_t* const out = a.out + ((int64_t)b_img * a.T + wy * a.win_h * a.grid_w + wx * a.win_w) * a.D +
                      h * a.hd;
  const int64_t rnd = (int64_t)1 << (a.pv_shift - 1);
  // tile t (channel group t / NF, fragment t % NF): a lane holds 4 channels of
  // one token
#pragma unroll
  for (int t0 = 0; t0 < 4 * NF; t0 += NW) {
    const int t = t0 + wave, g = t / NF, f = t % NF;
    if (t >= 4 * NF || g * 16 >= a.hd) break;  // channel group past the head dimension
    v4i s = part[t * 64 + lane];
#pragma unroll
    for (int q = 1; q < NW; ++q) s += part[(q * 4 * NF + t) * 64 + lane];
    const int32_t i = i0 + f * 16 + (lane & 15);
    if (i >= Tw) continue;
    const int32_t iy = fdiv(i, a.win_w, a.inv_ww);
    const int32_t tok = iy * (a.grid_w - a.win_w) + i;
    int32_t v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int32_t acc = min(max(s[r], -a.pv_clamp), a.pv_clamp);
      v[r] = min(max((int32_t)(((int64_t)acc * a.pv_mult + rnd) >> a.pv_shift), kQmin), kQmax);
    }
    *(uint32_t*)(out + (int64_t)tok * a.D + (g * 16 + (lane >> 4) * 4)) =
        pack_bytes((uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]);
  }
}

// [B, T, 3D] token-major QKV -> window-major Q, K and V (see QkvLayout).
// One thread per 16-byte chunk of Q and K; the values go in groups of 4
// consecutive keys: a thread loads a 16-channel chunk of each and stores 4
// keys of 4 channels per 16 bytes (byte stores of single keys made this 16.7 us
// against 7.0 at 4 x 1600 tokens of 384 channels).  n_qk and n_v are the two
// parts' thread counts.
__global__ __launch_bounds__(256) void qkv_relayout_kernel(const int8_t* qkv, QkvLayout L,
                                                           uint32_t n_qk, uint32_t n_v) {
  const uint32_t g = blockIdx.x * 256u + threadIdx.x;
  if (g < n_qk) {
    const uint32_t chunks = 2 * L.D / 16;
    const uint32_t m = g / chunks;
    const int32_t n = (int32_t)(g - m * chunks) * 16;
    const int32_t b = (int32_t)(m / (uint32_t)L.T), t = (int32_t)(m - (uint32_t)b * L.T);
    const int32_t ty = t / L.grid_w, tx = t - ty * L.grid_w;
    const int32_t wy = ty / L.win_h, wx = tx / L.win_w;
    const int32_t li = (ty - wy * L.win_h) * L.win_w + tx - wx * L.win_w;
    const int32_t part = n >= L.D, rem_n = n - part * L.D;
    const int32_t h = rem_n >> L.hs, c = rem_n & ((1 << L.hs) - 1);
    const int64_t slice = ((int64_t)b * L.nW + wy * L.nwx + wx) * L.H + h;
    *(v4i*)((part == 0 ? L.q : L.k) + (slice * L.Tw + li) * 64 + c) =
        *(const v4i*)(qkv + (int64_t)m * 3 * L.D + n);
    return;
  }
  const uint32_t v = g - n_qk;
  if (v >= n_v) return;
  // (window, key group, channel chunk), the chunks fastest
  const uint32_t chunks = L.D / 16, groups = (L.Tw + 3) / 4;
  const uint32_t kc = v / chunks, bw = kc / groups;
  const int32_t n = (int32_t)(v - kc * chunks) * 16, k0 = (int32_t)(kc - bw * groups) * 4;
  const int32_t b = (int32_t)(bw / (uint32_t)L.nW), w = (int32_t)(bw - (uint32_t)b * L.nW);
  const int32_t wy = w / L.nwx, wx = w - wy * L.nwx;
  v4i x[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int32_t li = min(k0 + r, L.Tw - 1);  // keys past the window carry no weight
    const int32_t iy = li / L.win_w;
    const int64_t m = (int64_t)b * L.T + (wy * L.win_h + iy) * L.grid_w + wx * L.win_w + li -
                      iy * L.win_w;
    x[r] = *(const v4i*)(qkv + m * 3 * L.D + 2 * L.D + n);
  }
  const int32_t h = n >> L.hs, c = n & ((1 << L.hs) - 1);
  int8_t* dst = L.vt + ((int64_t)bw * L.H + h) * 64 * L.Twp + vt_key(k0) + vt_channel(c);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    // 4 keys x 4 channels transposed: 16 consecutive bytes
    const uint32_t w[4] = {(uint32_t)x[0][q], (uint32_t)x[1][q], (uint32_t)x[2][q],
                           (uint32_t)x[3][q]};
    *(v4i*)(dst + vt_channel(4 * q)) = transpose4(w);
  }
}

template <int R, int NW, int NB, PForm P, bool HIGH>
hipError_t launch_variant(const AttnArgs& a, hipStream_t s) {
  const uint32_t nrb = (uint32_t)(a.Tw + R - 1) / R;
  const uint32_t ntiles = nrb * (uint32_t)(a.H * a.B * a.nW);
  hipLaunchKernelGGL((attention_kernel<R, NW, NB, P, HIGH>), dim3(ntiles), dim3(64 * NW), 0, s, a,
                     nrb, ntiles);
  return hipGetLastError();
}

// The instance with nb slots, LO <= nb <= HI.  A wave holds 16 nb keys of a
// row, a lane 4 nb, each of at most ShiftExp(0): their 32-bit sums are exact
// while that many ShiftExp(0) stay below 2^32.
template <int R, int NW, int LO, int HI>
hipError_t launch_slots(const AttnArgs& a, int32_t nb, PForm p, hipStream_t s) {
  if constexpr (LO < HI) {
    if (nb > LO) return launch_slots<R, NW, LO + 1, HI>(a, nb, p, s);
  }
  const int64_t lane = ((int64_t)a.I0 << a.k_inter) * 4 * LO;
  if (p == P_ANY || lane >= ((int64_t)1 << 32)) return launch_variant<R, NW, LO, P_ANY, true>(a, s);
  const bool high = a.score_shift >= 32;
  if (p == P_MUL && lane * 4 < ((int64_t)1 << 32))
    return high ? launch_variant<R, NW, LO, P_MUL, true>(a, s)
                : launch_variant<R, NW, LO, P_MUL, false>(a, s);
  return high ? launch_variant<R, NW, LO, P_SHIFT, true>(a, s)
              : launch_variant<R, NW, LO, P_SHIFT, false>(a, s);
}

// The cheapest form of P = floor(e F / 2^sh) that holds for every row of n
// keys (32-bit sums aside).  With E = ShiftExp(0) the sum S lies in [E, n E],
// sh = 32 - k_out + s_d, F = floor((2^31 - 1) / S_R).  The one-multiply forms
// need F < 2^sh where sh < 32, and P inside the output range without a clamp.
//  * s_d < k_out gives sh < 32: no shift after the multiply.
//  * Static s_d <= k_inter: E is a multiple of 2^s_d, so S_R >= E / 2^s_d (or
//    S_R is 2^31 - 1) and E F < 2^31 2^s_d = 2^(sh + k_out - 1), the limit.
//    S_R >= 2^(k_out - s_d) gives F < 2^(31 - k_out + s_d) = 2^(sh - 1).
//  * Dynamic s_d > 0 has S > 2^(31 - m_p) and S_R >= 2^(30 - m_p), F <=
//    2^(m_p + 1); with E <= 2^(30 - m_p) other keys make up half of S, and E F
//    stays below the limit by nearly a factor of two.  s_d = 0 is the static
//    case.
PForm p_form(const AttnArgs& a, int64_t n) {
  const int64_t E = (int64_t)a.I0 << a.k_inter;
  if (a.s_d >= 0) {
    if (a.s_d > a.k_inter || (a.s_d < a.k_out && (E >> a.s_d) < ((int64_t)1 << a.k_out)))
      return P_ANY;
    return a.s_d < a.k_out ? P_MUL : P_SHIFT;
  }
  if (E < ((int64_t)1 << a.k_out) || a.m_p + a.k_out > 30 || E > ((int64_t)1 << (30 - a.m_p)))
    return P_ANY;
  // the largest s_d: bit length of n E - 1, + m_p - 31
  const int32_t bits = 64 - __builtin_clzll((unsigned long long)(n * E));
  return bits + a.m_p - 31 < a.k_out ? P_MUL : P_SHIFT;
}

// Accumulator clamp of a requantization by m / 2^s: beyond |acc| = L the
// result saturates (|acc m| >= 129 2^s), and L m / 2^s stays far inside int32.
// (No accumulator here reaches 2^30.)
int32_t clamp_bound(int64_t am, int32_t shift) {
  if (shift > 54 || am == 0) return 1 << 30;
  const int64_t L = 129 * ((int64_t)1 << shift) / am + 1;
  return L > (1 << 30) ? 1 << 30 : (int32_t)L;
}

}  // namespace

hipError_t launch_attention(const AttnArgs& a, hipStream_t s) {
  if (a.B == 0) return hipSuccess;
  AttnArgs b = a;
  // Every score scale m / 2^s as one with s in [22, 54] and the same results,
  // |acc| <= 2^20.  A multiplier with room to spare takes a larger shift up to
  // 32 (the same value, so the same rounding), where the shift is that of the
  // product's high word.  One that stops short of 22 is at least 2^30: acc = 0
  // gives 0 and any other saturates, as with 2^30 / 2^22.  Past 54 every score
  // rounds to 0: |acc m| < 2^51.
  int64_t am = a.score_mult < 0 ? -(int64_t)a.score_mult : (int64_t)a.score_mult;
  while (b.score_shift < 32 && am < ((int64_t)1 << 30)) {
    b.score_mult *= 2;
    b.score_shift += 1;
    am *= 2;
  }
  if (b.score_shift < 22) {
    b.score_mult = b.score_mult < 0 ? -(1 << 30) : 1 << 30;
    b.score_shift = 22;
  } else if (b.score_shift > 54) {
    b.score_mult = 0;
    b.score_shift = 54;
  }
  b.pv_clamp = clamp_bound(a.pv_mult < 0 ? -(int64_t)a.pv_mult : (int64_t)a.pv_mult, a.pv_shift);
  b.inv_ww = 1.0f / (float)a.win_w;
  // floor(z / I0) = umulhi(z, ceil(2^32 / I0)) for z <= k_inter I0 <= 16 I0:
  // the excess z (I0 ceil(2^32 / I0) - 2^32) < 16 I0^2 <= 2^32
  b.inv_I0 = a.I0 == 1 ? 0 : (uint32_t)((((uint64_t)1 << 32) + a.I0 - 1) / (uint32_t)a.I0);
  const PForm p = p_form(a, a.Tw);
  const int32_t nkb = (a.Tw + 15) >> 4;  // 16-key blocks
  const int64_t wg32 = (int64_t)((a.Tw + 31) / 32) * a.H * a.B * a.nW;
  if (nkb <= 32) {
    // up to 512 keys: 4 waves, in 16-row blocks where 32-row blocks would
    // give fewer than two workgroups per CU (2 waves of twice the slots: the
    // medium encoder 1% slower)
    return wg32 < 512 ? launch_slots<16, 4, 1, 8>(b, (nkb + 3) / 4, p, s)
                      : launch_slots<32, 4, 1, 8>(b, (nkb + 3) / 4, p, s);
  }
  // Longer rows: 8 waves, two workgroups per CU, which fill each other's
  // barriers (16 waves, one workgroup: 53 against 40 us at 4 x 6 heads of
  // 1600 keys); grids of at most one workgroup per CU spread over 16 waves.
  if (wg32 <= 256) return launch_slots<32, 16, 3, 8>(b, (nkb + 15) / 16, p, s);
  return launch_slots<32, 8, 5, 16>(b, (nkb + 7) / 8, p, s);
}

hipError_t launch_qkv_relayout(const int8_t* qkv, int32_t B, const QkvLayout& L,
                               hipStream_t s) {
  // a launch holds fewer than 2^32 threads (over 68 GB of Q | K | V reach that)
  const int64_t n_qk = (int64_t)B * L.T * (2 * L.D / 16);
  const int64_t n_v = (int64_t)B * L.nW * ((L.Tw + 3) / 4) * (L.D / 16);
  if (n_qk == 0) return hipSuccess;
  if (n_qk + n_v + 255 >= ((int64_t)1 << 32)) return hipErrorInvalidValue;
  dim3 grid((unsigned)((n_qk + n_v + 255) / 256)), block(256);
  hipLaunchKernelGGL(qkv_relayout_kernel, grid, block, 0, s, qkv, L, (uint32_t)n_qk,
                     (uint32_t)n_v);
  return hipGetLastError();
}

}  // namespace ilw
