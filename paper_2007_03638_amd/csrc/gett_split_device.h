// GETT on the bf16 matrix cores with FP32 operands split into bf16 planes when a tile is staged.
//
// planes = 3 (the FP32 form): x = hi + mid + lo with hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid (8 significant
// bits each, 24 in all; both subtractions are exact). A bf16 denormal ends at 2^-133, so that an x below 2^-110 would lose
// low bits; both operands are therefore multiplied by 2^16 when they are staged, which makes the split exact for every x
// below 2^112, FP32 denormals included (denormals are kept by the conversions and by the matrix cores), and the sums of 16
// k's are divided by 2^32 as they are added to the accumulators. What is larger, or overflows so, is done again without the
// factor, element by element of the result (redo_block). The factor takes one multiplication per staged element, of which
// one operand's replaces the sign change below.
// A product a b is formed as the six plane products of relative weight down to 2^-18,
//   lo_a hi_b + hi_a lo_b + mid_a mid_b + mid_a hi_b + hi_a mid_b + hi_a hi_b,
// each exact in the matrix core, smallest first, into sums that start from zero for every 16 k's and are then added to
// the FP32 accumulators by vector additions. What is left out (mid lo, lo mid, lo lo) is below 2^-26 of |a b|, a
// quarter of the FP32 rounding of a single product. The fresh sums matter: a bf16 matrix instruction adds 8 products
// to its accumulator at a time, cut (towards minus infinity) at 2^-26 of the largest of them, so that products added
// straight to a long sum lose their low bits and leave a bias; measured over K = 13824, error against 64 bits 1.9e-6
// that way, 5.8e-7 with fresh sums and 2.2e-6 on the FP32 matrix instructions (K = 576: 3.8e-7, 1.3e-7, 4.5e-7). What
// bias the cut leaves within 16 k's is turned round in every other tile, of which one operand is staged negated and the
// sums subtracted (over K = 331776 of random signs it had been a third of the error).
// planes = 2 (the split-bf16 form): x ~ hi + lo, products lo hi, hi lo, hi hi.
//
// What bounds it: the bf16 matrix cores and the power they draw. 2.5 PFLOP/s / 6 = 417 TFLOP/s of contraction
// arithmetic in the FP32 form against 157 TFLOP/s on the FP32 matrix instructions; 833 in the split-bf16 form. At full
// load the card lowers its clock (1.7 GHz measured on the chi^9 steps at chi = 24, where the matrix cores are busy
// 0.57-0.64 of the time): a large bf16 library product reaches 1405 TFLOP/s on it, i.e. 234 and 468 per plane product. Measured: FP32 form 167-179
// TFLOP/s with 128 x 192 tiles (127 before, on the FP32 instructions with 192 x 192), split-bf16 form 310-322 with
// 192 x 192 tiles (221 before with 128 x 128 tiles and one barrier per 32 k's).
//
// Tile and waves: 4 waves of 64 x 64 to 96 x 96, two workgroups per CU (LDS up to 62 KB of 160), so that one's
// prologue, epilogue and waits hide behind the other's matrix instructions. Per 32 x 32 block and 16 k's: 6 (3) matrix
// instructions, 16 additions (FP32 form), and a share of the fragment reads, splitting, staging and loads, all spread
// over the blocks (slots) of the tile. The waves' issue slots are what these contend for: of the two staging teams the one
// with 192 rows sets the pace, 225 vector instructions a tile beside 36 matrix instructions (240 before its addresses were
// formed as they are now: chi^9 step 4 % slower; 201 without the factor of 2^16).
#pragma once

#include <algorithm>
#include <type_traits>

#include "gett_device.h"

namespace mera {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 16;  // one bf16 matrix instruction (32 x 32 x 16) deep
constexpr float kSplitScale = 0x1p16f;  // of both operands in the FP32 form

// plane products, smallest first: the planes of A and B in product q
template <int NP> constexpr int plane_a(int q) { return NP == 3 ? (q == 0 ? 2 : q == 2 || q == 3 ? 1 : 0) : (q == 0 ? 1 : 0); }
template <int NP> constexpr int plane_b(int q) { return NP == 3 ? (q == 1 ? 2 : q == 2 || q == 4 ? 1 : 0) : (q == 1 ? 1 : 0); }

// Two values as NP packed pairs of bf16 planes (value 0 in the low half), rounded to nearest even: one packed
// conversion per plane, and the residuals x - plane (exact) as two-element dot products with (-1, 0) and (0, -1),
// which need no unpacking. The two constants come through an empty asm statement: as a literal the compiler encodes
// (-1, 0) as the inline constant -1.0, which this instruction reads as the FP32 pattern, i.e. as (0, -1).
template <int NP>
__device__ inline void split_pair(float x0, float x1, uint32_t (&out)[NP]) {
  uint32_t m0 = 0x0000bf80u, m1 = 0xbf800000u;
  __asm__("" : "+s"(m0));
  __asm__("" : "+s"(m1));
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const bf16x2 w{(__bf16)x0, (__bf16)x1};
    out[p] = __builtin_bit_cast(uint32_t, w);
    if (p + 1 < NP) {
      x0 = __builtin_amdgcn_fdot2_f32_bf16(w, __builtin_bit_cast(bf16x2, m0), x0, false);
      x1 = __builtin_amdgcn_fdot2_f32_bf16(w, __builtin_bit_cast(bf16x2, m1), x1, false);
    }
  }
}

// LDS image of one operand's tile: two halves of 8 k's, in each the 8 k's of a row and plane side by side (8 bf16, 16
// bytes). A fragment of the matrix instruction (row = lane % 32, k half = lane / 32) is one 16-byte read per lane. Two
// planes: one behind the other, rows 16 bytes apart, so that 32 lanes read 512 contiguous bytes. Three planes: interleaved,
// rows 48 bytes apart (12 dwords, 3 * 4: 16 lanes' reads cover the 64 banks once), so that the places of a thread's four
// rows in all planes are within the reach of the two-word writes' 8-bit offsets from one address. The gap between the
// halves spreads the staging writes over the banks: a k-walking operand's 32 lanes write 8 bytes to 8 rows in each half
// (gap 32 dwords), a row-walking one's write 4 bytes to every fourth row, 4 k pairs in each half (gap 8 dwords).
template <bool KF, int R, int NP>
struct Image {
  static constexpr int ROW = NP == 3 ? 24 : 8;
  static constexpr int HALF = R * ROW + (KF ? 64 : 16);
  static constexpr int PLANE = NP == 3 ? 8 : 2 * HALF;
  static constexpr int SIZE = NP == 3 ? 2 * HALF : NP * PLANE;
};

// Loads one operand's R x 16 tile into registers and stages it split into the LDS image, by 128 threads (two
// waves; the other two load the other operand). VEC: 16-byte loads along the operand's unit-stride leg: 4 k's of one row
// (KF), or the same 4 rows at two neighbouring k's, which differ in the fastest contracted leg only (its extent is
// even). Otherwise for any layout and alignment: 4 k's of one row (KF), read at once at 4-byte alignment where they lie
// side by side for all lanes (RUN) and one by one elsewhere, or element by element 8 k's of one row with a wave's 64
// lanes on 64 consecutive rows and its k's, the same for all lanes, addressed in scalar registers. Rows past the
// extent read padded table entries (offset 0) and feed accumulator rows that are never stored; k's past the end are
// clamped for the address and zeroed when staged, in the last tile only.
template <bool KF, int R, int NKL, int NP, bool VEC>
struct SplitLoader {
  static constexpr int U = KF ? R / 32 : R / 64;       // units: rows per thread (VEC row-walking: quadruples of rows)
  static constexpr int NU = KF ? 4 : 8;                // elements per unit
  static constexpr int NO = VEC ? 1 : KF ? 4 : 8;      // k offsets per tile
  typedef Image<KF, R, NP> Im;
  struct Offsets {
    uint64_t o[NO];
    bool run;  // (not VEC, KF) wave-uniform: every lane's four k's are consecutive elements
  };
  const float* rowp[U];
  int r0, k0;
  float reg[U][NU];

  __device__ inline void init(const float* base, const int64_t* off_r, int64_t rbase, int t) {
    if (KF) {
      r0 = t / 4;
      k0 = 4 * (t % 4);
    } else if (VEC) {
      r0 = 4 * (t / 8);
      k0 = 2 * (t % 8);
    } else {
      r0 = t % 64;
      k0 = 8 * __builtin_amdgcn_readfirstlane(t / 64);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) rowp[i] = base + off_r[rbase + r0 + (KF ? 32 : 64) * i];
  }
  __device__ inline Offsets offsets(uint32_t kt, uint32_t K, const GettKLegs& kl, const uint32_t* stride) const {
    Offsets r;
    r.run = false;
    if (VEC) {
      const uint32_t k = kt + (uint32_t)k0, klast = K - (KF ? 4 : 2);
      r.o[0] = k_offset<NKL>(k < klast ? k : klast, kl, stride);
      // keeps the sum in one piece: otherwise each of its terms is added to every row's address
      __asm__("" : "+v"(r.o[0]));
      return r;
    }
    const uint32_t k = kt + (uint32_t)k0, klast = K - 1;
    r.o[0] = k_offset<NKL>(k < klast ? k : klast, kl, stride);
    if (KF) {
      // mag 0: a single leg, whose digit is k itself
      const uint32_t d = k - __umulhi(k, kl.mag[0]) * (kl.mag[0] ? kl.ext[0] : 0u);
      r.run = stride[0] == 1 && __all(k + 3 <= klast && d + 3 < kl.ext[0]);
      if (r.run) return r;
    }
#pragma unroll
    for (int e = 1; e < NO; ++e) r.o[e] = k_offset<NKL>(k + e < klast ? k + e : klast, kl, stride);
    return r;
  }
  __device__ inline void load_unit(int i, const Offsets& r, const uint32_t* stride) {
    if (VEC) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(rowp[i] + r.o[0]);
#pragma unroll
      for (int e = 0; e < 4; ++e) reg[i][e] = v[e];
      if (!KF) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(rowp[i] + r.o[0] + stride[0]);
#pragma unroll
        for (int e = 0; e < 4; ++e) reg[i][4 * (NU / 8) + e] = w[e];
      }
    } else if (KF && r.run) {
      const f32x4 v = *reinterpret_cast<const f32x4u*>(rowp[i] + r.o[0]);
#pragma unroll
      for (int e = 0; e < 4; ++e) reg[i][e] = v[e];
    } else {
#pragma unroll
      for (int e = 0; e < NU; ++e) reg[i][e] = rowp[i][r.o[e % NO]];
    }
  }
  __device__ inline void load(uint32_t kt, uint32_t K, const GettKLegs& kl, const uint32_t* stride) {
    const Offsets r = offsets(kt, K, kl, stride);
#pragma unroll
    for (int i = 0; i < U; ++i) load_unit(i, r, stride);
  }
  // Staging in pieces of two pairs per thread: four k's of a row (8 bytes per plane), or two of the four rows of a
  // vector row-walking operand (4 bytes per row and plane).
  static constexpr int PIECES = KF ? U : 2 * U;
  __device__ inline __bf16* at(__bf16* lds) const { return lds + (k0 >> 3) * Im::HALF + r0 * Im::ROW + (k0 & 7); }
  // `left`: k's of the range from this thread's first one on (zeros are written past them; K is a multiple of a
  // vector's or pair's length, so a vector is cut wholly or not at all). `scale`: factor of the three-plane form (a power
  // of two, negative to stage the negative)
  __device__ inline void stage_piece(int q, __bf16* dst, int left, float scale) const {
    auto val = [&](float v, bool in) {
      v = in ? v : 0.f;
      return NP == 3 ? v * scale : v;
    };
    uint32_t a[NP], b[NP];
    if (KF || !VEC) {
      const int i = KF ? q : q >> 1, e = KF ? 0 : 4 * (q & 1);
      float x[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) x[n] = val(reg[i][e + n], VEC ? left > 0 : e + n < left);
      split_pair<NP>(x[0], x[1], a);
      split_pair<NP>(x[2], x[3], b);
#pragma unroll
      for (int p = 0; p < NP; ++p)
        *reinterpret_cast<u32x2*>(dst + p * Im::PLANE + i * (KF ? 32 : 64) * Im::ROW + e) = u32x2{a[p], b[p]};
    } else {
      const int i = q >> 1, j = 2 * (q & 1), w = 4 * (NU / 8);
      const bool in = left > 0;
      split_pair<NP>(val(reg[i][j], in), val(reg[i][w + j], in), a);
      split_pair<NP>(val(reg[i][j + 1], in), val(reg[i][w + j + 1], in), b);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        *reinterpret_cast<uint32_t*>(dst + p * Im::PLANE + (i * 64 + j) * Im::ROW) = a[p];
        *reinterpret_cast<uint32_t*>(dst + p * Im::PLANE + (i * 64 + j + 1) * Im::ROW) = b[p];
      }
    }
  }
  // whether piece q is the last that reads its unit's registers, and that unit
  static constexpr bool frees(int q) { return KF || (q & 1); }
  static constexpr int unit_of(int q) { return KF ? q : q >> 1; }
};

// Elements of one wave's 32 x 32 block whose scaled sums were not finite (bit r of `todo`: register r of this lane), again
// from operands read straight from global memory: first the same products and sums without the scale. Of these, the
// elements that are no number (an infinite element, or one that bf16 rounds to infinity, splits into inf - inf, where FP32
// arithmetic may give an infinity or a number) or are below 2^60, in which an element that lost low bits may count (the
// loss is below 2^-134 times the other operand's element, together below 2^26 for K < 2^31), on the FP32 matrix
// instructions. One block at a time, which leaves the main loop its registers. An ascending map at chi = 16 whose operator
// lies beyond the scale's range takes 16 ms this way (ordinarily 4.5), one with a NaN in it 25 (by multiply-adds for each
// element 104); ternary at chi = 16 2.0 and 2.2 ms (0.67; 20).
template <int NKL>
__device__ inline void redo_block(const GettArgs& g, int grp, int64_t r0, int64_t c0, uint32_t kb, uint32_t ke, int lane,
                                  uint32_t todo) {
  // rows and columns past the extents read padded table entries (offset 0)
  const float* a = static_cast<const float*>(g.A[grp]) + g.a_m[r0 + (lane & 31)];
  const float* b = static_cast<const float*>(g.B[grp]) + g.b_n[c0 + (lane & 31)];
  auto load = [&](uint32_t k, float& x, float& y) {
    const bool in = k < ke;
    const uint32_t kc = in ? k : ke - 1;
    x = a[k_offset<NKL>(kc, g.kl, g.kl.sa)];
    y = b[k_offset<NKL>(kc, g.kl, g.kl.sb)];
    if (!in) x = y = 0.f;
  };
  f32x16 acc{};
  float sign = 1.f;
#pragma unroll 2
  for (uint32_t kt = kb; kt < ke; kt += BK, sign = -sign) {
    uint32_t pa[3][4], pb[3][4];
    float x[8], y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) load(kt + 8 * (lane >> 5) + e, x[e], y[e]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t u[3], v[3];
      split_pair<3>(sign * x[2 * j], sign * x[2 * j + 1], u);
      split_pair<3>(y[2 * j], y[2 * j + 1], v);
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        pa[p][j] = u[p];
        pb[p][j] = v[p];
      }
    }
    auto frag = [](const uint32_t (&w)[4]) { return __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]}); };
    f32x16 t{};
#pragma unroll
    for (int q = 0; q < 6; ++q)
      t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(pa[plane_a<3>(q)]), frag(pb[plane_b<3>(q)]), t, 0, 0, 0);
    acc += sign * t;
  }
  f32x16 plain{};
  uint32_t rest = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) rest |= fabsf(acc[r]) >= 0x1p60f ? 0u : 1u << r;
  rest &= todo;
  if (__any(rest != 0)) {
#pragma nounroll
    for (uint32_t kt = kb; kt < ke; kt += BK) {
      float x[BK / 2], y[BK / 2];
#pragma unroll
      for (int s = 0; s < BK / 2; ++s) load(kt + 2 * s + (lane >> 5), x[s], y[s]);
#pragma unroll
      for (int s = 0; s < BK / 2; ++s) plain = __builtin_amdgcn_mfma_f32_32x32x2f32(x[s], y[s], plain, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t row = r0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), col = c0 + (lane & 31);
    if (!((todo >> r) & 1) || row >= g.M || col >= g.N) continue;
    const float s = (rest >> r) & 1 ? plain[r] : acc[r];
    if (g.split) {
      (static_cast<float*>(g.partial[grp]) + (int64_t)blockIdx.z * g.M * g.N)[row * g.N + col] = s;
    } else {
      float* c = static_cast<float*>(g.C[grp]) + g.c_m[row] + g.c_n[col];
      const float v = float(g.alpha) * s;
      *c = g.beta != 0.0 ? v + float(g.beta) * *c : v;
    }
  }
}

template <int BM, int BN, bool AKF, bool BKF, int NKL, int NP, bool VEC>
__global__ void __launch_bounds__(256, 2) gett_split_kernel(GettArgs g) {
  constexpr int WM = BM / 2, WN = BN / 2, FM = WM / 32, FN = WN / 32;
  typedef Image<AKF, BM, NP> ImA;
  typedef Image<BKF, BN, NP> ImB;
  __shared__ __attribute__((aligned(16))) __bf16 As[2][ImA::SIZE];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[2][ImB::SIZE];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * WM;
  const int wn = (wave & 1) * WN;
  int64_t m0, n0;
  tile_origin<BM, BN>(xcd_tile(blockIdx.x, gridDim.x), g.M, g.N, m0, n0);
  // k in 32 bits (K < 2^31)
  const uint32_t K = (uint32_t)g.K, kb = blockIdx.z * (uint32_t)g.kchunk, ke = K - kb < g.kchunk ? K : kb + (uint32_t)g.kchunk;
  const int grp = blockIdx.y;

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x16{};

  constexpr int NQ = NP == 3 ? 6 : 3;

  auto left_of = [&](uint32_t k) { return (int)(ke - k) < BK ? (int)(ke - k) : BK; };

  // Wave tile in slots, one 32 x 32 block each, the blocks of a row one after another (of a column where the tile is
  // taller than wide). Fragments of the first block of a tile are read behind the barrier of the tile before; the
  // others two slots ahead of their use.
  constexpr bool ROWS = FM <= FN;                       // outer loop over block rows
  constexpr int NO = ROWS ? FM : FN, NI = ROWS ? FN : FM;
  constexpr int S = NO * NI;
  const int fa = (lane >> 5) * ImA::HALF + (wm + (lane & 31)) * ImA::ROW;
  const int fb = (lane >> 5) * ImB::HALF + (wn + (lane & 31)) * ImB::ROW;
  constexpr int PO = ROWS ? ImA::PLANE : ImB::PLANE, PI = ROWS ? ImB::PLANE : ImA::PLANE;
  constexpr int RO = NO == 3 ? 3 : 2;                    // the next tile's first fragments may not replace the last row's
  bf16x8 fro[RO][NP], fri[NI][NP];
  auto read_o = [&](int buf, int o) {
    const __bf16* at = (ROWS ? As[buf] + fa : Bs[buf] + fb) + o * 32 * ImA::ROW;
#pragma unroll
    for (int p = NP - 1; p >= 0; --p) fro[o % RO][p] = *reinterpret_cast<const bf16x8*>(at + p * PO);
  };
  auto read_i = [&](int buf, int i) {
    const __bf16* at = (ROWS ? Bs[buf] + fb : As[buf] + fa) + i * 32 * ImA::ROW;
#pragma unroll
    for (int p = NP - 1; p >= 0; --p) fri[i][p] = *reinterpret_cast<const bf16x8*>(at + p * PI);
  };
  static_assert(NP == 2 || S % 2 == 0, "slot 0 must not reuse the last slot's sums");
  f32x16 part[2] = {};
  auto multiply = [&](int s) {
    const int o = s / NI, i = s % NI;
    f32x16& c = acc[ROWS ? o : i][ROWS ? i : o];
    f32x16 t = NP == 3 ? f32x16{} : c;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const bf16x8 a = ROWS ? fro[o % RO][plane_a<NP>(q)] : fri[i][plane_a<NP>(q)];
      const bf16x8 b = ROWS ? fri[i][plane_b<NP>(q)] : fro[o % RO][plane_b<NP>(q)];
      t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, t, 0, 0, 0);
    }
    if (NP == 3) part[s & 1] = t;
    else c = t;
  };
  // adds the sums of block s of a tile, with the factor that undoes its scale and sign
  auto flush = [&](int s, float factor) {
    if (NP == 3) {
      const int o = s / NI, i = s % NI;
      acc[ROWS ? o : i][ROWS ? i : o] += factor * part[s & 1];
    }
  };

  // One tile t (one barrier, before the last slot): the matrix instructions read it from LDS buffer t & 1, while
  // tile t + 1, in registers since tile t - 1, is split and staged into the other buffer piece by piece over the
  // slots before the barrier (TAIL: with zeros past the end), each unit of registers being reloaded from tile t + 2
  // as soon as it is staged, so that a load has about a tile's time. Every wave runs the same number of barriers.
  // In the FP32 form one operand's odd tiles are staged negated (FLIP: by this wave).
  constexpr float unscale = 1.f / (kSplitScale * kSplitScale);
  auto signed_by = [](float x, uint32_t negative) { return __uint_as_float(__float_as_uint(x) | negative << 31); };  // x > 0
  auto tile = [&](auto tail_tag, auto flip_tag, auto& ld, uint32_t kt, uint32_t buf, __bf16* lds, const uint32_t* stride) {
    constexpr bool TAIL = decltype(tail_tag)::value;
    constexpr bool FLIP = NP == 3 && decltype(flip_tag)::value;
    typedef std::remove_reference_t<decltype(ld)> L;
    const auto off = ld.offsets(kt + 2 * BK, K, g.kl, stride);
    const int left = TAIL ? left_of(kt + BK + ld.k0) : BK;
    __bf16* const at = ld.at(lds + (buf ^ 1) * L::Im::SIZE);
    const float factor = signed_by(unscale, buf), scale = signed_by(kSplitScale, FLIP ? buf ^ 1 : 0);  // scale: of tile t + 1
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (s == S - 1) {
        __syncthreads();
        read_o(buf ^ 1, 0);
        read_i(buf ^ 1, 0);
      }
      // fragments: the inner ones during the first row, the next outer one in the middle of a row
      if (s + 1 < NI) read_i(buf, s + 1);
      if (s % NI == NI - 2 && s / NI + 1 < NO) read_o(buf, s / NI + 1);
      multiply(s);
      if (s > 0) flush(s - 1, factor);
      else flush(S - 1, -factor);  // the last block of the tile before
      if (s < S - 1) {
#pragma unroll
        for (int q = 0; q < L::PIECES; ++q)
          if (q * (S - 1) / L::PIECES == s) {
            ld.stage_piece(q, at, left, scale);
            if (ld.frees(q)) ld.load_unit(ld.unit_of(q), off, stride);
          }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto loop = [&](auto flip_tag, auto& ld, __bf16* lds, const uint32_t* stride) {
    if (kb >= ke) return;
    typedef std::remove_reference_t<decltype(ld)> L;
    ld.load(kb, K, g.kl, stride);
#pragma unroll
    for (int q = 0; q < L::PIECES; ++q) ld.stage_piece(q, ld.at(lds), left_of(kb + ld.k0), kSplitScale);
    ld.load(kb + BK, K, g.kl, stride);
    __syncthreads();
    read_o(0, 0);
    read_i(0, 0);
    uint32_t kt = kb, buf = 0;
    for (; kt + 2 * BK < ke; kt += BK, buf ^= 1) tile(std::false_type{}, flip_tag, ld, kt, buf, lds, stride);
    for (; kt < ke; kt += BK, buf ^= 1) tile(std::true_type{}, flip_tag, ld, kt, buf, lds, stride);
    flush(S - 1, signed_by(unscale, buf ^ 1));
  };
  const float* A = static_cast<const float*>(g.A[grp]);
  const float* B = static_cast<const float*>(g.B[grp]);
  // waves 0 and 1 stage A, waves 2 and 3 stage B (a wave-uniform choice)
  if (wave < 2) {
    SplitLoader<AKF, BM, NKL, NP, VEC> ld;
    ld.init(A, g.a_m, m0, tid & 127);
    loop(std::integral_constant<bool, (BM <= BN)>{}, ld, As[0], g.kl.sa);
  } else {
    SplitLoader<BKF, BN, NKL, NP, VEC> ld;
    ld.init(B, g.b_n, n0, tid & 127);
    loop(std::integral_constant<bool, (BM > BN)>{}, ld, Bs[0], g.kl.sb);
  }

  // Stores the elements for which take(value) holds; acc[i] -> row 8 (i / 4) + 4 (lane / 32) + i % 4,
  // column lane % 32.
  auto row_of = [&](int i, int r) { return m0 + wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); };
  auto col_of = [&](int j) { return n0 + wn + j * 32 + (lane & 31); };
  auto epilogue = [&](auto&& take) {
    if (g.split) {
      float* P = static_cast<float*>(g.partial[grp]) + (int64_t)blockIdx.z * g.M * g.N;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int64_t row = row_of(i, r), col = col_of(j);
            if (row < g.M && col < g.N && take(acc[i][j][r])) P[row * g.N + col] = acc[i][j][r];
          }
      return;
    }
    float* __restrict__ C = static_cast<float*>(g.C[grp]);
    const float alpha = float(g.alpha), beta = float(g.beta);
    int64_t cn[FN];
    bool cv[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      cn[j] = g.c_n[col_of(j)];
      cv[j] = col_of(j) < g.N;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      int64_t cm[16];
      bool rv[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        cm[r] = g.c_m[row_of(i, r)];
        rv[r] = row_of(i, r) < g.M;
      }
      if (g.beta != 0.0) {
        // per block, all reads of C first, unconditionally (padded table entries address element 0 of a valid row or
        // column), so they are in flight together; then the masked read-modify-write stores
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          float cold[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) cold[r] = C[cm[r] + cn[j]];
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (cv[j] && rv[r] && take(acc[i][j][r])) C[cm[r] + cn[j]] = alpha * acc[i][j][r] + beta * cold[r];
        }
      } else {
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (cv[j] && rv[r] && take(acc[i][j][r])) C[cm[r] + cn[j]] = alpha * acc[i][j][r];
      }
    }
  };
  if constexpr (NP == 3) {
    float zero = 0.f;  // NaN if any sum is not finite
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) zero = fmaf(acc[i][j][r], 0.f, zero);
    if (__any(zero != zero)) {
      uint32_t todo[FM * FN];
#pragma unroll
      for (int b = 0; b < FM * FN; ++b) {
        todo[b] = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) todo[b] |= fabsf(acc[b / FN][b % FN][r]) < INFINITY ? 0u : 1u << r;
      }
      epilogue([](float v) { return fabsf(v) < INFINITY; });
#pragma nounroll
      for (int b = 0; b < FM * FN; ++b) {
        uint32_t m = 0;
#pragma unroll
        for (int c = 0; c < FM * FN; ++c) m = b == c ? todo[c] : m;
        if (__any(m != 0)) redo_block<NKL>(g, grp, m0 + wm + b / FN * 32, n0 + wn + b % FN * 32, kb, ke, lane, m);
      }
      return;
    }
  }
  epilogue([](float) { return true; });
}

// Three planes without 16-byte loads: tiles with a 192 side exist for row-walking operands only. The branch between the
// two forms of a k-walking operand's loads costs registers that the larger tiles do not have (they spill 15 to 80: 82 to
// 104 TFLOP/s at chi = 21 and 22, 124 to 131 with 128 x 128).
template <bool VEC, int NP, int BM, int BN> constexpr bool kRowWalkingOnly = !VEC && NP == 3 && BM + BN > 256;

template <int BM, int BN, int NKL, int NP, bool VEC>
void launch_k(const GettArgs& a, dim3 grid, hipStream_t s, bool akf, bool bkf) {
  const dim3 block(256);
  if constexpr (!kRowWalkingOnly<VEC, NP, BM, BN>) {
    if (akf && bkf) hipLaunchKernelGGL((gett_split_kernel<BM, BN, true, true, NKL, NP, VEC>), grid, block, 0, s, a);
    else if (akf) hipLaunchKernelGGL((gett_split_kernel<BM, BN, true, false, NKL, NP, VEC>), grid, block, 0, s, a);
    else if (bkf) hipLaunchKernelGGL((gett_split_kernel<BM, BN, false, true, NKL, NP, VEC>), grid, block, 0, s, a);
    if (akf || bkf) return;
  } else if (akf || bkf) {
    throw Error(MERA_EINVAL, "gett: no split kernel of this tile");
  }
  hipLaunchKernelGGL((gett_split_kernel<BM, BN, false, false, NKL, NP, VEC>), grid, block, 0, s, a);
}

template <int BM, int BN, bool VEC>
void launch_tile(const GettArgs& a, int groups, int splits, hipStream_t s, bool akf, bool bkf, int planes) {
  const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const dim3 grid((unsigned)tiles, (unsigned)groups, (unsigned)splits);
  if (planes == 3) {
    constexpr int NP = BM + BN < 384 ? 3 : 2;  // no 192 x 192 tile of three planes: checked by the caller
    if (a.kl.n <= 2) launch_k<BM, BN, 2, NP, VEC>(a, grid, s, akf, bkf);
    else launch_k<BM, BN, 4, NP, VEC>(a, grid, s, akf, bkf);
  } else {
    if (a.kl.n <= 2) launch_k<BM, BN, 2, 2, VEC>(a, grid, s, akf, bkf);
    else launch_k<BM, BN, 4, 2, VEC>(a, grid, s, akf, bkf);
  }
}

template <bool VEC>
void launch_split(const GettArgs& a, int groups, int splits, hipStream_t s, bool akf, bool bkf, int bm, int bn, int planes) {
  if (bm == 192 && bn == 192 && planes == 2) launch_tile<192, 192, VEC>(a, groups, splits, s, akf, bkf, 2);
  else if (bm == 128 && bn == 192) launch_tile<128, 192, VEC>(a, groups, splits, s, akf, bkf, planes);
  else if (bm == 192 && bn == 128) launch_tile<192, 128, VEC>(a, groups, splits, s, akf, bkf, planes);
  else if (bm == 128 && bn == 128) launch_tile<128, 128, VEC>(a, groups, splits, s, akf, bkf, planes);
  else throw Error(MERA_EINVAL, "gett: no split kernel of this tile");
}

}  // namespace

}  // namespace mera
