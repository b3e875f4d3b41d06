// GETT for contractions too small to fill the chip with LDS tiles: 32 x 32 tiles, matrix-core fragments read straight
// from global memory, the four or eight waves of a workgroup sharing the tile's k range.
//
// Such a launch is bound by latency, not by any rate: the tables, the operands, the chain of matrix instructions, the
// stores. With 64 or 128-wide tiles a 144^3 product in FP64 occupies 6 of 256 CUs and walks its k range alone, staging
// each 16 k's through LDS between two barriers. Here it occupies 25, each wave walks every WAVES-th chunk of 16 k's,
// a chunk's loads are in flight together with the next chunk's behind them, and no barrier stands between them; the
// waves' sums meet once, in LDS, and are added in FP64. Operands come from L2 (they are small), in any layout and at any
// alignment. Measured, LDS tiles / this kernel: FP64 25 x 625 x 25 7.4 / 4.9 us, 144^3 18.2 / 6.4 us, 256^3 29.5 / 9.5 us,
// 4096 x 64 x 64 12.5 / 5.6 us, 100 x 100 x 10000 (split) 40 / 26 us; FP32 400^3 32 / 8 us, 144 x 144 x 20736 (split)
// 63 / 34 us.
#include "gett_device.h"

namespace mera {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Lane layouts: both 16x16x4 forms take A[m = lane % 16][k = lane / 16], B[k = lane / 16][n = lane % 16]
template <typename T> struct Mma16;
template <> struct Mma16<float> {
  typedef f32x4 acc_t;
  __device__ static inline acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int lane, int i) { return 4 * (lane >> 4) + i; }
};
template <> struct Mma16<double> {
  typedef f64x4 acc_t;
  __device__ static inline acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int lane, int i) { return (lane >> 4) + 4 * i; }
};

constexpr int TILE = kDirectTile, CHUNK = kDirectChunk;

// One lane's four consecutive k's of one row: 16-byte loads (V) or element by element
template <typename T, bool V>
__device__ inline void load4(T (&out)[4], const T* p, uint32_t stride) {
  if constexpr (V) {
    constexpr int W = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
#pragma unroll
    for (int e = 0; e < 4; e += W) {
      const vec v = *reinterpret_cast<const vec*>(p + e);
#pragma unroll
      for (int i = 0; i < W; ++i) out[e + i] = v[i];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = p[(uint64_t)e * stride];
  }
}

template <bool SPLIT, typename T>
__device__ inline T operand(T x) {
  if constexpr (SPLIT) {
    const float hi = (float)(__bf16)x;
    return hi + (float)(__bf16)(x - hi);
  }
  return x;
}

// QUADS: the fastest contracted leg's extent is a multiple of 4, and a lane takes four consecutive k's of a chunk (chosen
// from the layouts). AV, BV (only with QUADS): that leg is the operand's unit-stride leg and its addresses are 16-byte
// aligned, so that the four are read at once (chosen from the addresses too; the sums are the same either way).
// SPLIT: the split-bf16 form; each operand element is replaced by the sum of the two bf16 numbers it is split into.
template <typename T, int NKL, int WAVES, bool QUADS, bool AV, bool BV, bool SPLIT>
__global__ void __launch_bounds__(64 * WAVES) gett_direct_kernel(GettArgs g) {
  using F = Mma16<T>;
  static_assert(QUADS || !(AV || BV), "vectors of four k's");
  __shared__ T red[WAVES][TILE][TILE + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t tn = (g.N + TILE - 1) / TILE;
  const int64_t m0 = (int64_t)blockIdx.x / tn * TILE, n0 = (int64_t)blockIdx.x % tn * TILE;
  const int grp = blockIdx.y;
  const int64_t kb = (int64_t)blockIdx.z * g.kchunk;
  const int64_t ke = (g.K < kb + g.kchunk) ? g.K : kb + g.kchunk;
  const int r = lane & 15, kq = lane >> 4;
  // rows and columns past the extents read padded table entries (offset 0) and feed sums that are never stored
  const T* A = static_cast<const T*>(g.A[grp]);
  const T* B = static_cast<const T*>(g.B[grp]);
  const T* a[2] = {A + g.a_m[m0 + r], A + g.a_m[m0 + 16 + r]};
  const T* b[2] = {B + g.b_n[n0 + r], B + g.b_n[n0 + 16 + r]};

  // Where this thread's results go and, if they are added to C, what is there: on their way together with the operands
  constexpr int NE = TILE * TILE / (64 * WAVES);
  T* c[NE];
  T old[NE];
  bool live[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int id = tid + 64 * WAVES * e;
    const int64_t row = m0 + id / TILE, col = n0 + id % TILE;
    live[e] = row < g.M && col < g.N;
    c[e] = g.split ? static_cast<T*>(g.partial[grp]) + (int64_t)blockIdx.z * g.M * g.N + row * g.N + col
                   : static_cast<T*>(g.C[grp]) + g.c_m[row] + g.c_n[col];
    old[e] = T(0);
    if (!g.split && g.beta != 0.0 && live[e]) old[e] = *c[e];
  }

  typename F::acc_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = T(0);

  // Matrix instruction s of a chunk takes the k's 4 s + kq, in ascending order. With QUADS lane group kq takes
  // 4 kq + s instead: the order is free as long as both operands follow it, and a row's four k's can be one load.
  static_assert(CHUNK == 16, "four lane groups of four k's");
  T av[2][2][4], bv[2][2][4];  // two chunks: one multiplied, the next one on its way
  auto load = [&](int slot, int64_t k) {
    if constexpr (QUADS) {  // ke is a multiple of 4 then
      const uint32_t kc = (uint32_t)(k + 4 * kq < ke ? k + 4 * kq : ke - 4);
      const uint64_t oa = k_offset<NKL>(kc, g.kl, g.kl.sa), ob = k_offset<NKL>(kc, g.kl, g.kl.sb);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        load4<T, AV>(av[slot][i], a[i] + oa, g.kl.sa[0]);
        load4<T, BV>(bv[slot][i], b[i] + ob, g.kl.sb[0]);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint32_t kc = (uint32_t)(k + 4 * s + kq < ke ? k + 4 * s + kq : ke - 1);
        const uint64_t oa = k_offset<NKL>(kc, g.kl, g.kl.sa), ob = k_offset<NKL>(kc, g.kl, g.kl.sb);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          av[slot][i][s] = a[i][oa];
          bv[slot][i][s] = b[i][ob];
        }
      }
    }
  };
  auto mul = [&](int slot, int64_t k) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool in = k + (QUADS ? 4 * kq + s : 4 * s + kq) < ke;
      T x[2], y[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x[i] = in ? operand<SPLIT>(av[slot][i][s]) : T(0);
        y[i] = in ? operand<SPLIT>(bv[slot][i][s]) : T(0);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = F::mma(x[i], y[j], acc[i][j]);
    }
  };
  constexpr int STEP = CHUNK * WAVES;
  int64_t k = kb + CHUNK * wave;
  if (k < ke) load(0, k);
  while (k < ke) {
    if (k + STEP < ke) load(1, k + STEP);
    mul(0, k);
    k += STEP;
    if (k >= ke) break;
    if (k + STEP < ke) load(0, k + STEP);
    mul(1, k);
    k += STEP;
  }

#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][16 * i + F::row(lane, e)][16 * j + r] = acc[i][j][e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int id = tid + 64 * WAVES * e, i = id / TILE, j = id % TILE;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) v += (double)red[w][i][j];
    if (!g.split) v = g.beta != 0.0 ? g.alpha * v + g.beta * (double)old[e] : g.alpha * v;
    if (live[e]) *c[e] = (T)v;
  }
}

template <typename T, int NKL, int WAVES, bool SPLIT>
void launch_direct(const GettArgs& a, dim3 grid, hipStream_t s, bool quads, bool av, bool bv) {
  const dim3 block(64 * WAVES);
  if (!quads) hipLaunchKernelGGL((gett_direct_kernel<T, NKL, WAVES, false, false, false, SPLIT>), grid, block, 0, s, a);
  else if (av && bv) hipLaunchKernelGGL((gett_direct_kernel<T, NKL, WAVES, true, true, true, SPLIT>), grid, block, 0, s, a);
  else if (av) hipLaunchKernelGGL((gett_direct_kernel<T, NKL, WAVES, true, true, false, SPLIT>), grid, block, 0, s, a);
  else if (bv) hipLaunchKernelGGL((gett_direct_kernel<T, NKL, WAVES, true, false, true, SPLIT>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gett_direct_kernel<T, NKL, WAVES, true, false, false, SPLIT>), grid, block, 0, s, a);
}

template <typename T, bool SPLIT>
void launch_direct(const GettArgs& a, dim3 grid, hipStream_t s, int waves, bool quads, bool av, bool bv) {
  if (waves == 8) {
    if (a.kl.n <= 2) launch_direct<T, 2, 8, SPLIT>(a, grid, s, quads, av, bv);
    else launch_direct<T, 4, 8, SPLIT>(a, grid, s, quads, av, bv);
  } else {
    if (a.kl.n <= 2) launch_direct<T, 2, 4, SPLIT>(a, grid, s, quads, av, bv);
    else launch_direct<T, 4, 4, SPLIT>(a, grid, s, quads, av, bv);
  }
}

}  // namespace

void launch_gett_direct(const GettArgs& a, int groups, int splits, hipStream_t s, Prec prec, int waves, bool quads,
                        bool av, bool bv) {
  const int64_t tiles = ((a.M + TILE - 1) / TILE) * ((a.N + TILE - 1) / TILE);
  const dim3 grid((unsigned)tiles, (unsigned)groups, (unsigned)splits);
  quads = quads && a.kl.n >= 1 && a.kl.ext[0] % 4 == 0;
  av = av && quads;
  bv = bv && quads;
  if (prec == Prec::F64) launch_direct<double, false>(a, grid, s, waves, quads, av, bv);
  else if (prec == Prec::F32) launch_direct<float, false>(a, grid, s, waves, quads, av, bv);
  else launch_direct<float, true>(a, grid, s, waves, quads, av, bv);
}

}  // namespace mera
