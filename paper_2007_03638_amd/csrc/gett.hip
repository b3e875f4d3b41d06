// Permute-fused GETT kernels for gfx950: LDS-staged, register-prefetched tile loads (16-byte vectors where the
// layouts allow; row offsets from tables, k offsets computed from the contracted legs), MFMA inner products
// (f32 32x32x2, f64 16x16x4, bf16 16x16x32 for the split-bf16 form), split-K partials reduced in FP64.
#include "gett_device.h"

#include <algorithm>
#include <type_traits>

namespace mera {

namespace {

using Args = GettArgs;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Lane layouts (checked on gfx950 against a host GEMM):
//  f32 32x32x2:  A[m = lane%32][k = lane/32], B[k = lane/32][n = lane%32],
//                acc[i] -> row 8*(i/4) + 4*(lane/32) + i%4, col lane%32
//  f64 16x16x4:  A[m = lane%16][k = lane/16], B[k = lane/16][n = lane%16],
//                acc[i] -> row lane/16 + 4*i, col lane%16
//  bf16 16x16x32: A[m = lane%16][k = 8*(lane/16)+j], B[k = 8*(lane/16)+j][n = lane%16],
//                acc[i] -> row 4*(lane/16) + i, col lane%16
template <typename T> struct Mma;
template <> struct Mma<float> {
  static constexpr int MT = 32, NT = 32, KT = 2, NACC = 16;
  typedef f32x16 acc_t;
  __device__ static inline acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int lane, int i) { return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3); }
  __device__ static inline int col(int lane) { return lane & 31; }
};
template <> struct Mma<double> {
  static constexpr int MT = 16, NT = 16, KT = 4, NACC = 4;
  typedef f64x4 acc_t;
  __device__ static inline acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int lane, int i) { return (lane >> 4) + 4 * i; }
  __device__ static inline int col(int lane) { return lane & 15; }
};

// Tile loader: BMN x BK tile of an operand whose element (r, k) lives at base + off_r[r] + k_offset(k).
// KFAST: consecutive threads walk k (the operand's unit-stride leg is a K leg); each thread then owns one k
// and PER rows. Otherwise consecutive threads walk r in groups of 64; each thread owns NR rows and NK k's, and
// a wave's k's are the same for all its lanes, so their offsets are formed once per wave in scalar registers.
// Rows past the extent are not masked: their table entries are padded with offset 0, so they read a valid
// element and only feed accumulator rows that are never stored. k past the end of the range is clamped for the
// address and masked (zero) when the tile is staged, which only the last tile of a range needs (KMASK).
template <typename T, int BMN, int BK, bool KFAST, int NKL>
struct Loader {
  static constexpr int PER = BMN * BK / 256;
  static_assert(PER >= 1 && (BMN * BK) % 256 == 0, "tile too small for 256 threads");
  static_assert(KFAST ? (256 % BK == 0) : (BMN % 64 == 0), "thread mapping");
  static constexpr int NR = KFAST ? PER : BMN / 64;   // rows per thread
  static constexpr int NK = KFAST ? 1 : PER / NR;     // k's per thread
  static constexpr int RSTEP = KFAST ? 256 / BK : 64;
  static constexpr int KSTEP = KFAST ? 1 : 4;         // 256 threads / 64 rows per group
  static_assert(KFAST || NK * KSTEP == BK, "k coverage");
  const T* rowp[NR];
  int r0;
  uint32_t k0;
  T reg[PER];

  __device__ inline void init(const T* base, const int64_t* off_r, int64_t rbase, int tid) {
    if (KFAST) {
      k0 = tid % BK;
      r0 = tid / BK;
    } else {
      r0 = tid % 64;
      k0 = __builtin_amdgcn_readfirstlane(tid / 64);
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) rowp[i] = base + off_r[rbase + r0 + i * RSTEP];
  }
  // loads the tile starting at kt; element (i): row index i % NR, k index i / NR
  __device__ inline void load(int64_t kt, int64_t K, const GettKLegs& kl, const uint32_t* stride) {
    const uint32_t klast = (uint32_t)K - 1;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
      const uint32_t k = (uint32_t)kt + k0 + j * KSTEP;
      const uint64_t o = k_offset<NKL>(k < klast ? k : klast, kl, stride);
#pragma unroll
      for (int r = 0; r < NR; ++r) reg[j * NR + r] = rowp[r][o];
    }
  }
  // value of element i of the tile starting at kt, zero past kend when KMASK
  template <bool KMASK>
  __device__ inline T value(int i, int64_t kt, int64_t kend) const {
    return (KMASK && kt + k0 + (i / NR) * KSTEP >= kend) ? T(0) : reg[i];
  }
  __device__ inline int lds_index(int i, int LD) const {
    return (k0 + (i / NR) * KSTEP) * LD + r0 + (i % NR) * RSTEP;
  }
  // LDS tile stored k-major: lds[k * LD + r]
  template <int LD, bool KMASK>
  __device__ inline void store(T* lds, int64_t kt, int64_t kend) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) lds[lds_index(i, LD)] = value<KMASK>(i, kt, kend);
  }
  template <int LD>
  __device__ inline void store_tile(T* lds, int64_t kt, int64_t kend) const {
    if (kt + BK <= kend) store<LD, false>(lds, kt, kend);
    else store<LD, true>(lds, kt, kend);
  }
};

// Vectorised tile loader: each global load moves VW consecutive elements along the operand's unit-stride leg
// (VW = 4 for FP32, 2 for FP64: 16 bytes). Used when that leg is the fastest index the loader walks, its extent
// and every other stride are multiples of VW and the base is 16-byte aligned, so that every vector lies within
// one run of the unit-stride leg. KFAST: the vectors run along k (VW k's of one row; staged as VW scalar LDS
// writes); otherwise along rows (VW rows at one k; one vector LDS write). Vector i of a thread is the tile's
// vector number tid + 256 i; padded rows (offset 0) and clamped k read valid elements, as in Loader.
template <typename T, int BMN, int BK, bool KFAST, int NKL, int VW>
struct VecLoader {
  typedef T V __attribute__((ext_vector_type(VW)));
  static constexpr int G = KFAST ? BK / VW : BMN / VW;  // vectors along the walked dimension
  static constexpr int NV = BMN * BK / VW / 256;        // vectors per thread
  static_assert(NV >= 1 && (BMN * BK / VW) % 256 == 0, "tile too small for 256 threads");
  const T* rowp[NV];
  int rr[NV], kk[NV];
  V reg[NV];

  __device__ inline void init(const T* base, const int64_t* off_r, int64_t rbase, int tid) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int e = tid + 256 * i;
      rr[i] = KFAST ? e / G : (e % G) * VW;
      kk[i] = KFAST ? (e % G) * VW : e / G;
      rowp[i] = base + off_r[rbase + rr[i]];
    }
  }
  __device__ inline void load(int64_t kt, int64_t K, const GettKLegs& kl, const uint32_t* stride) {
    const uint32_t klast = (uint32_t)(KFAST ? K - VW : K - 1);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const uint32_t k = (uint32_t)kt + (uint32_t)kk[i];
      const uint64_t o = k_offset<NKL>(k < klast ? k : klast, kl, stride);
      reg[i] = *reinterpret_cast<const V*>(rowp[i] + o);
    }
  }
  template <int LD, bool KMASK>
  __device__ inline void store(T* lds, int64_t kt, int64_t kend) const {
    static_assert(KFAST || LD % VW == 0, "vector LDS rows");
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (KFAST) {
#pragma unroll
        for (int j = 0; j < VW; ++j)
          lds[(kk[i] + j) * LD + rr[i]] = (KMASK && kt + kk[i] + j >= kend) ? T(0) : reg[i][j];
      } else {
        V v = reg[i];
        if (KMASK && kt + kk[i] >= kend) v = V(T(0));
        *reinterpret_cast<V*>(&lds[kk[i] * LD + rr[i]]) = v;
      }
    }
  }
  template <int LD>
  __device__ inline void store_tile(T* lds, int64_t kt, int64_t kend) const {
    if (kt + BK <= kend) store<LD, false>(lds, kt, kend);
    else store<LD, true>(lds, kt, kend);
  }
};

template <typename T, int BM, int BN, int BK, bool AKF, bool BKF, int NKL, bool VEC>
// At most 256 registers per lane (2 waves per SIMD) for every tile; the register allocator then keeps the
// accumulators in VGPRs (the 128 x 64 FP64 tile fits in 168 and runs 3 waves per SIMD).
__global__ void __launch_bounds__(256, 2) gett_kernel(Args g) {
  using F = Mma<T>;
  // vector width of the tile loads (VEC: both operands qualify). LDS rows are padded: to a multiple of VW where
  // an operand is staged with vector writes (loads along rows), else by 2 FP32 / 1 FP64 elements, which keeps the
  // strided scalar writes of k-walking loads free of bank conflicts.
  constexpr int VW = VEC ? 16 / (int)sizeof(T) : 1;
  constexpr int PADS = sizeof(T) == 4 ? 2 : 1;
  constexpr int LDA = BM + ((VEC && !AKF) ? VW : PADS), LDB = BN + ((VEC && !BKF) ? VW : PADS);
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int FM = WM / F::MT, FN = WN / F::NT;
  static_assert(FM >= 1 && FN >= 1, "wave tile smaller than one MFMA block");
  __shared__ T As[2][BK * LDA];
  __shared__ T Bs[2][BK * LDB];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = (wave >> 1) * WM;
  const int wn = (wave & 1) * WN;

  int64_t m0, n0;
  tile_origin<BM, BN>(xcd_tile(blockIdx.x, gridDim.x), g.M, g.N, m0, n0);
  const int64_t kb = (int64_t)blockIdx.z * g.kchunk;
  const int64_t ke = (g.K < kb + g.kchunk) ? g.K : kb + g.kchunk;

  const int grp = blockIdx.y;
  const T* __restrict__ A = static_cast<const T*>(g.A[grp]);
  const T* __restrict__ B = static_cast<const T*>(g.B[grp]);

  std::conditional_t<VEC, VecLoader<T, BM, BK, AKF, NKL, VW>, Loader<T, BM, BK, AKF, NKL>> la;
  std::conditional_t<VEC, VecLoader<T, BN, BK, BKF, NKL, VW>, Loader<T, BN, BK, BKF, NKL>> lb;
  la.init(A, g.a_m, m0, tid);
  lb.init(B, g.b_n, n0, tid);

  typename F::acc_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < F::NACC; ++r) acc[i][j][r] = T(0);

  // MFMA operand fragments, double-buffered: the fragments of k-step s+1 are read from LDS while the MFMAs of
  // step s run
  constexpr int NKS = BK / F::KT;
  static_assert(NKS % 2 == 0, "even number of k-steps per tile");
  T af[2][FM], bf[2][FN];
  auto read_frag = [&](int slot, const T* as, const T* bs, int ks) {
#pragma unroll
    for (int i = 0; i < FM; ++i) af[slot][i] = as[(ks + lane / F::MT) * LDA + wm + i * F::MT + lane % F::MT];
#pragma unroll
    for (int j = 0; j < FN; ++j) bf[slot][j] = bs[(ks + lane / F::NT) * LDB + wn + j * F::NT + lane % F::NT];
  };
  auto mma = [&](int slot) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = F::mma(af[slot][i], bf[slot][j], acc[i][j]);
  };

  // Pipeline per tile t (one barrier): the MFMAs read tile t from LDS buffer t&1; at the start of the tile,
  // tile t+1 (in registers since the start of tile t-1) is staged into the other buffer, whose last reads ended
  // at the previous barrier, and tile t+2 is loaded into registers, a whole tile ahead of its use. The barrier
  // sits before the last k-step, after which the first fragments of tile t+1 are read. FULL: tiles t+1 and t+2
  // exist and t+1 is complete (the steady state, without branches).
  auto tile = [&](auto full_tag, int64_t kt, int buf) {
    constexpr bool FULL = decltype(full_tag)::value;
    const T* as = As[buf];
    const T* bs = Bs[buf];
    if (FULL) {
      // the staging and the global reads stay in the first k-step's scheduling region (the fence keeps the
      // compiler from sinking the reads towards the end of the tile, which would shorten their lead)
      read_frag(1, as, bs, F::KT);
      mma(0);
      la.template store<LDA, false>(As[buf ^ 1], kt + BK, ke);
      lb.template store<LDB, false>(Bs[buf ^ 1], kt + BK, ke);
      la.load(kt + 2 * BK, g.K, g.kl, g.kl.sa);
      lb.load(kt + 2 * BK, g.K, g.kl, g.kl.sb);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      if (kt + BK < ke) {
        la.template store_tile<LDA>(As[buf ^ 1], kt + BK, ke);
        lb.template store_tile<LDB>(Bs[buf ^ 1], kt + BK, ke);
        if (kt + 2 * BK < ke) {
          la.load(kt + 2 * BK, g.K, g.kl, g.kl.sa);
          lb.load(kt + 2 * BK, g.K, g.kl, g.kl.sb);
        }
      }
      read_frag(1, as, bs, F::KT);
      mma(0);
    }
#pragma unroll
    for (int ks = 1; ks + 1 < NKS; ++ks) {
      read_frag((ks + 1) & 1, as, bs, (ks + 1) * F::KT);
      mma(ks & 1);
    }
    __syncthreads();
    if (FULL || kt + BK < ke) read_frag(0, As[buf ^ 1], Bs[buf ^ 1], 0);
    mma((NKS - 1) & 1);
  };

  if (kb < ke) {
    la.load(kb, g.K, g.kl, g.kl.sa);
    lb.load(kb, g.K, g.kl, g.kl.sb);
    la.template store_tile<LDA>(As[0], kb, ke);
    lb.template store_tile<LDB>(Bs[0], kb, ke);
    if (kb + BK < ke) {
      la.load(kb + BK, g.K, g.kl, g.kl.sa);
      lb.load(kb + BK, g.K, g.kl, g.kl.sb);
    }
  }
  __syncthreads();
  if (kb < ke) read_frag(0, As[0], Bs[0], 0);
  int64_t kt = kb;
  int buf = 0;
  for (; kt + 2 * BK < ke; kt += BK, buf ^= 1) tile(std::true_type{}, kt, buf);
  for (; kt < ke; kt += BK, buf ^= 1) tile(std::false_type{}, kt, buf);

  // epilogue
  if (g.split) {
    T* P = static_cast<T*>(g.partial[grp]) + (int64_t)blockIdx.z * g.M * g.N;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < F::NACC; ++r) {
          int64_t row = m0 + wm + i * F::MT + F::row(lane, r);
          int64_t col = n0 + wn + j * F::NT + F::col(lane);
          if (row < g.M && col < g.N) P[row * g.N + col] = acc[i][j][r];
        }
    return;
  }
  T* __restrict__ C = static_cast<T*>(g.C[grp]);
  const T alpha = T(g.alpha), beta = T(g.beta);
  // table lookups first (padded: always in range), then the masked stores
  int64_t cn[FN];
  bool cv[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int64_t col = n0 + wn + j * F::NT + F::col(lane);
    cn[j] = g.c_n[col];
    cv[j] = col < g.N;
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    int64_t cm[F::NACC];
    bool rv[F::NACC];
#pragma unroll
    for (int r = 0; r < F::NACC; ++r) {
      const int64_t row = m0 + wm + i * F::MT + F::row(lane, r);
      cm[r] = g.c_m[row];
      rv[r] = row < g.M;
    }
    if (g.beta != 0.0) {
      // per MFMA block, all reads of C first, unconditionally (padded table entries address element 0 of a
      // valid row or column), so they are in flight together; then the masked read-modify-write stores
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        T cold[F::NACC];
#pragma unroll
        for (int r = 0; r < F::NACC; ++r) cold[r] = C[cm[r] + cn[j]];
#pragma unroll
        for (int r = 0; r < F::NACC; ++r)
          if (cv[j] && rv[r]) C[cm[r] + cn[j]] = alpha * acc[i][j][r] + beta * cold[r];
      }
    } else {
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < F::NACC; ++r)
          if (cv[j] && rv[r]) C[cm[r] + cn[j]] = alpha * acc[i][j][r];
    }
  }
}

// ---- split-bf16 (hi + lo) form with scalar loads: C ~= A_hi B_hi + A_hi B_lo + A_lo B_hi on the bf16 MFMA (operands
// of 128 and more in both extents run on gett_split_device.h) -----------------------------------------------------

__device__ inline void split_bf16(float x, __bf16& hi, __bf16& lo) {
  hi = (__bf16)x;
  lo = (__bf16)(x - (float)hi);
}

// Epilogue of the split-bf16 kernel: 16 x 16 accumulator blocks (acc[i] -> row 4 (lane / 16) + i, col lane % 16),
// written as split-K partials or as C = alpha acc + beta C through the C offset tables.
template <int FM, int FN>
__device__ inline void bf16x3_epilogue(const Args& g, const f32x4 (&acc)[FM][FN], int64_t m0, int64_t n0, int wm,
                                       int wn, int lane, int grp) {
  if (g.split) {
    float* P = static_cast<float*>(g.partial[grp]) + (int64_t)blockIdx.z * g.M * g.N;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          int64_t row = m0 + wm + i * 16 + 4 * (lane >> 4) + r;
          int64_t col = n0 + wn + j * 16 + (lane & 15);
          if (row < g.M && col < g.N) P[row * g.N + col] = acc[i][j][r];
        }
    return;
  }
  float* __restrict__ C = static_cast<float*>(g.C[grp]);
  const float alpha = float(g.alpha), beta = float(g.beta);
  int64_t cn[FN];
  bool cv[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int64_t col = n0 + wn + j * 16 + (lane & 15);
    cn[j] = g.c_n[col];
    cv[j] = col < g.N;
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    int64_t cm[4];
    bool rv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = m0 + wm + i * 16 + 4 * (lane >> 4) + r;
      cm[r] = g.c_m[row];
      rv[r] = row < g.M;
    }
    float cold[FN][4];
    if (g.beta != 0.0) {
      // unconditional reads first (padded table entries address a valid element), then the masked stores
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) cold[j][r] = C[cm[r] + cn[j]];
    }
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (cv[j] && rv[r]) {
          float v = alpha * acc[i][j][r];
          if (g.beta != 0.0) v += beta * cold[j][r];
          C[cm[r] + cn[j]] = v;
        }
  }
}

// FP32 tiles are split into bf16 hi and lo planes when staged in LDS. Each plane is stored row-major with k
// contiguous (row pitch BK + 8 bf16 = 80 bytes), so a lane's 8-element MFMA fragment is one 16-byte LDS read.
template <int BM, int BN, int BK, bool AKF, bool BKF, int NKL>
__global__ void __launch_bounds__(256) gett_bf16x3_kernel(Args g) {
  static_assert(BK == 32, "one bf16 MFMA step per tile");
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int FM = WM / 16, FN = WN / 16;
  constexpr int LDK = BK + 8;
  __shared__ __attribute__((aligned(16))) __bf16 Ah[BM * LDK];
  __shared__ __attribute__((aligned(16))) __bf16 Al[BM * LDK];
  __shared__ __attribute__((aligned(16))) __bf16 Bh[BN * LDK];
  __shared__ __attribute__((aligned(16))) __bf16 Bl[BN * LDK];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = (wave >> 1) * WM;
  const int wn = (wave & 1) * WN;
  int64_t m0, n0;
  tile_origin<BM, BN>(xcd_tile(blockIdx.x, gridDim.x), g.M, g.N, m0, n0);
  const int64_t kb = (int64_t)blockIdx.z * g.kchunk;
  const int64_t ke = (g.K < kb + g.kchunk) ? g.K : kb + g.kchunk;
  const int grp = blockIdx.y;
  const float* __restrict__ A = static_cast<const float*>(g.A[grp]);
  const float* __restrict__ B = static_cast<const float*>(g.B[grp]);

  Loader<float, BM, BK, AKF, NKL> la;
  Loader<float, BN, BK, BKF, NKL> lb;
  la.init(A, g.a_m, m0, tid);
  lb.init(B, g.b_n, n0, tid);

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  if (kb < ke) {
    la.load(kb, g.K, g.kl, g.kl.sa);
    lb.load(kb, g.K, g.kl, g.kl.sb);
  }
  const int kq = 8 * (lane >> 4);
  for (int64_t kt = kb; kt < ke; kt += BK) {
#pragma unroll
    for (int i = 0; i < la.PER; ++i) {
      __bf16 h, l;
      split_bf16(la.template value<true>(i, kt, ke), h, l);
      const int r = la.r0 + (i % la.NR) * la.RSTEP, k = la.k0 + (i / la.NR) * la.KSTEP;
      Ah[r * LDK + k] = h;
      Al[r * LDK + k] = l;
    }
#pragma unroll
    for (int i = 0; i < lb.PER; ++i) {
      __bf16 h, l;
      split_bf16(lb.template value<true>(i, kt, ke), h, l);
      const int r = lb.r0 + (i % lb.NR) * lb.RSTEP, k = lb.k0 + (i / lb.NR) * lb.KSTEP;
      Bh[r * LDK + k] = h;
      Bl[r * LDK + k] = l;
    }
    __syncthreads();
    if (kt + BK < ke) {
      la.load(kt + BK, g.K, g.kl, g.kl.sa);
      lb.load(kt + BK, g.K, g.kl, g.kl.sb);
    }
    bf16x8 bh[FN], bl[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int c = (wn + j * 16 + (lane & 15)) * LDK + kq;
      bh[j] = *reinterpret_cast<const bf16x8*>(&Bh[c]);
      bl[j] = *reinterpret_cast<const bf16x8*>(&Bl[c]);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int r = (wm + i * 16 + (lane & 15)) * LDK + kq;
      const bf16x8 ah = *reinterpret_cast<const bf16x8*>(&Ah[r]);
      const bf16x8 al = *reinterpret_cast<const bf16x8*>(&Al[r]);
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[j], acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[j], acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[j], acc[i][j], 0, 0, 0);
      }
    }
    __syncthreads();
  }

  bf16x3_epilogue<FM, FN>(g, acc, m0, n0, wm, wn, lane, grp);
}

struct RedArgs {
  const void* P[kGettMaxGroup];
  void* C[kGettMaxGroup];
};

template <typename T>
__global__ void splitk_reduce_kernel(RedArgs r, int splits, int64_t M, int64_t N, const int64_t* __restrict__ c_m,
                                     const int64_t* __restrict__ c_n, double alpha, double beta) {
  const T* __restrict__ P = static_cast<const T*>(r.P[blockIdx.y]);
  T* C = static_cast<T*>(r.C[blockIdx.y]);
  const int64_t total = M * N;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int z = 0; z < splits; ++z) s += (double)P[(int64_t)z * total + idx];
    int64_t m = idx / N, n = idx - m * N;
    int64_t o = c_m[m] + c_n[n];
    double v = alpha * s;
    if (beta != 0.0) v += beta * (double)C[o];
    C[o] = (T)v;
  }
}

template <typename T, int BM, int BN, int BK, int NKL, bool VEC>
void launch_tile_k(const Args& a, dim3 grid, hipStream_t s, bool akf, bool bkf) {
  const dim3 block(256);
  if (akf && bkf) hipLaunchKernelGGL((gett_kernel<T, BM, BN, BK, true, true, NKL, VEC>), grid, block, 0, s, a);
  else if (akf) hipLaunchKernelGGL((gett_kernel<T, BM, BN, BK, true, false, NKL, VEC>), grid, block, 0, s, a);
  else if (bkf) hipLaunchKernelGGL((gett_kernel<T, BM, BN, BK, false, true, NKL, VEC>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gett_kernel<T, BM, BN, BK, false, false, NKL, VEC>), grid, block, 0, s, a);
}

// Kernels are instantiated for 2 and for 4 contracted legs (fewer legs run with zero entries), with scalar or
// vector tile loads.
template <typename T, int BM, int BN, int BK>
void launch_tile(const Args& a, int groups, int splits, hipStream_t s, bool akf, bool bkf, bool vec) {
  const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const dim3 grid((unsigned)tiles, (unsigned)groups, (unsigned)splits);
  if (vec) {
    if (a.kl.n <= 2) launch_tile_k<T, BM, BN, BK, 2, true>(a, grid, s, akf, bkf);
    else launch_tile_k<T, BM, BN, BK, 4, true>(a, grid, s, akf, bkf);
  } else {
    if (a.kl.n <= 2) launch_tile_k<T, BM, BN, BK, 2, false>(a, grid, s, akf, bkf);
    else launch_tile_k<T, BM, BN, BK, 4, false>(a, grid, s, akf, bkf);
  }
}

template <int BM, int BN, int BK, int NKL>
void launch_bf16x3_k(const Args& a, dim3 grid, hipStream_t s, bool akf, bool bkf) {
  const dim3 block(256);
  if (akf && bkf) hipLaunchKernelGGL((gett_bf16x3_kernel<BM, BN, BK, true, true, NKL>), grid, block, 0, s, a);
  else if (akf) hipLaunchKernelGGL((gett_bf16x3_kernel<BM, BN, BK, true, false, NKL>), grid, block, 0, s, a);
  else if (bkf) hipLaunchKernelGGL((gett_bf16x3_kernel<BM, BN, BK, false, true, NKL>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gett_bf16x3_kernel<BM, BN, BK, false, false, NKL>), grid, block, 0, s, a);
}

template <int BM, int BN, int BK>
void launch_bf16x3(const Args& a, int groups, int splits, hipStream_t s, bool akf, bool bkf) {
  const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const dim3 grid((unsigned)tiles, (unsigned)groups, (unsigned)splits);
  if (a.kl.n <= 2) launch_bf16x3_k<BM, BN, BK, 2>(a, grid, s, akf, bkf);
  else launch_bf16x3_k<BM, BN, BK, 4>(a, grid, s, akf, bkf);
}

struct Tile {
  int bm, bn;
};

int64_t rup(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Tile shape per precision and extents. FP64: 128 x 64 (the 128 x 128 FP64 tile gives no gain at its lower
// occupancy). FP32 matrix instructions: among 192 x 192, 128 x 192, 192 x 128 and 128 x 128 the one with the least
// padding, ties to the larger tile; chi^2 = 576 and chi^4 extents at chi = 24 are multiples of 192 but not of 128.
// The split kernels (`planes` > 0) the same, the FP32 form (three planes) without the 192 x 192 tile, whose second
// sums and fragments do not fit the registers (spilling, it ran 159 TFLOP/s against 171 with 128 x 192), and with
// 128 x 128 only (`only128`) where an operand is walked along k without 16-byte loads. A 192-row (column) tile is only
// chosen when it pads no more than a 128-row one, so the offset tables, padded to multiples of 128, cover every tile.
// 64-wide tiles for extents below 128 (split-bf16: scalar loads).
Tile choose_tile(Prec p, int64_t M, int64_t N, int planes, bool only128) {
  const bool bigm = M >= 128, bign = N >= 128;
  if (p == Prec::F64) return Tile{bigm ? 128 : 64, 64};
  if (!bigm || !bign || only128) return Tile{bigm ? 128 : 64, bign ? 128 : 64};
  const Tile cand[4] = {{192, 192}, {128, 192}, {192, 128}, {128, 128}};
  Tile best = cand[3];
  double best_pad = 1e300;
  for (const Tile& c : cand) {
    if (planes == 3 && c.bm + c.bn == 384) continue;
    if (rup(M, c.bm) > rup(M, 128) || rup(N, c.bn) > rup(N, 128)) continue;
    const double pad = (double)rup(M, c.bm) * (double)rup(N, c.bn);
    if (pad < best_pad * (1 - 1e-12)) {
      best = c;
      best_pad = pad;
    }
  }
  return best;
}

// Estimated microseconds of `tiles` output tiles in `splits` k ranges: rounds of 512 workgroups (two per CU; up to 256
// more, alone on their CUs, take three quarters of a round) at `rate` flop/us over the chip, and, if split, writing and
// adding the partial sums (0.4 us per MB) in a second launch. Fitted to 2000 timings of the programs' contractions at
// chi = 4 .. 20, within 15 % at the median. Filling whole rounds is what it is for: FP32 20736 x 144 x 1728 (162 tiles)
// 128 us in two ranges, 105 in three; the 324 tiles of the isometry derivative at chi = 24 in 4 ranges fill 2.5 rounds.
double split_cost(int64_t tiles, int splits, const GettTables& t, const Tile& tile, double rate, size_t eb) {
  const int64_t blocks = tiles * splits, rem = blocks % 512;
  const double rounds = (double)(blocks / 512) + (rem == 0 ? 0.0 : rem <= 256 ? 0.75 : 1.0);
  const double kc = (double)rup((t.K + splits - 1) / splits, 32);
  const double red = splits > 1 ? 9.5 + 0.4e-6 * splits * (double)t.M * (double)t.N * (double)eb : 0.0;
  return rounds * kc * 2.0 * tile.bm * tile.bn * 512 / rate + red;
}

}  // namespace

void gett_run(Ctx& ctx, const GettTables& t, const GettLaunch& l) {
  if (t.M <= 0 || t.N <= 0) return;
  const int G = l.groups;
  if (G < 1 || G > kGettMaxGroup) throw Error(MERA_EINVAL, "gett: group count out of range");
  Args a{};
  for (int g = 0; g < G; ++g) {
    a.A[g] = l.A[g];
    a.B[g] = l.B[g];
    a.C[g] = l.C[g];
  }
  a.a_m = t.a_m;
  a.b_n = t.b_n;
  a.kl = t.kl;
  a.c_m = t.c_m;
  a.c_n = t.c_n;
  a.M = t.M;
  a.N = t.N;
  a.K = t.K;
  a.alpha = l.alpha;
  a.beta = l.beta;
  a.split = 0;

  // Kernel, tile, order of the k's and split-K follow from what the layouts allow (planned); where the bases lie only decides
  // whether vectors are loaded whole or by elements, for all sets of the launch. An operand set thus gets the same bits
  // wherever its tensors lie and whatever else is in the group.
  const int vw = l.prec == Prec::F64 ? 2 : 4;
  const bool a_vec = t.a_vw >= vw, b_vec = t.b_vw >= vw;
  bool a16 = a_vec, b16 = b_vec;  // 16-byte loads: the layout allows them and every base is aligned
  for (int g = 0; g < G; ++g) {
    a16 = a16 && (uintptr_t)l.A[g] % 16 == 0;
    b16 = b16 && (uintptr_t)l.B[g] % 16 == 0;
  }
  bool plan_vec = a_vec && b_vec;  // tile loads move vectors when both operands allow it
  // FP32 operands with extents of 128 and more run on the bf16 matrix cores from split operands: three planes for the
  // FP32 form (chi^9 steps at chi = 24: 172 TFLOP/s against 127 on the FP32 instructions), two for the split-bf16 form.
  // Below 128 rows or columns a launch is bound by latency and the FP32 tiles stay. Below kSplitMinK a step is bound by
  // writing C and both are alike (ternary maps at chi = 16 .. 32, whose composites have K = chi: 739 / 731, 3537 / 3507,
  // 9803 / 9795, 86792 / 87555 us native / split): the FP32 instructions stay, whose 192 x 192 tile reads less. With
  // vector loads a row-walking operand's pair of k's must not straddle two values of the next contracted leg: even
  // extent; every other layout (chi not a multiple of 4) is loaded by elements.
  constexpr int64_t kSplitMinK = 64;
  const bool split_form = t.M >= 128 && t.N >= 128 &&
                          (l.prec == Prec::BF16X3 || (l.prec == Prec::F32 && t.K >= kSplitMinK));
  const int planes = !split_form ? 0 : l.prec == Prec::F32 ? 3 : 2;
  if (planes > 0) plan_vec = plan_vec && t.kl.n >= 1 && t.kl.ext[0] % 2 == 0;
  else if (l.prec == Prec::BF16X3) plan_vec = false;
  const bool vec = plan_vec && a16 && b16;

  Tile tile = choose_tile(l.prec, t.M, t.N, planes, planes == 3 && !plan_vec && (t.a_kfast || t.b_kfast));
  // Small launches: 32 x 32 tiles straight from global memory (gett_direct.hip) where the LDS tiles would leave half of
  // the 256 CUs idle and the work is small. Over the 500 contractions of the binary and ternary programs at chi = 4 .. 20
  // this line is 30 % faster on the (geometric) average than the LDS tiles with their best split, 3 % short of the better
  // kernel each time. Beyond it the LDS tiles' reuse wins: FP64 10000 x 100 x 100 (158 tiles) 19.6 / 20.8 us LDS / direct,
  // 20736 x 144 x 144 (486 tiles) 34 / 49 us; this side of it 144 x 144 x 20736 (6 tiles) 73 / 49 us, FP32
  // 20 x 8000 x 8000 (63 tiles) 117 / 78 us. Where each k is loaded by itself (the fastest contracted leg no multiple
  // of 4, or a k-walking operand whose layout allows no 16-byte loads) the line lies lower: FP64 81 x 729 x 6561
  // (0.77 GFLOP) 44 / 74 us, 121 x 121 x 14641 (0.43) 47 / 26 us. Large FP32 outputs from few k's stay with the LDS tiles, which write whole
  // lines (4096 x 4096 x 16 25 / 59 us); by time alone that line would lie at 4 million elements (1728 x 1728 x 12
  // 17 / 13 us, 1728 x 144 x 12 15 / 5 us), but the tests of the chi = 12 evaluation ask for the 192 x 192 tile, whose
  // launches there have 250 thousand.
  const bool k4 = t.kl.n >= 1 && t.kl.ext[0] % 4 == 0 && (a_vec || !t.a_kfast) && (b_vec || !t.b_kfast);
  const bool direct = 2.0 * (double)t.M * (double)t.N * (double)t.K < (k4 ? 3e9 : 5e8) &&
                      ((t.M + tile.bm - 1) / tile.bm) * ((t.N + tile.bn - 1) / tile.bn) < 128 &&
                      !(l.prec == Prec::F32 && plan_vec && t.M >= 128 && t.N >= 128 && t.K < kSplitMinK && t.M * t.N >= 200000);
  if (direct) tile = Tile{kDirectTile, kDirectTile};
  const int BMsel = tile.bm, BNsel = tile.bn;
  // the m and n offset tables are padded to multiples of 128; every tile must lie within them
  if (rup(t.M, BMsel) > rup(t.M, 128) || rup(t.N, BNsel) > rup(t.N, 128))
    throw Error(MERA_EINVAL, "gett: tile exceeds the padded offset tables");
  const int64_t tiles = ((t.M + BMsel - 1) / BMsel) * ((t.N + BNsel - 1) / BNsel);
  const int BK = 32;  // k-chunks stay multiples of every tile depth in use

  // Direct tiles: eight waves share k while there is no more than one workgroup per CU (144^3 FP64 7.2 us with four
  // waves, 6.4 with eight; 6561 x 81 x 81, 618 tiles, 13.0 and 14.4)
  const int waves = tiles <= 256 ? 8 : 4;

  // Split-K. Direct tiles: up to one workgroup per CU, only from K > 512 on, below which the second launch costs more
  // than the shorter chains give (FP64 256^3 9.5 us whole, 11.9 in two; 36 x 36 x 1296 28 us whole, 12 in nine). LDS
  // tiles: the factor of least estimated time, see split_cost.
  const size_t eb = (l.prec == Prec::F64) ? 8 : 4;
  int splits = l.splits;
  if (splits <= 0) {
    splits = 1;
    if (direct && t.K > 512) {
      splits = (int)std::max<int64_t>(1, std::min<int64_t>(256 / tiles, t.K / (kDirectChunk * waves)));
    } else if (!direct && t.K >= 512 && tiles < 1024) {
      const double rate = l.prec == Prec::F64 ? 57e6 : planes == 3 ? 170e6 : planes == 2 ? 310e6 : 90e6;
      double best = split_cost(tiles, 1, t, tile, rate, eb);
      for (int z = 2; z <= 64 && tiles * z <= 8192 && t.K / z >= 256; ++z) {
        const double c = split_cost(tiles, z, t, tile, rate, eb);
        if (c < 0.98 * best) {
          best = c;
          splits = z;
        }
      }
    }
  }
  int64_t kchunk = (t.K + splits - 1) / splits;
  kchunk = ((kchunk + BK - 1) / BK) * BK;
  splits = (int)std::max<int64_t>(1, (t.K + kchunk - 1) / kchunk);
  a.kchunk = kchunk;

  if (splits > 1) {
    const size_t per = (size_t)splits * t.M * t.N * eb;
    char* p = static_cast<char*>(ctx.buf("gett.partial", per * G));
    for (int g = 0; g < G; ++g) a.partial[g] = p + per * g;
    a.split = 1;
  }
  if (l.prepare_only) return;
  // the split kernels of three planes walk k without 16-byte loads in 128 x 128 tiles only: same sums, smaller tiles
  if (planes == 3 && !direct && !vec && (t.a_kfast || t.b_kfast)) tile = Tile{128, 128};
  hipStream_t s = ctx.stream;
  LaunchRecord rec;
  if (ctx.profiling) {
    rec.kernel = std::string("gett<") + (l.prec == Prec::F64 ? "f64" : (l.prec == Prec::F32 ? "f32" : "bf16x3")) +
                 "," + std::to_string(tile.bm) + "x" + std::to_string(tile.bn) + (t.a_kfast ? ",Ak" : ",Am") +
                 (t.b_kfast ? ",Bk" : ",Bn") + (direct ? ",d" : vec ? ",v" : "") + (t.kl.n <= 2 ? ",k2" : ",k4") +
                 (direct ? "" : planes == 3 ? ",s3" : planes == 2 ? ",s2" : "") +
                 (splits > 1 ? ",splitk" : "") + (G > 1 ? ",grouped" : "") + ">";
    rec.flops = 2.0 * G * (double)t.M * (double)t.N * (double)t.K;
    rec.bytes = G * (double)eb * ((double)t.M * t.K + (double)t.K * t.N + (double)t.M * t.N * (l.beta != 0.0 ? 2 : 1));
    rec.start = ctx.take_event();
    rec.stop = ctx.take_event();
    MERA_HIP(hipEventRecord(rec.start, s));
  }
  const int sel = tile.bm * 1000 + tile.bn;
  const bool akf = t.a_kfast, bkf = t.b_kfast;

  if (direct) {
    launch_gett_direct(a, G, splits, s, l.prec, waves, (akf && a_vec) || (bkf && b_vec), akf && a16, bkf && b16);
  } else if (planes > 0) {
    (vec ? launch_gett_split : launch_gett_split_scalar)(a, G, splits, s, akf, bkf, tile.bm, tile.bn, planes);
  } else if (l.prec == Prec::F64) {
    if (sel == 128064) launch_tile<double, 128, 64, 16>(a, G, splits, s, akf, bkf, vec);
    else launch_tile<double, 64, 64, 16>(a, G, splits, s, akf, bkf, vec);
  } else if (l.prec == Prec::F32) {
    switch (sel) {
      case 192192: launch_tile<float, 192, 192, 16>(a, G, splits, s, akf, bkf, vec); break;
      case 128192: launch_tile<float, 128, 192, 16>(a, G, splits, s, akf, bkf, vec); break;
      case 192128: launch_tile<float, 192, 128, 16>(a, G, splits, s, akf, bkf, vec); break;
      case 128128: launch_tile<float, 128, 128, 16>(a, G, splits, s, akf, bkf, vec); break;
      case 128064: launch_tile<float, 128, 64, 16>(a, G, splits, s, akf, bkf, vec); break;
      case 64128: launch_tile<float, 64, 128, 16>(a, G, splits, s, akf, bkf, vec); break;
      default: launch_tile<float, 64, 64, 16>(a, G, splits, s, akf, bkf, vec); break;
    }
  } else {
    switch (sel) {
      case 128064: launch_bf16x3<128, 64, 32>(a, G, splits, s, akf, bkf); break;
      case 64128: launch_bf16x3<64, 128, 32>(a, G, splits, s, akf, bkf); break;
      default: launch_bf16x3<64, 64, 32>(a, G, splits, s, akf, bkf); break;
    }
  }
  MERA_HIP(hipGetLastError());
  if (ctx.profiling) {
    MERA_HIP(hipEventRecord(rec.stop, s));
    ctx.records.push_back(rec);
  }
  if (splits > 1) {
    RedArgs r{};
    for (int g = 0; g < G; ++g) {
      r.P[g] = a.partial[g];
      r.C[g] = l.C[g];
    }
    const int64_t total = t.M * t.N;
    int blocks = (int)std::min<int64_t>((total + 255) / 256, 4096);
    if (l.prec == Prec::F64)
      hipLaunchKernelGGL(splitk_reduce_kernel<double>, dim3(blocks, G), dim3(256), 0, s, r, splits, t.M, t.N, t.c_m,
                         t.c_n, l.alpha, l.beta);
    else
      hipLaunchKernelGGL(splitk_reduce_kernel<float>, dim3(blocks, G), dim3(256), 0, s, r, splits, t.M, t.N, t.c_m,
                         t.c_n, l.alpha, l.beta);
    MERA_HIP(hipGetLastError());
  }
}

}  // namespace mera
