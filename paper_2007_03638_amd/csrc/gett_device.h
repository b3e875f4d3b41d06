// Device-side pieces shared by the GETT kernels: launch arguments, k offsets, the workgroup-to-tile map.
#pragma once

#include "gett.h"

namespace mera {

// One launch runs the same contraction (same tables and extents) for up to kGettMaxGroup independent operand
// sets; blockIdx.y selects the set.
struct GettArgs {
  const void* A[kGettMaxGroup];
  const void* B[kGettMaxGroup];
  void* C[kGettMaxGroup];
  void* partial[kGettMaxGroup];  // splits x M x N partial sums per set (accumulator type); used when split != 0
  const int64_t* a_m;
  const int64_t* b_n;
  const int64_t* c_m;
  const int64_t* c_n;
  GettKLegs kl;
  int64_t M, N, K;
  int64_t kchunk;  // K range per split, a multiple of BK
  double alpha, beta;
  int split;       // 1: write partial sums, 0: write C
};

// Offset of the k-th index along the contracted legs (fastest leg first; see GettKLegs): NKL digit extractions
// by reciprocal multiplication, no memory access. Entries past kl.n are zero and contribute nothing.
template <int NKL>
__device__ inline uint64_t k_offset(uint32_t k, const GettKLegs& kl, const uint32_t* stride) {
  uint64_t off = 0;
  uint32_t q = k;
#pragma unroll
  for (int l = 0; l + 1 < NKL; ++l) {
    const uint32_t qn = __umulhi(q, kl.mag[l]);
    off += (uint64_t)(q - qn * kl.ext[l]) * stride[l];
    q = qn;
  }
  return off + (uint64_t)q * stride[NKL - 1];
}

// Workgroups are dispatched to the 8 XCDs round-robin (workgroup b runs on XCD b % 8). Remap so that each
// XCD processes a contiguous range of logical tiles: consecutive tiles share an A panel, which then stays in
// that XCD's L2 instead of being fetched by all eight. The tail (ntiles % 8 tiles) keeps the identity map.
__device__ inline int64_t xcd_tile(int64_t b, int64_t ntiles) {
  const int64_t full = ntiles / 8;
  return (b < full * 8) ? (b % 8) * full + b / 8 : b;
}

// Origin of logical tile `tile`. Tiles are taken in groups of kTileGroup panels of the dimension with more tiles
// (the larger operand); within a group that dimension runs fastest, then the other one. The 64 tiles an XCD runs
// at once then cover about 8 panels of each operand, which its L2 serves to all of them: each operand is fetched
// from beyond L2 about (tiles of the other dimension) / kTileGroup times instead of once per tile of the other
// dimension for the smaller operand.
constexpr int64_t kTileGroup = 8;
template <int BM, int BN>
__device__ inline void tile_origin(int64_t tile, int64_t M, int64_t N, int64_t& m0, int64_t& n0) {
  const int64_t tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
  const bool mgroups = tm >= tn;
  const int64_t tbig = mgroups ? tm : tn, tsmall = mgroups ? tn : tm;
  const int64_t grp = tile / (kTileGroup * tsmall), loc = tile % (kTileGroup * tsmall);
  const int64_t gsize = (tbig - grp * kTileGroup < kTileGroup) ? tbig - grp * kTileGroup : kTileGroup;
  const int64_t big = grp * kTileGroup + loc % gsize, small = loc / gsize;
  m0 = (mgroups ? big : small) * BM;
  n0 = (mgroups ? small : big) * BN;
}

// FP32 contraction on the bf16 matrix cores from split operands (gett_split_device.h): planes = 3 (FP32 form) or
// 2 (split-bf16 form); tile bm x bn with bm, bn in {128, 192}. The first needs operands that allow 16-byte loads and an
// even extent of the fastest contracted leg, the second takes any layout.
void launch_gett_split(const GettArgs& a, int groups, int splits, hipStream_t s, bool akf, bool bkf, int bm, int bn,
                       int planes);
void launch_gett_split_scalar(const GettArgs& a, int groups, int splits, hipStream_t s, bool akf, bool bkf, int bm,
                              int bn, int planes);

// Contraction in 32 x 32 tiles read straight from global memory, for launches too small to fill the chip with LDS tiles
// (gett_direct.hip); any layout and alignment. quads: the layout of an operand whose unit-stride leg is a contracted one
// allows 16-byte loads, so the k's are taken in quadruples (this fixes the order of the sums); av, bv: such an operand's
// bases are aligned too, so that it is read that way.
constexpr int kDirectTile = 32, kDirectChunk = 16;
void launch_gett_direct(const GettArgs& a, int groups, int splits, hipStream_t s, Prec prec, int waves, bool quads,
                        bool av, bool bv);

}  // namespace mera
