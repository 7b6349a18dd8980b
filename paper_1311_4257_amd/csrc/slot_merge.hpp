// The terms of a tile of the slot form for few right-hand sides (device code).
//
// A tile's 16 columns are (group, rhs) of neighbouring groups, and it walks the
// union of their terms, so that an operator is read and multiplied once for all of
// its groups that use it.  Every wave merges the groups' term lists as it goes: a
// lane holds its column's next term, the least key over the columns is the tile's,
// and the columns that hold it move on by one.  Lists merged ahead of the launches
// (80 bytes per merged term, one set per number of right-hand sides) had to be made,
// allocated and copied by the first apply: 3.4 ms for the first, 1.24 for the later
// ones on an adaptive K = 8 sphere of 65,536 points at one right-hand side, against
// 1.6 and 1.25 so; the same from 4 right-hand sides.
#pragma once

#include <hip/hip_runtime.h>

namespace dfmm {
namespace {

// Smallest of a row of 16 lanes, in all of them.
__device__ __forceinline__ unsigned row_min(unsigned v) {
#define DFMM_ROR(n) v = min(v, unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x120 + n, 0xF, 0xF, false)))
  DFMM_ROR(8);
  DFMM_ROR(4);
  DFMM_ROR(2);
  DFMM_ROR(1);
#undef DFMM_ROR
  return v;
}

struct TileTerm {
  bool any;  // false: past the last term
  int aoff;  // operator offset
  int K;     // its columns
  int kind;
  int src;   // source vector of column lane mod 16, -1: the column has no such term
};

// All waves of a workgroup see the same terms; the four rows of 16 lanes of a wave
// hold the same columns.  The lists are copied to LDS first: read from memory as
// they are walked, 16 lists of one tile missed the caches about every other term,
// and the next operator rows came in behind those loads (2% of that pass).
struct TileTerms {
  const int2* at;       // the column's next term in LDS: (source slot, key), key kNone past its last
  int2 v;               // that term
  int rhs, nrhs, lead;  // lead: the kind that the lists start with
  int out;              // output vector of the column (-1: none)
  int Mg;               // padded rows of the tile's groups
  // rec: the tile's records, one per group; for all waves of the workgroup
  __device__ __forceinline__ TileTerms(const int4* __restrict__ rec, int per, const int4* __restrict__ terms, int nrhs_,
                                       int lead_, int2* lds)
      : nrhs(nrhs_), lead(lead_) {
    const int j = int(threadIdx.x) & 15, c = j / nrhs;
    rhs = j - c * nrhs;
    // (first term, end, output vector or -1, padded rows | place in the lists << 12)
    const int4 r = rec[min(c, per - 1)];
    const bool has = c < per && r.z >= 0;
    Mg = __builtin_amdgcn_readfirstlane(r.w) & 0xFFF;
    out = has ? r.z * nrhs + rhs : -1;
    const int n = r.y - r.x;
    int2* const mine = lds + (r.w >> 12);
    at = has ? mine : mine + n;
    if (c < per && rhs == 0) {  // the rows of 16 lanes take a column's terms in turn
      const int row = int(threadIdx.x) >> 4, nrow = int(blockDim.x) >> 4;
      constexpr int UL = 4;  // terms in flight
      for (int i = row; i <= n; i += UL * nrow) {
        int2 w[UL];
#pragma unroll
        for (int u = 0; u < UL; ++u) {
          w[u] = make_int2(0, int(kNone));
          if (i + u * nrow < n) w[u] = reinterpret_cast<const int2*>(terms + r.x + i + u * nrow)[1];
        }
#pragma unroll
        for (int u = 0; u < UL; ++u)
          if (i + u * nrow <= n) mine[i + u * nrow] = w[u];
      }
    }
    __syncthreads();
    v = *at;
  }
  __device__ __forceinline__ TileTerm next() {
    const unsigned key = unsigned(v.y), k = unsigned(__builtin_amdgcn_readfirstlane(int(row_min(key))));
    TileTerm t;
    t.any = k != kNone;
    const bool mine = t.any && key == k;
    t.K = int(k % 32u + 1u) * 8;
    t.aoff = int(k & 0x7FFFFFE0u);
    t.kind = int(k >> 31) ^ lead;
    t.src = mine ? v.x * nrhs + rhs : -1;
    at += mine ? 1 : 0;  // columns that hold the term move on
    v = *at;
    return t;
  }

 private:
  static constexpr unsigned kNone = 0xFFFFFFFFu;
};

}  // namespace
}  // namespace dfmm
