// How the waves of a workgroup walk the columns of their rows in the products
// for up to 16 tokens.  Plain integer arithmetic, shared with a host-side check.
// A workgroup counts columns from its first one on and holds at most 2^31 of
// them (longer rows are always split), so no sum here wraps.
#pragma once
#include <cstdint>

#if defined(__HIP__)
#define DF11_HD __host__ __device__ __forceinline__
#else
#define DF11_HD inline
#endif

namespace df11gemm {

constexpr uint32_t kRowsWaves = 4;    // waves of a workgroup
constexpr uint32_t kSlabCols = 256;   // columns a wave takes at a time
constexpr uint32_t kRangeCols = 1024; // longest range, summed from zero

// Range of one wave: 1024 columns, or a quarter of the row where that is
// shorter (in whole slabs), so that every wave has one.
DF11_HD uint32_t rows_range(uint32_t cols) {
    constexpr uint32_t kAll = kRowsWaves * kSlabCols;
    const uint32_t quarter = (cols / kAll + (cols % kAll ? 1u : 0u)) * kSlabCols;
    return quarter < kRangeCols ? quarter : kRangeCols;
}

// Fewest workgroups that a row of `cols` columns is split over.
DF11_HD uint32_t least_ranges(uint32_t cols) { return cols > 0x80000000u ? 2u : 1u; }

// First column past `n` from `at` on, at most `end` (at <= end).
DF11_HD uint32_t past(uint32_t at, uint32_t n, uint32_t end) { return end - at > n ? at + n : end; }

// The slab [k, min(k + 256, k1)) of the range [k0, k1).
struct Slab {
    uint32_t k0, k1, k;
};

// The wave's first slab of [0, end); false when it has none.
DF11_HD bool first_slab(uint32_t end, uint32_t range, uint32_t wave, Slab *s) {
    s->k0 = s->k = wave * range;
    s->k1 = s->k0 + range < end ? s->k0 + range : end;
    return s->k0 < end;
}

// The range ends with this slab.
DF11_HD bool last_of_range(const Slab &s) { return s.k + kSlabCols >= s.k1; }

// The slab after s: in the range, or the first one of the wave's next range;
// false when there is none.
DF11_HD bool next_slab(uint32_t end, uint32_t range, const Slab &s, Slab *n) {
    const bool turn = last_of_range(s);
    n->k0 = turn ? s.k0 + kRowsWaves * range : s.k0;
    n->k = turn ? n->k0 : s.k + kSlabCols;
    n->k1 = n->k0 + range < end ? n->k0 + range : end;
    return n->k < end;
}

}  // namespace df11gemm
