// Fused decompression and matrix-vector products for one token: the weights
// of a transformer block are decoded on chip (Algorithm 1 of arXiv
// 2504.11651) and multiplied by the activations right away, so the 2 bytes
// per weight of BF16 are never written to memory and read back (the paper
// decompresses each block into a buffer right before its products,
// Sec. 2.3.3; with one token the products are bound by reading weights).
//
// Per 64-chunk block one wavefront decodes exactly as the decode kernel does
// (phase 1, prefix sum, phase 2 into LDS); then, in place of the stores, each
// lane takes its 8-weight groups, assembles the BF16 values, and accumulates
// their dot product with the matching 8 activations (v_dot2c_f32_bf16, fp32
// accumulation).  A block inside one matrix touches at most three of its rows
// (columns >= 2048), so every lane keeps three partial sums; a block at a
// boundary covers at most two matrices.  Wave-wide sums give at most 8
// partial sums per block, written to a workspace.  A second kernel adds, for
// every output row, the partial sums of the blocks that cover it, in a fixed
// order.  The result depends only on the stream and the inputs.
#include <hip/hip_runtime.h>

#include <array>
#include <cstdint>
#include <mutex>
#include <vector>

#include "df11.h"
#include "df11_decode_core.h"
#include "df11_tables.h"

namespace {

using namespace df11dec;

constexpr uint32_t kMaxM = DF11_MAX_MATRICES;
constexpr uint32_t kSegSlots = 4;              // partial sums per matrix segment (3 used)
constexpr uint32_t kSlots = 2 * kSegSlots;     // per block
constexpr uint32_t kMinCols = 2048;            // a block (<= 4096 weights) spans <= 3 rows
constexpr uint32_t kMaxBlockElems = 64u * 64u; // 64 chunks of at most 64 codes

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint64_t umin64(uint64_t a, uint64_t b) { return a < b ? a : b; }

// q = n / d for all 32-bit n, by the round-up multiply-and-shift method for
// division by an invariant integer (Granlund and Montgomery, 1994):
// t = mulhi(n, m), q = (t + ((n - t) >> 1)) >> (l - 1), l = ceil(log2 d).
struct Divider {
    uint32_t magic, shift;  // shift = l - 1
};

__host__ __device__ inline uint32_t divide(uint32_t n, Divider dv) {
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t t = __umulhi(n, dv.magic);
#else
    const uint32_t t = static_cast<uint32_t>((static_cast<uint64_t>(n) * dv.magic) >> 32);
#endif
    return (t + ((n - t) >> 1)) >> dv.shift;
}

Divider make_divider(uint32_t d) {  // d >= 2
    uint32_t l = 0;
    while ((uint64_t{1} << l) < d) ++l;
    const unsigned __int128 num = (static_cast<unsigned __int128>(1) << 32) *
                                  ((uint64_t{1} << l) - d);
    return Divider{static_cast<uint32_t>(num / d + 1), l - 1};
}

struct GemvArgs {
    DecodeArgs d;
    uint32_t n_mats;
    uint32_t off[kMaxM];  // first weight of each matrix (sorted, disjoint)
    uint32_t end[kMaxM];  // one past its last weight
    uint32_t cols[kMaxM];
    Divider div[kMaxM];   // division by cols
    const uint16_t *x[kMaxM];
    uint32_t row_base[kMaxM];  // index of the matrix's first row among all rows
    uint32_t boundary_grid;    // workgroups for the blocks at matrix boundaries
    // where matrices start and end inside the stream, ascending, each position
    // once; and the first matrix that a block around it can touch (a matrix is
    // at least as long as a block, so there is at most one more, the next)
    uint32_t n_bounds;
    uint32_t bound[2 * kMaxM];
    uint32_t bound_mat[2 * kMaxM];
    float *part;               // kSlots floats per block
    uint32_t *first_block;     // per row: the block holding its first weight
    uint32_t *last_block;      // per row: the block holding its last weight
};

struct ReduceArgs {
    const uint32_t *block_pos;  // B + 1 entries
    const float *part;
    const uint32_t *first_block;
    const uint32_t *last_block;
    uint32_t num_blocks;
    uint32_t n_mats;
    uint32_t row_start[kMaxM + 1];  // prefix sums of rows
    uint32_t off[kMaxM];
    uint32_t cols[kMaxM];
    float *y[kMaxM];
};

template <int kCtrl, int kRowMask, bool kBound>
__device__ __forceinline__ float dpp_f32(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x),
                                                                 kCtrl, kRowMask, 0xF, kBound));
}

// Same row-shift / row-broadcast pattern as the integer scan: lane 63 ends
// with the sum of all 64 lanes, added in a fixed order.
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_f32<0x111, 0xF, true>(v);
    v += dpp_f32<0x112, 0xF, true>(v);
    v += dpp_f32<0x114, 0xF, true>(v);
    v += dpp_f32<0x118, 0xF, true>(v);
    v += dpp_f32<0x142, 0xA, false>(v);
    v += dpp_f32<0x143, 0xC, false>(v);
    return v;
}

__device__ __forceinline__ float dot8(const uint4 &w, const uint4 &x) {
    float d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.x),
                                              __builtin_bit_cast(bf16x2, x.x), 0.f, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.y),
                                        __builtin_bit_cast(bf16x2, x.y), d, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.z),
                                        __builtin_bit_cast(bf16x2, x.z), d, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w.w),
                                        __builtin_bit_cast(bf16x2, x.w), d, false);
    return d;
}

// One block's weights [s, e) -- buffer bytes [lo_at, hi_at) from weight g0 on
// -- times the activations of the (at most two) matrices they belong to, m0 and
// the next one, one weight per lane and step: segment 0 is the matrix holding
// weight s, segment 1 the first matrix that starts inside (s, e).  For the few
// blocks at the matrices' boundaries.
constexpr uint32_t kAhead = 8;
__device__ __forceinline__ void dot_block(const GemvArgs &g, uint32_t g0, uint32_t lo_at,
                                          uint32_t hi_at, const uint8_t *buf, uint32_t lane,
                                          uint32_t b, uint32_t m0) {
    const uint32_t s = g0 + lo_at, e = g0 + hi_at;
    bool inside = false;
#pragma unroll 1
    for (uint32_t m = m0; m < umin(m0 + 2u, g.n_mats); ++m) {
        const uint32_t off = g.off[m], cols = g.cols[m];
        const uint32_t lo = umax(s, off), hi = umin(e, g.end[m]);
        if (lo >= hi || (off > s && inside)) continue;
        inside |= off > s;
        uint32_t row = (lo - off) / cols;
        float *slot = g.part + static_cast<uint64_t>(b) * kSlots + (off > s ? kSegSlots : 0u);
        // rows it touches: at most 3 (4096 weights, 2048 columns)
#pragma unroll 1
        for (uint32_t at = lo, i = 0; at < hi && i < kSegSlots; ++row, ++i) {
            const uint64_t start = uint64_t{off} + uint64_t{row} * cols;
            const uint32_t stop = static_cast<uint32_t>(umin64(hi, start + cols));
            float sum = 0.f;
            // kAhead weights of a lane requested at once (from memory, one after
            // the other they were the whole time of a short call)
            const uint32_t last = stop - 1u - at;
#pragma unroll 1
            for (uint32_t q0 = lane; q0 <= last; q0 += 64u * kAhead) {
                uint32_t sm[kAhead], x[kAhead];
#pragma unroll
                for (uint32_t k = 0; k < kAhead; ++k) {
                    const uint32_t q = at + umin(q0 + 64u * k, last);
                    sm[k] = g.d.sm[q];
                    x[k] = g.x[m][q - static_cast<uint32_t>(start)];
                }
#pragma unroll
                for (uint32_t k = 0; k < kAhead; ++k) {
                    const uint32_t q = umin(q0 + 64u * k, last);
                    const uint32_t ex = buf[at + q - g0];
                    const uint32_t w = ((sm[k] & 0x80u) << 24) | ((ex & 0x7Fu) << 24) |
                                       ((ex & 0x80u) << 16) | ((sm[k] & 0x7Fu) << 16);
                    const float v = __builtin_bit_cast(float, w) * __builtin_bit_cast(float, x[k] << 16);
                    sum += q0 + 64u * k <= last ? v : 0.f;
                }
            }
            sum = wave_sum(sum);
            if (lane == 63u) {
                slot[i] = sum;
                if (start >= lo) g.first_block[g.row_base[m] + row] = b;
                if (start + cols <= hi) g.last_block[g.row_base[m] + row] = b;
            }
            at = stop;
        }
    }
}

// The matrix a wave is in.  Its blocks come in stream order, so the matrix
// only ever moves on; its description stays in scalar registers (all eight
// would not fit beside the decoder's).
struct Current {
    uint32_t next;      // index of the next matrix
    uint32_t next_off;  // its first weight
    uint32_t off, end, cols, row_base;
    Divider div;
    const uint16_t *x;
};

__device__ __forceinline__ uint32_t matrix_start(const GemvArgs &g, uint32_t m) {
    return m < g.n_mats ? g.off[m] : 0xFFFFFFFFu;
}

// The last matrix that starts at or before weight s (none: an empty range).
__device__ __forceinline__ void advance(const GemvArgs &g, uint32_t s, Current &cur) {
    while (s >= cur.next_off && cur.next < g.n_mats) {
        const uint32_t m = cur.next++;
        cur.off = cur.next_off;
        cur.next_off = matrix_start(g, cur.next);
        cur.end = g.end[m];
        cur.cols = g.cols[m];
        cur.row_base = g.row_base[m];
        cur.div = g.div[m];
        cur.x = g.x[m];
    }
}

// A block inside one matrix (then it touches at most three of its rows): all
// but the few at the matrices' boundaries.
struct Span {
    bool plain;
    uint32_t rlo, cols;
    uint32_t col0;  // column of the block's first group
    uint32_t nrows;
};

__device__ __forceinline__ Span block_span(const Current &cur, const Range &r) {
    const uint32_t s = r.g0 + r.shift, e = r.g0 + r.lim;
    Span sp{};
    if (s < e && cur.off <= s && e <= cur.end) {
        sp.cols = cur.cols;
        sp.rlo = divide(s - cur.off, cur.div);
        sp.nrows = divide(e - 1u - cur.off, cur.div) - sp.rlo + 1u;
        sp.col0 = r.g0 - cur.off - sp.rlo * sp.cols;  // rows and groups start on multiples of 8
        sp.plain = true;
    }
    return sp;
}

// Column of byte `at` (a weight counted from the block's first group): c minus
// cols wraps to a large value while c is still in the row.
__device__ __forceinline__ uint32_t span_column(const Span &sp, uint32_t at) {
    uint32_t c = sp.col0 + at;
    c = umin(c, c - sp.cols);
    return umin(c, c - sp.cols);
}

// A plain block's weights times their activations: whole groups eight at a
// time; the elements of the (at most two) groups shared with the neighbours
// one per lane.
__device__ __forceinline__ void dot_plain(const GemvArgs &g, const Range &r, const Current &cur,
                                          const Span &sp, const uint8_t *buf, uint32_t lane,
                                          const Groups<kPre> &gr, const uint2 (&S)[kPre],
                                          uint32_t edge_sm, uint32_t b) {
    const uint32_t el = edge_byte(r, lane & 15u);
    uint2 E[kPre];
    uint4 X[kPre];
#pragma unroll
    for (int k = 0; k < kPre; ++k) E[k] = *reinterpret_cast<const uint2 *>(buf + gr.at[k]);
#pragma unroll
    for (int k = 0; k < kPre; ++k)
        X[k] = *reinterpret_cast<const uint4 *>(cur.x + span_column(sp, gr.at[k]));
    const uint32_t edge_x = cur.x[span_column(sp, el)];
    const uint32_t edge_e = buf[el];
    float t[3] = {0.f, 0.f, 0.f};
    // (rows past the block's are never reached: c stays below their start)
    auto add = [&](float v, uint32_t at) {
        const uint32_t c = sp.col0 + at;
        const bool second = c >= sp.cols, third = c >= 2u * sp.cols;
        t[0] += second ? 0.f : v;
        t[1] += second && !third ? v : 0.f;
        t[2] += third ? v : 0.f;
    };
    float d[kPre + 1];
#pragma unroll
    for (int k = 0; k < kPre; ++k) {
        const float v = dot8(assemble_group(E[k], S[k]), X[k]);
        // (a select: the product of a group that is not this lane's may be NaN)
        d[k] = full_group(r, lane + 64u * k) ? v : 0.f;
    }
    {
        const bool mine = lane < 16u && !full_group(r, el >> 3) && (lane < 8u || el >= 8u) &&
                          el >= r.shift && el < r.lim;
        const uint32_t w = ((edge_sm & 0x80u) << 24) | ((edge_e & 0x7Fu) << 24) |
                           ((edge_e & 0x80u) << 16) | ((edge_sm & 0x7Fu) << 16);
        const float v = __builtin_bit_cast(float, w) * __builtin_bit_cast(float, edge_x << 16);
        d[kPre] = mine ? v : 0.f;
    }
    if (sp.nrows == 1u) {  // uniform; three of five blocks with 4096 columns
#pragma unroll
        for (int k = 0; k <= kPre; ++k) t[0] += d[k];
    } else {
#pragma unroll
        for (int k = 0; k < kPre; ++k) add(d[k], gr.at[k]);
        add(d[kPre], el);
    }
    // blocks of more than 2048 weights (codes of less than two bits on average)
#pragma unroll 1
    for (uint32_t base = 64u * kPre; __builtin_expect(base < r.full_hi, 0); base += 64u * kPre) {
        const Groups<kPre> more = block_groups<kPre>(r, base + lane, 64u);
        uint2 T[kPre];
        prefetch_sm(g.d, r, more, T);
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            const float v = dot8(assemble_group(*reinterpret_cast<const uint2 *>(buf + more.at[k]), T[k]),
                                 *reinterpret_cast<const uint4 *>(cur.x + span_column(sp, more.at[k])));
            add(full_group(r, base + lane + 64u * k) ? v : 0.f, more.at[k]);
        }
    }
    t[0] = wave_sum(t[0]);
    if (sp.nrows > 1u) t[1] = wave_sum(t[1]);
    if (sp.nrows > 2u) t[2] = wave_sum(t[2]);
    if (lane == 63u)
        *reinterpret_cast<float4 *>(g.part + static_cast<uint64_t>(b) * kSlots) =
            make_float4(t[0], t[1], t[2], 0.f);
    // rows whose first or last weight is here (the first row's column 0 only
    // when the block starts there; always column 0 of the others)
    if (lane < sp.nrows) {
        const uint32_t row = cur.row_base + sp.rlo + lane;
        if (lane != 0u || sp.col0 + r.shift == 0u) g.first_block[row] = b;
        if (sp.col0 + r.lim >= (lane + 1u) * sp.cols) g.last_block[row] = b;
    }
}

// Last block that starts at or before weight `pos`: 64 probes at a time.
__device__ __forceinline__ uint32_t find_block(const DecodeArgs &a, uint32_t pos, uint32_t lane) {
    uint32_t lo = 0, n = a.num_blocks;  // the answer is in [lo, lo + n)
    while (n > 1u) {
        const uint32_t step = (n + 63u) / 64u;
        const bool le = lane * step < n && a.block_pos[lo + umin(lane * step, n - 1u)] <= pos;
        const uint32_t hits = static_cast<uint32_t>(__builtin_popcountll(__builtin_amdgcn_ballot_w64(le)));
        const uint32_t j = umax(hits, 1u) - 1u;
        lo += j * step;
        n = umin(step, n - j * step);
    }
    return lo;
}

// The block that has boundary q inside it (the first of its boundaries takes
// it): decoded by one wave like any other, multiplied by dot_block.
__device__ __forceinline__ void boundary_block(const GemvArgs &g, const Tables &tb, uint8_t *lds,
                                               uint32_t buf_off, uint32_t lane, uint32_t q) {
    const DecodeArgs &a = g.d;
    const uint32_t pos = g.bound[q], before = q ? g.bound[q - 1u] : 0u;
    const uint32_t b = static_cast<uint32_t>(
        __builtin_amdgcn_readfirstlane(static_cast<int>(find_block(a, pos, lane))));
    const ChunkWords cw = load_chunk<64>(a, b, lane);
    const Chunk ch[1] = {chunk_setup<64>(a, cw, b, lane)};
    const Range r = block_range(a, cw);
    const uint32_t s = r.g0 + r.shift, e = r.g0 + r.lim;
    if (pos <= s || pos >= e || before > s) return;  // (they ascend)
    for (uint32_t i = lane; i < (a.buf_bytes >> 4); i += 64u)
        reinterpret_cast<uint4 *>(lds + buf_off)[i] = make_uint4(0u, 0u, 0u, 0u);
    Trail<kKeep> tr[1];
    uint32_t state[1], out8[1];
    decode_count(tb, ch, tr, state, out8);
    const uint32_t excl8 = wave_inclusive_scan(out8[0]) - out8[0];
    wave_lds_sync();
    emit_exponents(tb, ch[0], tr[0], state[0], 8u * r.shift + excl8, buf_off, a.buf_bytes);
    wave_lds_sync();
    dot_block(g, r.g0, r.shift, r.lim, lds + buf_off + kBufLead, lane, b, g.bound_mat[q]);
}

// Same loop as the decode kernel's for 64-chunk blocks (persistent grid, one
// wave per block); the decoded weights go into their dot products instead of
// memory.  The activations are read through the caches.  (Staged in LDS, one
// set of matrices after the other, they cost scalar registers, LDS and a round
// trip per matrix, and were slower at every size: 8 matrices of 256 x 2048 14.4
// us against 13.5, of 2048 x 2048 31.0 against 26.2, a Llama-3-8B-sized block
// 115 against 109.5.)
//
// The blocks at the matrices' boundaries go to the first workgroups, a wave
// each: in the loop, their code would cost every block scalar registers
// (0.130 ms with it, 0.121 ms without).
//
// Bound: instruction issue and latency -- about 390 vector and 215 scalar
// instructions per block, six waves per SIMD.  A Llama-3-8B-sized block's
// compressed bytes alone take 57 us at the rate of a device copy; 109.5 us
// for the two kernels.
template <uint32_t W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(6))) void
df11_gemv_wave_kernel(GemvArgs g) {
    const DecodeArgs &a = g.d;
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // block indices stay scalar
    const uint32_t main_grid = gridDim.x - g.boundary_grid;
    const uint32_t buf_off = a.table_lds_bytes + wave * a.buf_bytes;
    if (blockIdx.x < g.boundary_grid) {
        stage_table_blob(a, lds, tid, 64 * W);
        __syncthreads();
        const Tables tb = staged_tables(a, lds);
        const uint32_t q = blockIdx.x * W + wave;
        if (q < g.n_bounds) boundary_block(g, tb, lds, buf_off, lane, q);
        return;
    }
    const uint32_t first_block = xcd_grouped_index(blockIdx.x - g.boundary_grid, main_grid) * W + wave;
    const uint32_t stride = main_grid * W;
    ChunkWords cw{};
    if (first_block < a.num_blocks) cw = load_chunk<64>(a, first_block, lane);
    stage_table_blob(a, lds, tid, 64 * W);
    uint8_t *buf = lds + buf_off + kBufLead;
    __syncthreads();
    if (first_block >= a.num_blocks) return;
    const Tables tb = staged_tables(a, lds);
    Chunk ch[1] = {chunk_setup<64>(a, cw, first_block, lane)};
    Range r = block_range(a, cw);
    Current cur{};
    cur.next_off = matrix_start(g, 0u);

    for (uint32_t b = first_block; b < a.num_blocks; b += stride) {
        ChunkWords nxt = cw;
        if (b + stride < a.num_blocks) nxt = load_chunk<64>(a, b + stride, lane);
        const Groups<kPre> gr = block_groups<kPre>(r, lane, 64u);
        uint2 S[kPre];
        prefetch_sm(a, r, gr, S);
        const uint32_t edge_sm = a.sm[r.g0 + edge_byte(r, lane & 15u)];

        wave_lds_sync();
        for (uint32_t i = lane; i < (a.buf_bytes >> 4); i += 64u)
            reinterpret_cast<uint4 *>(lds + buf_off)[i] = make_uint4(0u, 0u, 0u, 0u);

        Trail<kKeep> tr[1];
        uint32_t state[1], out8[1];
        decode_count(tb, ch, tr, state, out8);
        const uint32_t excl8 = wave_inclusive_scan(out8[0]) - out8[0];
        __builtin_amdgcn_s_setprio(1);
        wave_lds_sync();
        emit_exponents(tb, ch[0], tr[0], state[0], 8u * r.shift + excl8, buf_off, a.buf_bytes);
        wave_lds_sync();

        __builtin_amdgcn_s_setprio(2);
        advance(g, r.g0 + r.shift, cur);
        const Span sp = block_span(cur, r);
        if (__builtin_expect(sp.plain, 1)) dot_plain(g, r, cur, sp, buf, lane, gr, S, edge_sm, b);
        __builtin_amdgcn_s_setprio(0);
        cw = nxt;
        ch[0] = chunk_setup<64>(a, cw, b + stride, lane);
        r = block_range(a, cw);
    }
}

// Lanes per row in the reduction: the row's blocks (2 to 4 with 4096 columns,
// about 10 with 14336) are then all requested at once, and the sum costs two
// dependent round trips whatever their number (one thread per row took one
// per block: 8.5 us for the 43,008 rows of a Llama-3-8B-sized block).
constexpr uint32_t kRowLanes = 16;  // one DPP row

// y[m][row] = sum over the blocks covering the row of the block's partial sum
// for that row: lane q of the row's 16 adds blocks q, q+16, ... counted from
// the row's first, then the lanes' sums are added in a fixed order.
__global__ __launch_bounds__(256) void df11_gemv_reduce_kernel(ReduceArgs ra) {
    const uint32_t i = blockIdx.x * (256u / kRowLanes) + threadIdx.x / kRowLanes;
    const uint32_t q0 = threadIdx.x % kRowLanes;
    if (i >= ra.row_start[ra.n_mats]) return;  // whole 16-lane rows leave together
    uint32_t m = 0;
#pragma unroll
    for (uint32_t q = 1; q < kMaxM; ++q)
        if (q < ra.n_mats && i >= ra.row_start[q]) m = q;
    uint32_t rs = 0, off = 0, cols = 1;
    float *y = nullptr;
#pragma unroll
    for (uint32_t q = 0; q < kMaxM; ++q) {
        if (q == m) {
            rs = ra.row_start[q];
            off = ra.off[q];
            cols = ra.cols[q];
            y = ra.y[q];
        }
    }
    const uint32_t row = i - rs;
    // every block between the row's first and last holds at least one weight
    // (each 64-bit chunk starts a code), so all of them wrote partial sums
    const uint32_t fb = ra.first_block[i], lb = ra.last_block[i];
    // a block holds >= 128 weights (64 chunks, >= 2 codes each), so a row
    // spans at most cols / 128 + 2 blocks; indices outside that (not written
    // by the decode kernel) give NaN instead of reads out of range
    const bool bad = lb >= ra.num_blocks || fb > lb || lb - fb > cols / 128u + 2u;
    float sum = 0.f;
    if (!bad) {
        for (uint32_t b = fb + q0; b <= lb && b >= fb; b += kRowLanes) {
            const uint32_t bs = ra.block_pos[b];
            const uint32_t j = off <= bs ? 0u : 1u;
            const uint32_t seg_lo = bs > off ? bs : off;
            const uint32_t rlo = (seg_lo - off) / cols;
            const uint32_t rr = row - rlo;  // 0..2 by construction; checked to keep reads in range
            if (rr < 3u) sum += ra.part[static_cast<uint64_t>(b) * kSlots + j * kSegSlots + rr];
        }
    }
    // lane 15 of the row ends with the sum of its 16 lanes
    sum += dpp_f32<0x111, 0xF, true>(sum);
    sum += dpp_f32<0x112, 0xF, true>(sum);
    sum += dpp_f32<0x114, 0xF, true>(sum);
    sum += dpp_f32<0x118, 0xF, true>(sum);
    if (q0 == kRowLanes - 1u) y[row] = bad ? __builtin_nanf("") : sum;
}

using GemvFn = void (*)(GemvArgs);

GemvFn gemv_kernel(uint32_t W) {
    switch (W) {
        case 4: return df11_gemv_wave_kernel<4>;
        case 8: return df11_gemv_wave_kernel<8>;
        case 12: return df11_gemv_wave_kernel<12>;
        case 16: return df11_gemv_wave_kernel<16>;
        default: return nullptr;
    }
}

struct Shape {
    int dev;
    uint32_t tables, buf, W, per_cu;
};
std::mutex g_mu;
std::vector<Shape> g_shapes;
std::vector<std::array<uint32_t, 4>> g_lds_granted;  // per device and kernel: dynamic LDS allowed
constexpr size_t kMaxShapes = 64;

// Workgroup size and resident workgroups per CU for `tables` bytes of LDS per
// workgroup and `buf` per wave: the most resident waves, fewer per workgroup
// on a tie.
int gemv_shape(uint32_t tables, uint32_t buf, uint32_t *W_out, uint32_t *grid_max) {
    int dev = 0, cus = 0, max_lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return DF11_E_HIP;
    std::lock_guard<std::mutex> lk(g_mu);
    for (const Shape &sh : g_shapes) {
        if (sh.dev == dev && sh.tables == tables && sh.buf == buf) {
            *W_out = sh.W;
            *grid_max = sh.per_cu * static_cast<uint32_t>(cus);
            return DF11_OK;
        }
    }
    if (g_lds_granted.size() <= static_cast<size_t>(dev)) g_lds_granted.resize(dev + 1);
    std::array<uint32_t, 4> &granted = g_lds_granted[dev];
    uint32_t best_W = 0, best_pc = 0, best_waves = 0;
    for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t W = 4u * (i + 1u);
        const uint32_t lds = tables + W * buf;
        if (lds > static_cast<uint32_t>(max_lds)) continue;
        const void *fn = reinterpret_cast<const void *>(gemv_kernel(W));
        if (lds > 65536u && granted[i] < lds) {
            if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    static_cast<int>(lds)) != hipSuccess)
                return DF11_E_HIP;
            granted[i] = lds;
        }
        int pc = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&pc, fn, static_cast<int>(64 * W), lds) !=
            hipSuccess)
            return DF11_E_HIP;
        const uint32_t fits = lds_fit(static_cast<uint32_t>(max_lds), lds);
        if (static_cast<uint32_t>(pc) > fits) pc = static_cast<int>(fits);
        if (static_cast<uint32_t>(pc) * W > best_waves) {
            best_waves = static_cast<uint32_t>(pc) * W;
            best_W = W;
            best_pc = static_cast<uint32_t>(pc);
        }
    }
    if (!best_waves) return DF11_E_UNSUPPORTED;
    if (g_shapes.size() >= kMaxShapes) g_shapes.clear();
    g_shapes.push_back(Shape{dev, tables, buf, best_W, best_pc});
    *W_out = best_W;
    *grid_max = best_pc * static_cast<uint32_t>(cus);
    return DF11_OK;
}

// partial sums (kSlots floats per block), then first and last block per row
uint64_t workspace_bytes_for(const df11_stream *s, const df11_matrix *mats, uint32_t n_mats) {
    uint64_t rows = 0;
    for (uint32_t m = 0; m < n_mats; ++m) rows += mats[m].rows;
    return 4ull * kSlots * s->sizes.num_blocks + 8ull * rows;
}

int check_gemv(const df11_stream *s, const df11_matrix *mats, uint32_t n_mats) {
    int rc = check_stream(s);
    if (rc) return rc;
    if (s->layout.threads_per_block != 64) return DF11_E_UNSUPPORTED;
    if (!mats || n_mats == 0 || n_mats > kMaxM) return DF11_E_INVALID_ARG;
    uint64_t prev_end = 0;
    for (uint32_t m = 0; m < n_mats; ++m) {
        const df11_matrix &d = mats[m];
        if (d.rows == 0 || d.cols == 0) return DF11_E_INVALID_ARG;
        if (d.cols % 64 || d.cols < kMinCols || d.offset % 8) return DF11_E_UNSUPPORTED;
        const uint64_t size = static_cast<uint64_t>(d.rows) * d.cols;
        if (size < kMaxBlockElems) return DF11_E_UNSUPPORTED;  // a block spans <= 2 matrices
        if (d.offset < prev_end) return DF11_E_UNSUPPORTED;    // sorted and disjoint
        if (d.offset > s->sizes.n_elems || size > s->sizes.n_elems - d.offset)
            return DF11_E_INVALID_ARG;
        prev_end = d.offset + size;
    }
    return DF11_OK;
}

}  // namespace

extern "C" {

int df11_gemv_workspace_bytes(const df11_stream *dev, const df11_matrix *mats, uint32_t n_mats,
                              uint64_t *bytes) {
    if (!dev || !bytes || !mats || n_mats == 0 || n_mats > kMaxM) return DF11_E_INVALID_ARG;
    *bytes = workspace_bytes_for(dev, mats, n_mats);
    return DF11_OK;
}

int df11_block_gemv(const df11_stream *dev, const df11_matrix *mats, uint32_t n_mats,
                    const uint16_t *const *x, float *const *y, void *workspace,
                    uint64_t workspace_bytes, hipStream_t stream) {
    int rc = check_gemv(dev, mats, n_mats);
    if (rc) return rc;
    if (!x || !y) return DF11_E_INVALID_ARG;
    for (uint32_t m = 0; m < n_mats; ++m)
        if (!x[m] || !y[m] || (reinterpret_cast<uintptr_t>(x[m]) & 15u) ||
            (reinterpret_cast<uintptr_t>(y[m]) & 3u))
            return DF11_E_INVALID_ARG;
    const uint64_t need = workspace_bytes_for(dev, mats, n_mats);
    if (workspace_bytes < need) return DF11_E_BUFFER_TOO_SMALL;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 15u)) return DF11_E_INVALID_ARG;
    if (dev->sizes.n_elems == 0) return DF11_OK;

    GemvArgs g{};
    DecodeArgs &a = g.d;
    a.exp = dev->exp;
    a.sm = dev->sm;
    a.gaps = reinterpret_cast<const uint32_t *>(dev->gaps);
    a.block_pos = dev->block_pos;
    a.tables = dev->tables + df11tab::kHeaderBytes;
    a.out = nullptr;  // nothing is stored
    a.total_bits = dev->sizes.total_bits;
    a.n_elems = static_cast<uint32_t>(dev->sizes.n_elems);
    a.num_chunks = static_cast<uint32_t>(dev->sizes.num_chunks);
    a.num_blocks = static_cast<uint32_t>(dev->sizes.num_blocks);
    a.lut_bits = dev->layout.lut_bits;
    a.max_len = dev->sizes.max_code_len;
    a.table_lds_bytes = static_cast<uint32_t>(df11tab::lds_bytes(dev->layout.lut_bits));
    a.buf_bytes = buf_bytes_for(dev->sizes.max_elems_per_block);
    a.twin_bufs = a.hold = 0;  // not used by the fused kernel
    g.n_mats = n_mats;
    g.part = static_cast<float *>(workspace);
    ReduceArgs ra{};
    ra.block_pos = dev->block_pos;
    ra.part = static_cast<const float *>(workspace);
    ra.num_blocks = a.num_blocks;
    ra.n_mats = n_mats;
    uint64_t rows = 0;
    for (uint32_t m = 0; m < n_mats; ++m) {
        g.off[m] = ra.off[m] = static_cast<uint32_t>(mats[m].offset);
        g.end[m] = static_cast<uint32_t>(mats[m].offset + uint64_t{mats[m].rows} * mats[m].cols);
        g.cols[m] = ra.cols[m] = mats[m].cols;
        g.div[m] = make_divider(mats[m].cols);
        // the divider must agree with plain division at every row start and
        // just before it (a failed check means a bug here, not bad input)
        for (uint32_t t : {0u, 1u, mats[m].rows - 1u, mats[m].rows}) {
            const uint64_t n0 = uint64_t{t} * mats[m].cols;
            if (n0 <= 0xFFFFFFFFull && divide(static_cast<uint32_t>(n0), g.div[m]) != t)
                return DF11_E_UNSUPPORTED;
            if (n0 && n0 - 1 <= 0xFFFFFFFFull &&
                divide(static_cast<uint32_t>(n0 - 1), g.div[m]) != t - 1)
                return DF11_E_UNSUPPORTED;
        }
        g.x[m] = x[m];
        ra.y[m] = y[m];
        ra.row_start[m] = g.row_base[m] = static_cast<uint32_t>(rows);
        rows += mats[m].rows;
    }
    for (uint32_t m = n_mats; m <= kMaxM; ++m) ra.row_start[m] = static_cast<uint32_t>(rows);
    if (rows > 0xFFFFFFFFull) return DF11_E_UNSUPPORTED;
    uint32_t *row_blocks = reinterpret_cast<uint32_t *>(static_cast<uint8_t *>(workspace) +
                                                        4ull * kSlots * a.num_blocks);
    g.first_block = row_blocks;
    g.last_block = row_blocks + rows;
    ra.first_block = g.first_block;
    ra.last_block = g.last_block;

    uint32_t W = 0, grid_max = 0;
    rc = gemv_shape(a.table_lds_bytes, a.buf_bytes, &W, &grid_max);
    if (rc) return rc;
    for (uint32_t m = 0; m < n_mats; ++m) {
        if (g.off[m] > 0 && (m == 0 || g.off[m] > g.end[m - 1])) {
            g.bound[g.n_bounds] = g.off[m];
            g.bound_mat[g.n_bounds++] = m ? m - 1 : 0;
        }
        if (g.end[m] < a.n_elems) {
            g.bound[g.n_bounds] = g.end[m];
            g.bound_mat[g.n_bounds++] = m;
        }
    }
    g.boundary_grid = (g.n_bounds + W - 1) / W;
    uint32_t grid = (a.num_blocks + W - 1) / W;
    const uint32_t room = grid_max > g.boundary_grid ? grid_max - g.boundary_grid : 1u;
    if (grid > room) grid = room;
    if (!grid) grid = 1;
    grid += g.boundary_grid;
    const uint32_t lds = a.table_lds_bytes + W * a.buf_bytes;
    hipLaunchKernelGGL(gemv_kernel(W), dim3(grid), dim3(64 * W), lds, stream, g);
    if (hipGetLastError() != hipSuccess) return DF11_E_HIP;
    hipLaunchKernelGGL(df11_gemv_reduce_kernel, dim3(static_cast<uint32_t>((rows * kRowLanes + 255) / 256)),
                       dim3(256), 0, stream, ra);
    return hipGetLastError() == hipSuccess ? DF11_OK : DF11_E_HIP;
}

}  // extern "C"
