// Split-K paged grouped-query decode attention for gfx950 (data path 1 of the
// hot-cold hierarchy: every decode step reads the whole hot set).
//
// Work split.  A unit is one page (16 tokens) of one (row b, group of L KV
// heads); the units of all rows are laid end to end and cut into equal ranges,
// one per worker of a persistent grid, so long and short contexts balance
// exactly.  A worker is L consecutive waves, wave w taking KV head L hg + w of
// head group hg: with L = 4 the four waves of a worker read the four heads'
// tiles of each page side by side, which HBM serves faster than as many
// unrelated pages (DRAM row locality); L = 1 when the KV heads do not come in
// fours.  Where a worker's range meets the units of one (b, hg), each of its
// waves produces a partial result (running max m, weight sum l, unnormalised
// output o) for the query heads sharing its KV head; the combine kernel merges
// the partials of each (b, g) with the usual log-sum-exp rescaling.  Reduction
// order depends only on seq_lens, never on page placement, so results are
// bitwise independent of where pages sit in the pool.
//
// One wave processes one page of one KV head per step with matrix cores:
//   scores  S^T[t][h] = K[t][:] . Q[h][:]   v_mfma_f32_16x16x32_bf16 (f32: 16x16x4)
//           (16 tokens x 16 head slots; the group's heads fill the first slots)
//   output  O^T[d][h] += V^T[d][t] P^T[t][h] v_mfma_f32_16x16x16_bf16 (f32: 16x16x4)
// The score tile comes out of the first product in exactly the register layout
// the second product takes for P (lane l: head l % 16, tokens 4 (l / 16) + r),
// so the softmax needs no data movement besides two cross-lane max steps.
// Each query-head group reads every K/V byte once (the GQA reuse).
//
// Memory.  K tiles are stored as 16-byte groups of dims, token-minor, so the
// four 16-byte loads a lane issues for a K tile are each 1 KiB contiguous across
// the wave; V tiles are stored dims-major, token-minor, so each lane's slice of
// V^T for one 16-dim chunk is 8 contiguous bytes and a wave reads 512
// contiguous bytes per load.  Pages are addressed through buffer resources
// whose base is the page and whose size is its two tiles: an out-of-range page
// id becomes a zero-sized resource, reads return 0 and the row is flagged NaN.
// Each wave keeps a ring of page buffers in registers: while one page is
// computed, the loads of the next ring - 1 pages are in flight, whichever rows
// they belong to.

#include "device_common.h"
#include "kernels.h"

#include <math.h>

namespace hck {
namespace {

constexpr int kRsrcWord3 = 0x00020000;  // raw buffer, 32-bit data format (gfx9 family)

// Cache-policy bits of the K/V page loads: 2 = nontemporal (streaming).  Every
// K/V byte is read exactly once per call, so keeping it out of the caches'
// normal replacement leaves them to page ids, queries and partials.
#ifndef HCK_DECODE_LOAD_AUX
#define HCK_DECODE_LOAD_AUX 2
#endif
#ifndef HCK_RING_BF16_D128
#define HCK_RING_BF16_D128 3
#endif
// Waves per block of the split kernel.
#ifndef HCK_SPLIT_BLOCK_WAVES
#define HCK_SPLIT_BLOCK_WAVES 4
#endif
constexpr int kSplitBlockWaves = HCK_SPLIT_BLOCK_WAVES;
constexpr int kSplitBlockThreads = kSplitBlockWaves * kWave;

template <int D, bool BF16>
struct Shape {
    static constexpr int kElt = BF16 ? 2 : 4;
    static constexpr int kTile = kPageTokens * D * kElt;  // bytes of a K or V tile
    static constexpr int kKLoads = kTile / 1024;          // 16-byte K loads per lane
    static constexpr int kChunks = D / 16;                // 16-dim output chunks
};

template <bool BF16>
struct VSlice;
template <>
struct VSlice<true> {
    typedef u32x2 type;  // 4 bf16 tokens of one dim
};
template <>
struct VSlice<false> {
    typedef u32x4 type;  // 4 f32 tokens of one dim
};

template <int D, bool BF16>
struct PageRegs {
    u32x4 k[Shape<D, BF16>::kKLoads];
    typename VSlice<BF16>::type v[Shape<D, BF16>::kChunks];
};

__device__ __forceinline__ float wave_max_4(float x) {
    // max over lanes l, l^16, l^32, l^48 (the four token quarters of one head)
    x = fmaxf(x, __shfl_xor(x, 16));
    x = fmaxf(x, __shfl_xor(x, 32));
    return x;
}

__device__ __forceinline__ float wave_sum_4(float x) {
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    return x;
}

// Where a piece's pages live, already offset to its layer and KV head: hot
// pages, and for tiered entries the cold pool and this layer's staging slots.
struct PageSrc {
    const char* hot = nullptr;
    const char* cold = nullptr;
    const char* stage = nullptr;
    int64_t hot_stride = 0, cold_stride = 0, slice_bytes = 0;
    unsigned num_hot = 0, num_cold = 0, num_stage = 0;
};

// A (page, KV head)'s two tiles.  Page ids are wave-uniform, so the tier choice
// is scalar.  An id outside its pool (or a negative entry) reads nothing: the
// buffer resource gets no records and the row is marked bad (NaN).
struct PageAddr {
    const char* base;
    bool ok;
};

template <bool TIERED>
__device__ __forceinline__ PageAddr page_addr(const PageSrc& ps, int pid, unsigned head_off) {
    const char* lh_base = ps.hot;
    int64_t stride = ps.hot_stride;
    unsigned n = ps.num_hot;
    unsigned id = static_cast<unsigned>(pid);
    if constexpr (TIERED) {
        const unsigned tag = id >> 29;  // 0 hot, 1 staged, 2 cold, otherwise invalid
        id &= static_cast<unsigned>(kPageIdMask);
        if (tag == 1) {
            lh_base = ps.stage;
            stride = ps.slice_bytes;
            n = ps.num_stage;
        } else if (tag == 2) {
            lh_base = ps.cold;
            stride = ps.cold_stride;
            n = ps.num_cold;
        } else if (tag != 0) {
            n = 0;
        }
    }
    const bool ok = id < n;
    return PageAddr{lh_base + static_cast<int64_t>(ok ? id : 0) * stride + head_off, ok};
}

template <int D, bool BF16>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t page_rsrc(const PageAddr& p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p.base), static_cast<short>(0),
                                             p.ok ? 2 * Shape<D, BF16>::kTile : 0, kRsrcWord3);
}

// Offsets past the instruction's 12 bits go into the scalar offset: one VGPR of
// offsets for all K loads and one for all V loads.
template <int D, bool BF16>
__device__ __forceinline__ void load_page_k(PageRegs<D, BF16>& r, __amdgpu_buffer_rsrc_t rs, unsigned koff) {
#pragma unroll
    for (int i = 0; i < Shape<D, BF16>::kKLoads; ++i)
        r.k[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, koff + 1024u * (i % 4), 4096 * (i / 4), HCK_DECODE_LOAD_AUX);
}

template <int D, bool BF16>
__device__ __forceinline__ void load_page_v(PageRegs<D, BF16>& r, __amdgpu_buffer_rsrc_t rs, unsigned voff) {
    using S = Shape<D, BF16>;
#pragma unroll
    for (int c = 0; c < S::kChunks; ++c) {
        if constexpr (BF16)
            r.v[c] = __builtin_amdgcn_raw_buffer_load_b64(rs, voff + 512u * c, S::kTile, HCK_DECODE_LOAD_AUX);
        else
            r.v[c] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 1024u * (c % 4), S::kTile + 4096 * (c / 4),
                                                           HCK_DECODE_LOAD_AUX);
    }
}

// S^T tile of one page: lane l gets scores of head l % 16 for tokens 4 (l / 16) + r.
// Two accumulators halve the dependent MFMA chain; their sum is added once.
template <int D, bool BF16>
__device__ __forceinline__ f32x4 page_scores(const PageRegs<D, BF16>& r,
                                             const u32x4 (&q)[Shape<D, BF16>::kKLoads]) {
    using S = Shape<D, BF16>;
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < S::kKLoads; ++i) {
        f32x4& acc = (i & 1) ? s1 : s0;
        if constexpr (BF16) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.k[i]),
                                                          __builtin_bit_cast(bf16x8, q[i]), acc, 0,
                                                          0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(r.k[i][j]),
                                                           __uint_as_float(q[i][j]), acc, 0, 0, 0);
        }
    }
    return s0 + s1;
}

// Zero the V slice entries of tokens >= valid (this lane holds tokens 4 qg + j).
template <int D, bool BF16>
__device__ __forceinline__ void mask_v(PageRegs<D, BF16>& r, int valid, int qg) {
    using S = Shape<D, BF16>;
    const int t0 = 4 * qg;
    if constexpr (BF16) {
        const unsigned m0 = (t0 + 0 < valid ? 0x0000FFFFu : 0u) | (t0 + 1 < valid ? 0xFFFF0000u : 0u);
        const unsigned m1 = (t0 + 2 < valid ? 0x0000FFFFu : 0u) | (t0 + 3 < valid ? 0xFFFF0000u : 0u);
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c) {
            r.v[c][0] &= m0;
            r.v[c][1] &= m1;
        }
    } else {
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (t0 + j >= valid) r.v[c][j] = 0u;
    }
}

template <int D, bool BF16>
struct SegmentState {
    u32x4 q[Shape<D, BF16>::kKLoads];
    f32x4 o[Shape<D, BF16>::kChunks];
    float m;
    float l;
};

// Online-softmax update and weighted V for one page with `valid` tokens (1..16).
template <int D, bool BF16>
__device__ __forceinline__ void compute_page(SegmentState<D, BF16>& st, PageRegs<D, BF16>& pg,
                                             int valid, float scale_log2, int qg) {
    using S = Shape<D, BF16>;
    f32x4 s = page_scores<D, BF16>(pg, st.q);
    if (valid < kPageTokens) {
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = (4 * qg + r < valid) ? s[r] : -INFINITY;
        mask_v<D, BF16>(pg, valid, qg);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        s[r] *= scale_log2;
        mx = fmaxf(mx, s[r]);
    }
    // The running max m is the same on the four lanes of a head.  Only when some
    // lane sees a score above it is the page max reduced across lanes and the
    // accumulators rescaled; otherwise the reduced max would equal m and every
    // factor would be exactly 1, so skipping is bitwise identical.
    if (__builtin_amdgcn_ballot_w64(mx > st.m)) {
        const float m_new = fmaxf(st.m, wave_max_4(mx));
        const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
        st.l *= alpha;
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c) st.o[c] *= alpha;
        st.m = m_new;
    }
    float p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(s[r] - st.m);
    if constexpr (BF16) {
        __bf16 pb[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            pb[r] = static_cast<__bf16>(p[r]);
            st.l += static_cast<float>(pb[r]);
        }
        const s16x4 pv = {__builtin_bit_cast(short, pb[0]), __builtin_bit_cast(short, pb[1]),
                          __builtin_bit_cast(short, pb[2]), __builtin_bit_cast(short, pb[3])};
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c)
            st.o[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, pg.v[c]),
                                                                pv, st.o[c], 0, 0, 0);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) st.l += p[r];
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                st.o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    __uint_as_float(pg.v[c][j]), p[j], st.o[c], 0, 0, 0);
    }
}

// Fused merge: the split's partials cross between XCDs as device-scope
// stores and loads (cache-policy bit SC1 on gfx950).  The L2 of each XCD
// writes such stores through and does not serve such loads from its own
// lines, so neither the arrival nor the merge needs a whole-L2 write-back
// or invalidate.
constexpr int kScopeDevice = 16;  // SC1: device-scope coherence

// The workspace's partials through one buffer resource (offsets from part_o).
struct PartialsRsrc {
    __amdgpu_buffer_rsrc_t rs;
    const char* base;
    __device__ explicit PartialsRsrc(const DecodeArgs& a) : base(reinterpret_cast<const char*>(a.part_o)) {
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.part_o), static_cast<short>(0), 0x7FFFFFFF,
                                               kRsrcWord3);
    }
    __device__ unsigned off(const float* p) const {
        return static_cast<unsigned>(reinterpret_cast<const char*>(p) - base);
    }
    __device__ void store4(float* p, const f32x4& v) const {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, off(p), 0, kScopeDevice);
    }
    __device__ void store1(float* p, float v) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, off(p), 0, kScopeDevice);
    }
    __device__ f32x4 load4(const float* p) const {
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off(p), 0, kScopeDevice));
    }
    __device__ float load1(const float* p) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off(p), 0, kScopeDevice));
    }
};

__device__ __forceinline__ void lse_merge(float& M, float& den, f32x4& acc, float m2, float l2,
                                          const f32x4& o2) {
    const float Mn = fmaxf(M, m2);
    const float c1 = (M == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(M - Mn);
    const float c2 = (m2 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m2 - Mn);
    acc = acc * c1 + o2 * c2;
    den = den * c1 + l2 * c2;
    M = Mn;
}

// ceil-style worker of a unit: the worker that owns unit u - 1, for u >= 1.
__device__ __forceinline__ int unit_worker(int64_t u, int workers, int64_t total) {
    if (total * workers <= 0xFFFFFFFFll)
        return static_cast<int>((static_cast<unsigned>(u) * static_cast<unsigned>(workers) - 1u) /
                                static_cast<unsigned>(total));
    return static_cast<int>((u * workers - 1) / total);
}

// Partials of a segment of units [u_a, u_a + nb): one per worker that holds some
// of them, or one per unit with more workers than units.
__device__ __forceinline__ int seg_pieces(int64_t u_a, int nb, int64_t T, int N) {
    return N > T ? nb : unit_worker(u_a + nb, N, T) - unit_worker(u_a + 1, N, T) + 1;
}

template <int D, bool BF16>
__device__ __forceinline__ void store_quad(const DecodeArgs& a, int64_t orow, const f32x4& res) {
    if constexpr (BF16) {
        __bf16 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = static_cast<__bf16>(res[j]);
        *reinterpret_cast<u32x2*>(static_cast<__bf16*>(a.out) + orow) = __builtin_bit_cast(u32x2, v);
    } else {
        *reinterpret_cast<f32x4*>(static_cast<float*>(a.out) + orow) = res;
    }
}

// Every query head of (b, g) set to one value (rows with no pages, bad rows).
template <int D, bool BF16>
__device__ void fill_segment(const DecodeArgs& a, int b, int g, float value, int lane) {
    constexpr int kQuads = D / 4;
    for (int idx = lane; idx < a.group * kQuads; idx += kWave) {
        const int h = idx / kQuads, quad = idx % kQuads;
        store_quad<D, BF16>(a, (static_cast<int64_t>(b) * a.num_q_heads + g * a.group + h) * D + 4 * quad,
                            f32x4{value, value, value, value});
    }
}

// One wave merges every query head of segment (b, g): an item is (head, 4-dim
// quad), lane l takes items first + l + 64 it, in the order of the partials.  It
// is bound by the latency of device-scope loads, so kItems x kBatch of them are
// in flight together, and they are unconditional (past the end: the last item or
// partial again, unused): under a condition each waited for the ones before it.
// One row of 2K tokens (128 partials) 181 -> 65 us a call, 8 x 2K 50 -> 27 us;
// the merge before the unit stream, four partials at a time, 147 and 42 us.
template <int D, bool BF16, int kItems, int kBatch>
__device__ __forceinline__ void merge_items(const DecodeArgs& a, const PartialsRsrc& pr, int b, int g, int64_t u_a,
                                            int64_t T, int k_first, int count, int first, bool invalid, int lane) {
    constexpr int kQuads = D / 4;
    const int items = a.group * kQuads;
    const int gw = a.group_waves;
    const int64_t sseg = static_cast<int64_t>(b) * (a.num_kv_heads / gw) + g / gw;
    const int w = g % gw;
    const int N = a.waves / gw;
    int h[kItems], quad[kItems];
    float M[kItems], den[kItems];
    f32x4 acc[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int idx = first + it * kWave + lane < items ? first + it * kWave + lane : items - 1;
        h[it] = idx / kQuads;
        quad[it] = idx % kQuads;
        M[it] = -INFINITY;
        den[it] = 0.f;
        acc[it] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int i0 = 0; i0 < count; i0 += kBatch) {
        // lane j: the worker of partial i0 + j.  With more workers than units each
        // unit is a partial, held by the worker that owns it, else workers
        // k_first.. hold one each.
        const int i = i0 + lane < count ? i0 + lane : count - 1;
        const int k = N > T ? unit_worker(u_a + i + 1, N, T) : k_first + i;
        float mk[kBatch][kItems], lk[kBatch][kItems];
        f32x4 ok[kBatch][kItems];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int64_t slot = (static_cast<int64_t>(__builtin_amdgcn_readlane(k, j)) + sseg) * gw + w;
            const float* pml = a.part_ml + slot * 2 * a.group;
#pragma unroll
            for (int it = 0; it < kItems; ++it) {
                mk[j][it] = pr.load1(pml + h[it]);
                lk[j][it] = pr.load1(pml + a.group + h[it]);
                ok[j][it] = pr.load4(a.part_o + (slot * a.group + h[it]) * D + 4 * quad[it]);
            }
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (i0 + j < count)
#pragma unroll
                for (int it = 0; it < kItems; ++it) lse_merge(M[it], den[it], acc[it], mk[j][it], lk[j][it], ok[j][it]);
    }
    const float nan = __builtin_nanf("");
#pragma unroll
    for (int it = 0; it < kItems; ++it)
        if (first + it * kWave + lane < items)
            store_quad<D, BF16>(
                a, (static_cast<int64_t>(b) * a.num_q_heads + g * a.group + h[it]) * D + 4 * quad[it],
                invalid ? f32x4{nan, nan, nan, nan} : acc[it] / den[it]);
}

template <int D, bool BF16>
__device__ void combine_segment(const DecodeArgs& a, int b, int g, int64_t u_a, int nb, int64_t T,
                                int lane) {
    const PartialsRsrc pr(a);
    const int N = a.waves / a.group_waves;
    const int k_first = unit_worker(u_a + 1, N, T);
    const int count = seg_pieces(u_a, nb, T, N);
    const bool invalid = static_cast<int64_t>(a.seq_lens[b]) > kPageTokens * a.pt_stride;
    // all of a segment's items together where that leaves several partials in flight
    const int items = a.group * (D / 4);
    if (items <= kWave)
        merge_items<D, BF16, 1, 16>(a, pr, b, g, u_a, T, k_first, count, 0, invalid, lane);
    else if (items <= 2 * kWave)
        merge_items<D, BF16, 2, 8>(a, pr, b, g, u_a, T, k_first, count, 0, invalid, lane);
    else
        for (int first = 0; first < items; first += 4 * kWave)
            merge_items<D, BF16, 4, 4>(a, pr, b, g, u_a, T, k_first, count, first, invalid, lane);
}

// ---------------------------------------------------------------------------
// The unit stream.  A wave's units [u0, u1) are consecutive pages of one or
// more segments (row, head group).  Lane j of a chunk register holds unit
// base + j: its page id and a word saying which row and head group it belongs
// to and where it stands in its segment, so the loop needs one readlane per
// word and no arithmetic on rows.
constexpr unsigned kUnitRowMask = (1u << 13) - 1;  // row (kMaxDecodeBatch = 8192)
constexpr int kUnitGroupShift = 13;                // head group, 4 bits
constexpr unsigned kUnitFirst = 1u << 17;          // first unit of a piece: new queries, new accumulators
constexpr unsigned kUnitLast = 1u << 18;           // last unit of a piece: its result goes out
constexpr unsigned kUnitSegFirst = 1u << 19;       // the segment's first page
constexpr unsigned kUnitSegLast = 1u << 20;        // the segment's last page (the row's tail page)
constexpr unsigned kUnitNone = 1u << 27;           // past the end of the wave's units
// set by the load stage:
constexpr int kUnitTailShift = 21;                 // tokens of the page - 1, 4 bits (15 except on tail pages)
constexpr unsigned kUnitRowInvalid = 1u << 25;     // with kUnitSegLast: the length does not fit the table row
constexpr unsigned kUnitBad = 1u << 26;            // the page id names no page
constexpr unsigned kUnitQueries = 1u << 28;        // the piece's queries were loaded with this page
constexpr unsigned kUnitToken = 1u << 29;          // the row's new token was loaded with this page
static_assert(kMaxDecodeBatch <= (1 << 13), "row bits of a unit word");

struct UnitChunk {
    int pid;
    int len;  // the row's length
    unsigned word;
};

// Where a chunk starts: unit `off` of row b's units (heads * pages of them).
struct UnitPos {
    int b;
    unsigned off;
};

// Position of unit u (wave-uniform): a 64-way search of the row prefix, one LDS
// read per level.
__device__ __forceinline__ UnitPos unit_pos(const int32_t* s_pref, int batch, int heads, int64_t u, int lane) {
    const int64_t target = heads == 1 ? u
                           : (u >> 32) == 0 ? static_cast<int64_t>(static_cast<unsigned>(u) / static_cast<unsigned>(heads))
                                            : u / heads;
    int lo = 0, n = batch;  // the row is in [lo, lo + n)
    while (n > 1) {
        const int step = (n + kWave - 1) / kWave;
        const int i = lane * step;
        const bool le = i < n && s_pref[lo + i] <= target;
        const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(le)) - 1;  // row lo is always <= target
        lo += c * step;
        n = n - c * step < step ? n - c * step : step;
    }
    UnitPos p;
    p.b = lo;
    p.off = static_cast<unsigned>(u - static_cast<int64_t>(lds_uniform(s_pref + lo)) * heads);
    return p;
}

// Units [at, at + kUnits) of the stream, one per lane; `left` units remain from the
// chunk's start (lanes past them get kUnitNone).  Rows after the chunk's first are found by a
// galloping search: consecutive units are in the same or the next rows.
// A row has at most 2^27 pages (lengths are int32) and 16 head groups, so the
// offsets within a row fit 32 bits; `at` moves on to the next chunk.
template <int kUnits>
__device__ __forceinline__ UnitChunk load_units(const DecodeArgs& a, const int32_t* s_pref, int heads, UnitPos& at,
                                                int64_t left, bool worker_start, int lane) {
    const unsigned off = at.off + lane;
    const int32_t p0 = lds_uniform(s_pref + at.b);
    const bool in = lane < left && lane < kUnits;
    const int32_t q = static_cast<int32_t>(heads == 1 ? off : off / static_cast<unsigned>(heads));
    int b = at.b, step = 1;
    if (in) {
        while (b + step < a.batch && s_pref[b + step] - p0 <= q) {
            b += step;
            step <<= 1;
        }
        for (step >>= 1; step > 0; step >>= 1)
            if (b + step < a.batch && s_pref[b + step] - p0 <= q) b += step;
    }
    const int32_t first = s_pref[b];
    const unsigned nb = static_cast<unsigned>(s_pref[b + 1] - first);
    const unsigned rel = off - static_cast<unsigned>(heads) * static_cast<unsigned>(first - p0);
    const unsigned g = heads == 1 || !in ? 0u : rel / nb;
    const unsigned p = in ? rel - g * nb : 0u;
    // no branch around the loads (lanes past the end read their row's first
    // entry): they then land in the chunk's registers without a copy and its wait
    UnitChunk c;
    c.pid = a.page_table[static_cast<int64_t>(b) * a.pt_stride + p];
    c.len = a.seq_lens[b];
    unsigned word = static_cast<unsigned>(b) | (g << kUnitGroupShift);
    if (p == 0) word |= kUnitFirst | kUnitSegFirst;
    if (worker_start && lane == 0) word |= kUnitFirst;
    if (p == nb - 1) word |= kUnitLast | kUnitSegLast;
    if (lane == left - 1) word |= kUnitLast;
    c.word = in ? word : kUnitNone;
    at.b = __builtin_amdgcn_readlane(b, kUnits - 1);
    at.off = __builtin_amdgcn_readlane(rel, kUnits - 1) + 1;
    return c;
}

// Of 64-dim pages, a chunk's loads are waited for here.  Without this the first use
// in the page loop waits, in every round of the ring and so, from the second on,
// for nearly all pages in flight: one layer of 8 x 2K tokens, 16 heads of 64 dims,
// 17.6 us a call, now 16.6; 32 rows of 8K-32K, spilled pages and the append 431, now
// 404.  Pages of 128 dims keep the wait in the loop: they are twice as large, a round is
// two or three of them, and long rows stream slightly faster with fewer in flight
// (128 rows of 1K-256K, 32 query and 4 KV heads: 1,859 us a call with the wait in the
// loop, 1,871 here).
template <int D>
__device__ __forceinline__ void settle(UnitChunk& c) {
    if constexpr (D == 64) __asm__ volatile("" : "+v"(c.pid), "+v"(c.len));
}

// The V part of a row's new token (fused append): the element of each 16-dim
// chunk that the lane's V registers of the tail page take.
template <int D, bool BF16>
struct TokenV {
    unsigned v[Shape<D, BF16>::kChunks];
};

template <int D, bool BF16>
__device__ __forceinline__ void load_queries(u32x4* __restrict__ q, const DecodeArgs& a, int b, int g,
                                             int lane) {
    using S = Shape<D, BF16>;
    const int64_t row = static_cast<int64_t>(b) * a.num_q_heads + g * a.group;
    // lanes of head slots past the group read past the resource: zeros
    const __amdgpu_buffer_rsrc_t qr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(a.q) + row * (D * S::kElt)), static_cast<short>(0),
        a.group * D * S::kElt, kRsrcWord3);
    const unsigned off = static_cast<unsigned>((lane & 15) * D * S::kElt + 16 * (lane >> 4));
#pragma unroll
    for (int i = 0; i < S::kKLoads; ++i) q[i] = __builtin_amdgcn_raw_buffer_load_b128(qr, off + 64u * i, 0, 0);
}

template <int D, bool BF16>
__device__ __forceinline__ void load_token_v(TokenV<D, BF16>& t, const DecodeArgs& a, int b, int g, int lane) {
    const int64_t src = (static_cast<int64_t>(b) * a.num_kv_heads + g) * D + (lane & 15);
#pragma unroll
    for (int c = 0; c < Shape<D, BF16>::kChunks; ++c) {
        if constexpr (BF16)
            t.v[c] = static_cast<const unsigned short*>(a.v_new)[src + 16 * c];
        else
            t.v[c] = static_cast<const unsigned*>(a.v_new)[src + 16 * c];
    }
}

// Fused append (paged_decode_attention_append): row b's new token, k_new /
// v_new row b, is token L - 1 of the row, slot (L - 1) % 16 of its tail page.
// The lanes that hold the slot's K load it from k_new over the page's, and the
// lanes that hold its V put the new element in place of the page's, which may
// be the old or the new one by then; the same lanes store both to the page.
// So the append adds no wait.  No other wave reads that (page, KV head) in the
// launch.  Writing the token first and reading it back cost a load, a store and
// its acknowledgement before the row's first page load.  The page's K is loaded
// in any case: as two sides of a branch, the page's loads and the token's became
// two conditions in a row, and the token's waited for all pages in flight (16
// ragged rows up to 8K tokens, 16 heads of 64 dims, spilled pages, 67.5 us a
// call, now 64.4; 8 x 2K 20.7, now 19.9).
template <int D, bool BF16>
__device__ __forceinline__ void load_token_k(PageRegs<D, BF16>& pg, const DecodeArgs& a, int b, int g, int slot,
                                             int lane) {
    using S = Shape<D, BF16>;
    const char* ks = static_cast<const char*>(a.k_new) + (static_cast<int64_t>(b) * a.num_kv_heads + g) * D * S::kElt +
                     16 * (lane >> 4);
    if ((lane & 15) == slot) {
#pragma unroll
        for (int i = 0; i < S::kKLoads; ++i)
            pg.k[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ks + 64 * i));
    }
}

template <int D, bool BF16>
__device__ __forceinline__ void append_in_place(PageRegs<D, BF16>& pg, const TokenV<D, BF16>& t,
                                                __amdgpu_buffer_rsrc_t page, int slot, unsigned koff, unsigned voff,
                                                int lane) {
    using S = Shape<D, BF16>;
    if ((lane & 15) == slot) {
#pragma unroll
        for (int i = 0; i < S::kKLoads; ++i)
            __builtin_amdgcn_raw_buffer_store_b128(pg.k[i], page, koff + 1024u * (i % 4), 4096 * (i / 4), 0);
    }
    if ((lane >> 4) == slot >> 2) {
        const int j = slot & 3;
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c) {
            if constexpr (BF16) {
                const unsigned shift = (j & 1) * 16u, keep = ~(0xFFFFu << shift);
                const unsigned put = t.v[c] << shift;
                if (j >> 1)
                    pg.v[c][1] = (pg.v[c][1] & keep) | put;
                else
                    pg.v[c][0] = (pg.v[c][0] & keep) | put;
                __builtin_amdgcn_raw_buffer_store_b16(static_cast<unsigned short>(t.v[c]), page,
                                                      voff + 2u * j + 512u * c, S::kTile, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e == j) pg.v[c][e] = t.v[c];
                __builtin_amdgcn_raw_buffer_store_b32(t.v[c], page, voff + 4u * j + 1024u * (c % 4),
                                                      S::kTile + 4096 * (c / 4), 0);
            }
        }
    }
}

// Order this wave's LDS accesses: earlier writes complete before later reads,
// and the compiler moves no LDS access across it.
__device__ __forceinline__ void wave_lds_sync() { __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Holding results in LDS (calls with many rows: HOLD).  The counter that a
// wave's loads are waited for with also counts its stores, in order, and a store
// between the pages' reads is acknowledged late: each row written where it ended
// cost 2.4 us of the wave's stream (a ring run empty), a partial as much.  So a
// wave keeps the rows that it finishes in LDS, `out_slots` of them, and writes
// them together, as full 1 KiB stores, when the slots are full and when its
// range ends; the partial of the segment that its range starts inside of waits
// for the end too.  1,024 rows of 512 tokens: 186.7 -> 168.4 us a call (on other
// cards 177), of 256 to 768 tokens 189 -> 168 us, of 1,500 on average 498 -> 466 us
// (6.9 TB/s); 512 rows of 8 KV heads, 512 tokens on average, 183 -> 177 us; float32
// 192 -> 182 us.
constexpr int kLdsBudget = 60 << 10;  // of a 64 KiB launch, a few words of it static
constexpr int kMaxOutSlots = 8;
template <int D>
constexpr int kPartialBytes = 8 * (4 * D + 16);  // float32 rows of eight heads, 16 bytes past each other's banks

// Bytes of one slot: the group's output rows, laid out likewise.
__host__ __device__ __forceinline__ int out_slot_bytes(int group, int row_bytes) { return group * (row_bytes + 16); }

// A lane holds head lane % 16, dims 16 c + 4 (lane / 16) .. + 3 of chunk c,
// given by val(c): the group's rows into LDS.
template <int D, bool BF16, typename Val>
__device__ __forceinline__ void stage_heads(char* stage, int group, int lane, Val val) {
    constexpr int kElt = BF16 ? 2 : 4, kPitch = D * kElt + 16;
    if ((lane & 15) < group) {
        char* row = stage + (lane & 15) * kPitch + 4 * (lane >> 4) * kElt;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            const f32x4 x = val(c);
            if constexpr (BF16) {
                __bf16 v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = static_cast<__bf16>(x[j]);
                *reinterpret_cast<u32x2*>(row + 16 * c * kElt) = __builtin_bit_cast(u32x2, v);
            } else {
                *reinterpret_cast<f32x4*>(row + 16 * c * kElt) = x;
            }
        }
    }
}

// The staged rows to dst, where they follow each other.
template <int D, bool BF16>
__device__ __forceinline__ void write_heads(void* dst, const char* stage, int group, int lane) {
    constexpr int kRow = D * (BF16 ? 2 : 4), kPitch = kRow + 16;
    for (int o = 16 * lane; o < group * kRow; o += 16 * kWave)
        *reinterpret_cast<u32x4*>(static_cast<char*>(dst) + o) =
            *reinterpret_cast<const u32x4*>(stage + o / kRow * kPitch + o % kRow);
}

// What a wave holds: LDS with the partial's place, then the slots.
template <int D, bool BF16>
struct Held {
    static constexpr int kRow = D * Shape<D, BF16>::kElt;
    char* lds;
    int rows = 0;          // slots in use
    int row_seg = -1;      // lane i: the segment (b * KV heads + KV head) in slot i
    int part_slot = -1;    // the partial's slot in the workspace, or -1
    float part_m, part_l;

    __device__ __forceinline__ char* slot(const DecodeArgs& a, int i) const {
        return lds + kPartialBytes<D> + i * out_slot_bytes(a.group, kRow);
    }

    __device__ __forceinline__ void write_rows(const DecodeArgs& a, int lane) {
        wave_lds_sync();
        for (int i = 0; i < rows; ++i) {
            const int64_t seg = __builtin_amdgcn_readlane(row_seg, i);
            write_heads<D, BF16>(static_cast<char*>(a.out) + seg * a.group * kRow, slot(a, i), a.group, lane);
        }
        wave_lds_sync();
        rows = 0;
    }

    template <typename Val>
    __device__ __forceinline__ void row(const DecodeArgs& a, int seg, int lane, Val val) {
        if (rows == a.out_slots) write_rows(a, lane);
        stage_heads<D, BF16>(slot(a, rows), a.group, lane, val);
        row_seg = lane == rows ? seg : row_seg;
        ++rows;
    }

    __device__ __forceinline__ void write_all(const DecodeArgs& a, int lane) {
        if (part_slot >= 0) {
            wave_lds_sync();
            write_heads<D, false>(a.part_o + static_cast<int64_t>(part_slot) * a.group * D, lds, a.group, lane);
            if (lane < a.group) {
                float* pml = a.part_ml + static_cast<int64_t>(part_slot) * 2 * a.group;
                pml[lane] = part_m;
                pml[a.group + lane] = part_l;
            }
        }
        if (rows > 0) write_rows(a, lane);
    }
};

// A piece's result: the output rows themselves when the piece is its whole
// segment, else a partial (running max, weight sum, unnormalised output).
template <int D, bool BF16, bool FUSED, bool HOLD>
__device__ __forceinline__ void finish_piece(const DecodeArgs& a, Held<D, BF16>& held, SegmentState<D, BF16>& st,
                                             unsigned word, bool whole, bool bad, int worker, int heads, int w_in,
                                             int lane) {
    using S = Shape<D, BF16>;
    const int h = lane & 15, qg = lane >> 4;
    const int b = static_cast<int>(word & kUnitRowMask), hg = static_cast<int>((word >> kUnitGroupShift) & 15u);
    const int g = hg * a.group_waves + w_in;
    float l = wave_sum_4(st.l);
    if (bad) l = __builtin_nanf("");
    if (whole) {
        // (o + 0) / l is what merging this one partial gives
        if (word & kUnitRowInvalid) l = __builtin_nanf("");
        auto val = [&](int c) { return (st.o[c] + 0.f) / l; };
        if constexpr (HOLD) {
            held.row(a, b * a.num_kv_heads + g, lane, val);
        } else if (h < a.group) {
            const int64_t orow = (static_cast<int64_t>(b) * a.num_q_heads + g * a.group + h) * D + 4 * qg;
#pragma unroll
            for (int c = 0; c < S::kChunks; ++c) store_quad<D, BF16>(a, orow + 16 * c, val(c));
        }
        return;
    }
    const int64_t slot = (static_cast<int64_t>(worker) + static_cast<int64_t>(b) * heads + hg) * a.group_waves + w_in;
    if (HOLD && (word & kUnitSegLast) && a.group <= 8) {  // the range's first piece, at most one
        stage_heads<D, false>(held.lds, a.group, lane, [&](int c) { return st.o[c]; });
        held.part_m = st.m;
        held.part_l = l;
        held.part_slot = static_cast<int>(slot);
        return;
    }
    if (h < a.group) {
        float* po = a.part_o + (slot * a.group + h) * D + 4 * qg;
        float* pml = a.part_ml + slot * 2 * a.group;
        if constexpr (FUSED) {
            const PartialsRsrc pr(a);
#pragma unroll
            for (int c = 0; c < S::kChunks; ++c) pr.store4(po + 16 * c, st.o[c]);
            if (qg == 0) {
                pr.store1(pml + h, st.m);
                pr.store1(pml + a.group + h, l);
            }
        } else {
#pragma unroll
            for (int c = 0; c < S::kChunks; ++c) *reinterpret_cast<f32x4*>(po + 16 * c) = st.o[c];
            if (qg == 0) {
                pml[h] = st.m;
                pml[a.group + h] = l;
            }
        }
    }
}

// The segments (b * heads + head group) that a worker shares with others, or
// -1: the one its range starts inside of and finishes, and the one it does not
// finish, which it may also have started (it then is the first of that
// segment's workers).
struct SplitEnds {
    int first = -1, last = -1;
    bool last_starts = false;
};

// Fused merge: this wave's partials of the shared segments are stored; the wave
// that delivers a segment's last partial for its KV head merges them all.  The
// partials went out as device-scope stores: once they are acknowledged they are
// visible to every XCD, and the merging wave reads them back with device-scope
// loads.  Arrivals wait for the end of the worker's range, so that no ring is
// drained for them.
template <int D, bool BF16>
__device__ void merge_ends(const DecodeArgs& a, const int32_t* s_pref, const SplitEnds& ends, int heads, int w_in,
                           int64_t total_units, int lane) {
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
    for (int e = 0; e < 2; ++e) {
        const int seg = e ? ends.last : ends.first;
        if (seg < 0) continue;
        const int b = seg / heads, hg = seg % heads, g = hg * a.group_waves + w_in;
        const int nb = lds_uniform(s_pref + b + 1) - lds_uniform(s_pref + b);
        const int64_t seg_first = static_cast<int64_t>(lds_uniform(s_pref + b)) * heads + static_cast<int64_t>(hg) * nb;
        const int pieces = seg_pieces(seg_first, nb, total_units, a.waves / a.group_waves);
        int32_t* cnt = a.counters + b * a.num_kv_heads + g;
        int prev = 0;
        if (lane == 0) prev = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        prev = __builtin_amdgcn_readfirstlane(__shfl(prev, 0));
        if (prev + 1 == pieces) {
            combine_segment<D, BF16>(a, b, g, seg_first, nb, total_units, lane);
            if (lane == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next call
        }
    }
}

// Process units [u0, u1) of `worker`, KV head w_in of each unit's head group.
// R page buffers form a ring: step s issues unit s's loads and computes unit
// s - (R - 1), so R - 1 pages are in flight behind the one computed, across the
// ends of segments too: a new row costs its queries' registers and the old
// row's output, not a drained ring.  Every step issues exactly one page's loads
// (past the end with a resource of no records, which fetches nothing) and the
// loops have no exit inside a round of R steps, so that the compiler's waits
// for a page count just the pages ahead: with the loads under a condition, as with
// an early exit, they waited for nearly all of them (a chunk's list: see settle).  A piece's queries, and the V
// of a tail page's new token (fused append), are loaded ahead of their page into
// one set of registers each; where rows are so short that the set is still in
// use, they are loaded when their page is computed.
// Measured against one drained ring, row search and 64-bit division per piece
// (whole calls): 11 rows of up to 4K tokens, 16 heads of 64 dims, 33.2 -> 25.2
// us; 1,024 rows of 512 tokens 196 -> 187 us; 32 rows of 8K-32K tokens 211.8 ->
// 208.9 us (6.70 TB/s); a captured 48-layer step of 8 x 2K tokens with the fused
// append 955 -> 848 us.
template <int D, bool BF16, int R, bool TIERED, bool FUSED, bool APPEND, bool HOLD>
__device__ __forceinline__ SplitEnds run_units(const DecodeArgs& a, const int32_t* s_pref, int64_t u0, int64_t u1,
                                               int worker, int heads, int w_in, int lane, char* lds) {
    using S = Shape<D, BF16>;
    constexpr int kChunk = kWave / R * R;  // units per chunk: whole rounds of the ring
    SplitEnds ends;
    if (u1 <= u0) return ends;
    PageSrc ps;
    ps.hot = a.hot;
    ps.hot_stride = a.hot_stride;
    ps.num_hot = static_cast<unsigned>(a.num_pages);
    if constexpr (TIERED) {
        ps.cold = a.cold;
        ps.cold_stride = a.cold_stride;
        ps.stage = a.stage;
        ps.slice_bytes = a.slice_bytes;
        ps.num_cold = static_cast<unsigned>(a.num_cold_pages);
        ps.num_stage = static_cast<unsigned>(a.num_stage_slots);
    }
    const int qg = lane >> 4;
    const unsigned koff = 16u * lane;
    const unsigned voff = BF16 ? (32u * (lane & 15) + 8u * qg) : (64u * (lane & 15) + 16u * qg);

    PageRegs<D, BF16> ring[R];
    unsigned word[R];
    int pid[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        word[r] = kUnitNone;
        pid[r] = -1;
    }
    u32x4 q_next[S::kKLoads];
    TokenV<D, BF16> token;
    bool q_held = false, token_held = false;
    auto group_of = [&](unsigned w) { return static_cast<int>((w >> kUnitGroupShift) & 15u) * a.group_waves + w_in; };
    // the row takes a new token here: its tail page, and its length fits the table row
    auto takes_token = [](unsigned w) { return (w & (kUnitSegLast | kUnitRowInvalid)) == kUnitSegLast; };

    auto issue = [&](int r, const UnitChunk& c, int j) __attribute__((always_inline)) {
        pid[r] = __builtin_amdgcn_readlane(c.pid, j);
        unsigned w = __builtin_amdgcn_readlane(c.word, j);
        unsigned tail = kPageTokens - 1;
        if (w & kUnitSegLast) {
            const int len = __builtin_amdgcn_readlane(c.len, j);
            if (static_cast<int64_t>(len) > kPageTokens * a.pt_stride)
                w |= kUnitRowInvalid;
            else
                tail = static_cast<unsigned>(len - 1) % kPageTokens;
        }
        w |= tail << kUnitTailShift;
        const int b = static_cast<int>(w & kUnitRowMask), g = group_of(w);
        PageAddr page = page_addr<TIERED>(ps, pid[r], g * 2u * S::kTile);
        if (!page.ok) w |= kUnitBad;
        if (w & kUnitNone) page.ok = false;
        if ((w & kUnitFirst) && !q_held) {
            load_queries<D, BF16>(q_next, a, b, g, lane);
            w |= kUnitQueries;
            q_held = true;
        }
        const bool token_here = APPEND && takes_token(w) && !(w & kUnitNone);
        if (token_here && !token_held) {
            load_token_v<D, BF16>(token, a, b, g, lane);
            w |= kUnitToken;
            token_held = true;
        }
        const __amdgpu_buffer_rsrc_t rs = page_rsrc<D, BF16>(page);
        load_page_k<D, BF16>(ring[r], rs, koff);
        if (token_here) load_token_k<D, BF16>(ring[r], a, b, g, static_cast<int>(tail), lane);
        load_page_v<D, BF16>(ring[r], rs, voff);
        word[r] = w;
    };

    SegmentState<D, BF16> st;
    Held<D, BF16> held;
    held.lds = lds;
    bool bad = false, seg_first = false;
    // What a unit needs besides its page, taken before the step's own loads go
    // out: those may load the next queries or token into the same registers.
    auto begin = [&](int r) __attribute__((always_inline)) {
        const unsigned w = __builtin_amdgcn_readfirstlane(word[r]);
        if (w & kUnitNone) return;
        const int b = static_cast<int>(w & kUnitRowMask), g = group_of(w);
        if (w & kUnitFirst) {
            if (w & kUnitQueries) {
#pragma unroll
                for (int i = 0; i < S::kKLoads; ++i) st.q[i] = q_next[i];
                q_held = false;
            } else {  // q_next holds a later piece's
                load_queries<D, BF16>(st.q, a, b, g, lane);
                // waited for here, so that the usual way keeps its pages in flight
#pragma unroll
                for (int i = 0; i < S::kKLoads; ++i) __asm__ volatile("" : "+v"(st.q[i]));
            }
#pragma unroll
            for (int c = 0; c < S::kChunks; ++c) st.o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            st.m = -INFINITY;
            st.l = 0.f;
            bad = false;
            seg_first = (w & kUnitSegFirst) != 0;
        }
        if (APPEND && takes_token(w)) {
            const __amdgpu_buffer_rsrc_t page = page_rsrc<D, BF16>(
                page_addr<TIERED>(ps, __builtin_amdgcn_readfirstlane(pid[r]), g * 2u * S::kTile));
            const int slot = static_cast<int>((w >> kUnitTailShift) & 15u);
            if (w & kUnitToken) {
                append_in_place<D, BF16>(ring[r], token, page, slot, koff, voff, lane);
                token_held = false;
            } else {  // `token` holds a later row's
                TokenV<D, BF16> late;
                load_token_v<D, BF16>(late, a, b, g, lane);
                // waited for here, where they are loaded: not all lanes use them, and
                // with loads possibly left in flight every page of every row was waited
                // for before the next one's could go out (24 rows of 8K-32K tokens with
                // spilled pages, 16 heads of 64 dims: 490 us a call, now 297; 32 query and
                // 4 KV heads of 128: 161, now 137)
#pragma unroll
                for (int c = 0; c < S::kChunks; ++c) __asm__ volatile("" : "+v"(late.v[c]));
                append_in_place<D, BF16>(ring[r], late, page, slot, koff, voff, lane);
            }
        }
    };
    auto compute = [&](int r) __attribute__((always_inline)) {
        const unsigned w = __builtin_amdgcn_readfirstlane(word[r]);
        if (w & kUnitNone) return;
        bad |= (w & kUnitBad) != 0;
        const int tail = static_cast<int>((w >> kUnitTailShift) & 15u);  // last valid slot
        compute_page<D, BF16>(st, ring[r], tail + 1, a.scale_log2, qg);
        if (w & kUnitLast) {
            const int seg = static_cast<int>(w & kUnitRowMask) * heads + static_cast<int>((w >> kUnitGroupShift) & 15u);
            const bool seg_last = (w & kUnitSegLast) != 0;
            if (seg_last && !seg_first) ends.first = seg;
            if (!seg_last) {
                ends.last = seg;
                ends.last_starts = seg_first;
            }
            finish_piece<D, BF16, FUSED, HOLD>(a, held, st, w, seg_first && seg_last, bad, worker, heads, w_in, lane);
        }
    };

    UnitPos at = unit_pos(s_pref, a.batch, heads, u0, lane);
    UnitChunk nxt = load_units<kChunk>(a, s_pref, heads, at, u1 - u0, true, lane);
    settle<D>(nxt);
    // steps left: every unit is issued once and computed R - 1 steps later
    for (int64_t left = u1 - u0 + (R - 1); left > 0; left -= kChunk) {
        const UnitChunk cur = nxt;
        const int steps = __builtin_amdgcn_readfirstlane(static_cast<int>(left < kChunk ? left : kChunk));
        nxt = load_units<kChunk>(a, s_pref, heads, at, left - (R - 1) - kChunk, false, lane);
        for (int j = 0; j < steps; j += R) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                begin((r + 1) % R);
                issue(r, cur, j + r);
                compute((r + 1) % R);
            }
        }
        settle<D>(nxt);
    }
    if constexpr (HOLD) held.write_all(a, lane);
    return ends;
}

// ---------------------------------------------------------------------------
// Vector-ALU variant (bf16, at most 8 query heads per KV head).  Same work
// split, page loads, partial format and combine as the matrix-core path; both
// products run as v_dot2_f32_bf16 instead.  It exists to measure the choice of
// matrix cores on the same memory schedule.
//
// Scores: lane (t = l % 16, qq = l / 16) holds a quarter of token t's dims (the
// K loads are shared with the matrix-core path), so it forms partial dot
// products for all 8 head slots from the group's queries in LDS, and a
// reduce-scatter over the quarters leaves lane (t, qq) with the full scores of
// heads 2 qq and 2 qq + 1.  The bf16 weights cross to the output layout through
// 256 bytes of LDS.  Output: lane (dl, qg) holds dims 16 c + dl of tokens
// 4 qg .. 4 qg + 3 for every chunk c (the V loads of the matrix-core path) and
// accumulates all 8 head slots over its tokens; the four token quarters are
// summed once per piece.
constexpr int kValuMaxGroup = 8;

template <int D>
struct ValuLds {
    u32x4 q[(D / 8) * kValuMaxGroup];  // [load i][head][quarter qq]: dims 8 (4 i + qq) .. + 7
    unsigned p[kPageTokens * 4];       // [token][qq]: bf16 weights of heads 2 qq, 2 qq + 1
};

template <int D>
struct ValuState {
    float o[kValuMaxGroup][D / 16];  // lane (dl, qg): head h, dim 16 c + dl, over tokens 4 qg .. + 3
    float m[2], l[2];                // lane (t, qq): heads 2 qq + e; l over token t only
};

__device__ __forceinline__ float dot2_bf16(unsigned a, unsigned b, float c) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c,
                                           false);
}

__device__ __forceinline__ float readlane_f(float x, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// The value of lane ^ mask.  __shfl_xor computes the source lane's index anew,
// with a bound that a wave of 64 does not need, and the compiler leaves that in
// the page loop: 26 of the 260 instructions up to a page's weights.  32 rows of
// 8K-32K tokens, 32 query and 4 KV heads of 128 dims: 345 us a call with it, 339
// with the index taken from `lane`.
__device__ __forceinline__ float lane_xor(float x, int lane, int mask) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * (lane ^ mask), __builtin_bit_cast(int, x)));
}

template <int D>
__device__ __forceinline__ void compute_page_valu(ValuState<D>& st, PageRegs<D, true>& pg, int valid,
                                                  float scale_log2, int lane, ValuLds<D>& sm) {
    using S = Shape<D, true>;
    const int t = lane & 15, qq = lane >> 4, qg = lane >> 4;
    // partial scores of token t over this lane's dims, all 8 head slots
    float s[kValuMaxGroup];
#pragma unroll
    for (int h = 0; h < kValuMaxGroup; ++h) s[h] = 0.f;
#pragma unroll
    for (int i = 0; i < S::kKLoads; ++i) {
#pragma unroll
        for (int h = 0; h < kValuMaxGroup; ++h) {
            const u32x4 qv = sm.q[(i * kValuMaxGroup + h) * 4 + qq];
#pragma unroll
            for (int j = 0; j < 4; ++j) s[h] = dot2_bf16(pg.k[i][j], qv[j], s[h]);
        }
    }
    // reduce-scatter over the quarters: lanes l and l ^ 32 split heads 0-3 / 4-7,
    // then lanes l and l ^ 16 split each half in pairs
    const bool upper = lane >= 32, odd = (lane & 16) != 0;
    float k4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float send = upper ? s[j] : s[4 + j];
        k4[j] = (upper ? s[4 + j] : s[j]) + lane_xor(send, lane, 32);
    }
    float sh[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float send = odd ? k4[e] : k4[2 + e];
        sh[e] = (odd ? k4[2 + e] : k4[e]) + lane_xor(send, lane, 16);
    }
    // online softmax for heads 2 qq + e at token t (same lazy rescale as above)
#pragma unroll
    for (int e = 0; e < 2; ++e) sh[e] = t < valid ? sh[e] * scale_log2 : -INFINITY;
    if (__builtin_amdgcn_ballot_w64(sh[0] > st.m[0] || sh[1] > st.m[1])) {
        float mx[2] = {sh[0], sh[1]};
#pragma unroll
        for (int o = 1; o < 16; o <<= 1)
#pragma unroll
            for (int e = 0; e < 2; ++e) mx[e] = fmaxf(mx[e], lane_xor(mx[e], lane, o));
        float alpha[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float mn = fmaxf(st.m[e], mx[e]);
            alpha[e] = __builtin_amdgcn_exp2f(st.m[e] - mn);
            st.l[e] *= alpha[e];
            st.m[e] = mn;
        }
#pragma unroll
        for (int h = 0; h < kValuMaxGroup; ++h) {
            const float ah = readlane_f(alpha[h & 1], 16 * (h >> 1));
#pragma unroll
            for (int c = 0; c < S::kChunks; ++c) st.o[h][c] *= ah;
        }
    }
    __bf16 pb[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        pb[e] = static_cast<__bf16>(__builtin_amdgcn_exp2f(sh[e] - st.m[e]));
        st.l[e] += static_cast<float>(pb[e]);
    }
    sm.p[t * 4 + qq] = static_cast<unsigned>(__builtin_bit_cast(unsigned short, pb[0])) |
                       (static_cast<unsigned>(__builtin_bit_cast(unsigned short, pb[1])) << 16);
    wave_lds_sync();
    // w[j][hp] = weights of heads 2 hp, 2 hp + 1 at token 4 qg + j
    u32x4 w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = *reinterpret_cast<const u32x4*>(sm.p + 4 * (4 * qg + j));
    unsigned p01[kValuMaxGroup], p23[kValuMaxGroup];
#pragma unroll
    for (int hp = 0; hp < 4; ++hp) {
        p01[2 * hp] = (w[0][hp] & 0xFFFFu) | (w[1][hp] << 16);
        p01[2 * hp + 1] = (w[0][hp] >> 16) | (w[1][hp] & 0xFFFF0000u);
        p23[2 * hp] = (w[2][hp] & 0xFFFFu) | (w[3][hp] << 16);
        p23[2 * hp + 1] = (w[2][hp] >> 16) | (w[3][hp] & 0xFFFF0000u);
    }
    if (valid < kPageTokens) mask_v<D, true>(pg, valid, qg);
#pragma unroll
    for (int c = 0; c < S::kChunks; ++c)
#pragma unroll
        for (int h = 0; h < kValuMaxGroup; ++h) {
            st.o[h][c] = dot2_bf16(pg.v[c][0], p01[h], st.o[h][c]);
            st.o[h][c] = dot2_bf16(pg.v[c][1], p23[h], st.o[h][c]);
        }
    __asm__ volatile("" ::: "memory");  // the next page's weight writes stay after these reads
}

// Fused append, vector-ALU form: the piece holding a row's last
// page first writes the row's new token, k_new / v_new row b for this wave's
// KV head, into that page at slot (L - 1) % 16, then orders those stores before
// its own loads of the page (the same wave is the only reader of that page's
// tiles for this KV head in the launch).  Rows with L <= 0 or an invalid L, and
// tail entries that name no page (or a staging slot), write nothing.
template <int D, bool TIERED>
__device__ __forceinline__ void append_new_token(const DecodeArgs& a, const PageSrc& ps, const int32_t* row,
                                                 const Piece& pc, int nb, int seq_len, int lane) {
    using S = Shape<D, true>;
    if (!a.k_new || pc.p1 != nb || seq_len <= 0 || a.seq_lens[pc.b] != seq_len) return;
    unsigned id = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(row[nb - 1]));
    const char* base = ps.hot;
    int64_t stride = ps.hot_stride;
    unsigned n = ps.num_hot;
    if constexpr (TIERED) {
        const unsigned tag = id >> 29;  // 0 hot, 2 cold; a staged slot is a copy, not the page
        id &= static_cast<unsigned>(kPageIdMask);
        if (tag == 2) {
            base = ps.cold;
            stride = ps.cold_stride;
            n = ps.num_cold;
        } else if (tag != 0) {
            n = 0;
        }
    }
    if (id >= n) return;
    char* lh = const_cast<char*>(base) + static_cast<int64_t>(id) * stride;
    const int slot = (seq_len - 1) % kPageTokens;
    const int64_t src = (static_cast<int64_t>(pc.b) * a.num_kv_heads + pc.g) * D * S::kElt;
    const char* ks = static_cast<const char*>(a.k_new) + src;
    const char* vs = static_cast<const char*>(a.v_new) + src;
    constexpr int x = 16 / S::kElt;  // elements per 16-byte group of the K tile
    if (lane < D / x)
        *reinterpret_cast<u32x4*>(lh + (static_cast<int64_t>(lane) * kPageTokens + slot) * 16) =
            *reinterpret_cast<const u32x4*>(ks + 16 * lane);
    for (int d = lane; d < D; d += kWave) {
        char* vd = lh + S::kTile + (static_cast<int64_t>(d) * kPageTokens + slot) * S::kElt;
        *reinterpret_cast<unsigned short*>(vd) = reinterpret_cast<const unsigned short*>(vs)[d];
    }
    // Other lanes of this wave read these bytes back with the page's loads.  A
    // workgroup-scope release/acquire orders that in the memory model; waiting
    // for the stores to be acknowledged makes the order independent of how the
    // L1 treats the nontemporal loads (once per row's tail page: negligible).
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ int load_ids(const int32_t* __restrict__ row, int first, int end,
                                        int lane) {
    const int i = first + lane;
    return i < end ? row[i] : -1;
}

template <int D, bool TIERED>
__device__ __forceinline__ void load_page_id(PageRegs<D, true>& r, const PageSrc& ps, int pid, bool& bad,
                                             unsigned koff, unsigned voff) {
    const PageAddr page = page_addr<TIERED>(ps, pid, 0);
    const __amdgpu_buffer_rsrc_t rs = page_rsrc<D, true>(page);
    load_page_k<D, true>(r, rs, koff);
    load_page_v<D, true>(r, rs, voff);
    bad |= !page.ok;
}

// Pages [p0, p1) of row b, KV head g, into the partial's slot or the output.
template <int D, int R, bool TIERED>
__device__ void run_piece_valu(const DecodeArgs& a, const Piece& pc, int nb, int seq_len, bool row_invalid,
                               int lane, ValuLds<D>& sm) {
    using S = Shape<D, true>;
    constexpr int kGroups = D / 8;
    // the group's queries (zero beyond `group` heads) into LDS
    wave_lds_sync();  // the previous piece's reads are done
    {
        const __bf16* qrow = static_cast<const __bf16*>(a.q) +
                             (static_cast<int64_t>(pc.b) * a.num_q_heads + pc.g * a.group) * D;
        for (int e = lane; e < kGroups * kValuMaxGroup; e += kWave) {
            const int h = e / kGroups, grp = e % kGroups;
            const u32x4 v = h < a.group ? *reinterpret_cast<const u32x4*>(qrow + h * D + 8 * grp)
                                        : u32x4{0u, 0u, 0u, 0u};
            sm.q[((grp >> 2) * kValuMaxGroup + h) * 4 + (grp & 3)] = v;
        }
    }
    wave_lds_sync();
    ValuState<D> st;
#pragma unroll
    for (int h = 0; h < kValuMaxGroup; ++h)
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c) st.o[h][c] = 0.f;
    st.m[0] = st.m[1] = -INFINITY;
    st.l[0] = st.l[1] = 0.f;
    bool bad = false;

    const int32_t* row = a.page_table + static_cast<int64_t>(pc.b) * a.pt_stride;
    const int64_t head_off = static_cast<int64_t>(pc.g) * 2 * S::kTile;
    PageSrc ps;
    ps.hot = a.hot + head_off;
    ps.hot_stride = a.hot_stride;
    ps.num_hot = static_cast<unsigned>(a.num_pages);
    if constexpr (TIERED) {
        ps.cold = a.cold + head_off;
        ps.cold_stride = a.cold_stride;
        ps.stage = a.stage + head_off;
        ps.slice_bytes = a.slice_bytes;
        ps.num_cold = static_cast<unsigned>(a.num_cold_pages);
        ps.num_stage = static_cast<unsigned>(a.num_stage_slots);
    }
    append_new_token<D, TIERED>(a, ps, row, pc, nb, seq_len, lane);
    const int qg = lane >> 4;
    const unsigned koff = 16u * lane;
    const unsigned voff = 32u * (lane & 15) + 8u * qg;
    const int tail_valid = seq_len - kPageTokens * (nb - 1);

    int ids_cur = load_ids(row, pc.p0, pc.p1, lane);
    int ids_nxt = load_ids(row, pc.p0 + kWave, pc.p1, lane);
    int cur_chunk = 0;
    auto pid_at = [&](int i) -> int {
        const int rel = i - pc.p0;
        const int cc = rel >> 6;
        if (cc != cur_chunk) {
            ids_cur = ids_nxt;
            cur_chunk = cc;
            ids_nxt = load_ids(row, pc.p0 + kWave * (cc + 1), pc.p1, lane);
        }
        return __builtin_amdgcn_readlane(ids_cur, rel & 63);
    };

    PageRegs<D, true> buf[R];
#pragma unroll
    for (int r = 0; r < R - 1; ++r)
        if (pc.p0 + r < pc.p1) load_page_id<D, TIERED>(buf[r], ps, pid_at(pc.p0 + r), bad, koff, voff);
    for (int i = pc.p0; i < pc.p1; i += R) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int ip = i + r;
            if (ip < pc.p1) {
                const int ahead = ip + R - 1;
                if (ahead < pc.p1)
                    load_page_id<D, TIERED>(buf[(r + R - 1) % R], ps, pid_at(ahead), bad, koff, voff);
                compute_page_valu<D>(st, buf[r], ip == nb - 1 ? tail_valid : kPageTokens, a.scale_log2,
                                     lane, sm);
            }
        }
    }

    // outputs: reduce-scatter over the token quarters (lane (dl, qg) keeps heads
    // 2 qg, 2 qg + 1), then every lane writes its two heads' dims 16 c + dl
    const bool upper = lane >= 32, odd = (lane & 16) != 0;
    float o4[4][S::kChunks];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c) {
            const float send = upper ? st.o[j][c] : st.o[4 + j][c];
            o4[j][c] = (upper ? st.o[4 + j][c] : st.o[j][c]) + lane_xor(send, lane, 32);
        }
    float o2[2][S::kChunks];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int c = 0; c < S::kChunks; ++c) {
            const float send = odd ? o4[e][c] : o4[2 + e][c];
            o2[e][c] = (odd ? o4[2 + e][c] : o4[e][c]) + lane_xor(send, lane, 16);
        }
    // weight sums: lane (t, qq) holds token t's share of heads 2 qq + e
    float l[2] = {st.l[0], st.l[1]};
#pragma unroll
    for (int o = 1; o < 16; o <<= 1)
#pragma unroll
        for (int e = 0; e < 2; ++e) l[e] += lane_xor(l[e], lane, o);
    const int dl = lane & 15;
    if (pc.p0 == 0 && pc.p1 == nb) {
        // the whole segment: write its output (what merging one partial gives)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int h = 2 * qg + e;
            if (h < a.group) {
                const float den = bad ? __builtin_nanf("") : l[e];
                __bf16* orow = static_cast<__bf16*>(a.out) +
                               (static_cast<int64_t>(pc.b) * a.num_q_heads + pc.g * a.group + h) * D + dl;
#pragma unroll
                for (int c = 0; c < S::kChunks; ++c)
                    orow[16 * c] = static_cast<__bf16>(row_invalid ? __builtin_nanf("") : (o2[e][c] + 0.f) / den);
            }
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int h = 2 * qg + e;
        if (h < a.group) {
            float* po = a.part_o + (static_cast<int64_t>(pc.slot) * a.group + h) * D + dl;
#pragma unroll
            for (int c = 0; c < S::kChunks; ++c) po[16 * c] = o2[e][c];
            if (dl == 0) {
                float* pml = a.part_ml + static_cast<int64_t>(pc.slot) * 2 * a.group;
                pml[h] = st.m[e];
                pml[a.group + h] = bad ? __builtin_nanf("") : l[e];
            }
        }
    }
}

// Register budget of the split kernel: 512 / n registers, so that n waves fit a
// SIMD.  With 256 the shapes below keep everything in VGPRs; with 512 the
// compiler holds the accumulators in AGPRs and moves all of them in and out on
// every page.  The float32 128-dim shape needs more than 256.
template <int D, bool BF16>
constexpr int split_waves_per_eu() {
    return D == 128 && !BF16 ? 1 : 2;
}

// Dynamic LDS of the split: the row prefix, then (HOLD) what each wave holds, in
// 16-byte words: the array is declared with that alignment, which otherwise would
// depend on the sizes of the static arrays before it.
__host__ __device__ __forceinline__ int prefix_lds_bytes(int batch) { return (4 * (batch + 1) + 15) & ~15; }

template <int D>
__host__ __device__ __forceinline__ int held_lds_bytes(int group, int row_bytes, int out_slots) {
    return kPartialBytes<D> + out_slots * out_slot_bytes(group, row_bytes);
}

// What a wave of the split works on: its worker, its KV head within the
// worker's head group and its units [u0, u1).
struct WaveWork {
    int wave, worker, w_in, heads, lane;
    int64_t total, u0, u1;
};

// The row prefix into LDS (and by the first block to the workspace, where the
// combine reads it), then this wave's share; false for waves past the last.
__device__ __forceinline__ bool wave_work(const DecodeArgs& a, int32_t* s_pref, WaveWork& w) {
    block_prefix_pages<kSplitBlockThreads>(a.seq_lens, a.batch, a.pt_stride, s_pref);
    if (blockIdx.x == 0)
        for (int b = threadIdx.x; b <= a.batch; b += kSplitBlockThreads) a.row_pref[b] = s_pref[b];
    w.lane = threadIdx.x & (kWave - 1);
    w.wave = __builtin_amdgcn_readfirstlane(blockIdx.x * kSplitBlockWaves + threadIdx.x / kWave);
    if (w.wave >= a.waves) return false;
    const int gw = a.group_waves;
    w.heads = a.num_kv_heads / gw;
    w.worker = w.wave / gw;
    w.w_in = w.wave % gw;
    w.total = static_cast<int64_t>(lds_uniform(s_pref + a.batch)) * w.heads;
    wave_units(w.total, w.worker, a.waves / gw, w.u0, w.u1);
    return true;
}

// Rows with no pages get no pieces: their output is written here (0 for L = 0,
// NaN for L < 0), after the wave's own units.
template <int D, bool BF16>
__device__ __forceinline__ void fill_empty_rows(const DecodeArgs& a, const int32_t* s_pref, const WaveWork& w) {
    for (int seg = w.wave; seg < a.batch * a.num_kv_heads; seg += a.waves) {
        const int b = seg / a.num_kv_heads;
        if (lds_uniform(s_pref + b) == lds_uniform(s_pref + b + 1))
            fill_segment<D, BF16>(a, b, seg % a.num_kv_heads, a.seq_lens[b] == 0 ? 0.f : __builtin_nanf(""), w.lane);
    }
}

template <int D, bool BF16, int R, bool TIERED, bool FUSED, bool APPEND, bool HOLD>
__global__ __launch_bounds__(kSplitBlockThreads)
__attribute__((amdgpu_waves_per_eu(split_waves_per_eu<D, BF16>()))) void decode_split_kernel(DecodeArgs a) {
    extern __shared__ __align__(16) int32_t s_pref[];
    static_assert(__alignof__(s_pref) >= 16, "Held reads and writes 16-byte words behind the prefix");
    WaveWork w;
    if (!wave_work(a, s_pref, w)) return;
    const SplitEnds ends = run_units<D, BF16, R, TIERED, FUSED, APPEND, HOLD>(
        a, s_pref, w.u0, w.u1, w.worker, w.heads, w.w_in, w.lane,
        reinterpret_cast<char*>(s_pref) + prefix_lds_bytes(a.batch) +
            threadIdx.x / kWave * held_lds_bytes<D>(a.group, D * Shape<D, BF16>::kElt, a.out_slots));
    if constexpr (FUSED)
        merge_ends<D, BF16>(a, s_pref, ends, w.heads, w.w_in, w.total, w.lane);
    else if (w.w_in == 0 && w.lane == 0)
        a.split_segs[w.worker] = ends.last_starts ? ends.last : -1;
    fill_empty_rows<D, BF16>(a, s_pref, w);
}

// The vector-ALU form walks its range piece by piece.
template <int D, int R, bool TIERED>
__global__ __launch_bounds__(kSplitBlockThreads) void decode_split_valu_kernel(DecodeArgs a) {
    extern __shared__ __align__(16) int32_t s_pref[];
    __shared__ ValuLds<D> s_valu[kSplitBlockWaves];
    WaveWork w;
    if (!wave_work(a, s_pref, w)) return;
    int32_t split_seg = -1;
    int64_t u = w.u0;
    while (u < w.u1) {
        Piece pc = piece_at<true>(s_pref, a.batch, w.heads, w.worker, u, w.u1);
        if (pc.p1 <= pc.p0) break;  // cannot happen for a consistent prefix; never spin
        const int nb = lds_uniform(s_pref + pc.b + 1) - lds_uniform(s_pref + pc.b);
        const int32_t len = a.seq_lens[pc.b];
        const int seq_len = len < kPageTokens * nb ? len : kPageTokens * nb;
        const bool row_invalid = static_cast<int64_t>(len) > kPageTokens * a.pt_stride;
        if (pc.p0 == 0 && pc.p1 < nb) split_seg = pc.b * w.heads + pc.g;
        const int span = pc.p1 - pc.p0;
        pc.g = pc.g * a.group_waves + w.w_in;
        pc.slot = pc.slot * a.group_waves + w.w_in;
        run_piece_valu<D, R, TIERED>(a, pc, nb, seq_len, row_invalid, w.lane, s_valu[threadIdx.x / kWave]);
        u += span;
    }
    if (w.w_in == 0 && w.lane == 0) a.split_segs[w.worker] = split_seg;
    fill_empty_rows<D, true>(a, s_pref, w);
}

// Merge the partials of one (b, g) for one query head and write its output row.
// The D/4 lanes of a lane group each own four output dims, and lane groups take
// every stride-th partial; loads for four partials are issued before any of
// them is merged.  A head has kWaves waves: one (four heads per block) where
// segments have few partials, else a block of four or sixteen whose waves merge
// their results through LDS.  The partials of a segment are those of workers
// k_first..k_last when there are no more workers than units (each then holds
// at least one), and one per unit (the worker that owns it) otherwise.  Only
// segments split over several workers have partials (the split writes the
// others' output itself): the grid walks either all segments, skipping the
// rest, or, when workers are fewer than segments, the workers' split-segment
// entries.  The kernel is a chain of three memory latencies; dropping the
// 64-bit divisions between them (two of them per partial, for a condition that
// always holds) and giving long segments sixteen waves took the float32
// call of 16 ragged rows (48 partials each) from 25.0 to 23.1 us, one row of 32K
// tokens (192 partials) 11.8 -> 6.9 us in this kernel, and a captured 48-layer step
// of 8 x 2K tokens, with the shorter prefix sum, 848 -> 804 us (775 with the waves
// that `used` counts below and the append's waits gone).
constexpr int kWideCombinePieces = 12;   // partials per segment from which four waves share a head
constexpr int kWidestCombinePieces = 64; // and sixteen: 63 partials of 128 dims 9.6 us a captured call with four
                                         // waves, 9.3 with sixteen; 96 of 64 dims (float32) 10.6 and 10.3
constexpr int kCombineUnroll = 4;        // partials a lane loads before it merges any

template <int D, bool BF16, int kWaves>
__global__ __launch_bounds__(kWaves == 1 ? kBlockThreads : kWaves * kWave) void decode_combine_kernel(DecodeArgs a) {
    constexpr bool kWide = kWaves > 1;
    constexpr int kQuads = D / 4;
    constexpr int kGroups = kWave / kQuads;
    constexpr int kUnroll = kCombineUnroll;
    __shared__ float s_merge[kWaves][kQuads][6];
    const int wave = threadIdx.x / kWave;
    const int Lw = a.group_waves;
    const int heads = a.num_kv_heads / Lw;
    int b, g, hy;
    if (a.combine_by_worker) {
        // blockIdx.x: a worker; blockIdx.y: (KV head within the head group, head block)
        const int32_t e = a.split_segs[blockIdx.x];
        if (e < 0) return;  // whole block
        const int ny = kWide ? a.group : (a.group + kBlockWaves - 1) / kBlockWaves;
        b = e / heads;
        g = (e % heads) * Lw + static_cast<int>(blockIdx.y) / ny;
        hy = static_cast<int>(blockIdx.y) % ny;
    } else {
        b = static_cast<int>(blockIdx.x) / a.num_kv_heads;
        g = static_cast<int>(blockIdx.x) % a.num_kv_heads;
        hy = static_cast<int>(blockIdx.y);
    }
    const int h = kWide ? hy : hy * kBlockWaves + wave;
    if (h >= a.group) return;  // never taken by a wide block: its grid has one block per head
    const int lane = threadIdx.x & (kWave - 1);
    const int quad = lane % kQuads, grp = lane / kQuads;
    const int gid = kWide ? wave * kGroups + grp : grp;

    // pages of the rows before b, and of all rows (the split kernel's prefix)
    const int32_t before = a.row_pref[b], total = a.row_pref[a.batch];
    const int nb = a.row_pref[b + 1] - before;
    const int32_t len = a.seq_lens[b];
    // The split wrote rows with no pages and segments it did not split
    // (uniform over the block: a wide block holds one segment).
    if (nb == 0) return;
    const bool invalid = static_cast<int64_t>(len) > kPageTokens * a.pt_stride;
    // units of head group g / Lw over the workers' ranges; this head's partials
    // are slot (worker + b * heads + g / Lw) * Lw + g % Lw
    const int hg = g / Lw, w_in = g - hg * Lw;
    const int64_t sseg = static_cast<int64_t>(b) * heads + hg;
    const int64_t T = static_cast<int64_t>(total) * heads;
    const int64_t u_a = static_cast<int64_t>(before) * heads + static_cast<int64_t>(hg) * nb;
    const int N = a.waves / Lw;
    const int k_first = unit_worker(u_a + 1, N, T);
    const bool per_unit = N > T;  // every non-empty wave holds exactly one unit
    const int count = per_unit ? nb : unit_worker(u_a + nb, N, T) - k_first + 1;
    if (count == 1) return;
    // Waves that get partials: as many as have kUnroll per lane group.  With the
    // partials dealt to all sixteen, the fifteen merges through LDS cost more than
    // the shorter loop saves (captured calls, one row of 1K tokens: 63 partials
    // 9.7 -> 7.9 us a call with 64 dims, 10.6 -> 9.3 with 128; four waves took 8.2 and 10.9).
    const int used = kWide ? min(kWaves, (count + kUnroll * kGroups - 1) / (kUnroll * kGroups)) : 1;
    const int stride = used * kGroups;
    float M = -INFINITY, den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (!invalid && (!kWide || wave < used)) {
        for (int i0 = gid; i0 < count; i0 += kUnroll * stride) {
            float mk[kUnroll], lk[kUnroll];
            f32x4 ok[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int i = i0 + u * stride;
                const bool use = i < count;
                const int k = per_unit && use ? unit_worker(u_a + i + 1, N, T) : k_first + i;
                const int64_t slot = (static_cast<int64_t>(use ? k : k_first) + sseg) * Lw + w_in;
                const float* pml = a.part_ml + slot * 2 * a.group;
                const float m_raw = pml[h], l_raw = pml[a.group + h];
                const f32x4 o_raw =
                    *reinterpret_cast<const f32x4*>(a.part_o + (slot * a.group + h) * D + 4 * quad);
                mk[u] = use ? m_raw : -INFINITY;
                lk[u] = use ? l_raw : 0.f;
                ok[u] = use ? o_raw : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) lse_merge(M, den, acc, mk[u], lk[u], ok[u]);
        }
#pragma unroll
        for (int off = kQuads; off < kWave; off <<= 1) {
            const float M2 = __shfl_xor(M, off), den2 = __shfl_xor(den, off);
            f32x4 acc2;
#pragma unroll
            for (int j = 0; j < 4; ++j) acc2[j] = __shfl_xor(acc[j], off);
            lse_merge(M, den, acc, M2, den2, acc2);
        }
    }
    if constexpr (kWide) {
        // the block's waves took disjoint partials: merge their results in LDS
        if (grp == 0) {
            float* e = s_merge[wave][quad];
            e[0] = M;
            e[1] = den;
#pragma unroll
            for (int j = 0; j < 4; ++j) e[2 + j] = acc[j];
        }
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            if (w >= used) break;  // uniform
            const float* e = s_merge[w][quad];
            lse_merge(M, den, acc, e[0], e[1], f32x4{e[2], e[3], e[4], e[5]});
        }
    }
    f32x4 res;
    if (invalid) {
        const float nan = __builtin_nanf("");
        res = f32x4{nan, nan, nan, nan};
    } else {
        res = acc / den;
    }
    if (grp == 0)
        store_quad<D, BF16>(a, (static_cast<int64_t>(b) * a.num_q_heads + g * a.group + h) * D + 4 * quad, res);
}

// Ring depth per shape.  Deeper rings are no faster (bf16, 128 dims, layer
// workload: 203 us with 3 pages, 205 with 4, 254 with 5, which spills; 64 dims:
// 22.8 us with 5, 23 to 24.6 with 7 and 8), one of 2 pages is 11 us slower.
template <int D, bool BF16>
constexpr int ring_depth() {
    return BF16 ? (D == 128 ? HCK_RING_BF16_D128 : 5) : (D == 128 ? 2 : 3);
}

enum class Merge { kFused, kSeparate, kSeparateHold };  // how the split's results go out

template <int D, bool BF16, bool TIERED, bool APPEND>
const void* split_kernel_ptr(Merge m) {
    constexpr int R = ring_depth<D, BF16>();
    return m == Merge::kFused ? reinterpret_cast<const void*>(&decode_split_kernel<D, BF16, R, TIERED, true, APPEND, false>)
           : m == Merge::kSeparate
               ? reinterpret_cast<const void*>(&decode_split_kernel<D, BF16, R, TIERED, false, APPEND, false>)
               : reinterpret_cast<const void*>(&decode_split_kernel<D, BF16, R, TIERED, false, APPEND, true>);
}

template <int D, bool BF16>
const void* split_kernel_ptr(bool tiered, bool append, Merge m) {
    if (tiered) return append ? split_kernel_ptr<D, BF16, true, true>(m) : split_kernel_ptr<D, BF16, true, false>(m);
    return append ? split_kernel_ptr<D, BF16, false, true>(m) : split_kernel_ptr<D, BF16, false, false>(m);
}

template <int D>
const void* valu_kernel_ptr(bool tiered) {
    constexpr int R = ring_depth<D, true>();
    return tiered ? reinterpret_cast<const void*>(&decode_split_valu_kernel<D, R, true>)
                  : reinterpret_cast<const void*>(&decode_split_valu_kernel<D, R, false>);
}

// The vector-ALU variant exists for bf16 only.
const void* pick_split(int head_dim, int dtype, bool tiered, bool valu, bool append, Merge m) {
    if (valu) {
        if (dtype != kDtypeBf16) return nullptr;
        return head_dim == 128 ? valu_kernel_ptr<128>(tiered) : head_dim == 64 ? valu_kernel_ptr<64>(tiered) : nullptr;
    }
    if (dtype == kDtypeBf16) {
        if (head_dim == 128) return split_kernel_ptr<128, true>(tiered, append, m);
        if (head_dim == 64) return split_kernel_ptr<64, true>(tiered, append, m);
    } else {
        if (head_dim == 128) return split_kernel_ptr<128, false>(tiered, append, m);
        if (head_dim == 64) return split_kernel_ptr<64, false>(tiered, append, m);
    }
    return nullptr;
}

template <int D, bool BF16>
const void* combine_kernel_ptr(int waves) {
    return waves == 16  ? reinterpret_cast<const void*>(&decode_combine_kernel<D, BF16, 16>)
           : waves == 4 ? reinterpret_cast<const void*>(&decode_combine_kernel<D, BF16, 4>)
                        : reinterpret_cast<const void*>(&decode_combine_kernel<D, BF16, 1>);
}

const void* pick_combine(int head_dim, int dtype, int waves) {
    if (dtype == kDtypeBf16) {
        if (head_dim == 128) return combine_kernel_ptr<128, true>(waves);
        if (head_dim == 64) return combine_kernel_ptr<64, true>(waves);
    } else {
        if (head_dim == 128) return combine_kernel_ptr<128, false>(waves);
        if (head_dim == 64) return combine_kernel_ptr<64, false>(waves);
    }
    return nullptr;
}

}  // namespace

hipError_t launch_decode_split(const DecodeArgs& a, int head_dim, int dtype, hipStream_t s,
                               const LaunchEvents& ev) {
    if (a.valu && (a.group > kValuMaxGroup || a.fused)) return hipErrorInvalidValue;
    // a worker's waves must share a block and split the KV heads and waves evenly
    if (a.group_waves < 1 || kSplitBlockWaves % a.group_waves || a.num_kv_heads % a.group_waves ||
        a.waves % a.group_waves)
        return hipErrorInvalidValue;
    if (a.waves <= 0 || (head_dim != 64 && head_dim != 128)) return hipErrorInvalidValue;
    const int blocks = (a.waves + kSplitBlockWaves - 1) / kSplitBlockWaves;
    DecodeArgs c = a;
    c.out_slots = 0;
    int lds = prefix_lds_bytes(a.batch);
    Merge merge = a.fused ? Merge::kFused : Merge::kSeparate;
    // Results are held in LDS where segments (row, head group) are no fewer than
    // workers, so that waves finish whole rows, and where a segment's rows are at
    // least 1 KiB.  Below the first line nearly all segments are split, and the
    // larger kernel costs short calls up to 1% (8 x 2K); below the second a row
    // costs as much to hold as to store (16 heads of 64 dims, one query head
    // each: 1% slower).  As many slots as the budget leaves room for; no holding
    // without at least two (thousands of rows with wide groups).
    const int row = head_dim * (dtype == kDtypeBf16 ? 2 : 4);
    if (!a.valu && !a.fused && a.group * row >= 1024 &&
        static_cast<int64_t>(a.batch) * a.num_kv_heads >= a.waves) {
        const int slot = out_slot_bytes(a.group, row);
        const int base = head_dim == 128 ? held_lds_bytes<128>(a.group, row, 0) : held_lds_bytes<64>(a.group, row, 0);
        const int room = ((kLdsBudget - lds) / kSplitBlockWaves - base) / slot;
        if (room >= 2) {
            merge = Merge::kSeparateHold;
            c.out_slots = room < kMaxOutSlots ? room : kMaxOutSlots;
            lds += kSplitBlockWaves * (base + c.out_slots * slot);
        }
    }
    const void* k = pick_split(head_dim, dtype, a.tiered != 0, a.valu != 0, a.k_new != nullptr, merge);
    if (!k) return hipErrorInvalidValue;
    void* args[] = {&c};
    return launch_kernel(k, dim3(blocks), dim3(kSplitBlockThreads), args, lds, s, ev);
}

hipError_t launch_decode_combine(const DecodeArgs& a, int head_dim, int dtype, hipStream_t s,
                                 const LaunchEvents& ev) {
    const int segs = a.batch * a.num_kv_heads;
    if (segs == 0) return hipSuccess;
    if (a.group_waves < 1 || a.num_kv_heads % a.group_waves || a.waves % a.group_waves)
        return hipErrorInvalidValue;
    // Many partials per segment (waves well above segments): several waves per head.
    const int64_t pieces = a.waves / segs;
    int per_head = pieces >= kWidestCombinePieces ? 16 : pieces >= kWideCombinePieces ? 4 : 1;
    // A segment has at most a table row's pages as partials: no more waves than
    // they give work to (the merge is the same, see `used` in the kernel).  Rows
    // of one page, 2 KV heads of 64 dims: 6.3 us a call with sixteen waves, 5.7 with one.
    const int per_wave = kCombineUnroll * 4 * kWave / head_dim;
    while (per_head > 1 && a.pt_stride <= per_head / 4 * per_wave) per_head /= 4;
    const bool wide = per_head > 1;
    const void* k = pick_combine(head_dim, dtype, per_head);
    if (!k) return hipErrorInvalidValue;
    const unsigned ny = wide ? static_cast<unsigned>(a.group)
                             : static_cast<unsigned>((a.group + kBlockWaves - 1) / kBlockWaves);
    // Walk the workers' split-segment entries when they are fewer than the
    // segments (many short rows): each worker starts at most one split segment.
    DecodeArgs c = a;
    c.combine_by_worker = a.waves < segs ? 1 : 0;
    void* args[] = {&c};
    const dim3 grid = c.combine_by_worker
                          ? dim3(static_cast<unsigned>(a.waves / a.group_waves), ny * a.group_waves)
                          : dim3(static_cast<unsigned>(segs), ny);
    return launch_kernel(k, grid, dim3(wide ? per_head * kWave : kBlockThreads), args, 0, s, ev);
}

}  // namespace hck
