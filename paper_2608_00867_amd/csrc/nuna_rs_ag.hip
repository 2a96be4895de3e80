// nuna_rs_ag.hip -- gfx950 reduce-scatter and all-gather kernels (standalone,
// and the two phases of the two-kernel two-shot all-reduce), and their
// launchers.  Same numerics and 16-byte streaming accesses as the all-reduce
// kernels.
#include "device_common.h"
#include "shapes.h"

namespace nuna {
namespace {

// ---------------------------------------------------------------- reduce-scatter

struct RsShape {
    int64_t mv;   // vectors per shard
    int64_t wcs;  // chunks per shard
    int32_t P;
    int32_t pad;
};

// SEL: the output pointer of shard r is picked among the pinned pointers
// (direct kernel, up to 8 ranks) instead of loaded from the arguments.
template <int PT, int DT, int VPT, bool FULL, bool KEEP, int MAXP, bool SEL = false>
__device__ __forceinline__ void reduce_scatter_chunk(const Ptrs<MAXP>& p, const RankTable& tab, const RsShape& s,
                                                     int P, int64_t r, int64_t v0, int nt) {
    using A = Arith<DT>;
    float acc[VPT][A::kLanes];
    reduce_ranks<PT, DT, VPT, FULL, true>(p, tab, P, r * s.mv, v0, nt, s.mv, acc);
    uint4 y[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) y[j] = A::narrow(acc[j]);
    uint4* dst;
    if constexpr (SEL)
        dst = out_at(p, static_cast<int>(r));
    else
        dst = use_table<PT>() ? rank_out(tab, static_cast<int>(r)) : p.out[r];
    store_vecs<FULL, VPT, !KEEP>(dst, y, v0, nt, s.mv);
}

// KEEP: the shard is read again right away (the all-gather phase of a two-shot
// all-reduce), so it is stored through the caches instead of streamed.
template <int PT, int MAXP, int DT, int VPT, bool KEEP>
__global__ __launch_bounds__(kWG) void k_reduce_scatter(Ptrs<MAXP> p, RsShape s, Place pl) {
    __builtin_assume(pl.gsize > 0);  // the collectives always place uniform groups
    const int P = PT > 0 ? PT : s.P;
    const RankTable tab = use_table<PT>() ? load_rank_table(p, P) : RankTable{0u, 0u, 0u, 0u};
    // One use of every argument the item loop needs: their loads issue together.
    if constexpr (PT == 8)
        asm volatile("" ::"s"(p.in[0]), "s"(p.in[1]), "s"(p.in[2]), "s"(p.in[3]), "s"(p.in[4]), "s"(p.in[5]),
                     "s"(p.in[6]), "s"(p.in[7]), "s"(p.out[0]), "s"(p.out[1]), "s"(p.out[2]), "s"(p.out[3]),
                     "s"(p.out[4]), "s"(p.out[5]), "s"(p.out[6]), "s"(p.out[7]), "s"(s.mv), "s"(s.wcs),
                     "s"(pl.groups), "s"(pl.mode), "s"(pl.gsize), "s"(pl.gshift), "s"(blockDim.x));
    else
        asm volatile("" ::"s"(s.mv), "s"(s.wcs), "s"(pl.groups), "s"(pl.mode), "s"(pl.gsize), "s"(pl.gshift),
                     "s"(blockDim.x));
    const int nt = blockDim.x;
    const int64_t cv = static_cast<int64_t>(nt) * VPT;
    const ItemRange it = items_of(pl, blockIdx.x, gridDim.x);
    for (int64_t i = it.first; i < it.end; i += it.stride) {
        const int64_t w = item_at(pl, blockIdx.x, gridDim.x, i);
        const int64_t r = w / s.wcs;
        const int64_t c = w - r * s.wcs;
        const int64_t v0 = c * cv + threadIdx.x;
        if ((c + 1) * cv <= s.mv)
            reduce_scatter_chunk<PT, DT, VPT, true, KEEP>(p, tab, s, P, r, v0, nt);
        else
            reduce_scatter_chunk<PT, DT, VPT, false, KEEP>(p, tab, s, P, r, v0, nt);
    }
}

// Direct reduce-scatter: grid (chunks per shard, P), workgroup (c, r) reduces
// chunk c of shard r; everything it reads from its arguments sits at fixed
// offsets (see k_allreduce_direct; rank counts other than 2, 4, 8 and 16 as
// there).
template <int PT, int DT, int VPT, bool KEEP>
__global__ __launch_bounds__(kWG) void k_reduce_scatter_direct(Ptrs<rank_cap<PT>()> p, int64_t mv, int32_t ranks) {
    if constexpr (PT > 0)
        pin_args(p, mv, blockDim.x, blockIdx.y);
    else
        pin_args(p, mv, blockDim.x, blockIdx.y, ranks);
    if constexpr (PT == -16) pin_inputs16(p);
    const int nt = blockDim.x;
    const int64_t cv = static_cast<int64_t>(nt) * VPT;
    const int64_t c = blockIdx.x;
    const int64_t r = blockIdx.y;
    const int64_t v0 = c * cv + threadIdx.x;
    RsShape s{};
    s.mv = mv;
    const RankTable tab{0u, 0u, 0u, 0u};  // pointers come from the arguments
    constexpr int N = rank_cap<PT>();
    const int P = PT > 0 ? PT : ranks;
    if ((c + 1) * cv <= mv)
        reduce_scatter_chunk<PT, DT, VPT, true, KEEP, N, (N <= 8)>(p, tab, s, P, r, v0, nt);
    else
        reduce_scatter_chunk<PT, DT, VPT, false, KEEP, N, (N <= 8)>(p, tab, s, P, r, v0, nt);
}

// ---------------------------------------------------------------- ragged shards
//
// Shards that are no whole number of 16-byte vectors: shard r of a buffer
// then begins off a vector boundary.  The stores decide the cut, since they
// want whole aligned vectors: a shard's destination is `head` bytes up to the
// first boundary, `nv` aligned vectors, and the bytes after the last one.  The
// vectors are loaded from wherever they start in the source (load16_any).
// They are numbered from the 128-byte line the first one lies in (`lead`
// vectors into it), so that every wave but the first and last writes whole
// lines: with waves starting inside a line, their streamed partial lines cost
// the all-gather a third of its rate (8 ranks of bf16, 2 MiB shards: 35.1 us
// against 25.9 for aligned shards).  The head and tail, at most 14 elements,
// are moved element by element by one more workgroup per shard, so that no
// chunk waits for them.
// An element per thread with a 64-bit division for its shard, which now serves
// small shards only (below), took 15.4 us for the reduce-scatter of 8 ranks of
// bf16 at 512 KiB shards (now 8.0) and 55.1 us for the all-gather at 2 MiB shards
// (24.2).
constexpr int kLineVecs = 8;  // 16-byte vectors in a 128-byte line

struct RaggedCut {
    int64_t head;  // bytes before the first aligned vector (at most the shard)
    int64_t nv;    // aligned vectors
    int64_t lead;  // vectors of the first one's line that come before it
    int64_t tail;  // bytes after the last vector
};

__device__ __forceinline__ RaggedCut ragged_cut(uint64_t dst, int64_t bytes) {
    RaggedCut k;
    const int64_t to = static_cast<int64_t>((0 - dst) & 15u);
    k.head = to < bytes ? to : bytes;
    k.nv = (bytes - k.head) >> 4;
    k.lead = static_cast<int64_t>(((dst + k.head) >> 4) & (kLineVecs - 1));
    k.tail = (bytes - k.head) & 15;
    return k;
}

// Host: chunks of cv vectors that cover a shard of mv vectors and its lead.
inline int64_t ragged_chunks(int64_t mv, int64_t cv) { return mv > 0 ? (mv + kLineVecs - 1 + cv - 1) / cv : 0; }

// Byte offset of edge element e (head elements first), or -1 past the last.
template <int ES>
__device__ __forceinline__ int64_t edge_offset(const RaggedCut& k, int e) {
    const int64_t at = static_cast<int64_t>(e) * ES;
    if (at < k.head) return at;
    return at < k.head + k.tail ? at + k.nv * 16 : -1;
}

// acc[j] = sum over ranks in ascending order of the 16 bytes at off + 16 * (v0 + j*nt) of every
// input, for vectors from 0 to below `limit` (at least 1).  Lanes outside load the nearest vector
// inside and are never stored: a masked load would put a branch and its wait into every rank's test.
template <int PT, int DT, int VPT, bool FULL, int MAXP>
__device__ __forceinline__ void reduce_ranks_any(const Ptrs<MAXP>& p, const RankTable& tab, int P, int64_t off,
                                                 int64_t v0, int nt, int64_t limit,
                                                 float (&acc)[VPT][Arith<DT>::kLanes]) {
    using A = Arith<DT>;
    constexpr int B = rank_batch<PT>();
    for (int r0 = 0; r0 < (PT != 0 ? 1 : P); r0 += B) {
        uint4 buf[B][VPT];
#pragma unroll
        for (int q = 0; q < B; ++q)
            if (PT > 0 || r0 + q < P) {
                const char* src = reinterpret_cast<const char*>(in_ptr<PT>(p, tab, r0 + q)) + off;
#pragma unroll
                for (int j = 0; j < VPT; ++j) {
                    int64_t v = v0 + j * nt;
                    if (!FULL) v = v < 0 ? 0 : v < limit ? v : limit - 1;
                    buf[q][j] = load16_any(src + v * 16);
                }
            }
        // Loads first: the scheduler otherwise runs the ranks of a partial chunk one after another
        // (16 ranks of bf16, 8191 elements per shard, 4.58 us against 3.4).
        if constexpr (PT == 16 && DT == kDtBf16 && VPT == 1 && !FULL) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < B; ++q)
            if (PT > 0 || r0 + q < P) {
#pragma unroll
                for (int j = 0; j < VPT; ++j) {
                    if (r0 + q == 0)
                        A::init(acc[j], buf[q][j]);
                    else
                        A::add(acc[j], buf[q][j]);
                }
            }
    }
}

// Vectors within [0, limit) of a chunk's, to a destination that starts at vector 0.
template <bool FULL, int VPT, bool NT>
__device__ __forceinline__ void store_range(uint4* dst, const uint4 (&y)[VPT], int64_t v0, int nt, int64_t limit) {
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        if (FULL || (v0 + j * nt >= 0 && v0 + j * nt < limit)) {
            if constexpr (NT)
                store_stream(dst + v0 + j * nt, y[j]);
            else
                dst[v0 + j * nt] = y[j];
        }
    }
}

// Workgroup (c, r) reduces chunk c of shard r, c = wcs its edge elements (a
// capped grid walks on by the grid's size).  m elements per shard; the output
// pointer may sit at any element (a two-shot's shard inside an output).
template <int PT, int DT, int VPT, bool KEEP, int MAXP>
__global__ __launch_bounds__(kWG) void k_reduce_scatter_ragged(Ptrs<MAXP> p, int64_t m, int64_t wcs, int32_t ranks) {
    using A = Arith<DT>;
    if constexpr (PT != 0) pin_args(p, m, wcs, ranks, blockDim.x);
    if constexpr (PT == -16) pin_inputs16(p);
    const int P = PT > 0 ? PT : ranks;
    const RankTable tab = use_table<PT>() ? load_rank_table(p, P) : RankTable{0u, 0u, 0u, 0u};
    const int nt = blockDim.x;
    const int64_t cv = static_cast<int64_t>(nt) * VPT;
    for (int r = static_cast<int>(blockIdx.y); r < P; r += static_cast<int>(gridDim.y)) {
        char* dst;
        if constexpr (use_table<PT>())
            dst = reinterpret_cast<char*>(rank_out(tab, r));
        else if constexpr (MAXP <= 8)
            dst = reinterpret_cast<char*>(out_at(p, r));
        else
            dst = reinterpret_cast<char*>(p.out[r]);
        const int64_t bytes = m * A::kEsize;
        const RaggedCut k = ragged_cut(reinterpret_cast<uint64_t>(dst), bytes);
        const int64_t off = r * bytes + k.head;
        uint4* out = reinterpret_cast<uint4*>(dst + k.head);
        for (int64_t c = blockIdx.x; c <= wcs; c += gridDim.x) {
            if (c == wcs) {
                if (threadIdx.x < 64) {  // one wave; lanes without an element take the shard's first
                    const int64_t at = edge_offset<A::kEsize>(k, static_cast<int>(threadIdx.x & 15));
                    const float a = reduce_element<PT, DT>(p, tab, P, (r * bytes + (at < 0 ? 0 : at)) / A::kEsize);
                    if (at >= 0 && threadIdx.x < 16) A::store1(dst, at / A::kEsize, a);
                }
                break;
            }
            const int64_t v0 = c * cv - k.lead + threadIdx.x;
            float acc[VPT][A::kLanes];
            uint4 y[VPT];
            if (c * cv >= k.lead && (c + 1) * cv - k.lead <= k.nv) {
                reduce_ranks_any<PT, DT, VPT, true>(p, tab, P, off, v0, nt, k.nv, acc);
#pragma unroll
                for (int j = 0; j < VPT; ++j) y[j] = A::narrow(acc[j]);
                store_range<true, VPT, !KEEP>(out, y, v0, nt, k.nv);
            } else if (k.nv > 0) {
                reduce_ranks_any<PT, DT, VPT, false>(p, tab, P, off, v0, nt, k.nv, acc);
#pragma unroll
                for (int j = 0; j < VPT; ++j) y[j] = A::narrow(acc[j]);
                store_range<false, VPT, !KEEP>(out, y, v0, nt, k.nv);
            }
        }
    }
}

// Element by element, for small ragged shards of run-time rank counts: the
// kernel above tests for every rank there, and its longer code costs more than
// its wide loads save up to 512 Ki elements of input per rank (6 ranks of bf16:
// 2.3 against 2.7 us at 16 KiB shards, 10.1 against 6.4 at 512 KiB; 12 ranks of
// fp32 6.3 against 6.7 at 128 KiB, 19.6 against 15.7 at 512 KiB).
// 17 to 19 ranks of bf16, whose second batch of 16 holds 1 to 3, keep it up to
// 216 Ki (17 ranks at 16 KiB shards 3.74 against 4.17 us, at 32 KiB 6.1 against 4.7).
constexpr int64_t kRsRaggedElems = int64_t(1) << 19;

inline bool rs_ragged_elem(int P, int64_t total, int dtype) {
    if (P < 16) return P != 2 && P != 8 && total <= kRsRaggedElems;
    return P > 16 && P < 20 && dtype == kDtBf16 && total <= (216 << 10);
}

template <int DT, int MAXP>
__global__ __launch_bounds__(kWG) void k_reduce_scatter_elem(Ptrs<MAXP> p, int P, int64_t m) {
    using A = Arith<DT>;
    using Raw = typename A::Raw;
    const int64_t total = m * P;
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < total;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t r = i / m;
        float a = A::widen1(reinterpret_cast<const Raw*>(p.in[0])[i]);
        for (int q = 1; q < P; ++q) a = a + A::widen1(reinterpret_cast<const Raw*>(p.in[q])[i]);
        A::store1(p.out[r], i - r * m, a);
    }
}

template <int DT, int MAXP>
void launch_rs_elem(const void* const* in, void* const* out, int P, int64_t m, int64_t G, hipStream_t st) {
    hipLaunchKernelGGL((k_reduce_scatter_elem<DT, MAXP>), dim3(static_cast<unsigned>(G)), dim3(kWG), 0, st,
                       make_ptrs<MAXP>(in, out, P, P), P, m);
}

// ---------------------------------------------------------------- all-gather

struct AgShape {
    int64_t mv;   // vectors per shard
    int64_t wcs;  // chunks per shard
    int32_t P;
    int32_t dpi;  // destinations per item
    int32_t gap;  // store_gap between destinations
    int32_t pad;
};

// WT: write-through stores (store_vecs_wt); `cbase` is the chunk's first
// vector within the shard (v0 less the lane).
template <int VPT, bool FULL, bool NT, bool WT>
__device__ __forceinline__ void all_gather_chunk(const RankTable& tab, const AgShape& s, int64_t r, int64_t v0, int nt,
                                                 int g, int64_t cbase) {
    const uint4* src = rank_in(tab, static_cast<int>(r));
    uint4 y[VPT];
    load_vecs<FULL, VPT, NT>(y, src, v0, nt, s.mv);
    const int d0 = g * s.dpi;
    for (int d = d0; d < d0 + s.dpi; ++d) {
        uint4* dst = rank_out(tab, d) + r * s.mv;
        if (dst == src) continue;  // in-place shard
        if (d > d0) store_gap(s.gap);
        if constexpr (WT)
            store_vecs_wt<FULL, VPT>(dst + cbase, y, static_cast<int>(threadIdx.x), nt, s.mv - cbase);
        else
            store_vecs<FULL, VPT>(dst, y, v0, nt, s.mv);
    }
}

// CACHED: the sources were just written (two-shot all-gather phase) and may
// still sit in L2 or the Infinity Cache, so they are read through the caches.
// WT: write-through stores.
template <int MAXP, int VPT, bool CACHED, bool WT>
__global__ __launch_bounds__(kWG) void k_all_gather(Ptrs<MAXP> p, AgShape s, Place pl) {
    __builtin_assume(pl.gsize > 0);  // the collectives always place uniform groups
    const RankTable tab = load_rank_table(p, s.P);
    // One use of every scalar argument the item loop needs: their loads issue together.
    asm volatile("" ::"s"(s.mv), "s"(s.wcs), "s"(s.dpi), "s"(s.gap), "s"(pl.groups), "s"(pl.mode), "s"(pl.gsize),
                 "s"(pl.gshift), "s"(blockDim.x));
    const int nt = blockDim.x;
    const int64_t cv = static_cast<int64_t>(nt) * VPT;
    const ItemRange it = items_of(pl, blockIdx.x, gridDim.x);
    for (int64_t i = it.first; i < it.end; i += it.stride) {
        const int64_t w = item_at(pl, blockIdx.x, gridDim.x, i);
        int64_t grp;
        int g;
        split_item(w, pl.gsize, pl.gshift, grp, g);
        const int64_t r = grp / s.wcs;
        const int64_t c = grp - r * s.wcs;
        const int64_t v0 = c * cv + threadIdx.x;
        if (pl.gsize == 1 && !CACHED) {
            if ((c + 1) * cv <= s.mv)
                all_gather_chunk<VPT, true, true, WT>(tab, s, r, v0, nt, g, c * cv);
            else
                all_gather_chunk<VPT, false, true, WT>(tab, s, r, v0, nt, g, c * cv);
        } else {
            if ((c + 1) * cv <= s.mv)
                all_gather_chunk<VPT, true, false, WT>(tab, s, r, v0, nt, g, c * cv);
            else
                all_gather_chunk<VPT, false, false, WT>(tab, s, r, v0, nt, g, c * cv);
        }
    }
}

// Direct all-gather (every destination per work item): grid (chunks per
// shard, P), workgroup (c, r) copies chunk c of shard r to every destination.
// The source pointer is an argument indexed by the workgroup's y index; the
// destinations are compile-time offsets (see k_allreduce_direct).
template <int PT, int VPT, bool CACHED, bool WT>
__global__ __launch_bounds__(kWG) void k_all_gather_direct(Ptrs<rank_cap<PT>()> p, int64_t mv, int32_t gap,
                                                           int32_t ranks) {
    if constexpr (PT > 0)
        pin_args(p, mv, gap, blockDim.x);
    else
        pin_args(p, mv, gap, blockDim.x, ranks);
    if constexpr (PT == -16) pin_outputs16(p);
    const int nt = blockDim.x;
    const int64_t cv = static_cast<int64_t>(nt) * VPT;
    const int64_t c = blockIdx.x;
    const int r = static_cast<int>(blockIdx.y);
    const int64_t v0 = c * cv + threadIdx.x;
    const uint4* src = in_at(p, r);
    uint4 y[VPT];
    const bool full = (c + 1) * cv <= mv;
    if (full)
        load_vecs<true, VPT, !CACHED>(y, src, v0, nt, mv);
    else
        load_vecs<false, VPT, !CACHED>(y, src, v0, nt, mv);
#pragma unroll
    for (int d = 0; d < rank_cap<PT>(); ++d) {
        uint4* dst = p.out[d] + r * mv;
        if ((PT > 0 || d < ranks) && dst != src) {  // dst == src: in-place shard
            if (d > 0) store_gap(gap);
            if constexpr (WT) {
                if (full)
                    store_vecs_wt<true, VPT>(dst + c * cv, y, static_cast<int>(threadIdx.x), nt, mv - c * cv);
                else
                    store_vecs_wt<false, VPT>(dst + c * cv, y, static_cast<int>(threadIdx.x), nt, mv - c * cv);
            } else {
                if (full)
                    store_vecs<true, VPT>(dst, y, v0, nt, mv);
                else
                    store_vecs<false, VPT>(dst, y, v0, nt, mv);
            }
        }
    }
}

// Element by element, for up to 8 ranks and 512 Ki elements of output, where the
// kernel below is the slower one (fewer waves in flight for the same bytes): 8
// ranks of bf16 at 32 KiB shards 2.46 against 2.66 us and at 64 KiB 2.92 against
// 3.31, 4 ranks at 128 KiB 2.31 against 2.72; at 128 KiB shards and 8 ranks 4.18
// against 3.79.  With 9 to 16 ranks, where it has twice the stores per thread, in the
// middle of that range only (12 ranks of fp32 at 32 KiB shards 3.06 against 3.40 us, at
// 4 KiB 2.60 against 2.38, at 96 KiB 5.1 against 5.0).
constexpr int64_t kAgRaggedElems = int64_t(1) << 19;

inline bool ag_ragged_elem(int P, int64_t m, int64_t es) {
    if (P <= 8) return m * P <= kAgRaggedElems;
    const int64_t shard = m * es;
    if (P > 16 || shard < (20 << 10)) return false;
    if (es == 4) return shard <= (P <= 12 ? 72 << 10 : 42 << 10);
    return P <= 12 && shard >= (P <= 10 ? 20 << 10 : 30 << 10) && shard <= (42 << 10);
}

template <int ES, int MAXP>
__global__ __launch_bounds__(kWG) void k_all_gather_elem(Ptrs<MAXP> p, int P, int64_t m) {
    using E = typename std::conditional<ES == 2, uint16_t, uint32_t>::type;
    const int64_t total = m * P;
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < total;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t r = i / m;
        const int64_t j = i - r * m;
        const E* src = reinterpret_cast<const E*>(p.in[r]);
        const E v = src[j];
        for (int d = 0; d < P; ++d) {
            E* dst = reinterpret_cast<E*>(p.out[d]) + r * m;
            if (dst != src) dst[j] = v;
        }
    }
}

template <int ES, int MAXP>
void launch_ag_elem(const void* const* in, void* const* out, int P, int64_t m, int64_t G, hipStream_t st) {
    hipLaunchKernelGGL((k_all_gather_elem<ES, MAXP>), dim3(static_cast<unsigned>(G)), dim3(kWG), 0, st,
                       make_ptrs<MAXP>(in, out, P, P), P, m);
}

// All-gather of ragged shards: workgroup (c, r, g) copies chunk c of shard r,
// c = wcs its edge elements, to the destinations [g * dpi, (g + 1) * dpi).
// `bytes` per shard.
template <int PT, int ES, int VPT, int MAXP>
__global__ __launch_bounds__(kWG) void k_all_gather_ragged(Ptrs<MAXP> p, int64_t bytes, int64_t wcs, int32_t ranks,
                                                           int32_t dpi, int32_t gap) {
    using E = typename std::conditional<ES == 2, uint16_t, uint32_t>::type;
    if constexpr (PT != 0) pin_args(p, bytes, wcs, ranks, dpi, gap, blockDim.x);
    const int P = PT > 0 ? PT : ranks;
    const RankTable tab = use_table<PT>() ? load_rank_table(p, P) : RankTable{0u, 0u, 0u, 0u};
    const int nt = blockDim.x;
    const int64_t cv = static_cast<int64_t>(nt) * VPT;
    const int d0 = static_cast<int>(blockIdx.z) * dpi;
    const int d1 = d0 + dpi < P ? d0 + dpi : P;
    // The outputs' place within a line (any of them: it changes no result).
    const uint64_t out0 = reinterpret_cast<uint64_t>(out_ptr<PT>(p, tab, 0));
    auto each_destination = [&](auto&& put) {
        if constexpr (use_table<PT>()) {
            for (int d = d0; d < d1; ++d) {
                if (d > d0) store_gap(gap);
                put(reinterpret_cast<char*>(rank_out(tab, d)));
            }
        } else {
#pragma unroll
            for (int d = 0; d < rank_cap<PT>(); ++d)
                if (d >= d0 && d < d1) {
                    if (d > d0) store_gap(gap);
                    put(reinterpret_cast<char*>(p.out[d]));
                }
        }
    };
    for (int r = static_cast<int>(blockIdx.y); r < P; r += static_cast<int>(gridDim.y)) {
        const char* src;
        if constexpr (use_table<PT>())
            src = reinterpret_cast<const char*>(rank_in(tab, r));
        else if constexpr (MAXP <= 8)
            src = reinterpret_cast<const char*>(in_at(p, r));
        else
            src = reinterpret_cast<const char*>(p.in[r]);
        const int64_t base = r * bytes;
        const RaggedCut k = ragged_cut(out0 + static_cast<uint64_t>(base), bytes);
        for (int64_t c = blockIdx.x; c <= wcs; c += gridDim.x) {
            if (c == wcs) {
                const int64_t at = edge_offset<ES>(k, static_cast<int>(threadIdx.x));
                const E edge = at >= 0 ? *reinterpret_cast<const E*>(src + at) : E(0);
                each_destination([&](char* out) {
                    char* dst = out + base;
                    if (dst != src && at >= 0) *reinterpret_cast<E*>(dst + at) = edge;
                });
                break;
            }
            const int64_t v0 = c * cv - k.lead + threadIdx.x;
            const char* from = src + k.head;
            uint4 y[VPT];
            if (c * cv >= k.lead && (c + 1) * cv - k.lead <= k.nv) {
#pragma unroll
                for (int j = 0; j < VPT; ++j) y[j] = load16_any(from + (v0 + j * nt) * 16);
                each_destination([&](char* out) {
                    char* dst = out + base;
                    if (dst != src)  // else an in-place shard
                        store_range<true, VPT, true>(reinterpret_cast<uint4*>(dst + k.head), y, v0, nt, k.nv);
                });
            } else {
#pragma unroll
                for (int j = 0; j < VPT; ++j)
                    if (v0 + j * nt >= 0 && v0 + j * nt < k.nv) y[j] = load16_any(from + (v0 + j * nt) * 16);
                each_destination([&](char* out) {
                    char* dst = out + base;
                    if (dst != src)
                        store_range<false, VPT, true>(reinterpret_cast<uint4*>(dst + k.head), y, v0, nt, k.nv);
                });
            }
        }
    }
}

template <int PT, int MAXP, int DT, int VPT, bool KEEP>
void launch_rs_t(const void* const* in, void* const* out, int P, const RsShape& s, const Place& pl, int64_t G, int nt,
                 hipStream_t st) {
    Ptrs<MAXP> p = make_ptrs<MAXP>(in, out, P, P);
    hipLaunchKernelGGL((k_reduce_scatter<PT, MAXP, DT, VPT, KEEP>), dim3(static_cast<unsigned>(G)), dim3(nt), 0, st, p, s,
                       pl);
}

template <int DT, int VPT, bool KEEP>
void launch_rs_p(const void* const* in, void* const* out, int P, const RsShape& s, const Place& pl, int64_t G, int nt,
                 hipStream_t st) {
    switch (P) {
        case 2: launch_rs_t<2, 2, DT, VPT, KEEP>(in, out, P, s, pl, G, nt, st); break;
        case 4: launch_rs_t<4, 4, DT, VPT, KEEP>(in, out, P, s, pl, G, nt, st); break;
        case 8: launch_rs_t<8, 8, DT, VPT, KEEP>(in, out, P, s, pl, G, nt, st); break;
        case 16: launch_rs_t<16, 16, DT, VPT, KEEP>(in, out, P, s, pl, G, nt, st); break;
        default:
            if constexpr (VPT == 1) {
                if (P == 32) launch_rs_t<32, 64, DT, 1, KEEP>(in, out, P, s, pl, G, nt, st);
                else if (P == 64) launch_rs_t<64, 64, DT, 1, KEEP>(in, out, P, s, pl, G, nt, st);
                else launch_rs_t<0, 64, DT, 1, KEEP>(in, out, P, s, pl, G, nt, st);
            } else {
                launch_rs_t<0, 64, DT, VPT, KEEP>(in, out, P, s, pl, G, nt, st);  // other P up to 16 (above: VPT 1)
            }
            break;
    }
}

template <int PT, int DT, int VPT, bool KEEP>
void launch_rs_direct_t(const void* const* in, void* const* out, const RsShape& s, int nt, hipStream_t st) {
    const auto p = make_ptrs<rank_cap<PT>()>(in, out, s.P, s.P);
    hipLaunchKernelGGL((k_reduce_scatter_direct<PT, DT, VPT, KEEP>),
                       dim3(static_cast<unsigned>(s.wcs), static_cast<unsigned>(s.P)), dim3(nt), 0, st, p, s.mv, s.P);
}

template <int DT, int VPT, bool KEEP>
void launch_rs_direct_p(const void* const* in, void* const* out, const RsShape& s, int nt, hipStream_t st) {
    switch (s.P) {
        case 2: launch_rs_direct_t<2, DT, VPT, KEEP>(in, out, s, nt, st); break;
        case 4: launch_rs_direct_t<4, DT, VPT, KEEP>(in, out, s, nt, st); break;
        case 8: launch_rs_direct_t<8, DT, VPT, KEEP>(in, out, s, nt, st); break;
        case 16: launch_rs_direct_t<16, DT, VPT, KEEP>(in, out, s, nt, st); break;
        default:
            if (s.P < 4) launch_rs_direct_t<-4, DT, VPT, KEEP>(in, out, s, nt, st);
            else if (s.P < 8) launch_rs_direct_t<-8, DT, VPT, KEEP>(in, out, s, nt, st);
            else launch_rs_direct_t<-16, DT, VPT, KEEP>(in, out, s, nt, st);
            break;
    }
}

// Launch by dtype and vectors per thread.
template <bool KEEP>
void launch_rs(bool direct, const void* const* in, void* const* out, const RsShape& s, int dtype, int vpt,
               const Place& pl, int64_t G, int nt, hipStream_t st) {
    auto go = [&](auto dt, auto v) {
        if (direct)
            launch_rs_direct_p<dt(), v(), KEEP>(in, out, s, nt, st);
        else
            launch_rs_p<dt(), v(), KEEP>(in, out, s.P, s, pl, G, nt, st);
    };
    using F32 = std::integral_constant<int, kDtF32>;
    using Bf16 = std::integral_constant<int, kDtBf16>;
    using V1 = std::integral_constant<int, 1>;
    using V2 = std::integral_constant<int, 2>;
    using V4 = std::integral_constant<int, 4>;
    if (dtype == kDtF32) vpt == 4 ? go(F32{}, V4{}) : vpt == 2 ? go(F32{}, V2{}) : go(F32{}, V1{});
    else vpt == 4 ? go(Bf16{}, V4{}) : vpt == 2 ? go(Bf16{}, V2{}) : go(Bf16{}, V1{});
}

// Grid of a ragged launch: (chunks and edges, shards, destination groups), cut down to
// the workgroup cap; the kernels walk on over chunks and shards.
dim3 ragged_grid(int64_t wcs, int P, int groups) {
    ++wcs;  // and the edges
    const int64_t cap = max_workgroups() / groups > 0 ? max_workgroups() / groups : 1;
    const int64_t y = P < cap ? P : cap;
    const int64_t x = wcs < cap / y ? wcs : cap / y;
    return dim3(static_cast<unsigned>(x > 0 ? x : 1), static_cast<unsigned>(y), static_cast<unsigned>(groups));
}

template <int PT, int DT, int VPT, bool KEEP>
void launch_rs_ragged_t(const void* const* in, void* const* out, int P, int64_t m, int64_t wcs, int nt,
                        hipStream_t st) {
    constexpr int N = PT == 0 ? 64 : rank_cap<PT>();
    const auto p = make_ptrs<N>(in, out, P, P);
    hipLaunchKernelGGL((k_reduce_scatter_ragged<PT, DT, VPT, KEEP, N>), ragged_grid(wcs, P, 1), dim3(nt), 0, st, p, m,
                       wcs, P);
}

template <int DT, int VPT, bool KEEP>
void launch_rs_ragged_p(const void* const* in, void* const* out, int P, int64_t m, int64_t wcs, int nt,
                        hipStream_t st) {
    if (P > 16) launch_rs_ragged_t<0, DT, 1, KEEP>(in, out, P, m, wcs, nt, st);
    else if (P == 16) launch_rs_ragged_t<16, DT, VPT, KEEP>(in, out, P, m, wcs, nt, st);
    else if (P > 8) launch_rs_ragged_t<-16, DT, VPT, KEEP>(in, out, P, m, wcs, nt, st);
    else if (P == 8) launch_rs_ragged_t<8, DT, VPT, KEEP>(in, out, P, m, wcs, nt, st);
    else if (P > 4) launch_rs_ragged_t<-8, DT, VPT, KEEP>(in, out, P, m, wcs, nt, st);
    else if (P == 2) launch_rs_ragged_t<2, DT, VPT, KEEP>(in, out, P, m, wcs, nt, st);
    else launch_rs_ragged_t<-4, DT, VPT, KEEP>(in, out, P, m, wcs, nt, st);
}

template <bool KEEP>
void launch_rs_ragged(const void* const* in, void* const* out, int P, int64_t m, int64_t wcs, int dtype, int vpt,
                      int nt, hipStream_t st) {
    if (dtype == kDtF32) {
        if (vpt == 4) launch_rs_ragged_p<kDtF32, 4, KEEP>(in, out, P, m, wcs, nt, st);
        else if (vpt == 2) launch_rs_ragged_p<kDtF32, 2, KEEP>(in, out, P, m, wcs, nt, st);
        else launch_rs_ragged_p<kDtF32, 1, KEEP>(in, out, P, m, wcs, nt, st);
    } else {
        if (vpt == 4) launch_rs_ragged_p<kDtBf16, 4, KEEP>(in, out, P, m, wcs, nt, st);
        else if (vpt == 2) launch_rs_ragged_p<kDtBf16, 2, KEEP>(in, out, P, m, wcs, nt, st);
        else launch_rs_ragged_p<kDtBf16, 1, KEEP>(in, out, P, m, wcs, nt, st);
    }
}

template <int PT, int ES, int VPT>
void launch_ag_ragged_t(const void* const* in, void* const* out, int P, int64_t bytes, int64_t wcs, int nt, int dpi,
                        int gap, hipStream_t st) {
    constexpr int N = PT == 0 ? 64 : rank_cap<PT>();
    const auto p = make_ptrs<N>(in, out, P, P);
    hipLaunchKernelGGL((k_all_gather_ragged<PT, ES, VPT, N>), ragged_grid(wcs, P, (P + dpi - 1) / dpi), dim3(nt), 0,
                       st, p, bytes, wcs, P, dpi, gap);
}

template <int ES, int VPT>
void launch_ag_ragged(const void* const* in, void* const* out, int P, int64_t bytes, int64_t wcs, int nt, int dpi,
                      int gap, hipStream_t st) {
    // Split destinations: the rank table's loop runs the group's few stores only.
    if (P > 8 || (dpi < P && P > 4)) launch_ag_ragged_t<0, ES, VPT>(in, out, P, bytes, wcs, nt, dpi, gap, st);
    else if (P == 8) launch_ag_ragged_t<8, ES, VPT>(in, out, P, bytes, wcs, nt, dpi, gap, st);
    else if (P > 4) launch_ag_ragged_t<-8, ES, VPT>(in, out, P, bytes, wcs, nt, dpi, gap, st);
    else launch_ag_ragged_t<-4, ES, VPT>(in, out, P, bytes, wcs, nt, dpi, gap, st);
}

}  // namespace

hipError_t launch_reduce_scatter(const void* const* in, void* const* out, int P, size_t m, int dtype, int mode,
                                 bool keep_output, hipStream_t stream) {
    const size_t es = dtype_size(dtype);
    if ((m * es) % 16 != 0) {
        const int64_t mv = static_cast<int64_t>(m * es / 16);
        const int64_t total = static_cast<int64_t>(m) * P;
        if (rs_ragged_elem(P, total, dtype)) {
            const int64_t G = cap_grid((total + kWG - 1) / kWG);
            note_launch("k_reduce_scatter_elem", kMapLinear, 1, G, kWG, 0);
            const int64_t n = static_cast<int64_t>(m);
            if (P > 16) launch_rs_elem<kDtBf16, 64>(in, out, P, n, G, stream);
            else if (dtype == kDtF32) launch_rs_elem<kDtF32, 16>(in, out, P, n, G, stream);
            else launch_rs_elem<kDtBf16, 16>(in, out, P, n, G, stream);
            return hipGetLastError();
        }
        int nt, vpt;
        pick_rs_shape(mv * P, P, dtype, false, nt, vpt);
        if (P > 16) vpt = 1;
        if (vpt == 1 && !tuning().wg_threads) nt = 64;  // more workgroups for the small sizes
        const int64_t cv = static_cast<int64_t>(nt) * vpt;
        const int64_t wcs = ragged_chunks(mv, cv);
        const dim3 g = ragged_grid(wcs, P, 1);
        note_launch("k_reduce_scatter_ragged", kMapLinear, 1, int64_t(g.x) * g.y, nt, vpt);
        if (keep_output) launch_rs_ragged<true>(in, out, P, static_cast<int64_t>(m), wcs, dtype, vpt, nt, stream);
        else launch_rs_ragged<false>(in, out, P, static_cast<int64_t>(m), wcs, dtype, vpt, nt, stream);
        return hipGetLastError();
    }
    RsShape s{};
    s.mv = static_cast<int64_t>(m * es / 16);
    s.P = P;
    // Shape by the vectors each input rank holds (P shards of mv vectors).
    int nt, vpt;
    pick_rs_shape(s.mv * P, P, dtype, !keep_output, nt, vpt);
    const int64_t row_cv = static_cast<int64_t>(nt) * vpt;
    if (grid_capped((s.mv + row_cv - 1) / row_cv * P)) {
        pick_rs_capped_shape(s.mv * P, P, dtype, nt, vpt);
    } else if (keep_output && P <= 16 && !tuning().wg_threads && !tuning().vpt && s.mv * P >= (int64_t(1) << 17) &&
               s.mv * P < (int64_t(1) << 18) && row_cv != kWG) {
        // The all-gather that follows cuts these sizes (2-4 MiB per rank) into chunks of 256
        // vectors: cut alike, a chunk is read on the XCD that wrote it, from its L2.  Two-shot of two
        // kernels at 3 MiB, 6 ranks, 9.63 us with the standalone row's 64x1 and 9.15 with 256x1; 16 ranks
        // at 2 MiB 13.55 (256x2) and 12.72.
        nt = kWG;
        vpt = 1;
    }
    const int64_t cv = static_cast<int64_t>(nt) * vpt;
    s.wcs = (s.mv + cv - 1) / cv;
    const Place pl = make_place_uniform(mode, s.wcs * P, 1);
    const int64_t G = cap_grid(place_grid(pl));
    // Every work item is its own group: both placements run the linear map.
    const bool direct = G == s.wcs * P && G <= direct_max_grid() && P <= 16;
    note_launch(direct ? "k_reduce_scatter_direct" : "k_reduce_scatter", kMapLinear, 1, G, nt, vpt);
    if (keep_output) launch_rs<true>(direct, in, out, s, dtype, vpt, pl, G, nt, stream);
    else launch_rs<false>(direct, in, out, s, dtype, vpt, pl, G, nt, stream);
    return hipGetLastError();
}

// Write-through variants exist for the cached-source (two-shot) phase with 8 ranks.
template <int PT>
void launch_ag_direct_p(const void* const* in, void* const* out, const AgShape& s, int vpt, bool cached, bool wt,
                        dim3 g, dim3 b, hipStream_t st) {
    const auto p = make_ptrs<rank_cap<PT>()>(in, out, s.P, s.P);
    if constexpr (PT == 8) {
        if (cached && wt) {
            if (vpt == 4) hipLaunchKernelGGL((k_all_gather_direct<PT, 4, true, true>), g, b, 0, st, p, s.mv, s.gap, s.P);
            else if (vpt == 2) hipLaunchKernelGGL((k_all_gather_direct<PT, 2, true, true>), g, b, 0, st, p, s.mv, s.gap, s.P);
            else hipLaunchKernelGGL((k_all_gather_direct<PT, 1, true, true>), g, b, 0, st, p, s.mv, s.gap, s.P);
            return;
        }
    }
    if (cached) {
        if (vpt == 4) hipLaunchKernelGGL((k_all_gather_direct<PT, 4, true, false>), g, b, 0, st, p, s.mv, s.gap, s.P);
        else if (vpt == 2) hipLaunchKernelGGL((k_all_gather_direct<PT, 2, true, false>), g, b, 0, st, p, s.mv, s.gap, s.P);
        else hipLaunchKernelGGL((k_all_gather_direct<PT, 1, true, false>), g, b, 0, st, p, s.mv, s.gap, s.P);
    } else {
        if (vpt == 4) hipLaunchKernelGGL((k_all_gather_direct<PT, 4, false, false>), g, b, 0, st, p, s.mv, s.gap, s.P);
        else if (vpt == 2) hipLaunchKernelGGL((k_all_gather_direct<PT, 2, false, false>), g, b, 0, st, p, s.mv, s.gap, s.P);
        else hipLaunchKernelGGL((k_all_gather_direct<PT, 1, false, false>), g, b, 0, st, p, s.mv, s.gap, s.P);
    }
}

hipError_t launch_all_gather(const void* const* in, void* const* out, int P, size_t m, int dtype, int mode,
                             bool src_cached, hipStream_t stream) {
    const size_t es = dtype_size(dtype);
    if ((m * es) % 16 != 0) {
        const int64_t bytes = static_cast<int64_t>(m * es), mv = bytes / 16, total = static_cast<int64_t>(m) * P;
        if (ag_ragged_elem(P, static_cast<int64_t>(m), static_cast<int64_t>(es))) {
            const int64_t G = cap_grid((total + kWG - 1) / kWG);
            note_launch("k_all_gather_elem", kMapLinear, 1, G, kWG, 0);
            const int64_t n = static_cast<int64_t>(m);
            if (P <= 8) es == 4 ? launch_ag_elem<4, 8>(in, out, P, n, G, stream) : launch_ag_elem<2, 8>(in, out, P, n, G, stream);
            else es == 4 ? launch_ag_elem<4, 16>(in, out, P, n, G, stream) : launch_ag_elem<2, 16>(in, out, P, n, G, stream);
            return hipGetLastError();
        }
        int nt, vpt;
        pick_ag_shape(mv * P, P, nt, vpt);
        const int64_t cv = static_cast<int64_t>(nt) * vpt;
        const int64_t wcs = ragged_chunks(mv, cv);
        // Up to 4 groups while the launch is short of 1500 workgroups: 8 ranks of 128 KiB
        // shards 3.98 us against 4.73 with 8 groups and 4.60 with one.
        const int split = wcs * P < 1500 ? (P < 4 ? P : 4) : 1;
        const int dpi = split <= max_workgroups() ? (P + split - 1) / split : P;
        const int groups = (P + dpi - 1) / dpi, gap = store_gap_for(m * es * P);
        const dim3 g = ragged_grid(wcs, P, groups);
        note_launch("k_all_gather_ragged", kMapLinear, 1, int64_t(g.x) * g.y * g.z, nt, vpt);
        if (es == 4) {
            if (vpt == 4) launch_ag_ragged<4, 4>(in, out, P, bytes, wcs, nt, dpi, gap, stream);
            else if (vpt == 2) launch_ag_ragged<4, 2>(in, out, P, bytes, wcs, nt, dpi, gap, stream);
            else launch_ag_ragged<4, 1>(in, out, P, bytes, wcs, nt, dpi, gap, stream);
        } else {
            if (vpt == 4) launch_ag_ragged<2, 4>(in, out, P, bytes, wcs, nt, dpi, gap, stream);
            else if (vpt == 2) launch_ag_ragged<2, 2>(in, out, P, bytes, wcs, nt, dpi, gap, stream);
            else launch_ag_ragged<2, 1>(in, out, P, bytes, wcs, nt, dpi, gap, stream);
        }
        return hipGetLastError();
    }
    AgShape s{};
    s.mv = static_cast<int64_t>(m * es / 16);
    s.P = P;
    s.gap = store_gap_for(m * es * P);
    // Shape by the vectors each output rank receives (P shards of mv vectors).
    int nt, vpt;
    pick_ag_shape(s.mv * P, P, nt, vpt);
    const int64_t cv = static_cast<int64_t>(nt) * vpt;
    s.wcs = (s.mv + cv - 1) / cv;
    // Split destinations when there are few chunks, so that more workgroups
    // share the stores; each member re-reads its chunk (an L2 hit when the
    // group's members sit on one XCD).
    const int gsize = (s.wcs * P < 512) ? largest_divisor_upto(P, 8) : 1;
    s.dpi = P / gsize;
    // Each member loads the chunk once and stores it dpi times: gsize - 1 of
    // the group's gsize * (1 + dpi) transfers are re-reads.  The grouped map
    // from launches of more than 2 MiB, as for the split all-reduce: below, with
    // 8 ranks at 2-32 KiB shards, it was within 1 % of the linear map cold and
    // up to 2 % slower with warm inputs on MI355X.
    const int gmode = gsize > 1 ? group_mode(mode, gsize - 1, int64_t(gsize) * (1 + s.dpi),
                                             static_cast<int64_t>(P + 1) * P * static_cast<int64_t>(m * es),
                                             int64_t(2) << 20)
                                : mode;
    const Place pl = make_place_uniform(gmode, s.wcs * P, gsize);
    const int64_t G = cap_grid(place_grid(pl));
    // Write-through stores in the two-shot's all-gather phase (the shards were
    // just written and are read through the caches) with 8 ranks, at 1-2 MiB
    // shards.  Against streaming stores on MI355X, whole two-shot, back-to-back
    // cold calls: 4.3 % faster at 2 MiB shards, +0.2-0.5 % at 1-1.5 MiB; the
    // gain does not grow smoothly beyond (-4.7 % at 3 MiB, +3.4 % at 4 MiB,
    // -9 % at 6-8 MiB) and is -12 % at 0.5 MiB.
    const int wtf = tuning().write_through;
    const int64_t shard = static_cast<int64_t>(m * es);
    const bool wt = P == 8 && src_cached && gsize == 1 &&
                    (wtf == 2 || (wtf == 0 && shard >= (int64_t(1) << 20) && shard <= (int64_t(2) << 20)));
    // The direct kernel when every chunk item has its own workgroup.  With 8
    // ranks it takes grids beyond the direct-grid limit too: against the general
    // kernel's persistent loop it measured 6-10 % faster at 6-32 MiB shards on
    // MI355X (103 against 114 us at 8 MiB, 418 against 457 us at 32 MiB).
    // With 9 to 16 ranks only from 3 MiB per output: the 16-slot kernel loads its
    // pointers where it uses them, and below that the general kernel's rank
    // table is faster (16 ranks, 16 KiB shards 3.15 against 4.25 us; 12 ranks,
    // 512 KiB shards 14.2 against 13.4).
    const int64_t items = s.wcs * P;
    const bool direct = gsize == 1 && (P == 8 ? items <= grid_limit(kAgDirectMaxGrid8)
                                              : P <= 16 && G == items && G <= direct_max_grid() &&
                                                    (P < 8 || s.mv * P >= (int64_t(3) << 16)));
    if (direct) {
        note_launch("k_all_gather_direct", kMapLinear, 1, items, nt, vpt);
        const dim3 g(static_cast<unsigned>(s.wcs), static_cast<unsigned>(P)), b(nt);
        switch (P) {
            case 2: launch_ag_direct_p<2>(in, out, s, vpt, src_cached, false, g, b, stream); break;
            case 4: launch_ag_direct_p<4>(in, out, s, vpt, src_cached, false, g, b, stream); break;
            case 8: launch_ag_direct_p<8>(in, out, s, vpt, src_cached, wt, g, b, stream); break;
            default:
                if (P < 4) launch_ag_direct_p<-4>(in, out, s, vpt, src_cached, false, g, b, stream);
                else if (P < 8) launch_ag_direct_p<-8>(in, out, s, vpt, src_cached, false, g, b, stream);
                else launch_ag_direct_p<-16>(in, out, s, vpt, src_cached, false, g, b, stream);
                break;
        }
        return hipGetLastError();
    }
    note_launch("k_all_gather", pl.mode == kPlaceXcd && !linear_map(pl, G) ? kMapXcdGroups : kMapLinear, pl.gsize, G,
                nt, vpt);
    if (P <= 8) {
        Ptrs<8> p = make_ptrs<8>(in, out, P, P);
        const dim3 g(static_cast<unsigned>(G)), b(nt);
        if (src_cached && wt) {
            if (vpt == 4) hipLaunchKernelGGL((k_all_gather<8, 4, true, true>), g, b, 0, stream, p, s, pl);
            else if (vpt == 2) hipLaunchKernelGGL((k_all_gather<8, 2, true, true>), g, b, 0, stream, p, s, pl);
            else hipLaunchKernelGGL((k_all_gather<8, 1, true, true>), g, b, 0, stream, p, s, pl);
        } else if (src_cached) {
            if (vpt == 4) hipLaunchKernelGGL((k_all_gather<8, 4, true, false>), g, b, 0, stream, p, s, pl);
            else if (vpt == 2) hipLaunchKernelGGL((k_all_gather<8, 2, true, false>), g, b, 0, stream, p, s, pl);
            else hipLaunchKernelGGL((k_all_gather<8, 1, true, false>), g, b, 0, stream, p, s, pl);
        } else {
            if (vpt == 4) hipLaunchKernelGGL((k_all_gather<8, 4, false, false>), g, b, 0, stream, p, s, pl);
            else if (vpt == 2) hipLaunchKernelGGL((k_all_gather<8, 2, false, false>), g, b, 0, stream, p, s, pl);
            else hipLaunchKernelGGL((k_all_gather<8, 1, false, false>), g, b, 0, stream, p, s, pl);
        }
    } else {
        Ptrs<64> p = make_ptrs<64>(in, out, P, P);
        const dim3 g(static_cast<unsigned>(G)), b(nt);
        if (src_cached) {
            if (vpt == 4) hipLaunchKernelGGL((k_all_gather<64, 4, true, false>), g, b, 0, stream, p, s, pl);
            else if (vpt == 2) hipLaunchKernelGGL((k_all_gather<64, 2, true, false>), g, b, 0, stream, p, s, pl);
            else hipLaunchKernelGGL((k_all_gather<64, 1, true, false>), g, b, 0, stream, p, s, pl);
        } else {
            if (vpt == 4) hipLaunchKernelGGL((k_all_gather<64, 4, false, false>), g, b, 0, stream, p, s, pl);
            else if (vpt == 2) hipLaunchKernelGGL((k_all_gather<64, 2, false, false>), g, b, 0, stream, p, s, pl);
            else hipLaunchKernelGGL((k_all_gather<64, 1, false, false>), g, b, 0, stream, p, s, pl);
        }
    }
    return hipGetLastError();
}

}  // namespace nuna
