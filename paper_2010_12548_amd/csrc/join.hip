// join.hip -- polygon-polygon join over cells (Sec. 4: two rasterized
// canvases blended cell by cell, masked to the cells that hold a polygon of
// each, aggregated per polygon pair).
//
// Both canvases are Hilbert handles on one key grid, so each is a sorted
// list of runs (first key, code) that partitions [0, 4^L).  Blending them is
// a merge of the two run lists: the union of their first keys cuts the key
// range into elementary intervals on which both codes are constant.  Masking
// keeps the intervals whose two codes are both non-empty; every member pair
// of the two codes (polygon sets expand to their members) then shares the
// interval's cells.
//
// One kernel does all of it: tiles of the merged list go through LDS, the
// intervals' lengths are summed per pair of codes in an LDS table, and the
// table's entries, expanded to polygon pairs, are added to a table of all
// pairs in memory, whose entries are sorted at the end (polygons in layers: the
// LDS table is of polygon pairs).  What bounds it is the
// work in LDS, a search in the other list's part of the tile and an addition
// to the table for every run; the lists themselves are read once.  (Sorting
// the first keys of both lists, then a key for each pair of each interval
// with its lengths' sums: 8.1 ms for two lists of 31M runs together, 45M pairs
// of intervals; this way 0.43 ms, of them 0.3 in the tiles.)
#include <algorithm>

#include "sba_internal.h"

namespace {

struct CanvasView {
    const uint64_t *starts;
    const uint32_t *starts32;  // the same keys where they fit 32 bits, else null
    const uint32_t *code;
    int64_t n;
    const int64_t *set_off;
    const int32_t *set_ids;
    uint32_t np, n_sets;
};

__device__ __forceinline__ int64_t members(const CanvasView &C, uint32_t code)
{
    if (code == 0) return 0;
    if (code < CODE_SET_BASE) return code - 1u < C.np ? 1 : 0;
    const uint32_t k = code - CODE_SET_BASE;
    return k < C.n_sets ? C.set_off[k + 1] - C.set_off[k] : 0;
}

__device__ __forceinline__ uint32_t member(const CanvasView &C, uint32_t code, int64_t t)
{
    if (code < CODE_SET_BASE) return code - 1u;
    return (uint32_t)C.set_ids[C.set_off[code - CODE_SET_BASE] + t];
}

template <typename K>
__device__ __forceinline__ const K *starts_of(const CanvasView &C)
{
    if constexpr (sizeof(K) == 4) return C.starts32;
    else return C.starts;
}

#define JOIN_BLOCK 256
#define JOIN_TILE 2048     // runs of both lists at most
#define JOIN_SLOTS 1024    // code pairs, or polygon pairs, of a workgroup
#define JOIN_FILL 512      // taken slots after which the table goes out
#define JOIN_PROBES 8
#define JOIN_ASK 12        // taken slots of the table of all pairs before the question
#define JOIN_CELL_BITS 43  // a slot: cells (at most 4^21) below, intervals above
#define JOIN_MAX_TILES 256 // between two emptyings: fewer than 2^21 intervals
#define JOIN_EMPTY 0xffffffffffffffffull
#define JOIN_ALL ((uint64_t)1 << 17)     // possible pairs that get a slot each at once
#define JOIN_DIRECT ((uint64_t)1 << 22)  // slots up to which a second pass has enough for all

// Table of all pairs: open addressing, cap (a power of two) slots, at most
// `limit` further slots tried.
struct PairTab {
    unsigned long long *key;   // p << qbits | q, or JOIN_EMPTY
    unsigned long long *cells;
    uint64_t mask;
    uint64_t limit;
    int32_t qbits;
    unsigned long long *stat;  // intervals' pairs, then 1 if a pair found no slot
};

__device__ __forceinline__ uint64_t pair_hash(uint64_t k)
{
    k *= 0x9e3779b97f4a7c15ull;
    return k ^ (k >> 29);
}

// whether a pair has found no slot: the pass is made again with a larger table,
// and only counts from then on
__device__ __forceinline__ bool pair_full(const PairTab &T)
{
    return __hip_atomic_load(&T.stat[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// false: the table is too small
__device__ __forceinline__ bool pair_add(const PairTab &T, uint64_t key, uint64_t cells)
{
    uint64_t h = pair_hash(key) & T.mask;
    for (uint64_t k = 0; k <= T.limit; k++) {
        if (k == JOIN_ASK && pair_full(T)) return false;
        unsigned long long cur =
            __hip_atomic_load(&T.key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == JOIN_EMPTY) cur = atomicCAS(&T.key[h], JOIN_EMPTY, (unsigned long long)key);
        if (cur == JOIN_EMPTY || cur == key) {
            atomicAdd(&T.cells[h], (unsigned long long)cells);
            return true;
        }
        h = (h + 1) & T.mask;
    }
    atomicMax(&T.stat[1], 1ull);
    return false;
}

// add(p << qbits | q) for every member pair of two codes until it says false
// (nothing if `ok` does); returns their number
template <typename ADD>
__device__ __forceinline__ uint64_t codes_add(const PairTab &T, const CanvasView &A,
                                              const CanvasView &B, uint32_t a, uint32_t b, bool ok,
                                              ADD add)
{
    const int64_t ma = members(A, a), mb = members(B, b);
    for (int64_t x = 0; x < ma && ok; x++) {
        const uint64_t p = (uint64_t)member(A, a, x) << T.qbits;
        for (int64_t y = 0; y < mb && ok; y++) ok = add(p | member(B, b, y));
    }
    return (uint64_t)(ma * mb);
}

__global__ void k_pair_clear(PairTab T)
{
    const uint64_t t0 = (uint64_t)blockIdx.x * 1024 + threadIdx.x;
#pragma unroll
    for (int u = 0; u < 4; u++) {
        const uint64_t t = t0 + u * 256;
        if (t > T.mask) break;
        T.key[t] = JOIN_EMPTY;
        T.cells[t] = 0;
    }
    if (t0 < 3) T.stat[t0] = 0;
}

// The runs of A among the first t * tile of the merged list (of equal first keys
// B's comes first).
template <typename K>
__global__ void k_join_split(CanvasView A, CanvasView B, int tile, int64_t tiles, int64_t *split)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t > tiles) return;
    const K *ka = starts_of<K>(A), *kb = starts_of<K>(B);
    const int64_t d = min(t * tile, A.n + B.n);
    int64_t lo = max((int64_t)0, d - B.n), hi = min(d, A.n);
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (ka[mid] < kb[d - 1 - mid]) lo = mid + 1; else hi = mid;
    }
    split[t] = lo;
}

// LDS slot of key w, taken now if it has none (fill counts those); JOIN_SLOTS: no
// slot near
__device__ __forceinline__ uint32_t lds_slot(unsigned long long *tkey, uint32_t *fill,
                                             unsigned long long w)
{
    uint32_t h = (uint32_t)(pair_hash(w) >> 20) & (JOIN_SLOTS - 1);
    for (int q = 0; q < JOIN_PROBES; q++) {
        unsigned long long cur = tkey[h];
        if (cur == JOIN_EMPTY) {
            cur = atomicCAS(&tkey[h], JOIN_EMPTY, w);
            if (cur == JOIN_EMPTY) atomicAdd(fill, 1u);
        }
        if (cur == JOIN_EMPTY || cur == w) return h;
        h = (h + 1) & (JOIN_SLOTS - 1);
    }
    return JOIN_SLOTS;
}

// PAIRS: the LDS table is of polygon pairs, which every interval adds its cells
// to, else of pairs of codes, expanded when it goes out.  With sets of two, as
// along a partition's sides, code pairs take half the additions; where polygons
// lie in layers, nearly every interval has codes of its own and all of them meet
// the same pairs (3,000 by 3,000 rectangles, 5 by 5 of them a cell: 8.7 ms with
// pairs of codes, now 1.1; sorting all pairs of intervals took 4.5).
template <typename K, bool PAIRS>
__global__ __launch_bounds__(JOIN_BLOCK) void k_join(CanvasView A, CanvasView B, uint64_t total,
                                                     const int64_t *__restrict__ split, int tile,
                                                     int64_t tiles, PairTab T)
{
    // both lists' parts of the tile, each with the run before it and the first
    // key after it
    __shared__ K key[JOIN_TILE + 4];
    __shared__ uint32_t code[JOIN_TILE + 4];
    __shared__ unsigned long long tkey[JOIN_SLOTS], tval[JOIN_SLOTS];
    __shared__ uint32_t fill;
    __shared__ int full;  // a pair has found no slot: only count
    const K *gka = starts_of<K>(A), *gkb = starts_of<K>(B);
    for (int k = threadIdx.x; k < JOIN_SLOTS; k += JOIN_BLOCK) {
        tkey[k] = JOIN_EMPTY;
        tval[k] = 0;
    }
    if (threadIdx.x == 0) {
        fill = 0;
        full = 0;
    }
    uint64_t np = 0;
    int since = 0;
    const int64_t per = (tiles + gridDim.x - 1) / gridDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * per, t1 = min(t0 + per, tiles);
    for (int64_t t = t0; t < t1; t++) {
        const int64_t i0 = split[t], i1 = split[t + 1];
        const int64_t j0 = t * tile - i0, j1 = min((t + 1) * tile, A.n + B.n) - i1;
        const int na = (int)(i1 - i0), nb = (int)(j1 - j0);
        K *ka = key, *kb = key + na + 2;
        uint32_t *ca = code, *cb = code + na + 2;
        __syncthreads();
        for (int x = threadIdx.x; x < na + 2; x += JOIN_BLOCK) {
            const int64_t i = i0 - 1 + x;
            const bool in = i >= 0 && i < A.n;
            ka[x] = in ? gka[i] : (K)0;
            ca[x] = in ? A.code[i] : 0u;
        }
        for (int y = threadIdx.x; y < nb + 2; y += JOIN_BLOCK) {
            const int64_t j = j0 - 1 + y;
            const bool in = j >= 0 && j < B.n;
            kb[y] = in ? gkb[j] : (K)0;
            cb[y] = in ? B.code[j] : 0u;
        }
        __syncthreads();
        for (int z = threadIdx.x; z < na + nb; z += JOIN_BLOCK) {
            // the interval that starts with run x of A, or y of B: the other
            // list's last run that does not start after it (a run of B that
            // starts with one of A belongs to that one's interval)
            int x, y;
            uint64_t k;
            if (z < na) {
                x = z + 1;
                k = ka[x];
                int lo = 0, hi = nb;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (kb[mid + 1] <= (K)k) lo = mid + 1; else hi = mid;
                }
                y = lo;
            } else {
                y = z - na + 1;
                k = kb[y];
                int lo = 0, hi = na;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (ka[mid + 1] < (K)k) lo = mid + 1; else hi = mid;
                }
                x = lo;
                if (i0 + x < A.n && ka[x + 1] == (K)k) continue;
            }
            const uint32_t a = ca[x], b = cb[y];
            if (a == 0 || b == 0) continue;
            const uint64_t ea = i0 + x < A.n ? (uint64_t)ka[x + 1] : total;
            const uint64_t eb = j0 + y < B.n ? (uint64_t)kb[y + 1] : total;
            const uint64_t len = (ea < eb ? ea : eb) - k;
            auto ok = [&] { return *(volatile int *)&full == 0; };
            if (PAIRS) {
                np += codes_add(T, A, B, a, b, ok(), [&](uint64_t pair) {
                    const uint32_t h = lds_slot(tkey, &fill, pair);
                    if (h < JOIN_SLOTS) atomicAdd(&tval[h], (unsigned long long)len);
                    else if (!pair_add(T, pair, len)) return full = 1, false;
                    return true;
                });
            } else {
                const uint32_t h = lds_slot(tkey, &fill, (unsigned long long)a << 32 | b);
                if (h < JOIN_SLOTS) atomicAdd(&tval[h], 1ull << JOIN_CELL_BITS | len);
                else
                    np += codes_add(T, A, B, a, b, ok(), [&](uint64_t pair) {
                        return pair_add(T, pair, len) || (full = 1, false);
                    });
            }
        }
        __syncthreads();
        if (fill > JOIN_FILL || ++since == JOIN_MAX_TILES || t + 1 == t1) {
            if (threadIdx.x == 0 && pair_full(T)) full = 1;
            __syncthreads();
            for (int k = threadIdx.x; k < JOIN_SLOTS; k += JOIN_BLOCK) {
                const unsigned long long w = tkey[k], v = tval[k];
                if (w == JOIN_EMPTY) continue;
                tkey[k] = JOIN_EMPTY;
                tval[k] = 0;
                const bool ok = *(volatile int *)&full == 0;
                if (PAIRS) {
                    if (ok && !pair_add(T, w, v)) full = 1;
                } else {
                    const uint64_t cells = v & ((1ull << JOIN_CELL_BITS) - 1);
                    np += (v >> JOIN_CELL_BITS) *
                          codes_add(T, A, B, (uint32_t)(w >> 32), (uint32_t)w, ok,
                                    [&](uint64_t pair) {
                                        return pair_add(T, pair, cells) || (full = 1, false);
                                    });
                }
            }
            since = 0;
            __syncthreads();  // every lane has read the count
            if (threadIdx.x == 0) fill = 0;
        }
    }
    for (int o = 32; o > 0; o >>= 1) np += __shfl_xor((unsigned long long)np, o, 64);
    if ((threadIdx.x & 63) == 0 && np) atomicAdd(&T.stat[0], (unsigned long long)np);
}

// the taken slots of the table, in no order: key, place in this list, cells
__global__ __launch_bounds__(256) void k_pair_list(PairTab T, uint64_t *key, uint32_t *place,
                                                   uint64_t *cells)
{
    __shared__ uint32_t wc[4];
    __shared__ unsigned long long base;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t t0 = (uint64_t)blockIdx.x * 1024 + w * 256;
    unsigned long long k[4];
    uint64_t take[4];
    uint32_t c = 0;
#pragma unroll
    for (int u = 0; u < 4; u++) {
        const uint64_t t = t0 + u * 64 + lane;
        k[u] = t <= T.mask ? T.key[t] : JOIN_EMPTY;
        take[u] = __ballot(k[u] != JOIN_EMPTY);
        c += (uint32_t)__popcll(take[u]);
    }
    if (lane == 0) wc[w] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t all = wc[0] + wc[1] + wc[2] + wc[3];
        base = all ? atomicAdd(&T.stat[2], (unsigned long long)all) : 0;
    }
    __syncthreads();
    uint64_t at = base;
    for (int q = 0; q < w; q++) at += wc[q];
#pragma unroll
    for (int u = 0; u < 4; u++) {
        if (k[u] != JOIN_EMPTY) {
            const uint64_t o = at + __popcll(take[u] & ((1ull << lane) - 1));
            key[o] = k[u];
            place[o] = (uint32_t)o;
            cells[o] = T.cells[t0 + u * 64 + lane];
        }
        at += __popcll(take[u]);
    }
}

__global__ void k_pair_out(const uint64_t *key, const uint32_t *place, const uint64_t *sum,
                           int64_t nw, int32_t qbits, int32_t *pa, int32_t *pb, int64_t *cells)
{
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= nw) return;
    pa[u] = (int32_t)(key[u] >> qbits);
    pb[u] = (int32_t)(key[u] & (((uint64_t)1 << qbits) - 1));
    cells[u] = (int64_t)sum[place[u]];
}

CanvasView view_of(const sba_handle *h)
{
    return CanvasView{h->starts, h->starts32, h->run_code, h->n_runs, h->set_off, h->set_ids,
                      (uint32_t)h->n_polys, (uint32_t)h->n_sets};
}

}  // namespace

extern "C" int sba_join_pairs(const sba_handle *a, const sba_handle *b, int64_t cap, int32_t *pa,
                              int32_t *pb, int64_t *cells, int64_t *n_pairs, void *stream)
{
    if (!a || !b || !n_pairs || cap < 0 || (cap > 0 && (!pa || !pb || !cells))) return SBA_EINVAL;
    *n_pairs = 0;
    if (a->kind != SBA_KIND_HILBERT || b->kind != SBA_KIND_HILBERT || a->s != b->s)
        return SBA_EINVAL;
    if (a->n_polys == 0 || b->n_polys == 0 || a->n_runs == 0 || b->n_runs == 0) return 0;
    if (a->level != b->level || a->gi0 != b->gi0 || a->gj0 != b->gj0) return SBA_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    Workspace ws(st);
    const uint64_t total = (uint64_t)1 << (2 * a->level);
    const CanvasView A = view_of(a), B = view_of(b);

    // four workgroups a compute unit, as their LDS allows; smaller tiles where
    // there are too few runs for all of them
    const int64_t runs = a->n_runs + b->n_runs, wgs = (int64_t)cu_count() * 4;
    int tile = JOIN_TILE;
    while (tile > JOIN_BLOCK && runs < wgs * tile) tile >>= 1;
    const int64_t tiles = (runs + tile - 1) / tile;
    const bool k32 = a->starts32 && b->starts32;
    // sets of three polygons and more on average: layers
    const bool layers = a->n_set_ids >= 3 * std::max<int64_t>(a->n_sets, 1) ||
                        b->n_set_ids >= 3 * std::max<int64_t>(b->n_sets, 1);
    int64_t *split = nullptr;
    RC(ws.alloc(&split, tiles + 1));
    if (k32)
        hipLaunchKernelGGL(k_join_split<uint32_t>, dim3(grid_for(tiles + 1)), dim3(256), 0, st, A,
                           B, tile, tiles, split);
    else
        hipLaunchKernelGGL(k_join_split<uint64_t>, dim3(grid_for(tiles + 1)), dim3(256), 0, st, A,
                           B, tile, tiles, split);
    HIP_OK(hipGetLastError());

    // Two partitions meet in a few pairs a polygon, so the table starts at
    // eight slots or more a polygon, or with one for every pair there could be if
    // those are few; polygons that overlap many others take a
    // second pass with a larger one (at most two to four slots for each
    // pair of an interval, where every pair finds one).  The pass that finds its
    // table too small makes no further additions and counts the pairs.
    PairTab T{};
    T.qbits = bits_for((uint64_t)b->n_polys - 1);
    const int kbits = std::max(1, T.qbits + bits_for((uint64_t)a->n_polys - 1));
    const uint64_t could = (uint64_t)a->n_polys * (uint64_t)b->n_polys;
    uint64_t slots = (uint64_t)1 << std::max(13, bits_for((uint64_t)(a->n_polys + b->n_polys)) + 3);
    if (could <= JOIN_ALL) slots = std::max(slots, (uint64_t)2 << bits_for(could));
    const dim3 nb((unsigned)std::min<int64_t>(tiles, wgs));
    auto join = [&](auto kern) {
        hipLaunchKernelGGL(kern, nb, dim3(JOIN_BLOCK), 0, st, A, B, total, split, tile, tiles, T);
    };
    RC(ws.alloc(&T.stat, 3));
    uint64_t *key = nullptr, *sum = nullptr;
    uint32_t *place = nullptr;
    unsigned long long stat[3] = {0, 0, 0};
    for (uint64_t most = 0;;) {
        T.mask = slots - 1;
        T.limit = most && slots >= 2 * most ? T.mask : std::min<uint64_t>(T.mask, 256);
        RC(ws.alloc(&T.key, (int64_t)slots));
        RC(ws.alloc(&T.cells, (int64_t)slots));
        hipLaunchKernelGGL(k_pair_clear, dim3(grid_for((int64_t)slots, 1024)), dim3(256), 0, st, T);
        if (layers) {
            if (k32) join(k_join<uint32_t, true>);
            else join(k_join<uint64_t, true>);
        } else {
            if (k32) join(k_join<uint32_t, false>);
            else join(k_join<uint64_t, false>);
        }
        RC(ws.alloc(&key, (int64_t)slots));
        RC(ws.alloc(&sum, (int64_t)slots));
        RC(ws.alloc(&place, (int64_t)slots));
        hipLaunchKernelGGL(k_pair_list, dim3(grid_for((int64_t)slots, 1024)), dim3(256), 0, st, T, key,
                           place, sum);
        HIP_OK(hipGetLastError());
        RC(ws.read(stat, T.stat, sizeof(stat)));
        RC(ws.sync());
        const uint64_t NP = stat[0];
        if (NP == 0) return 0;
        if (NP >= ((uint64_t)1 << 32)) return SBA_ELIMIT;
        if (!stat[1]) break;
        ws.put(T.key);
        ws.put(T.cells);
        ws.put(key);
        ws.put(sum);
        ws.put(place);
        most = std::min(NP, could);  // different pairs
        const uint64_t all = (uint64_t)2 << bits_for(most);
        slots = all <= JOIN_DIRECT ? all : std::min(slots * 8, all);
    }
    const int64_t NU = (int64_t)stat[2];
    const int64_t nw = std::min(NU, cap);
    if (nw > 0) {
        RC(radix_sort_u64_ws(&key, &place, NU, kbits, ws));
        hipLaunchKernelGGL(k_pair_out, dim3(grid_for(nw)), dim3(256), 0, st, key, place, sum, nw,
                           T.qbits, pa, pb, cells);
        HIP_OK(hipGetLastError());
        HIP_OK(hipStreamSynchronize(st));
    }
    *n_pairs = NU;
    return 0;
}
