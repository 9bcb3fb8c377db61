// pindex.hip -- point-side pre-aggregation (Sec. 3, point indexing).
//
// The points are mapped to the cells of the same grid as the polygon
// approximations (side s(eps)), the cells linearised with the Hilbert curve,
// and the keys sorted; the values are permuted the same way and turned into
// an exclusive prefix-sum array.  Then for any key range [a, b)
//     COUNT = lb(b) - lb(a),   SUM = prefix[lb(b)] - prefix[lb(a)],
// with lb the lower bound in the sorted keys.  A Hilbert handle built on the
// index's key grid stores its approximation as runs of consecutive keys with
// one polygon set each, so a polygon query costs two lower bounds per run (a
// run is a union of aligned quadtree cells, the query cells of the method)
// and no pass over the points.
//
// Lower bounds come from a binary search or from a RadixSpline (Sec. 3):
// spline knots on the step function F(v) = lb(v) with every key's error at
// most E positions, and a radix table over the top bits of the key that
// narrows the knot search.  The estimate is followed by a binary search in a
// window of 2E + 3 positions, checked at both ends, and a full binary search
// if the check ever fails.
//
// Spline (greedy corridor, Neumann & Michel 2008, the construction RadixSpline
// uses): F is a step function, so it is enough to bound the error at the two
// ends of every step: for distinct keys D_0 < ... < D_{M-1} with first
// positions P_m, the corners (D_{m-1} + 1, P_m) and (D_m, P_m) (D_{-1} + 1 =
// 0), then (D_{M-1} + 1, n) and (4^L, n).  The distinct keys are cut into
// chunks; one thread runs the greedy corridor over the corners of each chunk
// from its first to its last corner (both become knots).  Two consecutive
// corners are exact on every integer key between them, so the chunk seams add
// no error.
#include <chrono>
#include <new>
#include <vector>

#include "sba_internal.h"
#include "wave.h"

struct sba_pindex {
    int device = 0;
    int64_t n = 0, eps = 0, s = 0;
    int64_t gi0 = 0, gj0 = 0;  // key grid origin (cells)
    int32_t L = 1;             // key grid side 2^L cells
    uint32_t mag = 0;
    int32_t shift = 0;
    uint64_t *keys = nullptr;  // [n] ascending Hilbert keys of the points' cells
    int64_t *psum = nullptr;   // [n + 1] exclusive prefix sums of the values (NULL: none)
    int64_t n_distinct = 0;
    // RadixSpline
    int32_t radix_bits = 0, spline_err = 0, rshift = 0;
    int64_t n_knots = 0;
    uint64_t *kx = nullptr;    // [n_knots] knot keys, kx[0] = 0, last = 4^L, non-decreasing
    int64_t *ky = nullptr;     // [n_knots] knot positions
    uint32_t *rtab = nullptr;  // [2^radix_bits + 2] knots whose key prefix is below p
    int64_t bytes = 0;
    double build_ms = 0;
    std::vector<DevBlock> owned;
};

template <typename T>
static int ix_alloc(sba_pindex *ix, T **p, int64_t n)
{
    DevBlock b{};
    const size_t bytes = (size_t)(n > 0 ? n : 1) * sizeof(T);
    RC(cache_get(bytes, &b));
    ix->owned.push_back(b);
    ix->bytes += (int64_t)bytes;
    *p = (T *)b.p;
    return 0;
}

static void ix_release(sba_pindex *ix)
{
    for (const DevBlock &b : ix->owned) cache_put(b);
    ix->owned.clear();
}

// ---------------------------------------------------------------- build kernels

// two points, or four keys (the caller's points are 8-byte aligned)
typedef int32_t pt2_t __attribute__((ext_vector_type(4), aligned(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

#define BOX_BLOCKS 1024

// min x, min y, max x, max y of each workgroup's points, then of all.  (One
// atomic a wavefront to four shared words: 435 us for 5e7 points; here 72,
// the time of a plain read.)
__global__ __launch_bounds__(512) void k_box(const int32_t *__restrict__ xy, int64_t n,
                                             int4 *__restrict__ part)
{
    __shared__ int4 wb[8];
    int32_t x0 = INT32_MAX, y0 = INT32_MAX, x1 = INT32_MIN, y1 = INT32_MIN;
    auto take = [&](pt2_t p) {
        x0 = min(x0, min(p.x, p.z));
        y0 = min(y0, min(p.y, p.w));
        x1 = max(x1, max(p.x, p.z));
        y1 = max(y1, max(p.y, p.w));
    };
    const pt2_t *p2 = (const pt2_t *)xy;
    const int64_t np = n >> 1, stride = (int64_t)gridDim.x * 512;
    int64_t t = (int64_t)blockIdx.x * 512 + threadIdx.x;
    for (; t + 3 * stride < np; t += 4 * stride) {
        pt2_t v[4];
#pragma unroll
        for (int u = 0; u < 4; u++) v[u] = p2[t + u * stride];
#pragma unroll
        for (int u = 0; u < 4; u++) take(v[u]);
    }
    for (; t < np; t += stride) take(p2[t]);
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        const int32_t x = xy[2 * (n - 1)], y = xy[2 * (n - 1) + 1];
        take(pt2_t{x, y, x, y});
    }
    for (int o = 32; o > 0; o >>= 1) {
        x0 = min(x0, __shfl_xor(x0, o, 64));
        y0 = min(y0, __shfl_xor(y0, o, 64));
        x1 = max(x1, __shfl_xor(x1, o, 64));
        y1 = max(y1, __shfl_xor(y1, o, 64));
    }
    if ((threadIdx.x & 63) == 0) wb[threadIdx.x >> 6] = make_int4(x0, y0, x1, y1);
    __syncthreads();
    if (threadIdx.x == 0) {
        int4 r = wb[0];
        for (int k = 1; k < 8; k++)
            r = make_int4(min(r.x, wb[k].x), min(r.y, wb[k].y), max(r.z, wb[k].z),
                          max(r.w, wb[k].w));
        part[blockIdx.x] = r;
    }
}

__global__ __launch_bounds__(BOX_BLOCKS) void k_box_all(const int4 *part, int nparts, int32_t *box)
{
    __shared__ int4 wb[BOX_BLOCKS / 64];
    int4 r = make_int4(INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN);
    if ((int)threadIdx.x < nparts) r = part[threadIdx.x];
    for (int o = 32; o > 0; o >>= 1) {
        r.x = min(r.x, __shfl_xor(r.x, o, 64));
        r.y = min(r.y, __shfl_xor(r.y, o, 64));
        r.z = max(r.z, __shfl_xor(r.z, o, 64));
        r.w = max(r.w, __shfl_xor(r.w, o, 64));
    }
    if ((threadIdx.x & 63) == 0) wb[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < BOX_BLOCKS / 64; k++)
            r = make_int4(min(r.x, wb[k].x), min(r.y, wb[k].y), max(r.z, wb[k].z),
                          max(r.w, wb[k].w));
        box[0] = r.x;
        box[1] = r.y;
        box[2] = r.z;
        box[3] = r.w;
    }
}

// Hilbert key of each point's cell (the box holds every point, so the
// offsets from the grid origin lie in [0, 2^31)).  Keys of up to 32 bits go
// through the table of four levels a step.
template <typename K>
__global__ __launch_bounds__(256) void k_point_keys(const int32_t *__restrict__ xy, int64_t n,
                                                    int64_t ox, int64_t oy, uint32_t mag,
                                                    int32_t shift, int L, K *__restrict__ keys)
{
    __shared__ uint16_t tab[HILBERT_TAB];
    if (sizeof(K) == 4) {
        for (int e = threadIdx.x; e < HILBERT_TAB; e += 256) tab[e] = hilbert_tab_entry((uint32_t)e);
        __syncthreads();
    }
    auto key = [&](int32_t x, int32_t y) {
        const uint32_t i = divmagic((uint32_t)((int64_t)x - ox), mag, shift);
        const uint32_t j = divmagic((uint32_t)((int64_t)y - oy), mag, shift);
        return sizeof(K) == 4 ? (K)hilbert_index_tab(L, i, j, tab) : (K)hilbert_index(L, i, j);
    };
    const int64_t nq = n >> 2;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < nq; t += (int64_t)gridDim.x * 256) {
        const pt2_t a = ((const pt2_t *)xy)[2 * t], b = ((const pt2_t *)xy)[2 * t + 1];
        K k[4] __attribute__((aligned(16))) = {key(a.x, a.y), key(a.z, a.w), key(b.x, b.y),
                                               key(b.z, b.w)};
#pragma unroll
        for (int u = 0; u < (int)sizeof(K) / 4; u++)
            ((u32x4_t *)(keys + 4 * t))[u] = ((const u32x4_t *)k)[u];
    }
    const int64_t r = 4 * nq + threadIdx.x;
    if (blockIdx.x == 0 && r < n) keys[r] = key(xy[2 * r], xy[2 * r + 1]);
}

// What the index keeps of the sorted keys and values, in two passes over
// tiles of IX_TILE: the tiles' numbers of distinct keys and sums of values,
// then (their scans between) the 64-bit keys, the values' exclusive prefix
// sums, and each distinct key with its first position.  A wavefront owns 512
// consecutive keys, 64 a round.  Both passes are bound by their traffic, 12
// bytes a key in each and up to 24 out: 5e7 keys take 0.15 and 0.36 ms (as
// separate kernels over arrays of 64-bit flags, copies and gathered values,
// 2.4 ms).
#define IX_BLOCK 512
#define IX_ROUNDS 8
#define IX_TILE (IX_BLOCK * IX_ROUNDS)

template <typename K, bool VALS>
__global__ __launch_bounds__(IX_BLOCK) void k_ix_count(const K *__restrict__ keys,
                                                       const int64_t *__restrict__ vals, int64_t n,
                                                       int64_t *__restrict__ tcnt,
                                                       int64_t *__restrict__ tsum)
{
    __shared__ uint32_t wc[IX_BLOCK / 64];
    __shared__ int64_t wv[IX_BLOCK / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * IX_TILE + w * (64 * IX_ROUNDS);
    uint32_t c = 0;
    int64_t sum = 0;
#pragma unroll
    for (int q = 0; q < IX_ROUNDS; q++) {
        const int64_t t = base + q * 64 + lane;
        if (t < n) {
            if (VALS) sum += vals[t];
            c += t == 0 || keys[t] != keys[t - 1];
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        c += (uint32_t)__shfl_xor((int)c, o, 64);
        if (VALS) sum += __shfl_xor((long long)sum, o, 64);
    }
    if (lane == 0) {
        wc[w] = c;
        wv[w] = sum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < IX_BLOCK / 64; k++) {
            c += wc[k];
            sum += wv[k];
        }
        tcnt[blockIdx.x] = c;
        if (VALS) tsum[blockIdx.x] = sum;
    }
}

template <typename K, bool VALS>
__global__ __launch_bounds__(IX_BLOCK) void k_ix_write(const K *__restrict__ keys,
                                                       const int64_t *__restrict__ vals, int64_t n,
                                                       const int64_t *__restrict__ tcnt,
                                                       const int64_t *__restrict__ tsum,
                                                       uint64_t *__restrict__ okeys,
                                                       int64_t *__restrict__ psum,
                                                       K *__restrict__ D, uint32_t *__restrict__ P)
{
    __shared__ uint32_t wc[IX_BLOCK / 64];
    __shared__ uint64_t wv[IX_BLOCK / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * IX_TILE + w * (64 * IX_ROUNDS);
    K key[IX_ROUNDS];
    uint64_t v[IX_ROUNDS], excl[IX_ROUNDS], head[IX_ROUNDS];
    bool first[IX_ROUNDS];
#pragma unroll
    for (int q = 0; q < IX_ROUNDS; q++) {
        const int64_t t = base + q * 64 + lane;
        key[q] = t < n ? keys[t] : (K)0;
        first[q] = t < n && (t == 0 || key[q] != keys[t - 1]);
        v[q] = (VALS && t < n) ? (uint64_t)vals[t] : 0;
    }
    uint32_t c = 0;
    uint64_t sum = 0;
#pragma unroll
    for (int q = 0; q < IX_ROUNDS; q++) {
        head[q] = __ballot(first[q]);
        c += (uint32_t)__popcll(head[q]);
        if (VALS) {
            const uint64_t incl = wave_scan<OpAdd>(v[q]);
            excl[q] = sum + incl - v[q];
            sum += (uint64_t)__shfl((unsigned long long)incl, 63, 64);
        }
    }
    if (lane == 0) {
        wc[w] = c;
        wv[w] = sum;
    }
    __syncthreads();
    int64_t at = tcnt[blockIdx.x];
    uint64_t before = VALS ? (uint64_t)tsum[blockIdx.x] : 0;
    for (int k = 0; k < w; k++) {
        at += wc[k];
        before += wv[k];
    }
    const uint64_t lt = lane ? ~0ull >> (64 - lane) : 0;
#pragma unroll
    for (int q = 0; q < IX_ROUNDS; q++) {
        const int64_t t = base + q * 64 + lane;
        if (t < n) {
            okeys[t] = (uint64_t)key[q];
            if (VALS) {
                psum[t] = (int64_t)(before + excl[q]);
                if (t == n - 1) psum[n] = (int64_t)(before + excl[q] + v[q]);
            }
            if (first[q]) {
                const int64_t m = at + __popcll(head[q] & lt);
                D[m] = key[q];
                P[m] = (uint32_t)t;
            }
        }
        at += __popcll(head[q]);
    }
}

// the distinct keys, ascending, and their first positions (M of them, on the
// device); both arrays have room for SPLINE_PF more entries than keys
template <typename K>
struct Corners {
    const K *D;
    const uint32_t *P;
    const int64_t *M;
    int64_t n;
    uint64_t total;
};

#define SPLINE_CHUNK 1024
#define SPLINE_PF 8
#define SPLINE_CAP 64     // knots kept from the first pass

// Greedy corridor over the corners of the distinct keys [c * SPLINE_CHUNK,
// min((c+1) * SPLINE_CHUNK, M)) (the last chunk also takes the two corners
// after the last key): the knot moves to the previous corner as soon as a
// corner's slope from the knot leaves the band of slopes that keeps every
// corner since the knot within E.  Slopes are compared as cross products (no
// divisions; positive run lengths).  One thread a chunk: what bounds it is the
// serial chain from corner to corner, so a step takes no branch but the knot's
// and the keys are read SPLINE_PF at a time, the next ones while these are
// used (16 or 32 at a time: the same).  5e7 keys: 2 x 470 us as a counting and
// a writing pass of branching steps, 288 here.
template <typename K, typename EMIT>
__device__ __forceinline__ void spline_chunk(const Corners<K> &C, int64_t M, double E, int64_t c,
                                             EMIT emit)
{
    const int64_t a = c * SPLINE_CHUNK, b = min(a + SPLINE_CHUNK, M);
    constexpr int DV = SPLINE_PF * sizeof(K) / 16, PV = SPLINE_PF / 4;
    struct Group {
        u32x4_t d[DV], p[PV];
        __device__ K key(int t) const
        {
            if (sizeof(K) == 4) return (K)d[t >> 2][t & 3];
            return (K)((uint64_t)d[(t >> 1) & (DV - 1)][2 * (t & 1)] |
                       (uint64_t)d[(t >> 1) & (DV - 1)][2 * (t & 1) + 1] << 32);
        }
    };
    auto load = [&](Group &g, int64_t m) {
#pragma unroll
        for (int u = 0; u < DV; u++) g.d[u] = ((const u32x4_t *)(C.D + m))[u];
#pragma unroll
        for (int u = 0; u < PV; u++) g.p[u] = ((const u32x4_t *)(C.P + m))[u];
    };
    Group g, gn;
    load(gn, a);
    // keys and positions are below 2^53, so differences of doubles are exact
    double x0 = a == 0 ? 0.0 : (double)((uint64_t)C.D[a - 1] + 1), lx = x0;
    double y0 = (double)C.P[a], ly = y0;
    emit(x0, y0);
    // band: slopes in [ln/ld, un/ud], none yet.  A corner fed again, or the
    // knot itself, changes nothing.
    const double INF = __builtin_inf();
    double un = INF, ud = 1, ln = -INF, ld = 1;
    auto feed = [&](double x, double y) {
        double dx = x - x0, dy = y - y0;
        if (dy * ud > un * dx || dy * ld < ln * dx) {
            emit(lx, ly);
            x0 = lx;
            y0 = ly;
            dx = x - x0;
            dy = y - y0;
            un = INF;
            ln = -INF;
            ud = ld = 1;
        }
        const double yu = dy + E, yl = dy - E;
        const bool up = yu * ud < un * dx, lo = yl * ld > ln * dx;
        un = up ? yu : un;
        ud = up ? dx : ud;
        ln = lo ? yl : ln;
        ld = lo ? dx : ld;
        lx = x;
        ly = y;
    };
    double prev = (double)C.D[a];
    feed(prev, y0);
    const int len = (int)(b - a);
    for (int j = 0; j < len; j += SPLINE_PF) {
        g = gn;
        if (j + SPLINE_PF < len) load(gn, a + j + SPLINE_PF);
#pragma unroll
        for (int t = 0; t < SPLINE_PF; t++) {
            if (j + t > 0 && j + t < len) {
                const double y = (double)g.p[t >> 2][t & 3], x = (double)g.key(t);
                feed(prev + 1, y);
                prev = x;
                feed(prev, y);
            }
        }
    }
    if (b == M) {
        feed(prev + 1, (double)C.n);
        feed((double)C.total, (double)C.n);
    }
    if (lx != x0) emit(lx, ly);
}

// knots of each chunk: their number, and the first SPLINE_CAP of them
template <typename K>
__global__ __launch_bounds__(64) void k_spline(Corners<K> C, double E, int64_t chunks, int64_t *cnt,
                                               uint64_t *tx, uint32_t *ty)
{
    const int64_t c = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (c >= chunks) return;
    const int64_t M = *C.M;
    int64_t k = 0;
    if (c * SPLINE_CHUNK < M) {
        spline_chunk<K>(C, M, E, c, [&](double x, double y) {
            if (k < SPLINE_CAP) {
                tx[c * SPLINE_CAP + k] = (uint64_t)x;
                ty[c * SPLINE_CAP + k] = (uint32_t)y;
            }
            k++;
        });
    }
    cnt[c] = k;
}

// the chunks' knots to their places, a wavefront each; a chunk of more than
// SPLINE_CAP walks its corridor again
template <typename K>
__global__ __launch_bounds__(256) void k_knots(Corners<K> C, double E, int64_t chunks,
                                               const int64_t *off, int64_t nk, const uint64_t *tx,
                                               const uint32_t *ty, uint64_t *kx, int64_t *ky)
{
    const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= chunks) return;
    const int64_t o = off[c], m = (c + 1 < chunks ? off[c + 1] : nk) - o;
    if (m <= SPLINE_CAP) {
        if (lane < m) {
            kx[o + lane] = tx[c * SPLINE_CAP + lane];
            ky[o + lane] = ty[c * SPLINE_CAP + lane];
        }
    } else if (lane == 0) {
        int64_t k = 0;
        spline_chunk<K>(C, *C.M, E, c, [&](double x, double y) {
            if (k < m) {  // the same number again
                kx[o + k] = (uint64_t)x;
                ky[o + k] = (int64_t)y;
            }
            k++;
        });
    }
}

// rtab[p] = number of knots whose key is below p << rshift
__global__ void k_radix_table(const uint64_t *kx, int64_t nk, int32_t rshift, int64_t entries,
                              uint32_t *rtab)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= entries) return;
    const uint64_t v = (uint64_t)p << rshift;
    int64_t lo = 0, hi = nk;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (kx[mid] < v) lo = mid + 1; else hi = mid;
    }
    rtab[p] = (uint32_t)lo;
}

// ---------------------------------------------------------------- query

struct IxView {
    const uint64_t *keys;
    const int64_t *psum;
    int64_t n;
    uint64_t total;  // 4^L
    const uint64_t *kx;
    const int64_t *ky;
    const uint32_t *rtab;
    int64_t nk;
    int32_t rshift, err;
};

struct RunsView {
    const uint64_t *starts;
    const uint32_t *code;
    int64_t n;
    const int64_t *set_off;
    const int32_t *set_ids;
    uint32_t np, n_sets;
};

// first position in [lo, hi) whose key is >= v (hi if none)
__device__ __forceinline__ int64_t lower_bound_in(const uint64_t *keys, int64_t lo, int64_t hi,
                                                  uint64_t v)
{
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int64_t rs_lower_bound(const IxView &V, uint64_t v,
                                                  unsigned long long *fallbacks = nullptr)
{
    // last knot with key <= v lies in [rtab[p] - 1, rtab[p+1] - 1]
    const uint64_t p = v >> V.rshift;
    int64_t lo = V.rtab[p], hi = (int64_t)V.rtab[p + 1] - 1;
    lo = lo > 0 ? lo - 1 : 0;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (V.kx[mid] <= v) lo = mid; else hi = mid - 1;
    }
    double y = (double)V.ky[lo];
    if (lo + 1 < V.nk)
        y += (double)(v - V.kx[lo]) * (double)(V.ky[lo + 1] - V.ky[lo]) /
             (double)(V.kx[lo + 1] - V.kx[lo]);
    const int64_t est = (int64_t)y;
    int64_t a = est - V.err - 1, b = est + V.err + 2;
    a = a < 0 ? 0 : (a > V.n ? V.n : a);
    b = b < a ? a : (b > V.n ? V.n : b);
    // the answer lies in [a, b] when the keys just outside the window agree
    if ((a == 0 || V.keys[a - 1] < v) && (b == V.n || V.keys[b] >= v))
        return lower_bound_in(V.keys, a, b, v);
    if (fallbacks) atomicAdd(fallbacks, 1ull);
    return lower_bound_in(V.keys, 0, V.n, v);
}

// (count, sum) of a run to its polygon or to every member of its set
template <bool VALS>
__device__ __forceinline__ void add_run(const RunsView &R, uint32_t code, unsigned long long c,
                                        unsigned long long sv, unsigned long long *counts,
                                        unsigned long long *sums)
{
    if (code < CODE_SET_BASE) {
        const uint32_t p = code - 1u;
        if (p >= R.np) return;
        atomicAdd(&counts[p], c);
        if (VALS) atomicAdd(&sums[p], sv);
    } else {
        const uint32_t k = code - CODE_SET_BASE;
        if (k >= R.n_sets) return;
        for (int64_t q = R.set_off[k], e = R.set_off[k + 1]; q < e; q++) {
            const uint32_t p = (uint32_t)R.set_ids[q];
            if (p >= R.np) continue;
            atomicAdd(&counts[p], c);
            if (VALS) atomicAdd(&sums[p], sv);
        }
    }
}

// A wavefront takes 63 consecutive runs: lane k finds the lower bound of
// start k (start R.n is 4^L), so run k's points are [lb_k, lb_{k+1}) with
// one search per lane.  Lanes with the same code then combine their counts
// and sums (runs along the curve meet few polygons), and one lane per code
// adds them to the outputs.
template <bool VALS, bool RS>
__global__ __launch_bounds__(256) void k_pindex_agg(IxView V, RunsView R,
                                                    unsigned long long *counts,
                                                    unsigned long long *sums)
{
    const int lane = threadIdx.x & 63;
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; w * 63 < R.n;
         w += nw) {
        const int64_t t = w * 63 + lane;
        int64_t lb = 0;
        if (t <= R.n) {
            const uint64_t v = t < R.n ? R.starts[t] : V.total;
            lb = RS ? rs_lower_bound(V, v) : lower_bound_in(V.keys, 0, V.n, v);
        }
        const int64_t ub = __shfl_down(lb, 1, 64);
        uint32_t code = 0;
        unsigned long long c = 0, sv = 0;
        if (lane < 63 && t < R.n) {
            code = R.code[t];
            c = (unsigned long long)(ub - lb);
            if (VALS && c) sv = (unsigned long long)(V.psum[ub] - V.psum[lb]);
            if (c == 0) code = 0;
        }
        unsigned long long todo = __ballot(code != 0);
        while (todo) {
            const int leader = __ffsll((long long)todo) - 1;
            const uint32_t lc = __shfl(code, leader, 64);
            const bool mine = code == lc;
            unsigned long long cc = mine ? c : 0ull, ss = mine ? sv : 0ull;
            for (int o = 32; o > 0; o >>= 1) {
                cc += __shfl_xor(cc, o, 64);
                if (VALS) ss += __shfl_xor(ss, o, 64);
            }
            if (lane == leader) add_run<VALS>(R, lc, cc, ss, counts, sums);
            todo &= ~__ballot(mine);
        }
    }
}

__global__ void k_pindex_zero(uint64_t *counts, int64_t *sums, int32_t np)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    counts[p] = 0;
    if (sums) sums[p] = 0;
}

// ---------------------------------------------------------------- build

// keys of K, sorted with the values, then everything that follows from them
template <typename K>
static int pindex_build_keys(const int32_t *xy, const int64_t *values, int64_t n, sba_pindex *ix,
                             Workspace &ws)
{
    hipStream_t st = ws.stream();
    const int L = ix->L;
    const double E = (double)ix->spline_err;
    K *keys = nullptr;
    int64_t *v = nullptr;
    RC(ws.alloc(&keys, n));
    hipLaunchKernelGGL(k_point_keys<K>, dim3(std::min<unsigned>(grid_for(n, 1024), 4096)),
                       dim3(256), 0, st, xy, n, ix->gi0 * ix->s, ix->gj0 * ix->s, ix->mag,
                       ix->shift, L, keys);
    HIP_OK(hipGetLastError());
    // the values move with their keys: a gather by sorted positions takes a
    // memory line for each (5e7 values: 1.06 ms)
    if (values) RC(radix_sort_vals_ws(&keys, values, &v, n, 2 * L, ws));
    else RC(radix_sort_keys_ws(&keys, n, 2 * L, ws));

    const int64_t tiles = (n + IX_TILE - 1) / IX_TILE;
    const int64_t chunks = (n + SPLINE_CHUNK - 1) / SPLINE_CHUNK;
    RC(ix_alloc(ix, &ix->keys, n));
    if (values) RC(ix_alloc(ix, &ix->psum, n + 1));
    int64_t *tcnt = nullptr, *tsum = nullptr, *tot = nullptr, *cnt = nullptr;
    K *D = nullptr;
    uint32_t *P = nullptr, *ty = nullptr;
    uint64_t *tx = nullptr;
    RC(ws.alloc(&tcnt, tiles));
    RC(ws.alloc(&tsum, tiles));
    RC(ws.alloc(&tot, 2));
    RC(ws.alloc(&D, n + SPLINE_PF));
    RC(ws.alloc(&P, n + SPLINE_PF));
    const dim3 nb((unsigned)tiles), blk(IX_BLOCK);
    if (values)
        hipLaunchKernelGGL((k_ix_count<K, true>), nb, blk, 0, st, keys, v, n, tcnt, tsum);
    else
        hipLaunchKernelGGL((k_ix_count<K, false>), nb, blk, 0, st, keys, v, n, tcnt, tsum);
    HIP_OK(hipGetLastError());
    const int64_t *const in[2] = {tcnt, tsum};
    int64_t *const out[2] = {tcnt, tsum}, *const total[2] = {tot, nullptr};
    const int64_t sizes[2] = {tiles, tiles};
    RC(scan_exclusive_i64_multi(values ? 2 : 1, in, out, sizes, total, st, &ws));
    if (values)
        hipLaunchKernelGGL((k_ix_write<K, true>), nb, blk, 0, st, keys, v, n, tcnt, tsum, ix->keys,
                           ix->psum, D, P);
    else
        hipLaunchKernelGGL((k_ix_write<K, false>), nb, blk, 0, st, keys, v, n, tcnt, tsum, ix->keys,
                           ix->psum, D, P);
    HIP_OK(hipGetLastError());
    ws.put(keys);
    if (v) ws.put(v);

    // RadixSpline knots over the corners of F, then the radix table
    const Corners<K> C{D, P, tot, n, (uint64_t)1 << (2 * L)};
    RC(ws.alloc(&cnt, chunks));
    RC(ws.alloc(&tx, chunks * SPLINE_CAP));
    RC(ws.alloc(&ty, chunks * SPLINE_CAP));
    hipLaunchKernelGGL(k_spline<K>, dim3(grid_for(chunks, 64)), dim3(64), 0, st, C, E, chunks, cnt,
                       tx, ty);
    HIP_OK(hipGetLastError());
    RC(scan_exclusive_i64(cnt, cnt, chunks, tot + 1, st, &ws));
    int64_t M = 0, nk = 0;
    RC(ws.read(&M, tot, sizeof(int64_t)));
    RC(ws.read(&nk, tot + 1, sizeof(int64_t)));
    RC(ws.sync());
    ix->n_distinct = M;
    ix->n_knots = nk;
    RC(ix_alloc(ix, &ix->kx, nk));
    RC(ix_alloc(ix, &ix->ky, nk));
    hipLaunchKernelGGL(k_knots<K>, dim3(grid_for(chunks, 4)), dim3(256), 0, st, C, E, chunks, cnt,
                       nk, tx, ty, ix->kx, ix->ky);
    HIP_OK(hipGetLastError());
    return 0;
}

static int pindex_build(const int32_t *xy, const int64_t *values, int64_t n, sba_pindex *ix,
                        hipStream_t st)
{
    Workspace ws(st);
    if (n == 0) return 0;
    int32_t *box = nullptr;
    int4 *part = nullptr;
    const unsigned nparts = std::min<unsigned>(grid_for(n, 1024), BOX_BLOCKS);
    RC(ws.alloc(&box, 4));
    RC(ws.alloc(&part, nparts));
    hipLaunchKernelGGL(k_box, dim3(nparts), dim3(512), 0, st, xy, n, part);
    hipLaunchKernelGGL(k_box_all, dim3(1), dim3(BOX_BLOCKS), 0, st, part, (int)nparts, box);
    HIP_OK(hipGetLastError());
    int32_t hb[4];
    RC(ws.read(hb, box, sizeof(hb)));
    RC(ws.sync());
    const int64_t s = ix->s;
    const int64_t gi0 = floordiv64(hb[0], s), gj0 = floordiv64(hb[1], s);
    const int64_t gw = floordiv64(hb[2], s) - gi0 + 1, gh = floordiv64(hb[3], s) - gj0 + 1;
    if (gw > MAX_GRID_SIDE || gh > MAX_GRID_SIDE) return SBA_ELIMIT;
    if (gw * s >= ((int64_t)1 << 31) || gh * s >= ((int64_t)1 << 31)) return SBA_ELIMIT;
    int L = 1;
    while (((int64_t)1 << L) < std::max(gw, gh)) L++;
    ix->gi0 = gi0;
    ix->gj0 = gj0;
    ix->L = L;
    // keys of 32 bits where they fit: a third of a sort pass's traffic less
    // than with 64
    if (2 * L <= 32) RC(pindex_build_keys<uint32_t>(xy, values, n, ix, ws));
    else RC(pindex_build_keys<uint64_t>(xy, values, n, ix, ws));
    ix->radix_bits = std::min(ix->radix_bits, 2 * L);
    ix->rshift = 2 * L - ix->radix_bits;
    const int64_t entries = ((int64_t)1 << ix->radix_bits) + 2;
    RC(ix_alloc(ix, &ix->rtab, entries));
    hipLaunchKernelGGL(k_radix_table, dim3(grid_for(entries)), dim3(256), 0, st, ix->kx,
                       ix->n_knots, ix->rshift, entries, ix->rtab);
    HIP_OK(hipGetLastError());
    HIP_OK(hipStreamSynchronize(st));
    return 0;
}

extern "C" int sba_pindex_build(const int32_t *xy, const int64_t *values, int64_t n, int64_t eps,
                                const sba_pindex_opts *opts, void *stream, sba_pindex **out)
{
    if (!out) return SBA_EINVAL;
    *out = nullptr;
    if (n < 0 || (n > 0 && !xy)) return SBA_EINVAL;
    if (((uintptr_t)xy & 7) != 0 || ((uintptr_t)values & 7) != 0) return SBA_EINVAL;
    if (eps < 2 || eps > ((int64_t)1 << 28)) return SBA_EINVAL;
    if (n >= ((int64_t)1 << 31)) return SBA_ELIMIT;
    sba_pindex_opts o{0, 0};
    if (opts) o = *opts;
    if (o.radix_bits == 0) o.radix_bits = 20;
    if (o.spline_err == 0) o.spline_err = 32;
    if (o.radix_bits < 1 || o.radix_bits > 28 || o.spline_err < 1 || o.spline_err > (1 << 20))
        return SBA_EINVAL;
    auto t0 = std::chrono::steady_clock::now();
    sba_pindex *ix = new (std::nothrow) sba_pindex();
    if (!ix) return SBA_ENOMEM;
    (void)hipGetDevice(&ix->device);
    ix->n = n;
    ix->eps = eps;
    ix->s = cell_side(eps);
    magic_for(ix->s, &ix->mag, &ix->shift);
    ix->radix_bits = o.radix_bits;
    ix->spline_err = o.spline_err;
    const int rc = pindex_build(xy, values, n, ix, (hipStream_t)stream);
    if (rc) {
        (void)hipStreamSynchronize((hipStream_t)stream);
        ix_release(ix);
        delete ix;
        return rc;
    }
    ix->build_ms =
        std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    *out = ix;
    return SBA_OK;
}

extern "C" int sba_pindex_info(const sba_pindex *ix, sba_pindex_info_t *info)
{
    if (!ix || !info) return SBA_EINVAL;
    sba_pindex_info_t o{};
    o.n = ix->n;
    o.eps = ix->eps;
    o.s = ix->s;
    o.key_i0 = ix->gi0;
    o.key_j0 = ix->gj0;
    o.key_level = ix->L;
    o.has_values = ix->psum != nullptr || ix->n == 0 ? 1 : 0;
    o.n_distinct = ix->n_distinct;
    o.n_knots = ix->n_knots;
    o.radix_bits = ix->radix_bits;
    o.spline_err = ix->spline_err;
    o.bytes = ix->bytes;
    o.build_ms = ix->build_ms;
    *info = o;
    return SBA_OK;
}

extern "C" int sba_pindex_aggregate(const sba_pindex *ix, const sba_handle *h, int32_t search,
                                    uint64_t *counts, int64_t *sums, void *stream)
{
    if (!ix || !h) return SBA_EINVAL;
    if (search != SBA_SEARCH_BINARY && search != SBA_SEARCH_LEARNED) return SBA_EINVAL;
    if (h->n_polys > 0 && !counts) return SBA_EINVAL;
    if (sums && ix->n > 0 && !ix->psum) return SBA_EINVAL;
    if (h->n_polys == 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    if (h->kind != SBA_KIND_HILBERT || h->s != ix->s) return SBA_EINVAL;
    const bool has_cells = h->gw > 0 && h->n_runs > 0;
    if (has_cells && (h->level != ix->L || h->gi0 != ix->gi0 || h->gj0 != ix->gj0))
        return SBA_EINVAL;
    hipLaunchKernelGGL(k_pindex_zero, dim3(grid_for(h->n_polys)), dim3(256), 0, st, counts, sums,
                       h->n_polys);
    HIP_OK(hipGetLastError());
    if (!has_cells || ix->n == 0) return 0;
    const IxView V{ix->keys, ix->psum, ix->n, (uint64_t)1 << (2 * ix->L), ix->kx, ix->ky,
                   ix->rtab, ix->n_knots, ix->rshift, ix->spline_err};
    const RunsView R{h->starts, h->run_code, h->n_runs, h->set_off, h->set_ids,
                     (uint32_t)h->n_polys, (uint32_t)h->n_sets};
    const dim3 grid(std::min<unsigned>(grid_for((h->n_runs + 62) / 63 * 64), 8192));
    unsigned long long *c = (unsigned long long *)counts, *sv = (unsigned long long *)sums;
    const bool vals = sums != nullptr;
    if (search == SBA_SEARCH_LEARNED) {
        if (vals) hipLaunchKernelGGL((k_pindex_agg<true, true>), grid, dim3(256), 0, st, V, R, c, sv);
        else hipLaunchKernelGGL((k_pindex_agg<false, true>), grid, dim3(256), 0, st, V, R, c, sv);
    } else {
        if (vals) hipLaunchKernelGGL((k_pindex_agg<true, false>), grid, dim3(256), 0, st, V, R, c, sv);
        else hipLaunchKernelGGL((k_pindex_agg<false, false>), grid, dim3(256), 0, st, V, R, c, sv);
    }
    HIP_OK(hipGetLastError());
    return 0;
}

__global__ void k_debug_lb(IxView V, const uint64_t *v, int64_t n, int32_t rs, int64_t *out,
                           unsigned long long *fallbacks)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const uint64_t q = v[t] < V.total ? v[t] : V.total;
    out[t] = rs ? rs_lower_bound(V, q, fallbacks) : lower_bound_in(V.keys, 0, V.n, q);
}

extern "C" int sba_debug_pindex_lb(const sba_pindex *ix, const uint64_t *v, int64_t n,
                                   int32_t search, int64_t *out, int64_t *fallbacks, void *stream)
{
    if (!ix || n < 0 || (n > 0 && (!v || !out))) return SBA_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    if (fallbacks) *fallbacks = 0;
    if (n == 0) return 0;
    if (ix->n == 0) {
        HIP_OK(hipMemsetAsync(out, 0, sizeof(int64_t) * n, st));
        HIP_OK(hipStreamSynchronize(st));
        return 0;
    }
    Workspace ws(st);
    unsigned long long *fb = nullptr;
    RC(ws.alloc(&fb, 1));
    HIP_OK(hipMemsetAsync(fb, 0, sizeof(unsigned long long), st));
    const IxView V{ix->keys, ix->psum, ix->n, (uint64_t)1 << (2 * ix->L), ix->kx, ix->ky,
                   ix->rtab, ix->n_knots, ix->rshift, ix->spline_err};
    hipLaunchKernelGGL(k_debug_lb, dim3(grid_for(n)), dim3(256), 0, st, V, v, n,
                       search == SBA_SEARCH_LEARNED ? 1 : 0, out, fb);
    HIP_OK(hipGetLastError());
    unsigned long long h = 0;
    RC(ws.read(&h, fb, sizeof(h)));
    RC(ws.sync());
    if (fallbacks) *fallbacks = (int64_t)h;
    return 0;
}

extern "C" void sba_pindex_free(sba_pindex *ix)
{
    if (!ix) return;
    ix_release(ix);
    delete ix;
}
