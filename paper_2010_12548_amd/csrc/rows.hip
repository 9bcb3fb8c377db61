// rows.hip -- coverage of the rows of cells: from the polygons' edges to the
// maximal row segments of constant polygon set (steps 1 to 4 of the build,
// see build.hip), one workgroup per row.
//
// An edge touches a handful of rows, and everything a row's segments depend
// on is the edges that touch it.  So the (edge, row) pairs are bucketed by
// row (count, scan, emit: k_edge_rows twice around k_row_scan), and one
// workgroup then sweeps each row in LDS (k_row_sweep): it sorts the row's
// pairs by (polygon, first cell), takes each polygon's coverage from their
// running end and crossing parity, sorts the changes of coverage by x, and
// writes the pieces between them that hold a polygon.  Nothing but the
// buckets (16 B a pair) and the segments goes through memory; sorting the
// same events globally by (polygon, row, x) and their toggles by (row, x)
// took 10 radix passes over 8 + 4 B each at 1 m (1.9 of the 2.2 ms build of
// 260 polygons on 57,143 rows).
//
// Rows with more pairs or toggles than a workgroup's LDS holds send the build
// back to the global sorts (build.hip).
#include <vector>

#include "sba_internal.h"
#include "wave.h"
#include "build_state.h"
#include "sets.h"

// ---------------------------------------------------------------- geometry

struct RowGeo {
    int64_t s;
    uint32_t mag;
    int32_t shift;
    int64_t ox, oy;          // coordinate of the box's first cell
    int64_t extx, exty;      // box extent in coordinate units (< 2^31)
    int64_t gi0, gj0;
    int32_t gw, gh;
    int use_b;               // boundary intervals count as covered
    int use_c;               // crossings are taken
    int need_b;              // pairs for every touched row (else crossed rows only)
    int centre;              // crossings of the centre lines
};

struct PolyView {
    const int32_t *ring_off;
    const int64_t *vert_off;
    const int32_t *xy;
    const int4 *bbox;
    const int32_t *hint;     // [ceil(nv / 64)] polygon of vertex 64 k
    int32_t np;
    int64_t nv;
};

// floor(d / s) for an offset d from the box's first cell, clamped to [-1, g]
__device__ __forceinline__ int32_t rel_cell(int64_t d, int64_t ext, int32_t g, const RowGeo &G)
{
    if (d < 0) return -1;
    if (d >= ext) return g;
    return (int32_t)divmagic((uint32_t)d, G.mag, G.shift);
}

struct Edge {
    int32_t x1, y1, x2, y2, p;
    bool first;              // first edge of its ring
};

// the edge that starts at vertex v < nv: its polygon is that of the first
// vertex of its 64, or one of the next
__device__ __forceinline__ Edge edge_of(const PolyView &P, int64_t v)
{
    int32_t p = P.hint[v >> 6];
    int32_t ra = P.ring_off[p], rb = P.ring_off[p + 1];
    int64_t end = P.vert_off[rb];
    while (end <= v) {  // ends at the last polygon: v < nv
        p++;
        ra = rb;
        rb = P.ring_off[p + 1];
        end = P.vert_off[rb];
    }
    // last ring of the polygon that starts at or before v
    int32_t lo = ra, len = rb - ra;
    while (len > 1) {
        const int32_t half = len >> 1;
        if (P.vert_off[lo + half] <= v) {
            lo += half;
            len -= half;
        } else {
            len = half;
        }
    }
    const int64_t r0 = P.vert_off[lo], r1 = lo + 1 == rb ? end : P.vert_off[lo + 1];
    const int64_t w = v + 1 < r1 ? v + 1 : r0;
    Edge E;
    E.p = p;
    E.x1 = P.xy[2 * v];
    E.y1 = P.xy[2 * v + 1];
    E.x2 = P.xy[2 * w];
    E.y2 = P.xy[2 * w + 1];
    E.first = v == r0;
    return E;
}

// The rows of an edge inside the box: pairs for rows [ra, ra + n), crossings
// of rows [ka, kb]; nb, nc: its boundary strips and crossings (the handle's
// figures).  An edge strictly inside one cell gives no pair unless it opens
// its ring: the edge before it ends in that cell, so that cell is marked by
// it, or by the first edge back along the ring that was kept.
__device__ __forceinline__ void edge_rows(const Edge &E, const PolyView &P, const RowGeo &G,
                                          int32_t *ra, int32_t *n, int32_t *ka, int32_t *kb,
                                          uint32_t *nb, uint32_t *nc)
{
    *ra = *n = 0;
    *ka = 0;
    *kb = -1;
    *nb = *nc = 0;
    const int4 bb = P.bbox[E.p];
    if ((int64_t)bb.z - G.ox < 0 || (int64_t)bb.x - 1 - G.ox >= G.extx) return;
    const int64_t y0 = (int64_t)min(E.y1, E.y2) - G.oy, y1 = (int64_t)max(E.y1, E.y2) - G.oy;
    const int32_t j0 = rel_cell(y0 - 1, G.exty, G.gh, G), j1 = rel_cell(y1, G.exty, G.gh, G);
    if (G.use_c && E.y1 != E.y2) {
        if (G.centre) {
            const int64_t s2 = 2 * G.s, a = min(E.y1, E.y2), b = max(E.y1, E.y2);
            *ka = (int32_t)(max(ceildiv64(2 * a - G.s, s2), G.gj0) - G.gj0);
            *kb = (int32_t)(min(ceildiv64(2 * b - G.s, s2) - 1, G.gj0 + G.gh - 1) - G.gj0);
        } else {
            *ka = j0 + 1;
            *kb = min(rel_cell(y1 - 1, G.exty, G.gh, G), G.gh - 1);
        }
        if (*kb >= *ka) *nc = (uint32_t)(*kb - *ka + 1);
    }
    if (!G.need_b) {
        *ra = *ka;
        *n = (int32_t)*nc;
        return;
    }
    const int32_t a = max(j0, 0), b = min(j1, G.gh - 1);
    if (b < a) return;
    *nb = (uint32_t)(b - a + 1);
    if (j0 == j1 && !G.centre && !E.first) {
        const int64_t x0 = (int64_t)min(E.x1, E.x2) - G.ox, x1 = (int64_t)max(E.x1, E.x2) - G.ox;
        if (rel_cell(x0 - 1, G.extx, G.gw, G) == rel_cell(x1, G.extx, G.gw, G)) return;
    }
    *ra = a;
    *n = b - a + 1;
}

// floor(a / b) and its remainder for b > 0, |a / b| < 2^32: a quotient in
// double (off by one at most) put right in integers; rb = 1.0 / b
__device__ __forceinline__ int64_t floordiv_est(int64_t a, int64_t b, double rb, int64_t *rem)
{
    int64_t q = (int64_t)floor((double)a * rb);
    int64_t r = a - q * b;
    while (r < 0) {
        q--;
        r += b;
    }
    while (r >= b) {
        q++;
        r -= b;
    }
    *rem = r;
    return q;
}

#define NO_CROSS 0xffffffffu

// The pair of edge E and row j (relative): its boundary cells [c0, c1] of the
// row cut to the box, as c0 and c1 + 1 (both 0, or both gw + 1, when they lie
// wholly before or after it), and its crossing cell k, cut to [0, gw]
// (NO_CROSS: none).  An edge's crossing of the row's lower line lies in its
// boundary interval: c0 < k <= c1 + 1.
__device__ __forceinline__ uint4 edge_row_item(const Edge &E, int32_t j, bool cross,
                                               const RowGeo &G)
{
    const int64_t x1 = E.x1, y1 = E.y1, x2 = E.x2, y2 = E.y2, s = G.s;
    const int64_t gi1 = G.gi0 + G.gw - 1, J = G.gj0 + j;
    int64_t c0, c1, k = -1;
    if (y1 == y2) {
        c0 = ceildiv64(min(x1, x2), s) - 1;
        c1 = floordiv64(max(x1, x2), s);
    } else {
        const int64_t ya = max(min(y1, y2), J * s), yb = min(max(y1, y2), (J + 1) * s);
        int64_t den = y2 - y1;
        // x(y) = (x1 den + (y - y1)(x2 - x1)) / den ; |numerator| < 2^63
        int64_t na = x1 * den + (ya - y1) * (x2 - x1);
        int64_t nz = x1 * den + (yb - y1) * (x2 - x1);
        if (den < 0) {
            den = -den;
            na = -na;
            nz = -nz;
        }
        const int64_t ds = den * s;
        const double rds = 1.0 / (double)ds;
        int64_t rema, remz;
        const int64_t qa = floordiv_est(na, ds, rds, &rema), qz = floordiv_est(nz, ds, rds, &remz);
        c0 = na <= nz ? qa - (rema == 0) : qz - (remz == 0);
        c1 = na <= nz ? qz : qa;
        // a crossed row line y = J s lies inside the edge: ya is that line
        if (cross && !G.centre) k = qa + (rema != 0);
        if (cross && G.centre) {
            // centre line y = (J + 1/2) s; with 2 xc = num / den the centre of
            // cell i lies left of the crossing iff (2i + 1) s den < num
            const int64_t d0 = y2 - y1;
            int64_t num = 2 * x1 * d0 + ((2 * J + 1) * s - 2 * y1) * (x2 - x1);
            if (d0 < 0) num = -num;
            k = ceildiv64(num - ds, 2 * ds);
        }
    }
    uint4 it;
    it.x = (uint32_t)E.p;
    if (c1 < G.gi0) {
        it.y = it.z = 0;
    } else if (c0 > gi1) {
        it.y = it.z = (uint32_t)G.gw + 1;
    } else {
        it.y = (uint32_t)(max(c0, G.gi0) - G.gi0);
        it.z = (uint32_t)(min(c1, gi1) + 1 - G.gi0);
    }
    it.w = cross ? (uint32_t)(min(max(k, G.gi0), gi1 + 1) - G.gi0) : NO_CROSS;
    return it;
}

// ---------------------------------------------------------------- buckets

#define EB 256       // lanes per workgroup, at most one edge each
#define EROWS 1024   // rows a workgroup's edges may span to share LDS counters

// inclusive scan over a workgroup of BLOCK lanes; *tot receives the whole.
// wsum: BLOCK / 64 words of LDS.
template <int BLOCK, typename OP = OpAdd, typename T>
__device__ __forceinline__ T wg_scan_incl(T v, T *wsum, T *tot)
{
    v = wave_scan<OP>(v);
    if constexpr (BLOCK == 64) {
        *tot = __shfl(v, 63, 64);
        return v;
    } else {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        if (lane == 63) wsum[w] = v;
        __syncthreads();
        T before = 0, all = 0;
#pragma unroll
        for (int k = 0; k < BLOCK / 64; k++) {
            const T c = wsum[k];
            if (k < w) before = OP::f(before, c);
            all = OP::f(all, c);
        }
        __syncthreads();
        *tot = all;
        return OP::f(before, v);
    }
}

// hint[k] = polygon of vertex 64 k (a wavefront per polygon); rowdiff, stat and
// the rows' figures of large sets zeroed, the set table (if any) emptied
__global__ void k_rows_init(const int32_t *ring_off, const int64_t *vert_off, int32_t np,
                            int32_t *hint, int32_t *rowdiff, int64_t nrow, unsigned long long *stat,
                            int nstat, uint32_t *row_large, uint64_t *tab, int64_t ntab)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t k = t; k < ntab; k += (int64_t)gridDim.x * blockDim.x) tab[k] = ~0ull;
    if (t < nrow) rowdiff[t] = 0;
    if (t < nrow - 1) row_large[t] = row_large[t + nrow - 1] = 0;
    if (t < nstat) stat[t] = 0;
    const int64_t p = t >> 6;
    if (p >= np) return;
    const int64_t v0 = vert_off[ring_off[p]], v1 = vert_off[ring_off[p + 1]];
    for (int64_t k = ((v0 + 63) >> 6) + (t & 63); (k << 6) < v1; k += 64) hint[k] = (int32_t)p;
}

// COUNT: rowdiff[r] += pairs that begin at row r less pairs that end before
// it (the row's pair count is the prefix sum), and the boundary strips and
// crossings go to one of ROW_STATS pairs of counters, each in a cache line of
// its own (additions to one line take about 10 ns each, one after another).
// EMIT: every pair to its row's bucket, rowdiff (zero on entry) counting the
// pairs placed so far.  A workgroup whose edges lie within EROWS rows, as
// neighbouring edges of a polygon do, counts in LDS and touches each row's
// global word once.  epw edges a workgroup (its lanes share their pairs).
// Workgroups whose edges have more than EPAIRS_MAX pairs, as edges across
// thousands of rows make, leave them to others when they emit: COUNT lists them
// (big: their numbers; bigfig: how many, the most pairs of one), and the first
// nbig * parts workgroups share their pairs, EPAIRS at a time.  (The four edges of
// a box over 57,143 rows, by one workgroup: 587 us.)
#define ROW_STATS 64
#define ROW_STAT_STEP 16  // words between counter pairs: a cache line of their own
#define EPAIRS_MAX 4096
#define EPAIRS 1024

template <bool EMIT>
__global__ __launch_bounds__(EB) void k_edge_rows(PolyView P, RowGeo G, int epw, int32_t *rowdiff,
                                                  const int64_t *rowoff, uint4 *items,
                                                  unsigned long long *stat, uint32_t *big,
                                                  unsigned long long *bigfig, int nbig, int parts)
{
    __shared__ int32_t hist[EROWS + 1];
    __shared__ uint32_t base[EMIT ? EROWS : 1];
    __shared__ uint32_t off[EMIT ? EB : 1];
    __shared__ Edge se[EMIT ? EB : 1];
    __shared__ int32_t sra[EMIT ? EB : 1], ska[EMIT ? EB : 1], skb[EMIT ? EB : 1];
    __shared__ uint32_t wsum[EB / 64];
    __shared__ int32_t lo_s, hi_s;
    __shared__ uint32_t sb[3];  // of 256 edges, each over at most 2^21 rows
    const int tid = threadIdx.x;
    const uint32_t shared = EMIT ? (uint32_t)(nbig * parts) : 0u;
    const bool sharing = EMIT && blockIdx.x < shared;
    const uint32_t part = sharing ? blockIdx.x % (uint32_t)parts : 0u;
    const int64_t v =
        (int64_t)(sharing ? big[blockIdx.x / (uint32_t)parts] : blockIdx.x - shared) * epw + tid;
    if (tid == 0) {
        lo_s = INT32_MAX;
        hi_s = -1;
        sb[0] = sb[1] = sb[2] = 0;
    }
    for (int k = tid; k <= EROWS; k += EB) hist[k] = 0;
    __syncthreads();
    int32_t ra = 0, n = 0, ka = 0, kb = -1;
    uint32_t nb = 0, nc = 0;
    Edge E{};
    if (tid < epw && v < P.nv) {
        E = edge_of(P, v);
        edge_rows(E, P, G, &ra, &n, &ka, &kb, &nb, &nc);
    }
    int32_t lo = n ? ra : INT32_MAX, hi = n ? ra + n - 1 : -1;
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o, 64));
        hi = max(hi, __shfl_xor(hi, o, 64));
    }
    if (!EMIT) {
        const uint32_t tb = wave_scan<OpAdd>(nb), tc = wave_scan<OpAdd>(nc),
                       tn = wave_scan<OpAdd>((uint32_t)n);
        if ((tid & 63) == 63 && (tb | tc)) {
            atomicAdd(&sb[0], tb);
            atomicAdd(&sb[1], tc);
            atomicAdd(&sb[2], tn);
        }
    }
    if ((tid & 63) == 0) {
        atomicMin(&lo_s, lo);
        atomicMax(&hi_s, hi);
    }
    __syncthreads();
    const int32_t r0 = lo_s, span = hi_s - lo_s + 1;
    if (!EMIT && tid == 0 && (sb[0] | sb[1])) {
        unsigned long long *st = stat + ROW_STAT_STEP * (blockIdx.x & (ROW_STATS - 1));
        atomicAdd(&st[0], (unsigned long long)sb[0]);
        atomicAdd(&st[1], (unsigned long long)sb[1]);
        if (sb[2] > EPAIRS_MAX) {
            big[atomicAdd(&bigfig[0], 1ull)] = blockIdx.x;
            atomicMax(&bigfig[1], (unsigned long long)sb[2]);
        }
    }
    if (hi_s < 0) return;  // no pair in the whole workgroup
    const bool local = span <= EROWS;
    if (!EMIT) {
        if (n && local) {
            atomicAdd(&hist[ra - r0], 1);
            atomicAdd(&hist[ra + n - r0], -1);
        } else if (n) {
            atomicAdd(&rowdiff[ra], 1);
            atomicAdd(&rowdiff[ra + n], -1);
        }
        __syncthreads();
        if (local)
            for (int k = tid; k <= span; k += EB)
                if (hist[k]) atomicAdd(&rowdiff[r0 + k], hist[k]);
        return;
    }
    uint32_t total;
    const uint32_t incl = wg_scan_incl<EB>((uint32_t)n, wsum, &total);
    off[tid] = incl;
    se[tid] = E;
    sra[tid] = ra;
    ska[tid] = ka;
    skb[tid] = kb;
    __syncthreads();
    // pair t belongs to the first edge whose inclusive count exceeds t
    auto edge_at = [&](uint32_t t) {
        int a = 0, len = EB;
        while (len > 0) {
            const int half = len >> 1;
            if (off[a + half] <= t) {
                a += half + 1;
                len -= half + 1;
            } else {
                len = half;
            }
        }
        return a;
    };
    auto row_at = [&](uint32_t t, int e) {
        return sra[e] + (int32_t)(t - (e ? off[e - 1] : 0u));
    };
    if (!sharing && total > EPAIRS_MAX) return;
    const uint32_t step = sharing ? (uint32_t)parts * EPAIRS : EPAIRS_MAX;
    for (uint32_t t0 = part * EPAIRS; t0 < total; t0 += step) {
        const uint32_t t1 = sharing ? min(t0 + EPAIRS, total) : total;
        if (local) {
            for (uint32_t t = t0 + tid; t < t1; t += EB) {
                const int e = edge_at(t);
                atomicAdd(&hist[row_at(t, e) - r0], 1);
            }
            __syncthreads();
            for (int k = tid; k < span; k += EB) {
                const int32_t c = hist[k];
                base[k] = c ? (uint32_t)atomicAdd(&rowdiff[r0 + k], c) : 0u;
                hist[k] = 0;
            }
            __syncthreads();
        }
        for (uint32_t t = t0 + tid; t < t1; t += EB) {
            const int e = edge_at(t);
            const int32_t j = row_at(t, e);
            const uint32_t at = local ? base[j - r0] + (uint32_t)atomicAdd(&hist[j - r0], 1)
                                      : (uint32_t)atomicAdd(&rowdiff[j], 1);
            items[rowoff[j] + at] = edge_row_item(se[e], j, j >= ska[e] && j <= skb[e], G);
        }
        if (local && sharing) {
            __syncthreads();
            for (int k = tid; k < span; k += EB) hist[k] = 0;
            __syncthreads();
        }
    }
}

// Rows by their number of pairs: class c takes up to ROW_MAX[c]
#define ROW_CLASSES 4
__device__ __forceinline__ int row_class(uint32_t n)
{
    return n <= 64 ? 0 : (n <= 256 ? 1 : (n <= 1024 ? 2 : (n <= 4096 ? 3 : 4)));
}

// a place in its class for each lane's row (class c, none if negative): one
// addition to the workgroup's counters n a class and wavefront
__device__ __forceinline__ uint32_t class_slot(int c, uint32_t *n)
{
    const int lane = threadIdx.x & 63;
    uint32_t at = 0;
    for (int q = 0; q < ROW_CLASSES; q++) {
        const uint64_t b = __ballot(c == q);
        if (c != q) continue;
        const uint32_t rank = (uint32_t)__popcll(b & ((1ull << lane) - 1));
        uint32_t first = 0;
        if (rank == 0) first = atomicAdd(&n[q], (uint32_t)__popcll(b));
        at = (uint32_t)__shfl((int)first, __ffsll((long long)b) - 1, 64) + rank;
    }
    return at;
}

// One workgroup, or many (PARTS): from rowdiff (see k_edge_rows) the rows' pair counts and
// their exclusive scan rowoff[0..gh] (pairs < 2^31); rowdiff goes back to
// zero.  out[0]: pairs, out[1]: the most in a row, out[6], out[7]: boundary
// strips and crossings (the sums over stat).  The rows come and go by threads
// (a lane of eight consecutive rows would touch a line an access) and are
// summed eight to a lane, the next chunk loaded meanwhile.
#define RSCAN 1024
#define RSCAN_PER 8
#define RS_PAD(i) ((i) + ((i) >> 3))  // a lane's eight in banks of their own
// Up to RSCAN_LISTS rows it makes the rows' lists as well (see k_row_lists),
// and copies the host's values: two launches less.
#define RSCAN_LISTS (RSCAN * RSCAN_PER)
// From RSCAN_PARTS times as many rows on, a workgroup for each RSCAN_LISTS of them
// (one workgroup takes 3 us for so many: 1,048,577 rows 393 us, now 10 and
// less than 5 for the parts' sums).
#define RSCAN_PARTS 4
// a row's figures, [gh] each: multi-polygon segments and their members, then
// those of more than three polygons and theirs
#define ROW_FIGS 4
struct RowLists {
    int32_t *list;
    int64_t *seg_beg, *seg_end;
    uint32_t *row_stat;
};

// Of each RSCAN_LISTS rows (a workgroup): the sum of their differences, and of
// their pairs had no row before them any.
__global__ __launch_bounds__(RSCAN) void k_row_parts(const int32_t *rowdiff, int64_t gh, uint2 *parts)
{
    __shared__ uint32_t wsum[RSCAN / 64];
    const int64_t c0 = (int64_t)blockIdx.x * RSCAN_LISTS;
    const int64_t c1 = min(c0 + RSCAN_LISTS, gh);
    uint32_t d = 0, sum = 0;
    for (int64_t r = c0 + threadIdx.x; r < c1; r += RSCAN) {
        const uint32_t v = (uint32_t)rowdiff[r];
        d += v;
        sum += v * (uint32_t)(c1 - r);
    }
    uint32_t td, ts;
    wg_scan_incl<RSCAN>(d, wsum, &td);
    wg_scan_incl<RSCAN>(sum, wsum, &ts);
    if (threadIdx.x == 0) parts[blockIdx.x] = make_uint2(td, ts);
}

// PARTS (of k_row_parts; no lists): workgroup c scans the c-th RSCAN_LISTS rows,
// after the sums of the parts before it.
template <bool PARTS>
__global__ __launch_bounds__(RSCAN) void k_row_scan(int32_t *rowdiff, int64_t gh, int64_t *rowoff,
                                                    const unsigned long long *stat,
                                                    unsigned long long *out, const uint2 *parts,
                                                    RowLists Q, ReadSet R)
{
    __shared__ uint32_t ncls[ROW_CLASSES];
    __shared__ uint32_t wd[RSCAN / 64];
    __shared__ uint32_t chunk[RS_PAD(RSCAN * RSCAN_PER)];
    __shared__ uint32_t smax;
    __shared__ unsigned long long sst[2];
    if (threadIdx.x == 0) smax = 0;
    if (threadIdx.x < 2) sst[threadIdx.x] = 0;
    if (threadIdx.x < ROW_CLASSES) ncls[threadIdx.x] = 0;
    uint32_t next[RSCAN_PER];
    auto load = [&](int64_t c0) {
#pragma unroll
        for (int k = 0; k < RSCAN_PER; k++) {
            const int64_t r = c0 + k * RSCAN + threadIdx.x;
            next[k] = r <= gh ? (uint32_t)rowdiff[r] : 0u;
        }
    };
    const int64_t beg = PARTS ? (int64_t)blockIdx.x * RSCAN_LISTS : 0;
    const int64_t end = PARTS ? min(beg + RSCAN_LISTS - 1, gh) : gh;
    load(beg);
    __syncthreads();
    if (threadIdx.x < 2 * ROW_STATS)
        atomicAdd(&sst[threadIdx.x & 1],
                  stat[ROW_STAT_STEP * (threadIdx.x >> 1) + (threadIdx.x & 1)]);
    uint32_t cd = 0, cs = 0, m = 0;
    if constexpr (PARTS) {  // at most RSCAN of them: MAX_GRID_SIDE rows
        static_assert(MAX_GRID_SIDE / RSCAN_LISTS < RSCAN, "a part a thread");
        const uint2 p = threadIdx.x < blockIdx.x ? parts[threadIdx.x] : make_uint2(0, 0);
        const uint32_t before = wg_scan_incl<RSCAN>(p.x, wd, &cd) - p.x;
        wg_scan_incl<RSCAN>(threadIdx.x < blockIdx.x ? p.y + before * RSCAN_LISTS : 0u, wd, &cs);
    }
    for (int64_t c0 = beg; c0 <= end; c0 += RSCAN * RSCAN_PER) {
        const int64_t b = c0 + (int64_t)threadIdx.x * RSCAN_PER;
#pragma unroll
        for (int k = 0; k < RSCAN_PER; k++) chunk[RS_PAD(k * RSCAN + threadIdx.x)] = next[k];
        __syncthreads();
        uint32_t d[RSCAN_PER], run = 0;
#pragma unroll
        for (int k = 0; k < RSCAN_PER; k++) {
            run += chunk[RS_PAD(threadIdx.x * RSCAN_PER + k)];  // modulo 2^32
            d[k] = run;
        }
        if (!PARTS) load(c0 + RSCAN * RSCAN_PER);
        uint32_t totd;
        const uint32_t before = cd + wg_scan_incl<RSCAN>(run, wd, &totd) - run;
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < RSCAN_PER; k++) {
            d[k] = b + k < gh ? d[k] + before : 0u;
            sum += d[k];
            m = max(m, d[k]);
        }
        uint32_t tots;
        uint32_t o = cs + wg_scan_incl<RSCAN>(sum, wd, &tots) - sum;
#pragma unroll
        for (int k = 0; k < RSCAN_PER; k++) {
            chunk[RS_PAD(threadIdx.x * RSCAN_PER + k)] = o;
            if (!PARTS && Q.list) {
                const int64_t r = b + k;
                int c = -1;
                if (r < gh && d[k] == 0) {
                    Q.seg_beg[r] = Q.seg_end[r] = 2 * (int64_t)o;
                    Q.row_stat[r] = Q.row_stat[gh + r] = 0;
                } else if (r < gh) {
                    c = row_class(d[k]);
                }
                const uint32_t at = class_slot(c, ncls);
                if (c >= 0 && c < ROW_CLASSES) Q.list[(int64_t)c * gh + at] = (int32_t)r;
            }
            o += d[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < RSCAN_PER; k++) {
            const int64_t r = c0 + k * RSCAN + threadIdx.x;
            if (r <= gh) {
                rowoff[r] = chunk[RS_PAD(k * RSCAN + threadIdx.x)];
                rowdiff[r] = 0;
            }
        }
        __syncthreads();
        cd += totd;
        cs += tots;
    }
    for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(&smax, m);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (end == gh) out[0] = cs;
        if (PARTS) atomicMax(&out[1], (unsigned long long)smax);
        else out[1] = smax;
        out[6] = sst[0];
        out[7] = sst[1];
    }
    if (!PARTS && Q.list && threadIdx.x < ROW_CLASSES) out[2 + threadIdx.x] = ncls[threadIdx.x];
    read_back(R);
}

// The rows by class: list[c gh ..] holds class c's, cnt[c] of them (zero on
// entry), one reservation a class and workgroup.  Empty rows get their (empty)
// segment range and figures at once.
__global__ __launch_bounds__(256) void k_row_lists(const int64_t *rowoff, int64_t gh, int32_t *list,
                                                   int64_t *seg_beg, int64_t *seg_end,
                                                   uint32_t *row_stat, unsigned long long *cnt)
{
    __shared__ uint32_t n[ROW_CLASSES], base[ROW_CLASSES];
    const int tid = threadIdx.x;
    const int64_t r = (int64_t)blockIdx.x * 256 + tid;
    if (tid < ROW_CLASSES) n[tid] = 0;
    __syncthreads();
    int c = -1;
    if (r < gh) {
        const int64_t o = rowoff[r];
        const uint32_t d = (uint32_t)(rowoff[r + 1] - o);
        if (d == 0) {
            seg_beg[r] = seg_end[r] = 2 * o;
            row_stat[r] = row_stat[gh + r] = 0;
        } else {
            c = row_class(d);
        }
    }
    const uint32_t at = class_slot(c, n);
    __syncthreads();
    if (tid < ROW_CLASSES && n[tid]) base[tid] = (uint32_t)atomicAdd(&cnt[tid], (unsigned long long)n[tid]);
    __syncthreads();
    if (c >= 0 && c < ROW_CLASSES) list[(int64_t)c * gh + base[c] + at] = (int32_t)r;
}

// ---------------------------------------------------------------- sweep

// one step between lanes M apart
template <int M, int R, typename K>
__device__ __forceinline__ void sort_step(K (&v)[R], bool up)
{
    const bool small = ((threadIdx.x & M) == 0) == up;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const K o = lane_xor<M>(v[r]);
        v[r] = (v[r] < o) == small ? v[r] : o;
    }
}

// Ascending bitonic sort of BLOCK R words by one workgroup, R consecutive ones
// a lane: steps inside a lane take registers only, steps inside a wavefront
// one exchange a word in the vector ALU, and only steps between wavefronts go
// through LDS (buf, BLOCK R words) and a barrier.  The chain of steps is what
// bounds it: exchanges through LDS made a sweep of rows of 257 to 1,024 pairs
// (260 polygons at 10 m) 31 us, these 24.
template <int BLOCK, int R, typename K>
__device__ __forceinline__ void wg_sort(K (&v)[R], K *buf)
{
    const int tid = threadIdx.x;
    for (int k = 2; k <= BLOCK * R; k <<= 1) {
        // the lane keeps the smaller words when its place in the pair and the
        // direction of its sequence agree (R divides j and k)
        const bool up = (tid * R & k) == 0;
        for (int m = (k >> 1) / R; m >= 64; m >>= 1) {
            const bool small = ((tid & m) == 0) == up;
#pragma unroll
            for (int r = 0; r < R; r++) buf[r * BLOCK + tid] = v[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; r++) {
                const K o = buf[r * BLOCK + (tid ^ m)];
                v[r] = (v[r] < o) == small ? v[r] : o;
            }
            __syncthreads();
        }
        if (k >= 64 * R) sort_step<32, R>(v, up);
        if (k >= 32 * R) sort_step<16, R>(v, up);
        if (k >= 16 * R) sort_step<8, R>(v, up);
        if (k >= 8 * R) sort_step<4, R>(v, up);
        if (k >= 4 * R) sort_step<2, R>(v, up);
        if (k >= 2 * R) sort_step<1, R>(v, up);
#pragma unroll
        for (int j = R >> 1; j > 0; j >>= 1) {
            if (j >= k) continue;
#pragma unroll
            for (int r = 0; r < R; r++) {
                if (r & j) continue;
                const bool up = ((tid * R + r) & k) == 0;
                const K a = v[r], b = v[r | j];
                const bool swap = (a > b) == up;
                v[r] = swap ? b : a;
                v[r | j] = swap ? a : b;
            }
        }
    }
}

__host__ __device__ inline int pow2_at_least(int n)
{
    int p = 2;
    while (p < n) p *= 2;
    return p;
}

struct SweepArgs {
    const uint4 *items;
    const int64_t *rowoff;
    int32_t gh;
    const int32_t *list;     // the launch's rows
    int32_t gw;
    int xbits, tbits;        // bits of a column (0 .. gw + 1); of a toggle index
    int use_b;
    int fb;                  // bits of an id + 1 in a set key
    int nmax, tc;            // pairs and toggles the workgroup's LDS holds
    int64_t *seg_beg, *seg_end;
    int32_t *seg_x0, *seg_x1;
    uint32_t *seg_code;
    uint64_t *seg_key;       // set keys of multi-polygon segments (list mode), or NULL
    uint32_t *row_stat;      // the rows' figures (ROW_FIGS)
    uint64_t *memloc;        // members of the sets of more than three polygons
    int32_t *mem_ids;
    unsigned long long *memcnt;
    int64_t memcap;
    SetTab tab;              // tab.tab NULL: list mode
    int *err;
};

#define ERR_DEPTH 8
#define ERR_ROW 16   // a row does not fit the workgroup

// LDS of a sweep workgroup: the sorted pairs, later the pieces (start,
// smallest, largest and sum of the polygon ids, depth); the toggles; each
// toggle's polygon and piece
static __host__ __device__ inline int sweep_lds_a(int nmax, int tc)
{
    const int a = 8 * nmax, b = 18 * tc;
    return ((a > b ? a : b) + 15) & ~15;
}

template <typename P, typename K2>
struct SweepLds {
    uint64_t *S;
    uint32_t *E, *pmin, *pmax, *psum;
    uint16_t *D;
    K2 *tog;
    uint32_t *tpoly;
    uint16_t *rank;
    uint32_t *wsum;
    P *wmax;
    int *err;  // set when a polygon's crossings of the row are odd in number
    int *large;  // set when a piece holds more than three polygons
};

// The row's n pairs to its toggles: x and polygon of every change of a
// polygon's coverage, in (polygon, x) order, on and off in turn.
//
// The pairs are sorted by polygon, then first cell, then last cell (larger
// first).  Runs of pairs that touch or overlap (running largest end, which a
// prefix maximum over (polygon, end) gives for every polygon at once) are
// covered; between two runs of a polygon the cells are covered when the
// crossings so far are odd in number, since a pair's crossing never lies past
// its end.  Pairs without a cell (cut away by the box, or crossings of centre
// lines) make runs of their own, where only the parity changes.
template <int BLOCK, int R, typename P, typename K2>
__device__ __forceinline__ int sweep_toggles(const SweepArgs &A, const SweepLds<P, K2> &L,
                                             int64_t i0, int n)
{
    const int tid = threadIdx.x, xb = A.xbits;
    const uint32_t xm = (1u << xb) - 1u;
    uint64_t v[R];
    uint32_t mine = 0, ne;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = r * BLOCK + tid;
        v[r] = ~(uint64_t)0;
        if (i < n) {
            const uint4 it = A.items[i0 + i];
            const bool c = it.w != NO_CROSS;
            const uint32_t c0 = A.use_b ? it.y : it.w, c1 = A.use_b ? it.z : it.w;
            if (c || (A.use_b && c0 < c1)) {
                v[r] = ((uint64_t)it.x << (2 * xb + 1)) | ((uint64_t)c0 << (xb + 1)) |
                       ((uint64_t)(xm - c1) << 1) | (c ? 1u : 0u);
                mine++;
            }
        }
    }
    wg_scan_incl<BLOCK>(mine, L.wsum, &ne);
    wg_sort<BLOCK, R, uint64_t>(v, L.S);
#pragma unroll
    for (int r = 0; r < R; r++) L.S[tid * R + r] = v[r];
    __syncthreads();
    // (polygon, end) maximum and crossings before each pair
    const int b = tid * R;
    P mx = 0;
    uint32_t cr = 0;
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (b + r < (int)ne) {
            const P e = ((P)(v[r] >> (2 * xb + 1)) << xb) | (P)(xm - ((uint32_t)(v[r] >> 1) & xm));
            mx = mx > e ? mx : e;
            cr += (uint32_t)v[r] & 1u;
        }
    }
    P tm;
    uint32_t tc;
    P im = wg_scan_incl<BLOCK, OpMax>(mx, L.wmax, &tm);
    const uint32_t ic = wg_scan_incl<BLOCK>(cr, L.wsum, &tc);
    // exclusive maximum: that of the lanes before
    {
        P up;
        if constexpr (sizeof(P) == 4) up = (P)__shfl_up((int)im, 1, 64);
        else up = (P)__shfl_up((unsigned long long)im, 1, 64);
        if constexpr (BLOCK > 64) {
            if ((tid & 63) == 63) L.wmax[tid >> 6] = im;
            __syncthreads();
            if ((tid & 63) == 0) up = tid ? L.wmax[(tid >> 6) - 1] : (P)0;
            __syncthreads();
        } else if (tid == 0) {
            up = 0;
        }
        im = up;
    }
    uint32_t c = ic - cr;
    uint32_t fl = 0, cnt = 0, clx[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = b + r;
        clx[r] = 0;
        if (i >= (int)ne) continue;
        const uint32_t poly = (uint32_t)(v[r] >> (2 * xb + 1));
        const uint32_t c0 = (uint32_t)(v[r] >> (xb + 1)) & xm;
        const uint32_t c1 = xm - ((uint32_t)(v[r] >> 1) & xm);
        const bool newp = i == 0 || (uint32_t)(im >> xb) != poly;
        const bool start = newp || c0 > ((uint32_t)im & xm);
        const bool sb = !newp && (c & 1u);  // covered just before a run here
        const P e = ((P)poly << xb) | (P)c1;
        im = im > e ? im : e;
        c += (uint32_t)v[r] & 1u;
        const uint32_t M = (uint32_t)im & xm;
        const uint64_t nx = i + 1 < (int)ne ? L.S[i + 1] : ~(uint64_t)0;
        const bool lastp = i + 1 >= (int)ne || (uint32_t)(nx >> (2 * xb + 1)) != poly;
        const bool last = lastp || ((uint32_t)(nx >> (xb + 1)) & xm) > M;
        const bool se = (c & 1u) != 0;  // covered just past a run that ends here
        if (lastp && se) *L.err = 1;
        const bool empty = !A.use_b || M == 0 || M > (uint32_t)A.gw;
        if (start && c0 < c1 && !sb) {
            fl |= 1u << (2 * r);
            cnt++;
        }
        if (last && !empty && !se) {
            fl |= 2u << (2 * r);
            clx[r] = M;
            cnt++;
        }
        if (last && empty) {
            // a run without a cell: the parity changes with its pairs (all of
            // them crossings at one place)
            int a = i;
            while (a > 0 && (L.S[a - 1] >> (xb + 1)) == (v[r] >> (xb + 1))) a--;
            if ((i - a + 1) & 1) {
                fl |= 2u << (2 * r);
                clx[r] = min(M, (uint32_t)A.gw);
                cnt++;
            }
        }
    }
    uint32_t nt;
    int at = (int)(wg_scan_incl<BLOCK>(cnt, L.wsum, &nt) - cnt);
    if ((int)nt > A.tc) return (int)nt;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const uint32_t poly = (uint32_t)(v[r] >> (2 * xb + 1));
        if (fl & (1u << (2 * r))) {
            L.tog[at] = ((K2)((v[r] >> (xb + 1)) & xm) << A.tbits) | (K2)at;
            L.tpoly[at++] = poly;
        }
        if (fl & (2u << (2 * r))) {
            L.tog[at] = ((K2)clx[r] << A.tbits) | (K2)at;
            L.tpoly[at++] = poly;
        }
    }
    return (int)nt;
}

// The toggles sorted by x: the distinct positions E[0..nd) cut the row, piece
// k = [E[k], E[k+1]) lies under D[k] intervals; each toggle learns its piece.
// Returns nd.
template <int BLOCK, int R, typename P, typename K2>
__device__ __forceinline__ int sweep_pieces(const SweepArgs &A, const SweepLds<P, K2> &L, int nt)
{
    const int tid = threadIdx.x, tb = A.tbits;
    K2 v[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = r * BLOCK + tid;
        v[r] = i < nt ? L.tog[i] : (K2)~(K2)0;
    }
    __syncthreads();
    wg_sort<BLOCK, R, K2>(v, L.tog);
#pragma unroll
    for (int r = 0; r < R; r++) L.tog[tid * R + r] = v[r];
    __syncthreads();
    const int b = tid * R;
    const K2 tm = ((K2)1 << tb) - 1;
    // positions above bit 16, open intervals below it (never negative: at one
    // position at least as many intervals were open as close)
    uint32_t sum = 0, w[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = b + r;
        w[r] = 0;
        if (i < nt) {
            const K2 pv = r ? v[r - 1] : (i ? L.tog[i - 1] : (K2)0);
            const bool first = i == 0 || (pv >> tb) != (v[r] >> tb);
            w[r] = (first ? 0x10000u : 0u) + ((v[r] & 1) ? 0xffffffffu : 1u);
        }
        sum += w[r];
    }
    uint32_t tot;
    uint32_t S = wg_scan_incl<BLOCK>(sum, L.wsum, &tot) - sum;
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = b + r;
        if (i >= nt) continue;
        const uint32_t p0 = S >> 16;
        S += w[r];
        const uint32_t k = (S >> 16) - 1;
        const K2 nx = r + 1 < R ? v[r + 1 < R ? r + 1 : r] : (i + 1 < nt ? L.tog[i + 1] : (K2)~(K2)0);
        L.rank[(int)(v[r] & tm)] = (uint16_t)k;
        if (p0 != (S >> 16)) {
            L.E[k] = (uint32_t)(v[r] >> tb);
            L.pmin[k] = 0xffffffffu;
            L.pmax[k] = 0;
            L.psum[k] = 0;
        }
        if (i + 1 >= nt || (nx >> tb) != (v[r] >> tb)) {
            L.D[k] = (uint16_t)(S & 0xffffu);
            if ((S & 0xffffu) > 3) *L.large = 1;
        }
    }
    __syncthreads();
    return (int)(tot >> 16);
}

// One workgroup per row.  RN, RT: the most pairs and toggles a lane holds.
template <int BLOCK, int RN, int RT, typename P, typename K2>
__global__ __launch_bounds__(BLOCK) void k_row_sweep(const SweepArgs A)
{
    extern __shared__ __align__(16) unsigned char sweep_lds[];
    __shared__ uint32_t wsum[BLOCK / 64];
    __shared__ P wmax[BLOCK / 64];
    __shared__ uint32_t s_stat[2];
    __shared__ int s_err, s_large;
    __shared__ unsigned long long s_mem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int row = A.list[blockIdx.x];
    const int64_t i0 = A.rowoff[row];
    const int n = (int)(A.rowoff[row + 1] - i0);
    const int64_t sbase = 2 * i0;
    SweepLds<P, K2> L;
    L.S = (uint64_t *)sweep_lds;
    L.E = (uint32_t *)sweep_lds;
    L.pmin = L.E + A.tc;
    L.pmax = L.pmin + A.tc;
    L.psum = L.pmax + A.tc;
    L.D = (uint16_t *)(L.psum + A.tc);
    L.tog = (K2 *)(sweep_lds + sweep_lds_a(A.nmax, A.tc));
    L.tpoly = (uint32_t *)(L.tog + BLOCK * RT);
    L.rank = (uint16_t *)(L.tpoly + A.tc);
    L.wsum = wsum;
    L.wmax = wmax;
    L.err = &s_err;
    L.large = &s_large;
    if (tid == 0) {
        s_stat[0] = s_stat[1] = 0;
        s_err = s_large = 0;
    }
    __syncthreads();
    int nt;
    if (RN >= 4 && n > 2 * BLOCK) nt = sweep_toggles<BLOCK, RN >= 4 ? 4 : 1, P, K2>(A, L, i0, n);
    else if (RN >= 2 && n > BLOCK) nt = sweep_toggles<BLOCK, RN >= 2 ? 2 : 1, P, K2>(A, L, i0, n);
    else nt = sweep_toggles<BLOCK, 1, P, K2>(A, L, i0, n);
    __syncthreads();  // the pairs are done with: their space takes the pieces
    if (nt > A.tc || s_err) {
        if (tid == 0) atomicOr(A.err, nt > A.tc ? ERR_ROW : 2);
        return;
    }
    int nd;
    if (RT >= 4 && nt > 2 * BLOCK) nd = sweep_pieces<BLOCK, RT >= 4 ? 4 : 1, P, K2>(A, L, nt);
    else if (RT >= 2 && nt > BLOCK) nd = sweep_pieces<BLOCK, RT >= 2 ? 2 : 1, P, K2>(A, L, nt);
    else nd = sweep_pieces<BLOCK, 1, P, K2>(A, L, nt);
    // places for the members of the row's large sets (more than three polygons):
    // each piece's first one in psum, and how many it has in pmin
    const bool large = s_large != 0;
    bool fits = false;  // all of them, in mem_ids
    uint32_t places = 0;
    if (large) {
        for (int b = 0; b < nd; b += BLOCK) {
            const int k = b + tid, d = k < nd ? L.D[k] : 0;
            const uint32_t need = d > 3 && d <= MAX_DEPTH ? (uint32_t)d : 0u;
            uint32_t tot;
            const uint32_t at = places + wg_scan_incl<BLOCK>(need, wsum, &tot) - need;
            if (need) {
                L.psum[k] = at;
                L.pmin[k] = 0;
            }
            places += tot;
        }
        if (tid == 0) s_mem = atomicAdd(A.memcnt, (unsigned long long)places);
        __syncthreads();
        fits = (int64_t)s_mem + places <= A.memcap;
    }
    int32_t *const mem = large ? A.mem_ids + s_mem : nullptr;
    // members: each covered interval (toggles 2m, 2m + 1) adds its polygon to
    // the pieces it spans, a lane an interval, or a wavefront those of more than 64
    // pieces; up to three ids come back from their smallest, largest and sum
    const int ni = nt >> 1;
    // small classes: a wavefront looks through the row's intervals, at most four
    // steps of 64, for each large set (its members, written to memory, read again
    // and sorted took a row of 64 pairs 2.5 us more)
    constexpr bool SCAN = BLOCK <= 256;
    auto join = [&](int k, uint32_t p) {
        const int d = L.D[k];
        if (d == 1) {
            L.pmin[k] = p;
        } else if (d <= 3) {
            atomicMin(&L.pmin[k], p);
            atomicMax(&L.pmax[k], p);
            atomicAdd(&L.psum[k], p);
        } else if (!SCAN && fits && d <= MAX_DEPTH) {
            mem[L.psum[k] + atomicAdd(&L.pmin[k], 1u)] = (int32_t)p;
        }
    };
    for (int m0 = 0; m0 < ni; m0 += BLOCK) {
        const int m = m0 + tid;
        const int ka = m < ni ? L.rank[2 * m] : 0, kb = m < ni ? L.rank[2 * m + 1] : 0;
        const uint32_t p = m < ni ? L.tpoly[2 * m] : 0u;
        uint64_t wide = __ballot(kb - ka > 64);
        if (kb - ka <= 64)
            for (int k = ka; k < kb; k++) join(k, p);
        while (wide) {
            const int l = __ffsll((unsigned long long)wide) - 1;
            wide &= wide - 1;
            const int a = __shfl(ka, l), b = __shfl(kb, l);
            const uint32_t q = (uint32_t)__shfl((int)p, l);
            for (int k = a + lane; k < b; k += 64) join(k, q);
        }
    }
    __syncthreads();
    // the members of large sets into ascending order, half a wavefront a set (each
    // its place by the members below it).  (A wavefront that looked through all
    // of the row's intervals for each set: the two sweeps of 300,000 rectangles in
    // layers 23.3 ms, 17.9 this way.)
    if (SCAN && large && fits) {
        for (int b = 0; b < nd; b += BLOCK) {
            const int k = b + tid, d = k < nd ? L.D[k] : 0;
            uint64_t sets = __ballot(d > 3 && d <= MAX_DEPTH);
            while (sets) {
                const int l = __ffsll((unsigned long long)sets) - 1;
                sets &= sets - 1;
                const int kk = __shfl(k, l), dd = __shfl(d, l);
                int32_t *const set = mem + L.psum[kk];
                // intervals are in polygon order: the ids come out ascending
                for (int m0 = 0, q = 0; m0 < ni && q < dd; m0 += 64) {
                    const int m = m0 + lane;
                    const bool in = m < ni && (int)L.rank[2 * m] <= kk &&
                                    kk < (int)L.rank[2 * m + 1];
                    const uint64_t who = __ballot(in);
                    const int at = q + __popcll(who & ((1ull << lane) - 1));
                    if (in && at < dd) set[at] = (int32_t)L.tpoly[2 * m];
                    q += __popcll(who);
                }
            }
        }
    } else if (large && fits) {
        static_assert(MAX_DEPTH == 32, "half a wavefront");
        for (int k0 = (tid >> 6) * 2; k0 < nd; k0 += BLOCK / 32) {
            const int k = k0 + (lane >> 5), d = k < nd ? L.D[k] : 0, q = lane & 31;
            const bool in = d > 3 && q < d && d <= MAX_DEPTH;
            if (!__any(in)) continue;
            int32_t *const set = mem + (in ? L.psum[k] : 0u);
            const int32_t v = in ? set[q] : INT32_MAX;
            int below = 0;
            // (all 32 at once took 80 registers, and a wavefront a SIMD)
#pragma unroll 4
            for (int j = 0; j < 32; j++) below += __shfl(v, (lane & 32) | j) < v ? 1 : 0;
            if (in) set[below] = v;
        }
    }
    // segments: the pieces that hold a polygon
    uint32_t nseg = 0, nm = 0, nmem = 0, nlarge = 0;
    const bool hash = A.tab.tab != nullptr;
    for (int b = 0; b < nd; b += BLOCK) {
        const int k = b + tid;
        const int d = k < nd ? L.D[k] : 0;
        // segments, and above bit 16 those of more than three polygons (at most
        // 1024 a step)
        uint32_t tot;
        const uint32_t at_once = wg_scan_incl<BLOCK>((d ? 1u : 0u) | (d > 3 ? 1u << 16 : 0u), wsum,
                                                     &tot);
        const uint32_t o = nseg + (at_once & 0xffffu) - 1, g = nlarge + (at_once >> 16) - 1;
        nseg += tot & 0xffffu;
        nlarge += tot >> 16;
        if (!d) continue;
        const int64_t at = sbase + o;
        A.seg_x0[at] = (int32_t)L.E[k];
        A.seg_x1[at] = (int32_t)L.E[k + 1];
        if (d == 1) {
            A.seg_code[at] = L.pmin[k] + 1u;
            continue;
        }
        nm++;
        nmem += (uint32_t)d;
        uint64_t key;
        const uint64_t lo = (uint64_t)L.pmin[k] + 1, hi = (uint64_t)L.pmax[k] + 1;
        if (d == 2) {
            key = lo | (hi << A.fb);
        } else if (d == 3) {
            const uint64_t mid = (uint64_t)(L.psum[k] - L.pmin[k] - L.pmax[k]) + 1;
            key = lo | (mid << A.fb) | (hi << (2 * A.fb));
        } else {
            if (d > MAX_DEPTH) {
                atomicOr(A.err, ERR_DEPTH);
                continue;
            }
            A.memloc[at] = ((uint64_t)(s_mem + L.psum[k]) << 6) | (uint64_t)d;
            key = (1ull << (3 * A.fb)) + (uint64_t)at;
        }
        if (hash && d > 3) {
            // not shared, so no place in the table (which they filled, so that
            // the sweep was made again for keys to be sorted: 64 stars in layers
            // 192 us of sweeps, now 62)
            A.seg_code[at] = SEG_SLOT | SEG_LARGE | g;
            const uint64_t of = (s_mem + L.psum[k]) >> 2;  // a set has at least four members
            if (of < LARGE_FEW) A.tab.large[of] = key;
        } else if (hash) {
            A.seg_code[at] = SEG_SLOT | set_insert(A.tab, key, (uint32_t)d);
        } else {
            A.seg_key[at] = key;
            A.seg_code[at] = SEG_SLOT;
        }
    }
    if (nm) {
        atomicAdd(&s_stat[0], nm);
        atomicAdd(&s_stat[1], nmem);
    }
    __syncthreads();
    if (tid == 0) {
        A.seg_beg[row] = sbase;
        A.seg_end[row] = sbase + nseg;
        A.row_stat[row] = s_stat[0];
        A.row_stat[A.gh + row] = s_stat[1];
        if (large) {
            A.row_stat[2 * (int64_t)A.gh + row] = nlarge;
            A.row_stat[3 * (int64_t)A.gh + row] = places;
        }
    }
}

// out[0..2] += segments, multi-polygon segments and their members of all rows,
// *large += those of more than three polygons
// (the rows' own figures, added up once: an addition to a shared counter by
// every row took 10 ns a row)
// (as one workgroup it copies the host's values too)
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_row_totals(const int64_t *seg_beg, const int64_t *seg_end,
                                                      const uint32_t *row_stat, int64_t gh,
                                                      unsigned long long *out,
                                                      unsigned long long *large, ReadSet R)
{
    __shared__ unsigned long long sum[3];
    if (threadIdx.x < 3) sum[threadIdx.x] = 0;
    __syncthreads();
    // (b: multi-polygon segments, and above bit 32 those of more than three
    // polygons: below 2^32 each, as two segments a pair are)
    unsigned long long a = 0, b = 0, c = 0;
    // four rows' loads together: the chain of them is what one workgroup takes
    const int64_t step = (int64_t)gridDim.x * BLOCK;
    for (int64_t r0 = (int64_t)blockIdx.x * BLOCK + threadIdx.x; r0 < gh; r0 += 4 * step) {
        int64_t e[4], s[4];
        uint32_t m[4], f[4], l[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int64_t r = r0 + k * step;
            const bool in = r < gh;
            const int64_t q = in ? r : r0;
            e[k] = seg_end[q];
            s[k] = in ? seg_beg[q] : e[k];
            m[k] = in ? row_stat[q] : 0u;
            f[k] = in ? row_stat[gh + q] : 0u;
            l[k] = in ? row_stat[2 * gh + q] : 0u;
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            a += (unsigned long long)(e[k] - s[k]);
            b += m[k] + ((unsigned long long)l[k] << 32);
            c += f[k];
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
        c += __shfl_xor(c, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&sum[0], a);
        atomicAdd(&sum[1], b);
        atomicAdd(&sum[2], c);
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const unsigned long long v = threadIdx.x == 3 ? sum[1] >> 32
                                     : threadIdx.x == 1 ? (uint32_t)sum[1] : sum[threadIdx.x];
        if (v) atomicAdd(threadIdx.x < 3 ? &out[threadIdx.x] : large, v);
    }
    read_back(R);
}

// list mode: the multi-polygon segments of all rows, in row order
__global__ __launch_bounds__(256) void k_multi_list(const int64_t *seg_beg, const int64_t *seg_end,
                                                    const uint32_t *seg_code,
                                                    const uint64_t *seg_key,
                                                    const int64_t *row_moff, int32_t gh,
                                                    uint64_t *mkey, uint32_t *mval)
{
    const int lane = threadIdx.x & 63;
    const int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (r >= gh) return;
    int64_t o = row_moff[r];
    const int64_t b = seg_beg[r], e = seg_end[r];
    for (int64_t q0 = b; q0 < e; q0 += 64) {
        const int64_t q = q0 + lane;
        const bool m = q < e && (seg_code[q] & SEG_SLOT);
        const uint64_t bal = __ballot(m);
        if (m) {
            const int64_t at = o + __popcll(bal & ((1ull << lane) - 1));
            mkey[at] = seg_key[q];
            mval[at] = (uint32_t)q;
        }
        o += __popcll(bal);
    }
}

__global__ void k_widen(const uint32_t *a, int64_t n, int64_t *b)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) b[t] = a[t];
}

// ---------------------------------------------------------------- boundary cells (Hilbert layout)

// The row's distinct boundary cells, found as a bitmap of the row in LDS
// (CELL_BITS columns at a time).  COUNT: their number.  WRITE: each cell's
// Hilbert key and the segment that holds it (NO_SEG if none does: centre-
// sampled cells) from rowcell[row] on: the bits are first listed in LDS, so
// that each lane then takes one cell, with the row's segment starts in LDS to
// search (a lane walking a word's bits against the segments in memory kept a
// row of 500 cells and 350 segments busy four times as long).  With `border`
// (clip windows) the cells on the box's border belong to them.
//
// That is for rows of more than CELL_PAIRS pairs, or CELLS_FEW cells; of a row
// of fewer a wavefront sorts the pairs instead, whatever the box's width.  (One
// ring over 1.0M rows and columns, two pairs a row: the bitmaps alone took 35 ms
// of a build that now takes 1.8.)
#define CELL_BITS 65536
#define CELL_LIST 4096
#define CELL_SEGS 1536
#define NO_SEG 0xffffffffu
#define CELL_PAIRS 64
#define CELLS_FEW 128
// Many rows of few pairs each, a ring's over a large box, take a lane each: rows of
// up to TINY_PAIRS pairs and TINY_CELLS cells, where there are TINY_ROWS rows or
// more and no more than TINY_PAIRS pairs a row on average (a ring of 64 edges over
// 1,048,577 rows: COUNT 296 us with a wavefront a row, 80 so, WRITE 908 and 243;
// over fewer rows than wavefronts in flight, 8 a SIMD, a wavefront each is better).
#define TINY_PAIRS 4
#define TINY_CELLS 16
#define TINY_ROWS (1 << 17)

// The rows that get a bitmap: those of the classes above CELL_PAIRS pairs, then
// with a border the first and the last, then listed ones of many cells.  WRITE
// gives the rows of more than CELL_LIST cells `parts` workgroups each, before all
// others: a partition's outer sides are such rows, and by one workgroup those of
// 260 polygons at 0.5 m, 114,286 cells, made the launch take 1,330 us; 293 now.
struct CellRows {
    const int32_t *list;  // by class, see k_row_lists
    int32_t gh;
    int32_t n1, n2, n3;   // rows of classes 1 to 3
    int32_t border;       // 0, or how many of row 0 and row gh - 1 there are
    int32_t *many, *large;                 // rows listed by COUNT
    unsigned long long *fig;               // their numbers, the most cells of a row
    int32_t nlarge, parts;                 // WRITE
};

// the block's row; -1: a border row, which has a block of its own
__device__ __forceinline__ int32_t cell_row(const CellRows &C, int *part)
{
    int32_t b = (int32_t)blockIdx.x, r;
    const int64_t gh = C.gh;
    *part = -1;
    if (b < C.nlarge * C.parts) {
        *part = b % C.parts;
        return C.large[b / C.parts];
    }
    b -= C.nlarge * C.parts;
    if (b < C.n1) {
        r = C.list[gh + b];
    } else if ((b -= C.n1) < C.n2) {
        r = C.list[2 * gh + b];
    } else if ((b -= C.n2) < C.n3) {
        r = C.list[3 * gh + b];
    } else if ((b -= C.n3) < C.border) {
        return b ? C.gh - 1 : 0;
    } else {
        return C.many[b - C.border];
    }
    return C.border && (r == 0 || r == C.gh - 1) ? -1 : r;
}

__device__ __forceinline__ void cells_large(const CellRows &C, int32_t row, int64_t cells)
{
    C.large[atomicAdd(&C.fig[1], 1ull)] = row;
    atomicMax(&C.fig[2], (unsigned long long)cells);
}

// ascending over a wavefront
__device__ __forceinline__ void wave_sort(uint64_t (&v)[1])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 2; k <= 64; k <<= 1) {
        const bool up = k == 64 || (lane & k) == 0;
        if (k >= 64) sort_step<32, 1>(v, up);
        if (k >= 32) sort_step<16, 1>(v, up);
        if (k >= 16) sort_step<8, 1>(v, up);
        if (k >= 8) sort_step<4, 1>(v, up);
        if (k >= 4) sort_step<2, 1>(v, up);
        sort_step<1, 1>(v, up);
    }
}

// A row of at most CELL_PAIRS pairs by a wavefront: its intervals in order of
// their first cells, each less what the ones before it reach.  COUNT lists the
// rows of more than CELLS_FEW cells, which WRITE leaves to a bitmap.
template <bool WRITE, typename K>
__device__ __forceinline__ void row_cells_few(int32_t row, const uint4 *items,
                                              const int64_t *rowoff, int32_t gw, int32_t gh,
                                              int border, int64_t *rowcell, const int64_t *seg_beg,
                                              const int64_t *seg_end, const int32_t *seg_x0,
                                              const int32_t *seg_x1, int L, K *keys, uint32_t *bseg,
                                              const CellRows &C)
{
    const int lane = threadIdx.x & 63;
    if (row >= gh || (border && (row == 0 || row == gh - 1))) return;
    const int64_t i0 = rowoff[row];
    const int n = (int)(rowoff[row + 1] - i0);
    if (n > CELL_PAIRS) return;
    const int64_t done = WRITE ? rowcell[row] : 0;
    if (WRITE && (rowcell[row + 1] == done || rowcell[row + 1] - done > CELLS_FEW)) return;
    uint64_t v[1] = {~(uint64_t)0};
    if (lane < n) {
        const uint4 it = items[i0 + lane];
        const uint32_t end = min(it.z, (uint32_t)gw);
        if (it.y < end) v[0] = ((uint64_t)it.y << 32) | end;
    }
    wave_sort(v);
    const bool in = v[0] != ~(uint64_t)0;
    const uint32_t a = in ? (uint32_t)(v[0] >> 32) : 0xffffffffu, b = in ? (uint32_t)v[0] : 0u;
    const uint32_t reach = wave_scan<OpMax>(b);  // of the intervals up to this one
    // (every lane takes part: a lane that does not reads as 0)
    const uint32_t up = (uint32_t)__shfl_up((int)reach, 1, 64), before = lane ? up : 0u;
    const uint32_t from = max(a, before), len = in && b > from ? b - from : 0u;
    const uint32_t incl = wave_scan<OpAdd>(len);
    const uint32_t cells = (uint32_t)__shfl((int)incl, 63, 64);
    // the border's cells, where no interval holds them
    const uint32_t lowest = (uint32_t)__shfl((int)a, 0, 64);
    const uint32_t highest = (uint32_t)__shfl((int)reach, 63, 64);
    const uint32_t first = border && lowest != 0 ? 1u : 0u;
    const uint32_t last = border && highest != (uint32_t)gw && gw > 1 ? 1u : 0u;
    const uint32_t all = cells + first + last;
    if (!WRITE) {
        if (lane == 0) {
            rowcell[row] = all;
            if (all > CELL_LIST) cells_large(C, row, all);
            else if (all > CELLS_FEW) C.many[atomicAdd(&C.fig[0], 1ull)] = row;
        }
        return;
    }
    const int64_t sb = seg_beg[row];
    const int ns = (int)(seg_end[row] - sb);
    for (uint32_t t0 = 0; t0 < all; t0 += 64) {
        const uint32_t t = t0 + lane;
        // the interval of cell t: the first whose inclusive count exceeds it
        int i = 0;
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) {
            const uint32_t u = (uint32_t)__shfl((int)incl, i + step - 1, 64);
            i += u <= t ? step : 0;
        }
        i = i > 63 ? 63 : i;
        uint32_t x = (uint32_t)__shfl((int)from, i, 64) +
                     (t - (uint32_t)__shfl((int)(incl - len), i, 64));
        if (t >= cells) x = t == cells && first ? 0u : (uint32_t)gw - 1;
        if (t >= all) continue;
        int lo = 0, hi = ns;  // segments that start at or before x
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (seg_x0[sb + mid] <= (int32_t)x) lo = mid + 1; else hi = mid;
        }
        const bool held = lo > 0 && (int32_t)x < seg_x1[sb + lo - 1];
        keys[done + t] = (K)hilbert_index(L, x, (uint32_t)row);
        bseg[done + t] = held ? (uint32_t)(sb + lo - 1) : NO_SEG;
    }
}

// A row of at most TINY_PAIRS pairs and TINY_CELLS cells by one lane; false: not
// such a row (or, WRITE, none of a wavefront's).
template <bool WRITE, typename K>
__device__ __forceinline__ bool row_cells_tiny(int32_t row, const uint4 *items,
                                               const int64_t *rowoff, int32_t gw, int32_t gh,
                                               int border, int64_t *rowcell, const int64_t *seg_beg,
                                               const int64_t *seg_end, const int32_t *seg_x0,
                                               const int32_t *seg_x1, int L, K *keys, uint32_t *bseg)
{
    if (row >= gh || (border && (row == 0 || row == gh - 1))) return true;  // none, or a bitmap's
    const int64_t i0 = rowoff[row];
    const int n = (int)(rowoff[row + 1] - i0);
    if (n > TINY_PAIRS) return false;
    const int64_t done = WRITE ? rowcell[row] : 0;
    const int64_t total = WRITE ? rowcell[row + 1] - done : 0;
    if (WRITE && total > TINY_CELLS) return false;
    if (WRITE && total == 0) return true;
    uint64_t v[TINY_PAIRS];
#pragma unroll
    for (int k = 0; k < TINY_PAIRS; k++) {
        v[k] = ~(uint64_t)0;
        if (k >= n) continue;
        const uint4 it = items[i0 + k];
        const uint32_t end = min(it.z, (uint32_t)gw);
        if (it.y < end) v[k] = ((uint64_t)it.y << 32) | end;
    }
#pragma unroll
    for (int i = 0; i < TINY_PAIRS; i++)
#pragma unroll
        for (int k = 0; k + 1 < TINY_PAIRS - i; k++) {
            const uint64_t a = min(v[k], v[k + 1]), b = max(v[k], v[k + 1]);
            v[k] = a;
            v[k + 1] = b;
        }
    uint32_t reach = 0, cells = 0;
    const uint32_t lowest = (uint32_t)(v[0] >> 32);
    const int64_t sb = WRITE ? seg_beg[row] : 0;
    const int ns = WRITE ? (int)(seg_end[row] - sb) : 0;
    int lo = 0;  // segments that start at or before the cell
    auto put = [&](uint32_t x) {
        while (lo < ns && seg_x0[sb + lo] <= (int32_t)x) lo++;
        const bool held = lo > 0 && (int32_t)x < seg_x1[sb + lo - 1];
        keys[done + cells] = (K)hilbert_index(L, x, (uint32_t)row);
        bseg[done + cells] = held ? (uint32_t)(sb + lo - 1) : NO_SEG;
    };
    const uint32_t first = border && lowest != 0 ? 1u : 0u;
    if (WRITE && first) put(0);
    cells += first;
#pragma unroll
    for (int k = 0; k < TINY_PAIRS; k++) {
        if (v[k] == ~(uint64_t)0) continue;
        const uint32_t b = (uint32_t)v[k], a = max((uint32_t)(v[k] >> 32), reach);
        if (b <= a) continue;
        reach = b;
        if (WRITE)
            for (uint32_t x = a; x < b; x++, cells++) put(x);
        else
            cells += b - a;
    }
    const uint32_t last = border && reach != (uint32_t)gw && gw > 1 ? 1u : 0u;
    if (WRITE && last) put((uint32_t)gw - 1);
    cells += last;
    if (!WRITE) {
        if (cells > TINY_CELLS) return false;
        rowcell[row] = cells;
    }
    return true;
}

template <bool WRITE, typename K>
__global__ __launch_bounds__(256) void k_row_cells(const uint4 *items, const int64_t *rowoff,
                                                   int32_t gw, int32_t gh, int border,
                                                   int64_t *rowcell, const int64_t *seg_beg,
                                                   const int64_t *seg_end, const int32_t *seg_x0,
                                                   const int32_t *seg_x1, int L, K *keys,
                                                   uint32_t *bseg, CellRows C, int bitmaps,
                                                   int tiny)
{
    // the first workgroups a row's bitmap each, the others rows of few pairs: a
    // wavefront one, or (tiny) a lane one and the wavefront those left
    if ((int)blockIdx.x >= bitmaps) {
        const unsigned b = blockIdx.x - (unsigned)bitmaps;
        const int32_t row = (int32_t)(tiny ? b * 256 + threadIdx.x : b * 4 + (threadIdx.x >> 6));
        const bool rest = !tiny || !row_cells_tiny<WRITE, K>(row, items, rowoff, gw, gh, border,
                                                             rowcell, seg_beg, seg_end, seg_x0,
                                                             seg_x1, L, keys, bseg);
        for (uint64_t m = tiny ? __ballot(rest) : 1ull; m; m &= m - 1) {
            const int32_t r = tiny ? row - (int32_t)(threadIdx.x & 63) + __ffsll((long long)m) - 1 : row;
            row_cells_few<WRITE, K>(r, items, rowoff, gw, gh, border, rowcell, seg_beg, seg_end,
                                    seg_x0, seg_x1, L, keys, bseg, C);
        }
        return;
    }
    __shared__ uint32_t bits[CELL_BITS / 32];
    __shared__ uint16_t cells[WRITE ? CELL_LIST : 1];
    __shared__ int32_t sx[WRITE ? CELL_SEGS : 1];
    __shared__ uint16_t htab[WRITE ? HILBERT_TAB : 1];
    __shared__ uint32_t wsum[4];
    __shared__ uint32_t taken;  // chunks of CELL_BITS columns that hold a cell
    static_assert(MAX_GRID_SIDE <= 32 * CELL_BITS, "a bit a chunk");
    int part;
    const int row = cell_row(C, &part), tid = threadIdx.x;
    if (row < 0) return;
    const int64_t i0 = rowoff[row];
    const int n = (int)(rowoff[row + 1] - i0);
    int64_t done = WRITE ? rowcell[row] : 0;
    if (WRITE && rowcell[row + 1] == done) return;
    if (WRITE && part < 0 && rowcell[row + 1] - done > CELL_LIST) return;  // in parts
    int batch = 0;  // of CELL_LIST cells
    const int64_t sb = WRITE ? seg_beg[row] : 0;
    const int ns = WRITE ? (int)(seg_end[row] - sb) : 0;
    const bool staged = ns <= CELL_SEGS;
    if (WRITE) {
        if (staged)
            for (int k = tid; k < ns; k += 256) sx[k] = seg_x0[sb + k];
        for (int e = tid; e < HILBERT_TAB; e += 256) htab[e] = hilbert_tab_entry((uint32_t)e);
    }
    const bool all = border && (row == 0 || row == gh - 1);
    if (gw > CELL_BITS && !all) {
        if (tid == 0) taken = border ? 1u | 1u << ((gw - 1) / CELL_BITS) : 0u;
        __syncthreads();
        uint32_t m = 0;
        for (int i = tid; i < n; i += 256) {
            const uint4 it = items[i0 + i];
            const int32_t b = min((int32_t)it.z, gw);
            if ((int32_t)it.y >= b) continue;
            const int ca = (int32_t)it.y / CELL_BITS, cb = (b - 1) / CELL_BITS;
            m |= (0xffffffffu << ca) & (0xffffffffu >> (31 - cb));
        }
        if (m) atomicOr(&taken, m);
        __syncthreads();
    }
    for (int32_t w0 = 0; w0 < gw; w0 += CELL_BITS) {
        if (gw > CELL_BITS && !all && !(taken >> (w0 / CELL_BITS) & 1u)) continue;
        const int32_t wn = min(CELL_BITS, gw - w0);
        const int words = (wn + 31) >> 5;
        for (int k = tid; k < words; k += 256) {
            uint32_t v = 0;
            if (all) v = (k + 1) * 32 <= wn ? 0xffffffffu : (1u << (wn & 31)) - 1u;
            bits[k] = v;
        }
        __syncthreads();
        for (int i = tid; i < n; i += 256) {
            const uint4 it = items[i0 + i];
            const int32_t a = max((int32_t)it.y - w0, 0), b = min((int32_t)it.z - w0, wn);
            if (a >= b) continue;
            const int ka = a >> 5, kb = (b - 1) >> 5;
            for (int k = ka; k <= kb; k++) {
                const int x0 = k == ka ? (a & 31) : 0, x1 = k == kb ? ((b - 1) & 31) : 31;
                const uint32_t m = (0xffffffffu << x0) & (0xffffffffu >> (31 - x1));
                if ((bits[k] & m) != m) atomicOr(&bits[k], m);
            }
        }
        if (border && !all && tid == 0) {
            if (w0 == 0) atomicOr(&bits[0], 1u);
            if (w0 + wn == gw) atomicOr(&bits[(wn - 1) >> 5], 1u << ((wn - 1) & 31));
        }
        __syncthreads();
        // each lane takes consecutive words
        const int per = (words + 255) >> 8, k0 = min(tid * per, words), k1 = min(k0 + per, words);
        uint32_t c = 0, tot;
        for (int k = k0; k < k1; k++) c += (uint32_t)__popc(bits[k]);
        const uint32_t first = wg_scan_incl<256>(c, wsum, &tot) - c;
        if (WRITE) {
            for (uint32_t base = 0; base < tot; base += CELL_LIST) {
                if (part >= 0 && batch++ % C.parts != part) continue;
                uint32_t o = first;
                for (int k = k0; k < k1 && o < base + CELL_LIST; k++) {
                    for (uint32_t v = bits[k]; v; v &= v - 1, o++)
                        if (o >= base && o < base + CELL_LIST)
                            cells[o - base] = (uint16_t)(32 * k + __ffs((int)v) - 1);
                }
                __syncthreads();
                const uint32_t m = min(tot - base, (uint32_t)CELL_LIST);
                for (uint32_t i = tid; i < m; i += 256) {
                    const int32_t x = w0 + (int32_t)cells[i];
                    // last segment that starts at or before x
                    int lo = 0, len = ns;
                    while (len > 0) {
                        const int half = len >> 1;
                        const int32_t s = staged ? sx[lo + half] : seg_x0[sb + lo + half];
                        if (s <= x) {
                            lo += half + 1;
                            len -= half + 1;
                        } else {
                            len = half;
                        }
                    }
                    const bool in = lo > 0 && x < seg_x1[sb + lo - 1];
                    const int64_t at = done + base + i;
                    keys[at] = sizeof(K) == 4
                                   ? (K)hilbert_index_tab(L, (uint32_t)x, (uint32_t)row, htab)
                                   : (K)hilbert_index(L, (uint32_t)x, (uint32_t)row);
                    bseg[at] = in ? (uint32_t)(sb + lo - 1) : NO_SEG;
                }
                __syncthreads();
            }
        }
        done += tot;
        __syncthreads();
    }
    if (!WRITE && tid == 0) {
        rowcell[row] = done;
        if (done > CELL_LIST) cells_large(C, row, done);
    }
}

template <typename K>
static int row_cells_write(BuildState &B, const sba_handle *h, const uint4 *items,
                           const int64_t *rowoff, int64_t *rowcell, int64_t nc, const CellRows &C,
                           unsigned rows, int tiny, K **keys, hipStream_t st)
{
    RC(B.alloc(keys, nc));
    RC(B.alloc(&B.bseg, nc));
    const int32_t gw = (int32_t)h->gw, gh = (int32_t)h->gh;
    const int border = B.window ? 1 : 0;
    hipLaunchKernelGGL((k_row_cells<true, K>), dim3(rows + grid_for(gh, tiny ? 256 : 4)), dim3(256),
                       0, st, items, rowoff, gw, gh, border, rowcell, B.seg_beg, B.seg_end, B.seg_x0,
                       B.seg_x1, h->level, *keys, B.bseg, C, (int)rows, tiny);
    HIP_OK(hipGetLastError());
    return 0;
}

// ---------------------------------------------------------------- host

// A class of rows: workgroup, pairs and toggles it takes.  A covered interval
// starts at a pair of its own, so n pairs leave at most 2 n toggles, which the
// first two classes hold; in larger rows toggles outnumber the pairs only when
// most edges stand alone, and a row that does not fit takes the global sorts.
// A small row wants many rows in flight (3.6 KB of LDS a wavefront), a large
// one many wavefronts.
struct SweepClass {
    int block, nmax, rt, tc;
};
static const SweepClass SWEEP[ROW_CLASSES] = {
    {64, 64, 2, 128}, {256, 256, 2, 512}, {512, 1024, 4, 1408}, {1024, 4096, 4, 4096}};

template <int BLOCK, int RN, int RT, typename P, typename K2>
static int sweep_class(const SweepArgs &A0, int c, int64_t rows, hipStream_t st)
{
    SweepArgs A = A0;
    A.list += (int64_t)c * A.gh;
    A.nmax = SWEEP[c].nmax;
    A.tc = SWEEP[c].tc;
    const int lds = sweep_lds_a(A.nmax, A.tc) + BLOCK * RT * (int)sizeof(K2) + 6 * A.tc;
    auto kern = k_row_sweep<BLOCK, RN, RT, P, K2>;
    if (lds > 64 * 1024) {
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  lds);
        (void)hipGetLastError();
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)rows), dim3(BLOCK), lds, st, A);
    HIP_OK(hipGetLastError());
    return 0;
}

// rows[c]: rows of class c (the largest first: its workgroups take longest)
template <typename P, typename K2>
static int sweep_launch(const SweepArgs &A, const int64_t *rows, hipStream_t st)
{
    if (rows[3]) RC((sweep_class<1024, 4, 4, P, K2>(A, 3, rows[3], st)));
    if (rows[2]) RC((sweep_class<512, 2, 4, P, K2>(A, 2, rows[2], st)));
    if (rows[1]) RC((sweep_class<256, 1, 2, P, K2>(A, 1, rows[1], st)));
    if (rows[0]) RC((sweep_class<64, 1, 2, P, K2>(A, 0, rows[0], st)));
    return 0;
}

int rows_coverage(const sba_polygons *polys, const int4 *bbox, int64_t nv,
                  hipStream_t st, sba_handle *h, BuildState &B, int paths_off, bool *taken,
                  bool *one_wg)
{
    *taken = *one_wg = false;
    const int32_t np = polys->n_polys;
    const int32_t gh = (int32_t)h->gh;
    RowGeo G{};
    G.s = h->s;
    G.mag = h->mag;
    G.shift = h->shift;
    G.gi0 = h->gi0;
    G.gj0 = h->gj0;
    G.gw = (int32_t)h->gw;
    G.gh = gh;
    G.ox = h->gi0 * h->s;
    G.oy = h->gj0 * h->s;
    G.extx = h->gw * h->s;
    G.exty = h->gh * h->s;
    const bool hilbert = h->kind == SBA_KIND_HILBERT;
    G.use_b = B.centre ? 0 : 1;
    G.use_c = B.boundary_only ? 0 : 1;
    G.need_b = (!B.centre || hilbert) ? 1 : 0;
    G.centre = B.centre ? 1 : 0;
    int32_t *hint = nullptr;
    RC(B.alloc(&hint, (nv + 63) / 64));
    const PolyView P{polys->ring_off, polys->vert_off, polys->xy, bbox, hint, np, nv};

    // pairs per row, their offsets
    int32_t *rowdiff = nullptr;
    int64_t *rowoff = nullptr;
    unsigned long long *stat = nullptr;
    // the pair counters, then the figures that the host reads: k_row_scan's
    // and k_row_lists' eight, the sweep's totals (k_row_totals), the members of
    // large sets, k_edge_rows' workgroups of many pairs, k_row_cells' listed rows
    // (three), the number of large sets
    constexpr int NFIG = 18, NST = ROW_STATS * ROW_STAT_STEP + NFIG;
    RC(B.alloc(&rowdiff, (int64_t)gh + 1));
    RC(B.alloc(&rowoff, (int64_t)gh + 1));
    RC(B.alloc(&stat, NST));
    int32_t *list = nullptr;
    uint32_t *row_stat = nullptr;
    RC(B.alloc(&list, (int64_t)gh * ROW_CLASSES));
    RC(B.alloc(&row_stat, (int64_t)gh * ROW_FIGS));
    RC(B.alloc(&B.seg_beg, gh));
    RC(B.alloc(&B.seg_end, gh));
    unsigned long long *fig = stat + ROW_STATS * ROW_STAT_STEP;
    bool hash = !(paths_off & 4);
    SetStage S{};
    if (hash) RC(sets_table(S, B, np, false));
    hipLaunchKernelGGL(k_rows_init, dim3(grid_for(std::max<int64_t>((int64_t)np * 64, std::max<int64_t>(gh + 1, NST)))),
                       dim3(256), 0, st, polys->ring_off, polys->vert_off, np, hint, rowdiff,
                       (int64_t)gh + 1, stat, NST, row_stat + 2 * (int64_t)gh, S.tab.tab,
                       hash ? set_tab_words(S.tab) : (int64_t)0);
    // few edges: fewer a workgroup, so that their pairs (each two 64-bit
    // divisions) spread over the chip (512 edges of 55 rows: 80 us with 256 a
    // workgroup)
    int epw = EB;
    while (epw > 4 && nv < (int64_t)1024 * epw) epw >>= 1;
    const dim3 egrid((unsigned)((nv + epw - 1) / epw));
    uint32_t *big = nullptr;
    RC(B.alloc(&big, egrid.x));
    hipLaunchKernelGGL(k_edge_rows<false>, egrid, dim3(EB), 0, st, P, G, epw, rowdiff,
                       (const int64_t *)nullptr, (uint4 *)nullptr, stat, big, fig + 12, 0, 1);
    const bool few_rows = gh < RSCAN_LISTS;  // the scan has gh + 1 entries
    unsigned long long hs[NFIG];
    RC(B.ws.read(hs, fig, sizeof(hs)));
    const RowLists lists{few_rows ? list : nullptr, B.seg_beg, B.seg_end, row_stat};
    uint2 *parts = nullptr;
    const unsigned nparts = (unsigned)(gh / RSCAN_LISTS + 1);
    if (nparts >= RSCAN_PARTS) {
        RC(B.alloc(&parts, nparts));
        hipLaunchKernelGGL(k_row_parts, dim3(nparts), dim3(RSCAN), 0, st, rowdiff, (int64_t)gh,
                           parts);
    }
    hipLaunchKernelGGL(parts ? k_row_scan<true> : k_row_scan<false>, dim3(parts ? nparts : 1),
                       dim3(RSCAN), 0, st, rowdiff, (int64_t)gh, rowoff, stat, fig, parts, lists,
                       few_rows ? B.ws.reads() : ReadSet{});
    HIP_OK(hipGetLastError());
    if (few_rows) {
        RC(B.ws.wait());
    } else {
        hipLaunchKernelGGL(k_row_lists, dim3(grid_for(gh)), dim3(256), 0, st, rowoff, (int64_t)gh,
                           list, B.seg_beg, B.seg_end, row_stat, fig + 2);
        HIP_OK(hipGetLastError());
        RC(B.ws.sync());
    }
    const int64_t items_n = (int64_t)hs[0], max_n = (int64_t)hs[1];
    const int64_t NB = (int64_t)hs[6], NC = (int64_t)hs[7];
    int64_t rows[ROW_CLASSES];
    for (int c = 0; c < ROW_CLASSES; c++) rows[c] = (int64_t)hs[2 + c];
    if (NC % 2) return SBA_EDEVICE;
    h->n_boundary = NB;
    if (2 * NB + NC >= ((int64_t)1 << 32)) return SBA_ELIMIT;
    auto leave = [&]() {
        for (void *p : {(void *)rowdiff, (void *)rowoff, (void *)stat, (void *)list, (void *)hint,
                        (void *)parts, (void *)big, (void *)row_stat, (void *)B.seg_beg, (void *)B.seg_end})
            B.release(p);
        B.seg_beg = B.seg_end = nullptr;
        sets_release(S, B);
        return 0;
    };
    const int pbits = std::max(bits_for((uint64_t)(np - 1)), 1);
    const int xbits = bits_for((uint64_t)h->gw + 1);
    if (max_n > SWEEP[ROW_CLASSES - 1].nmax || items_n >= ((int64_t)1 << 31) ||
        pbits + 2 * xbits + 1 > 63 || (paths_off & 2))
        return leave();

    uint4 *items = nullptr;
    RC(B.alloc(&items, items_n));
    if (items_n) {
        const int64_t nbig = (int64_t)hs[12], most = (int64_t)hs[13];
        // as many workgroups as have a part, or a few for each compute unit
        const int64_t parts = nbig ? std::min<int64_t>((most + EPAIRS - 1) / EPAIRS,
                                                       std::max<int64_t>(8192 / nbig, 1))
                                   : 1;
        hipLaunchKernelGGL(k_edge_rows<true>, dim3(egrid.x + (unsigned)(nbig * parts)), dim3(EB), 0,
                           st, P, G, epw, rowdiff, rowoff, items, (unsigned long long *)nullptr, big,
                           (unsigned long long *)nullptr, (int)nbig, (int)parts);
        HIP_OK(hipGetLastError());
    }
    B.release(rowdiff);
    B.release(hint);
    B.release(big);
    B.release(parts);
    rowdiff = hint = nullptr;
    big = nullptr;
    parts = nullptr;

    // the sweep; again when the members of large sets outgrew their array,
    // or with set keys instead of the hash table when that overflowed
    const int64_t slots = std::max<int64_t>(2 * items_n, 1);
    const int fb = std::min(pbits + 1, 21);  // ids + 1 < 2^21
    int tbits = 0;
    const int64_t tmax = std::min<int64_t>(2 * max_n, SWEEP[ROW_CLASSES - 1].tc);
    while (((int64_t)1 << tbits) < tmax) tbits++;
    RC(B.alloc(&B.seg_x0, slots));
    RC(B.alloc(&B.seg_x1, slots));
    RC(B.alloc(&B.seg_code, slots));
    SweepArgs A{};
    S.fb = fb;
    A.row_stat = row_stat;
    A.list = list;
    A.gw = G.gw;
    RC(B.alloc(&S.memloc, slots));
    A.items = items;
    A.rowoff = rowoff;
    A.gh = gh;
    A.xbits = xbits;
    A.tbits = tbits;
    A.use_b = G.use_b;
    A.fb = fb;
    A.seg_beg = B.seg_beg;
    A.seg_end = B.seg_end;
    A.seg_x0 = B.seg_x0;
    A.seg_x1 = B.seg_x1;
    A.seg_code = B.seg_code;
    A.memloc = S.memloc;
    A.memcnt = fig + 11;
    A.err = (int *)B.sc;
    A.memcap = std::max<int64_t>(1 << 16, items_n);
    RC(B.alloc(&A.mem_ids, A.memcap));
    int64_t NS = 0, NM = 0, NMEM = 0, nset = 0, nids = 0;
    for (int attempt = 0;; attempt++) {
        if (attempt > 0) {
            HIP_OK(hipMemsetAsync(fig + 8, 0, 4 * sizeof(unsigned long long), st));
            HIP_OK(hipMemsetAsync(fig + 17, 0, sizeof(unsigned long long), st));
            HIP_OK(hipMemsetAsync(B.sc + SC_SET_N, 0, sizeof(int64_t), st));
        }
        if (hash && attempt > 0)
            HIP_OK(hipMemsetAsync(S.tab.tab, 0xff, sizeof(uint64_t) * set_tab_words(S.tab), st));
        A.tab = hash ? S.tab : SetTab{};
        if (!hash && !A.seg_key) RC(B.alloc(&A.seg_key, slots));
        const bool p32 = pbits + xbits <= 32, t32 = xbits + tbits <= 31;
        if (p32 && t32) RC((sweep_launch<uint32_t, uint32_t>(A, rows, st)));
        else if (t32) RC((sweep_launch<uint64_t, uint32_t>(A, rows, st)));
        else RC((sweep_launch<uint64_t, uint64_t>(A, rows, st)));
        int64_t hsc[SC_READ];
        RC(B.ws.read(hs, fig, sizeof(hs)));
        RC(B.ws.read(hsc, B.sc, sizeof(hsc)));
        if (few_rows) {
            hipLaunchKernelGGL(k_row_totals<1024>, dim3(1), dim3(1024), 0, st, B.seg_beg, B.seg_end,
                               row_stat, (int64_t)gh, fig + 8, fig + 17, B.ws.reads());
            HIP_OK(hipGetLastError());
            RC(B.ws.wait());
        } else {
            hipLaunchKernelGGL(k_row_totals<256>,
                               dim3((unsigned)std::min<int64_t>((gh + 255) / 256, 64)), dim3(256),
                               0, st, B.seg_beg, B.seg_end, row_stat, (int64_t)gh, fig + 8,
                               fig + 17, ReadSet{});
            HIP_OK(hipGetLastError());
            RC(B.ws.sync());
        }
        const int herr = (int)(uint32_t)hsc[0];
        if (herr & ERR_DEPTH) return SBA_ELIMIT;
        if (herr & ~ERR_ROW) return SBA_EDEVICE;
        if (herr & ERR_ROW) {  // a row does not fit after all: the global sorts
            HIP_OK(hipMemsetAsync(B.sc, 0, sizeof(int64_t) * SC_SLOTS, st));
            for (void *p : {(void *)items, (void *)B.seg_x0, (void *)B.seg_x1, (void *)B.seg_code,
                            (void *)A.mem_ids, (void *)A.seg_key})
                B.release(p);
            sets_release(S, B);
            B.seg_x0 = B.seg_x1 = nullptr;
            B.seg_code = nullptr;
            return leave();
        }
        NS = (int64_t)hs[8];
        NM = (int64_t)hs[9];
        NMEM = (int64_t)hs[10];
        const int64_t mem = (int64_t)hs[11];
        nset = set_count(hsc[SC_SET_N]);
        nids = set_ids_count(hsc[SC_SET_N]);
        bool again = false;
        if (mem > A.memcap) {
            B.release(A.mem_ids);
            A.memcap = mem;
            RC(B.alloc(&A.mem_ids, A.memcap));
            again = true;
        }
        if (hash && nset > (int64_t)S.tab.cap) {
            hash = false;
            again = true;
        }
        if (!again) break;
        if (attempt > 2) return SBA_EDEVICE;
    }
    if (NS >= ((int64_t)1 << 31)) return SBA_ELIMIT;
    h->n_segments = NS;
    B.NS = NS;
    S.mem_ids = A.mem_ids;

    // polygon sets
    if (NM > 0) {
        if (hash) {
            RC(sets_from_table(S, B, h, NM, NMEM, nset, nids, slots, (int64_t)hs[17],
                               (int64_t)hs[11], row_stat + 2 * (int64_t)gh, st));
        } else {
            uint64_t *mkey = nullptr;
            uint32_t *mval = nullptr;
            int64_t *moff = nullptr;
            RC(B.alloc(&mkey, NM));
            RC(B.alloc(&mval, NM));
            RC(B.alloc(&moff, (int64_t)gh));
            hipLaunchKernelGGL(k_widen, dim3(grid_for(gh)), dim3(256), 0, st, row_stat,
                               (int64_t)gh, moff);
            HIP_OK(hipGetLastError());
            RC(scan_exclusive_i64(moff, moff, gh, nullptr, st, &B.ws));
            hipLaunchKernelGGL(k_multi_list, dim3(grid_for((int64_t)gh * 64)), dim3(256), 0, st,
                               B.seg_beg, B.seg_end, B.seg_code, A.seg_key, moff, gh, mkey, mval);
            HIP_OK(hipGetLastError());
            B.release(moff);
            RC(sets_from_list(S, B, h, mkey, mval, NM, NMEM, slots, st));
        }
    }
    *one_wg = S.one_workgroup;
    B.release(A.seg_key);
    B.release(row_stat);
    B.release(A.mem_ids);
    sets_release(S, B);

    // the Hilbert layout's boundary cells
    if (hilbert) {
        RC(hilbert_level(B, h));
        int64_t *rowcell = nullptr;
        RC(B.alloc(&rowcell, (int64_t)gh + 1));
        const int border = B.window ? 1 : 0;
        CellRows C{list, gh, (int32_t)rows[1], (int32_t)rows[2], (int32_t)rows[3],
                   border ? std::min(gh, 2) : 0, nullptr, nullptr, fig + 14, 0, 1};
        RC(B.alloc(&C.many, gh));
        RC(B.alloc(&C.large, gh));
        const unsigned bitmaps = (unsigned)(rows[1] + rows[2] + rows[3] + C.border);
        const int tiny = gh >= TINY_ROWS && items_n <= (int64_t)TINY_PAIRS * gh ? 1 : 0;
        hipLaunchKernelGGL((k_row_cells<false, uint64_t>),
                           dim3(bitmaps + grid_for(gh, tiny ? 256 : 4)), dim3(256), 0, st, items, rowoff, (int32_t)h->gw, gh, border, rowcell,
                           (const int64_t *)nullptr, (const int64_t *)nullptr,
                           (const int32_t *)nullptr, (const int32_t *)nullptr, 0,
                           (uint64_t *)nullptr, (uint32_t *)nullptr, C, (int)bitmaps, tiny);
        HIP_OK(hipGetLastError());
        RC(scan_exclusive_i64(rowcell, rowcell, gh, rowcell + gh, st, &B.ws));
        int64_t nc = 0;
        unsigned long long hc[3] = {0, 0, 0};
        RC(B.ws.read(&nc, rowcell + gh, sizeof(int64_t)));
        RC(B.ws.read(hc, C.fig, sizeof(hc)));
        RC(B.ws.sync());
        B.nbkeys = nc;
        if (nc > 0) {
            C.nlarge = (int32_t)hc[1];
            if (C.nlarge)
                C.parts = (int32_t)std::min<int64_t>(((int64_t)hc[2] + CELL_LIST - 1) / CELL_LIST,
                                                     std::max<int64_t>(4096 / C.nlarge, 1));
            const unsigned all = (unsigned)(C.nlarge * C.parts) + bitmaps + (unsigned)hc[0];
            if (2 * h->level <= 32) {
                RC(row_cells_write<uint32_t>(B, h, items, rowoff, rowcell, nc, C, all, tiny,
                                             &B.bkeys32, st));
                RC(radix_sort_u32_ws(&B.bkeys32, &B.bseg, nc, 2 * h->level, B.ws));
            } else {
                RC(row_cells_write<uint64_t>(B, h, items, rowoff, rowcell, nc, C, all, tiny,
                                             &B.bkeys, st));
                RC(radix_sort_u64_ws(&B.bkeys, &B.bseg, nc, 2 * h->level, B.ws));
            }
        }
        B.release(C.many);
        B.release(C.large);
        B.release(rowcell);
    }
    B.release(list);
    B.release(items);
    B.release(rowoff);
    B.release(stat);
    *taken = true;
    return 0;
}
