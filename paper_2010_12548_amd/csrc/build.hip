// build.hip -- construction of the conservative eps-approximation on the GPU.
//
// Sec. 2.2 of the paper defines the approximation: cells of side
// eps/sqrt(2) along the boundary, every cell that touches the boundary kept
// (conservative raster), interior cells kept whole.  In integers, cell (i,j)
// is in A(P) when its closed square [is,(i+1)s]x[js,(j+1)s] meets an edge of
// P, or when it meets none and its corner (is,js) is inside P by the
// crossing-number rule.
//
// The build never visits a cell that is not on a boundary.  It works on
// rows of cells:
//   1. per edge and per row strip the edge touches: the closed x-range of the
//      edge inside the strip gives one interval of boundary cells;
//   2. per edge and per row line y = js it crosses (half-open rule): the
//      crossing's cell index k = ceil(xc/s); in order per (polygon, row), the
//      crossings pair up into the intervals [k1,k2), [k3,k4) ... of cells
//      whose corner is inside;
//   3. boundary intervals and crossings become events keyed (polygon, row,
//      x); one scan over them in key order yields each polygon's coverage
//      count, whose changes give its maximal covered intervals per row;
//   4. the distinct interval ends of a row cut it into pieces; each covered
//      interval adds its polygon to the pieces it spans, and the non-empty
//      pieces are the maximal row segments of constant polygon set;
//   5. sets of two or more polygons are deduplicated into a set table;
// Steps 1 to 4 run row by row in LDS (rows.hip); the kernels here that sort
// all events and toggles globally take the builds whose rows do not fit.
// Step 5 is in sets.hip.
//   6. the segments are written into the chosen layout: a two-level tiled
//      grid (uniform tiles stored once in a directory, mixed tiles as fine
//      blocks) or, in hilbert.hip, the runs of the Hilbert order.
#include <atomic>
#include <chrono>
#include <vector>

#include "sba_internal.h"
#include "build_state.h"
#include "sets.h"

// ---------------------------------------------------------------- kernels

// event kinds (payload of the (polygon, row, x) event keys)
#define EV_OPEN 0u   // first cell of a boundary interval
#define EV_CLOSE 1u  // one past the last cell of a boundary interval
#define EV_CROSS 2u  // crossing of the row line y = j s

__global__ void k_edges(const int32_t *ring_off, int32_t n_polys, const int64_t *vert_off,
                        int32_t n_rings, const int32_t *xy, int64_t n_verts, int4 *edges,
                        int32_t *epoly)
{
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n_verts) return;
    int lo = 0, hi = n_rings;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (vert_off[mid] <= v) lo = mid + 1; else hi = mid;
    }
    int r = lo - 1;
    lo = 0;
    hi = n_polys;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (ring_off[mid] <= r) lo = mid + 1; else hi = mid;
    }
    int p = lo - 1;
    int64_t w = (v + 1 < vert_off[r + 1]) ? v + 1 : vert_off[r];
    edges[v] = make_int4(xy[2 * v], xy[2 * v + 1], xy[2 * w], xy[2 * w + 1]);
    epoly[v] = p;
}

// offsets: ring_off[0] = 0 and non-decreasing; sizes[0] = n_rings (err bit 2)
__global__ void k_check_rings(const int32_t *ring_off, int32_t n_polys, int64_t *sizes, int *err)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p > n_polys) return;
    if (p == 0 && ring_off[0] != 0) atomicOr(err, 2);
    if (p < n_polys && ring_off[p + 1] < ring_off[p]) atomicOr(err, 2);
    if (p == n_polys) sizes[0] = ring_off[n_polys];
}

// vert_off[0] = 0 and non-decreasing over the n_rings+1 entries; sizes[1] =
// n_verts.  Reads nothing if the ring offsets were already refused.
__global__ void k_check_verts(const int64_t *vert_off, int64_t *sizes, int *err)
{
    if (*err) return;
    const int64_t nr = sizes[0];
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= nr;
         r += (int64_t)gridDim.x * blockDim.x) {
        if (r == 0 && vert_off[0] != 0) atomicOr(err, 2);
        if (r < nr && vert_off[r + 1] < vert_off[r]) atomicOr(err, 2);
        if (r == nr) sizes[1] = vert_off[nr];
    }
}

// k_check_rings and k_check_verts by one workgroup, which zeroes the scalars
// first: for up to CHECK_POLYS polygons, where a launch each (3.4 us of the
// host's time) costs more than the checks
#define CHECK_POLYS 8192
__global__ __launch_bounds__(1024) void k_check_offsets(const int32_t *ring_off,
                                                        const int64_t *vert_off, int32_t n_polys,
                                                        int64_t *sc, int n_sc)
{
    __shared__ int bad;
    if (threadIdx.x == 0) bad = ring_off[0] != 0;
    __syncthreads();
    const int32_t nr = ring_off[n_polys];
    bool b = false;
    for (int32_t p = threadIdx.x; p < n_polys; p += 1024) b |= ring_off[p + 1] < ring_off[p];
    if (b) atomicOr(&bad, 1);
    __syncthreads();
    int64_t nv = 0;
    if (!bad) {  // the same in every lane: read again only after a barrier
        nv = vert_off[nr];
        b = threadIdx.x == 0 && vert_off[0] != 0;
        int64_t r = threadIdx.x;
        for (; r + 7 * 1024 < nr; r += 8 * 1024) {  // 3.2M rings: 1456 us one by one
            int64_t v[8], w[8];  // and 531 with eight rings' loads together
#pragma unroll
            for (int k = 0; k < 8; k++) {
                v[k] = vert_off[r + k * 1024];
                w[k] = vert_off[r + k * 1024 + 1];
            }
#pragma unroll
            for (int k = 0; k < 8; k++) b |= w[k] < v[k];
        }
        for (; r < nr; r += 1024) b |= vert_off[r + 1] < vert_off[r];
    }
    __syncthreads();
    if (b) atomicOr(&bad, 1);
    __syncthreads();
    for (int k = threadIdx.x; k < n_sc; k += 1024)
        sc[k] = k == 0 ? (bad ? 2 : 0) : (k == 1 ? nr : (k == 2 ? nv : 0));
}

#define BOX_BLOCK 1024
#define BOX_GRID 512  // workgroups at most

// the extremes over a workgroup, in thread 0
__device__ __forceinline__ int4 box_reduce(int4 v)
{
    __shared__ int4 red[BOX_BLOCK / 64];
    for (int o = 32; o > 0; o >>= 1) {
        v.x = min(v.x, __shfl_xor(v.x, o, 64));
        v.y = min(v.y, __shfl_xor(v.y, o, 64));
        v.z = max(v.z, __shfl_xor(v.z, o, 64));
        v.w = max(v.w, __shfl_xor(v.w, o, 64));
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int q = 1; q < BOX_BLOCK / 64; q++)
            v = make_int4(min(v.x, red[q].x), min(v.y, red[q].y), max(v.z, red[q].z),
                          max(v.w, red[q].w));
    return v;
}

// one wavefront per polygon: coordinate bounding box, range check (err bit
// 1), empty polygon (err bit 2); skipped when the offsets were refused.  The
// workgroup that ends last (ticket, zero on entry) forms the union of the cell
// boxes, {min over p of ceil(xmin/s) - 1, same for y, max over p of
// floor(xmax/s), same for y} (ceil and floor are monotone, so the extremes of
// the coordinates are found first and divided once), and copies the host's
// values.  The workgroups' extremes pass through memory as single words that
// bypass the caches of their XCD, the ticket after them: a fence a workgroup,
// which empties its L2, took 80 us for 250 of them.
__global__ __launch_bounds__(BOX_BLOCK) void k_poly_bbox(const int32_t *ring_off,
                                                         const int64_t *vert_off, const int32_t *xy,
                                                         int32_t n_polys, int64_t s, int4 *bbox,
                                                         int32_t *part, int *err, int64_t *box,
                                                         unsigned long long *ticket, ReadSet R)
{
    const int lane = threadIdx.x & 63;
    const bool refused = (*err & 2) != 0;
    int4 u = make_int4(INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN);
    for (int64_t p = ((int64_t)blockIdx.x * BOX_BLOCK + threadIdx.x) >> 6; p < n_polys && !refused;
         p += (int64_t)gridDim.x * (BOX_BLOCK / 64)) {
        int64_t v0 = vert_off[ring_off[p]], v1 = vert_off[ring_off[p + 1]];
        if (v1 == v0 && lane == 0) atomicOr(err, 2);
        int xmin = INT32_MAX, ymin = INT32_MAX, xmax = INT32_MIN, ymax = INT32_MIN;
        bool bad = false;
        for (int64_t v = v0 + lane; v < v1; v += 64) {
            int x = xy[2 * v], y = xy[2 * v + 1];
            bad |= (x <= -(1 << 30)) | (x >= (1 << 30)) | (y <= -(1 << 30)) | (y >= (1 << 30));
            xmin = min(xmin, x); ymin = min(ymin, y);
            xmax = max(xmax, x); ymax = max(ymax, y);
        }
        for (int o = 32; o > 0; o >>= 1) {
            xmin = min(xmin, __shfl_xor(xmin, o, 64));
            ymin = min(ymin, __shfl_xor(ymin, o, 64));
            xmax = max(xmax, __shfl_xor(xmax, o, 64));
            ymax = max(ymax, __shfl_xor(ymax, o, 64));
        }
        if (bad) atomicOr(err, 1);
        if (lane == 0) bbox[p] = make_int4(xmin, ymin, xmax, ymax);
        u = make_int4(min(u.x, xmin), min(u.y, ymin), max(u.z, xmax), max(u.w, ymax));
    }
    u = box_reduce(u);
    __shared__ bool last;
    __builtin_amdgcn_s_waitcnt(0);  // the error bits have arrived
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t *q = part + 4 * (int64_t)blockIdx.x;
        __hip_atomic_store(q, u.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(q + 1, u.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(q + 2, u.z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(q + 3, u.w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0);
        last = atomicAdd(ticket, 1ull) + 1 == gridDim.x;
    }
    __syncthreads();
    if (!last) return;
    u = make_int4(INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN);
    for (unsigned k = threadIdx.x; k < gridDim.x; k += BOX_BLOCK) {
        int32_t *q = part + 4 * (int64_t)k;
        const int32_t x0 = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int32_t y0 = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int32_t x1 = __hip_atomic_load(q + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int32_t y1 = __hip_atomic_load(q + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        u = make_int4(min(u.x, x0), min(u.y, y0), max(u.z, x1), max(u.w, y1));
    }
    u = box_reduce(u);
    if (threadIdx.x == 0) {
        box[0] = ceildiv64(u.x, s) - 1;
        box[1] = ceildiv64(u.y, s) - 1;
        box[2] = floordiv64(u.z, s);
        box[3] = floordiv64(u.w, s);
    }
    read_back(R);
}

// per edge: number of boundary row strips and of row-line crossings inside
// the stored box [gi0,gi1] x [gj0,gj1] (the box is the union of the cell
// boxes, cut by the clip window if there is one); polygons whose cell box
// misses the box in x contribute nothing inside it
__global__ void k_edge_counts(const int4 *edges, const int32_t *epoly, const int4 *bbox,
                              int64_t n_edges, int64_t s, int64_t gi0, int64_t gj0, int64_t gi1,
                              int64_t gj1, int centre, int64_t *nb, int64_t *nc)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_edges) return;
    int4 E = edges[e];
    int4 bb = bbox[epoly[e]];
    if (floordiv64(bb.z, s) < gi0 || ceildiv64(bb.x, s) - 1 > gi1) {
        nb[e] = 0;
        nc[e] = 0;
        return;
    }
    int64_t ey0 = min(E.y, E.w), ey1 = max(E.y, E.w);
    int64_t ja = max(ceildiv64(ey0, s) - 1, gj0), jb = min(floordiv64(ey1, s), gj1);
    nb[e] = jb >= ja ? jb - ja + 1 : 0;
    // row lines y = js (corners) or y = (j+1/2)s (centres) crossed under the
    // half-open rule: ey0 <= y < ey1
    int64_t ka, kb;
    if (centre) {
        ka = max(ceildiv64(2 * ey0 - s, 2 * s), gj0);
        kb = min(ceildiv64(2 * ey1 - s, 2 * s) - 1, gj1);
    } else {
        ka = max(ceildiv64(ey0, s), gj0);
        kb = min(ceildiv64(ey1, s) - 1, gj1);
    }
    nc[e] = (E.y != E.w && kb >= ka) ? kb - ka + 1 : 0;
}

__device__ __forceinline__ int64_t upper_bound_i64(const int64_t *a, int64_t n, int64_t v)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] <= v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// boundary item t -> interval of cells [c0, c1] of row j touched by its edge,
// cut to the stored box, written as a start and an end event keyed
// (polygon, row, x) (an interval cut away entirely becomes an empty
// start/end pair at x = 0)
__global__ void k_emit_boundary(const int4 *edges, const int32_t *epoly, int64_t n_edges,
                                const int64_t *boff, int64_t nb_total, int64_t s, int64_t gi0,
                                int64_t gj0, int64_t gi1, int xbits, int rbits, uint64_t *evkey,
                                uint32_t *evpay)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nb_total) return;
    int64_t e = upper_bound_i64(boff, n_edges, t) - 1;
    int4 E = edges[e];
    int64_t x1 = E.x, y1 = E.y, x2 = E.z, y2 = E.w;
    int64_t ey0 = min(y1, y2), ey1 = max(y1, y2);
    int64_t j = max(ceildiv64(ey0, s) - 1, gj0) + (t - boff[e]);
    int64_t c0, c1;
    if (y1 == y2) {
        c0 = ceildiv64(min(x1, x2), s) - 1;
        c1 = floordiv64(max(x1, x2), s);
    } else {
        int64_t ya = max(ey0, j * s), yb = min(ey1, (j + 1) * s);
        int64_t den = y2 - y1;
        // x(y) = (x1*den + (y - y1)*(x2 - x1)) / den ; |numerator| < 2^63
        int64_t na = x1 * den + (ya - y1) * (x2 - x1);
        int64_t nbv = x1 * den + (yb - y1) * (x2 - x1);
        if (den < 0) { den = -den; na = -na; nbv = -nbv; }
        int64_t lo = min(na, nbv), hi = max(na, nbv);
        c0 = ceildiv64(lo, den * s) - 1;
        c1 = floordiv64(hi, den * s);
    }
    c0 = max(c0, gi0);
    c1 = min(c1, gi1);
    if (c0 > c1) { c0 = gi0; c1 = gi0 - 1; }
    uint64_t pr = ((uint64_t)epoly[e] << (rbits + xbits)) | ((uint64_t)(j - gj0) << xbits);
    evkey[2 * t] = pr | (uint64_t)(c0 - gi0);
    evpay[2 * t] = EV_OPEN;
    evkey[2 * t + 1] = pr | (uint64_t)(c1 + 1 - gi0);
    evpay[2 * t + 1] = EV_CLOSE;
}

// crossing item t -> event (polygon, row, k) with k = ceil(xc / s), k cut to
// [gi0, gi1 + 1] (inside spans are then cut to the stored box)
__global__ void k_emit_cross(const int4 *edges, const int32_t *epoly, int64_t n_edges,
                             const int64_t *coff, int64_t nc_total, int64_t s, int64_t gi0,
                             int64_t gj0, int64_t gi1, int centre, int xbits, int rbits,
                             uint64_t *evkey, uint32_t *evpay)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nc_total) return;
    int64_t e = upper_bound_i64(coff, n_edges, t) - 1;
    int4 E = edges[e];
    int64_t x1 = E.x, y1 = E.y, x2 = E.z, y2 = E.w;
    int64_t ey0 = min(y1, y2);
    int64_t den = y2 - y1, k;
    if (centre) {
        // centre line y = (j+1/2)s; with 2 xc = num / den the centre of cell i
        // lies left of the crossing iff (2i+1) s den < num (den > 0).  The
        // terms stay below 2^63 for coordinates under 2^30 in magnitude.
        int64_t j = max(ceildiv64(2 * ey0 - s, 2 * s), gj0) + (t - coff[e]);
        int64_t num = 2 * x1 * den + ((2 * j + 1) * s - 2 * y1) * (x2 - x1);
        if (den < 0) { den = -den; num = -num; }
        k = ceildiv64(num - s * den, 2 * s * den);
        k = min(max(k, gi0), gi1 + 1);
        evkey[t] = ((uint64_t)epoly[e] << (rbits + xbits)) | ((uint64_t)(j - gj0) << xbits) |
                   (uint64_t)(k - gi0);
        evpay[t] = EV_CROSS;
        return;
    }
    int64_t j = max(ceildiv64(ey0, s), gj0) + (t - coff[e]);
    int64_t num = x1 * den + (j * s - y1) * (x2 - x1);
    if (den < 0) { den = -den; num = -num; }
    k = ceildiv64(num, den * s);
    k = min(max(k, gi0), gi1 + 1);
    evkey[t] = ((uint64_t)epoly[e] << (rbits + xbits)) | ((uint64_t)(j - gj0) << xbits) |
               (uint64_t)(k - gi0);
    evpay[t] = EV_CROSS;
}

// ------------------------------------------------ coverage of each row
//
// Events carry the key (polygon, row, x) and one of three kinds: the start
// of a boundary interval, one past its end, or a crossing of the row line.
// Sorted by key, each (polygon, row) group holds matched starts and ends and
// an even number of crossings; cells from the 2m-th to the (2m+1)-th
// crossing have their corner inside (Sec. 2.2, crossing-number rule).  The
// polygon covers x when a boundary interval is open there or the crossings
// seen so far are odd in number.  One global scan gives both counts at every
// event: starts and ends add +1/-1 to the low 32 bits, crossings add 1 to
// the high bits.  Groups before the current one are balanced, so the prefix
// equals the prefix within the group.
__device__ __forceinline__ int64_t ev_value(uint32_t kind)
{
    return kind == EV_CROSS ? ((int64_t)1 << 32) : (kind == EV_OPEN ? 1 : -1);
}

// coverage count of the event's polygon just after event t (cex = exclusive
// scan of ev_value); the low part never goes negative because the sort is
// stable and every interval's start precedes its end
__device__ __forceinline__ int64_t cov_after(const int64_t *cex, const uint32_t *kind, int64_t t)
{
    int64_t S = cex[t] + ev_value(kind[t]);
    return (S & 0xffffffffll) + ((S >> 32) & 1);
}

__global__ void k_ev_values(const uint32_t *kind, int64_t n, int64_t *v)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) v[t] = ev_value(kind[t]);
}

// flag[t] = 1 when t is the last event of its (polygon, row, x) group and
// the polygon's membership at x differs from its membership just before x
// (a toggle).  Toggles of one (polygon, row) alternate on/off, starting with
// on, so consecutive pairs are the maximal covered intervals [a, b).  The
// group's first event comes from a ballot of the wavefront's group heads; only
// a group that began in an earlier wavefront is walked back in memory.
__global__ __launch_bounds__(256) void k_toggle_flags(const uint64_t *key, const uint32_t *kind,
                                                      const int64_t *cex, int64_t n, int xbits,
                                                      int64_t *flag, int *err)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool in = t < n;
    const uint64_t k = in ? key[t] : 0;
    const bool head = in && (t == 0 || key[t - 1] != k);
    const uint64_t heads = __ballot(head);
    if (!in) return;
    int64_t f = 0;
    if (t + 1 == n || key[t + 1] != k) {
        // heads at or before this lane (2 << 63 wraps to 0: all lanes)
        const uint64_t le = heads & ((2ull << lane) - 1);
        int64_t a = t - lane;
        if (le) {
            a += 63 - __clzll(le);
        } else {
            while (a > 0 && key[a - 1] == k) a--;
        }
        uint64_t g = k >> xbits;
        int64_t before = (a > 0 && (key[a - 1] >> xbits) == g) ? cov_after(cex, kind, a - 1) : 0;
        int64_t after = cov_after(cex, kind, t);
        f = (before > 0) != (after > 0);
        if ((t + 1 == n || (key[t + 1] >> xbits) != g) && after != 0) atomicOr(err, 2);
    }
    flag[t] = f;
}

__global__ void k_toggle_emit(const uint64_t *key, const int64_t *toff, int64_t n, int64_t nt,
                              int rxbits, uint64_t *tkey, int32_t *tpoly)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    int64_t o = toff[t];
    int64_t o1 = t + 1 < n ? toff[t + 1] : nt;
    if (o1 == o) return;
    uint64_t k = key[t];
    tkey[o] = k & ((1ull << rxbits) - 1);
    tpoly[o] = (int32_t)(k >> rxbits);
}

__global__ void k_iota_u32(uint32_t *v, int64_t n)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) v[t] = (uint32_t)t;
}

// One pass over the toggles sorted by position (row << xbits | x), each
// carrying its original slot src[t] (slot 2m opens covered interval m, slot
// 2m + 1 closes it).  pos is the exclusive count of first occurrences, nu
// its total (the number of distinct positions).  Writes
//  * E: the sorted distinct positions, which cut every row into elementary
//    pieces [E[k], E[k+1]) of constant polygon set;
//  * rank[slot]: the index in E of every toggle;
//  * diff[k]: intervals opening at E[k] less intervals closing there (the
//    depth of piece k is the prefix sum), formed by the first toggle of each
//    distinct position over its run of equal positions; entries nu..n are
//    zeroed here.
__global__ void k_unique_rank(const uint64_t *keys, int64_t n, const int64_t *pos,
                              const int64_t *nu_p, const uint32_t *src, uint64_t *E,
                              int64_t *rank, int64_t *diff)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const uint64_t k = keys[t];
    const bool first = t == 0 || k != keys[t - 1];
    const int64_t r = pos[t] - (first ? 0 : 1);
    rank[src[t]] = r;
    if (first) {
        E[r] = k;
        int64_t d = 0;
        for (int64_t u = t; u < n && keys[u] == k; u++) d += (src[u] & 1u) ? -1 : 1;
        diff[r] = d;
    }
    const int64_t nu = *nu_p;
    if (t >= nu) diff[t] = 0;
    if (t == n - 1) diff[n] = 0;
}

// Covered interval m spans pieces [ka, kb), the indices in E of its two
// toggles.
__global__ void k_interval_span(const int64_t *rank, int64_t nint, int64_t *ika, int64_t *cnt)
{
    int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= nint) return;
    const int64_t ka = rank[2 * m], kb = rank[2 * m + 1];
    ika[m] = ka;
    cnt[m] = kb - ka;
}

// per piece: packed counters (non-empty << 32 | multi) and multi member count
__global__ void k_piece_classify(const int64_t *dex, const int64_t *diff, int64_t n, int64_t *segc,
                                 int64_t *mm, int *err)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int64_t d = dex[k] + diff[k];
    if (d > MAX_DEPTH) atomicOr(err, 8);
    segc[k] = (d >= 1 ? ((int64_t)1 << 32) : 0) | (d >= 2 ? 1 : 0);
    mm[k] = d >= 2 ? d : 0;
}

// one thread per (interval, piece) pair: record the interval's polygon in
// the piece (a piece of depth 1 keeps its polygon directly)
__global__ void k_piece_members(const int64_t *xoff, int64_t nint, int64_t nx, const int64_t *ika,
                                const int32_t *tpoly, const int64_t *dex, const int64_t *diff,
                                const int64_t *mmoff, int32_t *sid, int32_t *fill, int32_t *mem_ids)
{
    int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= nx) return;
    int64_t lo = 0, hi = nint;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (xoff[mid] <= u) lo = mid + 1; else hi = mid;
    }
    int64_t m = lo - 1;
    int64_t k = ika[m] + (u - xoff[m]);
    int32_t p = tpoly[2 * m];
    if (dex[k] + diff[k] == 1) {
        sid[k] = p;
    } else {
        int32_t r = atomicAdd(&fill[k], 1);
        mem_ids[mmoff[k] + r] = p;
    }
}

// non-empty pieces become the row segments; members of multi-polygon
// segments are put in ascending order (the set's canonical form)
__global__ void k_piece_emit(const uint64_t *E, int64_t n, const int64_t *dex, const int64_t *diff,
                             const int64_t *segc, const int64_t *mmoff, const int32_t *sid,
                             int xbits, int32_t *seg_x0, int32_t *seg_x1, uint32_t *seg_code,
                             uint32_t *seg_row, int64_t *multi_seg, int64_t *multi_mem,
                             int32_t *mem_ids)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int64_t d = dex[k] + diff[k];
    if (d < 1) return;
    const uint64_t xm = (1ull << xbits) - 1;
    int64_t sc = segc[k];
    int64_t o = sc >> 32;
    uint64_t e0 = E[k], e1 = E[k + 1];
    seg_x0[o] = (int32_t)(e0 & xm);
    seg_x1[o] = (int32_t)(e1 & xm);
    seg_row[o] = (uint32_t)(e0 >> xbits);
    if (d == 1) {
        seg_code[o] = (uint32_t)sid[k] + 1u;
        return;
    }
    int64_t a = mmoff[k];
    for (int64_t i = a + 1; i < a + d; i++) {
        int32_t v = mem_ids[i];
        int64_t j = i;
        while (j > a && mem_ids[j - 1] > v) { mem_ids[j] = mem_ids[j - 1]; j--; }
        mem_ids[j] = v;
    }
    int64_t mi = sc & 0xffffffffll;
    multi_seg[mi] = o;
    multi_mem[mi] = a;
    seg_code[o] = 0xffffffffu;
}

__global__ void k_seg_row_off(const uint32_t *seg_row, int64_t ns, int64_t gh, int64_t *row_off)
{
    int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r > gh) return;
    int64_t lo = 0, hi = ns;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if ((int64_t)seg_row[mid] < r) lo = mid + 1; else hi = mid;
    }
    row_off[r] = lo;
}

// ------------------------------------------------ multi-polygon segments

// set key of multi segment m (sets.h); members of larger sets stay where
// k_piece_emit sorted them
__global__ void k_multi_keys(const int64_t *multi_mem, const int64_t *multi_seg, int64_t n_multi,
                             int64_t n_mem, const int32_t *mem_ids, int fb, uint64_t *key,
                             uint32_t *val, uint64_t *memloc)
{
    int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n_multi) return;
    int64_t a = multi_mem[m], b = (m + 1 < n_multi) ? multi_mem[m + 1] : n_mem;
    const int64_t o = multi_seg[m];
    uint64_t k = 0;
    if (b - a <= 3) {
        for (int64_t t = a; t < b; t++) k |= (uint64_t)(mem_ids[t] + 1) << (fb * (t - a));
    } else {
        k = (1ull << (3 * fb)) + (uint64_t)o;
        memloc[o] = ((uint64_t)a << 6) | (uint64_t)(b - a);
    }
    key[m] = k;
    val[m] = (uint32_t)o;
}

__global__ void k_flag_new(const uint64_t *key, int64_t n, int64_t *flag)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    flag[t] = (t == 0 || key[t] != key[t - 1]) ? 1 : 0;
}

// ------------------------------------------------ tiled grid
//
// The grid is stored in up to three levels: a directory of tiles of 2^tl
// cells a side, for mixed tiles a sub-directory of sub-tiles of 2^sl cells a
// side (sl < tl), and for mixed sub-tiles (or mixed tiles when sl == tl) a
// fine block of one code per cell.  A uniform square stores its code once.

// 16-bit short code of a cell code: 0 none, p+1 polygon p, np+1+k set k
__device__ __forceinline__ uint32_t short_code(uint32_t c, uint32_t np)
{
    return c < CODE_SET_BASE ? c : np + 1 + (c - CODE_SET_BASE);
}

// origin (first column, first row) of square u: a tile (mt == NULL), or
// sub-tile u % Q of mixed tile mt[u / Q]
__device__ __forceinline__ void square_origin(int64_t u, const int64_t *mt, int tl, int sl,
                                              int64_t tw, int32_t *x0, int64_t *r0)
{
    if (!mt) {
        *x0 = (int32_t)((u % tw) << tl);
        *r0 = (u / tw) << tl;
        return;
    }
    const int qs = tl - sl;  // sub-tiles per tile side: 2^qs
    int64_t q = u & (((int64_t)1 << (2 * qs)) - 1);
    int64_t tile = mt[u >> (2 * qs)];
    *x0 = (int32_t)(((tile % tw) << tl) + ((q & (((int64_t)1 << qs) - 1)) << sl));
    *r0 = ((tile / tw) << tl) + ((q >> qs) << sl);
}

// G lanes per square (G = min(side, 64)): uniform code of the square, or
// 0xffffffff and mixed[u] = 1
template <int G>
__global__ void k_square_classify(const int64_t *seg_beg, const int64_t *seg_end,
                                  const int32_t *seg_x0, const int32_t *seg_x1,
                                  const uint32_t *seg_code, int64_t gw,
                                  int64_t gh, const int64_t *mt, int tl, int sl, int64_t tw,
                                  int64_t n_sq, uint32_t *code, int64_t *mixed)
{
    int64_t u = ((int64_t)xcd_block() * blockDim.x + threadIdx.x) / G;
    int lane = threadIdx.x & (G - 1);
    if (u >= n_sq) return;  // whole groups leave together (G divides the block)
    const int side_log2 = mt ? sl : tl;
    int32_t x0;
    int64_t r0;
    square_origin(u, mt, tl, sl, tw, &x0, &r0);
    int32_t x1 = (int32_t)min((int64_t)x0 + (1 << side_log2), gw);
    int64_t r1 = min(r0 + (1 << side_log2), gh);
    uint32_t lo_c = 0xffffffffu, hi_c = 0;
    if (x0 >= gw || r0 >= gh) {  // square wholly outside the stored box
        lo_c = hi_c = 0;
    }
    for (int64_t r = r0 + lane; r < r1 && x0 < gw; r += G) {
        int64_t a = seg_beg[r], lo = a, hi = seg_end[r], e = hi;
        while (lo < hi) {
            int64_t mid = (lo + hi) >> 1;
            if (seg_x0[mid] <= x0) lo = mid + 1; else hi = mid;
        }
        uint32_t c;
        if (lo > a && x0 < seg_x1[lo - 1]) {
            c = (seg_x1[lo - 1] >= x1) ? seg_code[lo - 1] : 0xffffffffu;
        } else {
            c = (lo >= e || seg_x0[lo] >= x1) ? 0u : 0xffffffffu;
        }
        lo_c = min(lo_c, c);
        hi_c = max(hi_c, c);
    }
    // a square cut by the edge of the box is uniform only if its stored part
    // is; cells beyond the box read as 0 through the probe's range test
    for (int o = G / 2; o > 0; o >>= 1) {
        lo_c = min(lo_c, (uint32_t)__shfl_xor((int)lo_c, o, 64));
        hi_c = max(hi_c, (uint32_t)__shfl_xor((int)hi_c, o, 64));
    }
    if (lane == 0) {
        bool uni = (lo_c == hi_c) && (hi_c != 0xffffffffu);
        code[u] = uni ? hi_c : 0xffffffffu;
        mixed[u] = uni ? 0 : 1;
    }
}

// The same for big tiles (2^tl >= 64 cells): a workgroup takes regions of 2^tl
// rows and Q squares side by side -- the sub-tiles of a mixed tile (mt), or 16
// tiles of a tile row -- 256 rows at a time.  Each row is searched once for the
// region's first cell, a lane a row, its next SQ_WIN segments go to LDS, and
// the squares find theirs there (rows with more segments in the region fall
// back to a search in memory).  What bounds it is those searches' and windows'
// lines from beyond the L2, so neighbouring regions go to one XCD.  49,000 tiles
// of 256 x 256 cells and 1.95M sub-tiles of 16 x 16 over 56,590 rows: 245 and 295
// us with a search in memory for every row of every square; 114 and 132 with one
// a row and region; 79 and 109 with regions in order on each XCD (windows of 8:
// 78 and 151).
#define SQ_WIN 4
#define SQ_MAX 2048   // squares of a workgroup
#define SQ_Q 16       // tiles side by side of one region

struct SquareGeo {
    const int64_t *seg_beg, *seg_end;
    const int32_t *seg_x0, *seg_x1;
    const uint32_t *seg_code;
    int64_t gw, gh, tw, th;
    const int64_t *mt;
    int tl, sl;
    int qlog;        // log2 of the squares side by side in a region
    int64_t regions; // mixed tiles, or tile rows times groups of tiles
};

__global__ __launch_bounds__(256) void k_squares(SquareGeo G, uint32_t *code, int64_t *mixed)
{
    __shared__ int32_t wx0[256][SQ_WIN + 1], wx1[256][SQ_WIN + 1];
    __shared__ uint32_t wcode[256][SQ_WIN + 1];
    __shared__ int64_t sfirst[256], send[256];
    extern __shared__ uint32_t sq_lds[];
    const uint32_t block = xcd_block();
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int rows = 1 << G.tl, side = G.mt ? G.sl : G.tl;
    const int Q = 1 << G.qlog, strips = rows >> side;
    const int rpb = rows < 256 ? 256 >> G.tl : 1;       // regions of a workgroup
    const int nsq = rpb * strips << G.qlog;
    const uint32_t groups = (uint32_t)((G.tw + SQ_Q - 1) / SQ_Q);
    uint32_t *lo_s = sq_lds, *hi_s = sq_lds + nsq;
    for (int k = tid; k < nsq; k += 256) {
        lo_s[k] = 0xffffffffu;
        hi_s[k] = 0;
    }
    // first cell and row of region g of the workgroup
    // (tiles and regions are fewer than 2^31, rows and columns at most 2^21)
    auto origin = [&](int g, int32_t *x0, int32_t *r0) {
        const uint32_t k = block * (uint32_t)rpb + (uint32_t)g;
        if (k >= (uint32_t)G.regions) {
            *x0 = (int32_t)G.gw;
            *r0 = (int32_t)G.gh;
            return false;
        }
        const uint32_t t = G.mt ? (uint32_t)G.mt[k] : k, m = G.mt ? (uint32_t)G.tw : groups;
        const uint32_t ty = t / m, tx = t - ty * m;
        *x0 = (int32_t)((G.mt ? tx : tx * SQ_Q) << G.tl);
        *r0 = (int32_t)(ty << G.tl);
        return true;
    };
    for (int c0 = 0; c0 < (rows < 256 ? 256 : rows); c0 += 256) {
        __syncthreads();
        {   // each lane a row: its last segment at or before the region's first cell
            const int g = rows < 256 ? tid >> G.tl : 0;
            int32_t X, R;
            origin(g, &X, &R);
            const int32_t r = R + (rows < 256 ? tid & (rows - 1) : c0 + tid);
            int64_t a = 0, e = 0;
            if (r < G.gh && X < G.gw) {
                a = G.seg_beg[r];
                e = G.seg_end[r];
                int64_t lo = a, hi = e;
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (G.seg_x0[mid] <= X) lo = mid + 1; else hi = mid;
                }
                a = lo > a ? lo - 1 : a;
            }
            sfirst[tid] = a;
            send[tid] = e;
        }
        __syncthreads();
        for (int k = tid; k < 256 * SQ_WIN; k += 256) {
            const int row = k / SQ_WIN, u = k % SQ_WIN;
            const int64_t t = sfirst[row] + u;
            const bool in = t < send[row];
            wx0[row][u] = in ? G.seg_x0[t] : INT32_MAX;
            wx1[row][u] = in ? G.seg_x1[t] : 0;
            wcode[row][u] = in ? G.seg_code[t] : 0u;
        }
        __syncthreads();
        // a wavefront takes 64 rows, 64 / Q a pass, a lane a square
        const int q = lane & (Q - 1), rw = 64 >> G.qlog;
        const int g = rows < 256 ? (w * 64) >> G.tl : 0;
        int32_t X, R;
        origin(g, &X, &R);
        const int32_t gw = (int32_t)G.gw, gh = (int32_t)G.gh;
        const int32_t cx0 = X + (q << side), cx1 = min(cx0 + (1 << side), gw);
        const int rin = (rows < 256 ? (w * 64) & (rows - 1) : c0 + w * 64);  // in the region
        uint32_t lo_c = 0xffffffffu, hi_c = 0;
        for (int p = 0; p < 64; p += rw) {
            const int y = p + (lane >> G.qlog), row = w * 64 + y;
            if (R + rin + y < gh && cx0 < gw) {
                // segments of the window that start at or before the square
                int n = 0;
#pragma unroll
                for (int b = SQ_WIN / 2; b > 0; b >>= 1)
                    if (wx0[row][n + b - 1] <= cx0) n += b;
                if (wx0[row][n] <= cx0) n++;
                uint32_t c;
                if (n == SQ_WIN && sfirst[row] + SQ_WIN < send[row]) {
                    const int64_t e = send[row];
                    int64_t lo = sfirst[row] + SQ_WIN, hi = e;
                    while (lo < hi) {
                        const int64_t mid = (lo + hi) >> 1;
                        if (G.seg_x0[mid] <= cx0) lo = mid + 1; else hi = mid;
                    }
                    if (cx0 < G.seg_x1[lo - 1])
                        c = G.seg_x1[lo - 1] >= cx1 ? G.seg_code[lo - 1] : 0xffffffffu;
                    else
                        c = (lo >= e || G.seg_x0[lo] >= cx1) ? 0u : 0xffffffffu;
                } else if (n > 0 && cx0 < wx1[row][n - 1]) {
                    c = wx1[row][n - 1] >= cx1 ? wcode[row][n - 1] : 0xffffffffu;
                } else {
                    c = (n == SQ_WIN || wx0[row][n] >= cx1) ? 0u : 0xffffffffu;
                }
                lo_c = min(lo_c, c);
                hi_c = max(hi_c, c);
            }
            if (((rin + p + rw) & ((1 << side) - 1)) == 0 || p + rw == 64) {  // the strip ends
                for (int o = 32; o >= Q; o >>= 1) {
                    lo_c = min(lo_c, (uint32_t)__shfl_xor((int)lo_c, o, 64));
                    hi_c = max(hi_c, (uint32_t)__shfl_xor((int)hi_c, o, 64));
                }
                if (lane < Q) {
                    const int k = ((g * strips + ((rin + p) >> side)) << G.qlog) + q;
                    atomicMin(&lo_s[k], lo_c);
                    atomicMax(&hi_s[k], hi_c);
                }
                lo_c = 0xffffffffu;
                hi_c = 0;
            }
        }
    }
    __syncthreads();
    for (int k = tid; k < nsq; k += 256) {
        const int q = k & (Q - 1), strip = (k >> G.qlog) & (strips - 1);
        const int g = k >> (G.qlog + G.tl - side);
        int32_t X, R;
        if (!origin(g, &X, &R)) continue;
        const int32_t x0 = X + (q << side), r0 = R + (strip << side);
        int64_t u;
        if (G.mt) {
            u = (((int64_t)block * rpb + g) << (2 * G.qlog)) +
                (k & ((strips << G.qlog) - 1));
        } else {
            if ((x0 >> G.tl) >= G.tw) continue;  // past the row's last tile
            u = (int64_t)(r0 >> G.tl) * G.tw + (x0 >> G.tl);
        }
        uint32_t lo_c = lo_s[k], hi_c = hi_s[k];
        if (x0 >= G.gw || r0 >= G.gh) lo_c = hi_c = 0;  // wholly outside the stored box
        const bool uni = lo_c == hi_c && hi_c != 0xffffffffu;
        code[u] = uni ? hi_c : 0xffffffffu;
        mixed[u] = uni ? 0 : 1;
    }
}

// list[pos[u]] = u for every flagged u (pos = exclusive scan of the flags)
__global__ void k_flag_list(const int64_t *pos, int64_t n, int64_t total, int64_t *list)
{
    int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    int64_t o = pos[u], o1 = u + 1 < n ? pos[u + 1] : total;
    if (o1 != o) list[o] = u;
}

// Fine blocks: one thread per (block, row, run of up to 16 cells): one
// binary search for the run's first cell, then a walk along the row's
// segments.  Block k holds square sq[k] of side 2^side_log2 (sq indexes the
// squares of k_square_classify).  OUT = uint32_t full codes or uint16_t
// short codes.
template <typename OUT>
__global__ __launch_bounds__(256) void k_block_fill(const int64_t *seg_beg, const int64_t *seg_end,
                             const int32_t *seg_x0, const int32_t *seg_x1, const uint32_t *seg_code, int64_t gw,
                             int64_t gh, const int64_t *sq, int64_t nblk, const int64_t *mt,
                             int tl, int sl, int64_t tw, int side_log2, uint32_t np, OUT *blocks)
{
    const int side = 1 << side_log2;
    const int runs = side > 16 ? side >> 4 : 1;
    const int rlen = side > 16 ? 16 : side;
    int64_t t = (int64_t)xcd_block() * 256 + threadIdx.x;
    if (t >= nblk * side * runs) return;
    int64_t k = t / ((int64_t)side * runs);
    int rem = (int)(t - k * side * runs);
    int row = rem / runs, run = rem - row * runs;
    int32_t x0;
    int64_t r0;
    square_origin(sq[k], mt, tl, sl, tw, &x0, &r0);
    OUT *out = blocks + (k << (2 * side_log2)) + ((int64_t)row << side_log2) + run * rlen;
    int64_t r = r0 + row;
    int32_t xa = x0 + run * rlen;
    if (r >= gh) {
        for (int c = 0; c < rlen; c++) out[c] = 0;
        return;
    }
    const int64_t lo = seg_beg[r], hi = seg_end[r];
    int64_t a = lo, e = hi;
    while (a < e) {
        int64_t mid = (a + e) >> 1;
        if (seg_x0[mid] <= xa) a = mid + 1; else e = mid;
    }
    const int64_t q0 = a - 1;  // last segment starting at or before xa (lo-1 if none)
    // the run's codes go to registers first and leave in 16-byte stores (a
    // run starts at a multiple of 16 bytes: blocks and rows are multiples of
    // 8 bytes long and runs of 16 codes are 32 or 64 bytes)
    OUT buf[16] __attribute__((aligned(16)));
    // Segments q0 .. q0 + 3 are loaded at once (no chain of dependent loads
    // along the row); they cover the run unless segment q0 + 4 starts inside
    // it, and then the run walks the row's segments one by one.  Segments of
    // a row are disjoint, so at most one holds a cell.
    constexpr int W = 4;
    int32_t wx0[W], wx1[W];
    uint32_t wc[W];
#pragma unroll
    for (int j = 0; j < W; j++) {
        const int64_t q = q0 + j;
        const bool in = q >= lo && q < hi;
        wx0[j] = in ? seg_x0[q] : INT32_MAX;
        wx1[j] = in ? seg_x1[q] : INT32_MIN;
        wc[j] = in ? seg_code[q] : 0u;
    }
    if (!(q0 + W < hi && seg_x0[q0 + W] < xa + rlen)) {
#pragma unroll
        for (int c = 0; c < 16; c++) {
            if (c >= rlen) break;
            const int32_t x = xa + c;
            uint32_t v = 0;
#pragma unroll
            for (int j = 0; j < W; j++) v = (wx0[j] <= x && x < wx1[j]) ? wc[j] : v;
            if (x >= gw) v = 0;
            buf[c] = sizeof(OUT) == 2 ? (OUT)short_code(v, np) : (OUT)v;
        }
    } else {
        int64_t q = q0;
#pragma unroll
        for (int c = 0; c < 16; c++) {
            if (c >= rlen) break;
            int32_t x = xa + c;
            while (q + 1 < hi && seg_x0[q + 1] <= x) q++;
            uint32_t v = 0;
            if (x < gw && q >= lo && x < seg_x1[q]) v = seg_code[q];
            buf[c] = sizeof(OUT) == 2 ? (OUT)short_code(v, np) : (OUT)v;
        }
    }
    // constant indices only, so buf stays in registers (a dynamically
    // indexed array would be moved to LDS, which the kernel then reserves)
    const int bytes = rlen * (int)sizeof(OUT);
    if (bytes % 16 == 0) {
        uint4 *o4 = (uint4 *)out;
        const uint4 *b4 = (const uint4 *)buf;
#pragma unroll
        for (int k = 0; k < (int)sizeof(OUT); k++)  // 16 codes = sizeof(OUT) x 16 bytes
            if (k < bytes / 16) o4[k] = b4[k];
    } else {
#pragma unroll
        for (int c = 0; c < 16; c++)
            if (c < rlen) out[c] = buf[c];
    }
}

// final directory / sub-directory entries: the square's code (short codes
// in the compact format), or TILE_MIXED | index of its fine block or
// sub-directory.  Compact directory entries are 16-bit: 0x8000 | index.
__global__ void k_entries(const uint32_t *code, const int64_t *pos, int64_t n, int64_t n_pad,
                          uint32_t np, int mode, uint32_t *out32, uint16_t *out16)
{
    int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n_pad) return;
    if (u >= n) { out16[u] = 0; return; }  // padding exists only in mode 2
    uint32_t c = code[u];
    bool mixed = c == 0xffffffffu;
    uint32_t idx = (uint32_t)pos[u];
    if (mode == 0) out32[u] = mixed ? (TILE_MIXED | idx) : c;                   // wide
    else if (mode == 1) out32[u] = mixed ? (TILE_MIXED | idx) : short_code(c, np);  // compact sub
    else out16[u] = (uint16_t)(mixed ? (0x8000u | idx) : short_code(c, np));   // compact dir
}

// Scan, entries, list and read-back in one launch for up to NUMBER_MAX squares:
// the mixed squares numbered in order, their total to *tot, list[number] =
// square, and the entries as k_entries writes them (nothing in mode 2 when the
// numbers do not fit 16 bits).  Each workgroup takes NUMBER_TILE squares and
// counts the mixed ones among all by itself (at most 256 KB, read from the L2),
// so none waits for another, and the first can send the total to the host.
// (One workgroup for all squares was bound by its instructions: 25 us for
// 48,000; this way 9.  As five launches, tile sums, their scan, entries, list and read-back,
// the kernels took 16 us and the gaps between them as much.)
#define NUMBER_MAX 65536
#define NUMBER_BLOCK 256
#define NUMBER_PER 8
#define NUMBER_TILE (NUMBER_BLOCK * NUMBER_PER)
__global__ __launch_bounds__(NUMBER_BLOCK) void k_number(const uint32_t *__restrict__ code, int n,
                                                         int n_pad, uint32_t np, int mode,
                                                         uint32_t *__restrict__ out32,
                                                         uint16_t *__restrict__ out16,
                                                         int64_t *__restrict__ list, int64_t *tot,
                                                         ReadSet R)
{
    constexpr int WAVES = NUMBER_BLOCK / 64;
    __shared__ uint32_t sb[WAVES], sa[WAVES], sc[WAVES];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int start = (int)blockIdx.x * NUMBER_TILE;
    uint32_t c[NUMBER_PER], cnt = 0;
#pragma unroll
    for (int k = 0; k < NUMBER_PER; k++) {
        const int u = start + (w * NUMBER_PER + k) * 64 + lane;
        c[k] = u < n ? code[u] : 0u;
    }
    // four codes a load; start is a multiple of four
    const uint4 *c4 = (const uint4 *)code;
    auto count = [&](int a, int b) {
        uint32_t m = 0;
#pragma unroll 8
        for (int t = a + (int)threadIdx.x; t < b; t += NUMBER_BLOCK) {
            const uint4 v = c4[t];
            m += (v.x == 0xffffffffu) + (v.y == 0xffffffffu) + (v.z == 0xffffffffu) +
                 (v.w == 0xffffffffu);
        }
        return m;
    };
    const int s4 = min(start, n) >> 2, n4 = n >> 2;
    uint32_t before = count(0, s4), after = count(s4, n4);
    if ((int)threadIdx.x < (n & 3)) {  // the last one to three, not before any start
        const bool m = code[4 * n4 + threadIdx.x] == 0xffffffffu;
        if (4 * n4 < start) before += m;
        else after += m;
    }
    for (int o = 32; o > 0; o >>= 1) {
        before += (uint32_t)__shfl_xor((int)before, o, 64);
        after += (uint32_t)__shfl_xor((int)after, o, 64);
    }
#pragma unroll
    for (int k = 0; k < NUMBER_PER; k++) cnt += (uint32_t)__popcll(__ballot(c[k] == 0xffffffffu));
    if (lane == 0) {
        sb[w] = before;
        sa[w] = after;
        sc[w] = cnt;
    }
    __syncthreads();
    uint32_t at = 0, all = 0;
#pragma unroll
    for (int k = 0; k < WAVES; k++) {
        at += sb[k] + (k < w ? sc[k] : 0u);
        all += sb[k] + sa[k];
    }
    const bool entries = mode != 2 || all < 0x8000u;
#pragma unroll
    for (int k = 0; k < NUMBER_PER; k++) {
        const int u = start + (w * NUMBER_PER + k) * 64 + lane;
        const bool mixed = c[k] == 0xffffffffu;
        const uint64_t m = __ballot(mixed);
        const uint32_t idx = at + (uint32_t)__popcll(m & ((1ull << lane) - 1));
        at += (uint32_t)__popcll(m);
        if (mixed) list[idx] = u;
        if (!entries || u >= n_pad) continue;
        if (mode == 0) out32[u] = mixed ? (TILE_MIXED | idx) : c[k];
        else if (mode == 1) out32[u] = mixed ? (TILE_MIXED | idx) : short_code(c[k], np);
        else out16[u] = (uint16_t)(mixed ? (0x8000u | idx) : short_code(c[k], np));
    }
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) *tot = all;
        read_back(R);
    }
}

// ---------------------------------------------------------------- host side

void magic_for(int64_t s, uint32_t *mag, int32_t *shift)
{
    int l = 0;
    while (((int64_t)1 << l) < s) l++;  // l = ceil(log2 s)
    // m = ceil(2^(31+l) / s)
    unsigned __int128 num = (unsigned __int128)1 << (31 + l);
    uint64_t m = (uint64_t)((num + (unsigned __int128)(s - 1)) / (unsigned __int128)s);
    *mag = (uint32_t)m;  // < 2^32 (== 2^31 for s == 1)
    *shift = 31 + l;
}

static unsigned box_grid(int32_t np)
{
    return std::min<unsigned>(grid_for((int64_t)np * 64, BOX_BLOCK), BOX_GRID);
}

int pool_setup()
{
    static bool done[64] = {false};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return SBA_EDEVICE;
    if (done[dev]) return 0;
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, dev) != hipSuccess) {
        (void)hipGetLastError();
        return SBA_EDEVICE;
    }
    uint64_t keep = ~0ull;
    if (hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess) {
        (void)hipGetLastError();
        return SBA_EDEVICE;
    }
    done[dev] = true;
    return 0;
}

// Hilbert key grid covering the cell boxes of several polygon sets: each
// set's offsets are checked and its union cell box found by the kernels of
// the build (k_check_rings, k_check_verts, k_poly_bbox); the
// grid is anchored at the first cell of the union of the boxes and has the
// smallest level L >= 1 with 2^L cells covering the union's longer side,
// the level the Hilbert layout takes for a stored box of that size.
int key_grid_launch(const sba_polygons *sets, int32_t n_sets, int64_t eps, hipStream_t st,
                    int32_t *level, int64_t *i0, int64_t *j0)
{
    const int64_t s = cell_side(eps);
    constexpr int SLOTS = 8;  // per set: [0] error bits, [1..2] sizes, [3..6] cell box
    Workspace ws(st);
    int64_t *sc = nullptr;
    RC(ws.alloc(&sc, (int64_t)n_sets * SLOTS));
    HIP_OK(hipMemsetAsync(sc, 0, sizeof(int64_t) * SLOTS * n_sets, st));
    std::vector<int4 *> bbox(n_sets, nullptr);
    for (int32_t k = 0; k < n_sets; k++) {
        const sba_polygons &P = sets[k];
        const int32_t np = P.n_polys;
        if (np == 0) continue;
        int *err = (int *)(sc + SLOTS * k);
        int64_t *sizes = sc + SLOTS * k + 1, *dbox = sc + SLOTS * k + 3;
        hipLaunchKernelGGL(k_check_rings, dim3(grid_for(np + 1)), dim3(256), 0, st, P.ring_off, np,
                           sizes, err);
        hipLaunchKernelGGL(k_check_verts, dim3(1024), dim3(256), 0, st, P.vert_off, sizes, err);
        RC(ws.alloc(&bbox[k], np));
        int32_t *part = nullptr;
        RC(ws.alloc(&part, 4 * BOX_GRID));
        hipLaunchKernelGGL(k_poly_bbox, dim3(box_grid(np)), dim3(BOX_BLOCK), 0, st,
                           P.ring_off, P.vert_off, P.xy, np, s, bbox[k], part, err, dbox,
                           (unsigned long long *)(sc + SLOTS * k + 7), ReadSet{});
        HIP_OK(hipGetLastError());
    }
    std::vector<int64_t> hsc((size_t)SLOTS * n_sets);
    RC(ws.read(hsc.data(), sc, sizeof(int64_t) * SLOTS * n_sets));
    RC(ws.sync());
    bool any = false;
    int64_t bi0 = 0, bj0 = 0, bi1 = 0, bj1 = 0;
    for (int32_t k = 0; k < n_sets; k++) {
        if (sets[k].n_polys == 0) continue;
        const int64_t *v = hsc.data() + SLOTS * k;
        const int herr = (int)(uint32_t)v[0];
        if (herr & 2) return SBA_EINVAL;
        if (herr & 1) return SBA_ERANGE;
        bi0 = any ? std::min(bi0, v[3]) : v[3];
        bj0 = any ? std::min(bj0, v[4]) : v[4];
        bi1 = any ? std::max(bi1, v[5]) : v[5];
        bj1 = any ? std::max(bj1, v[6]) : v[6];
        any = true;
    }
    if (!any) return SBA_EINVAL;
    const int64_t side = std::max(bi1 - bi0 + 1, bj1 - bj0 + 1);
    int L = 1;
    while (L <= 21 && ((int64_t)1 << L) < side) L++;
    if (L > 21) return SBA_ELIMIT;
    *level = L;
    *i0 = bi0;
    *j0 = bj0;
    return 0;
}

// paths of the coverage stages: bits set in g_build_paths_off turn a path
// off (1: the pairs of edges and rows counted per row, 2: the rows swept in
// LDS, 4: the set table through a hash); the last build's paths taken, same
// bits (tests of both sides of each choice)
static std::atomic<int> g_build_paths_off{0}, g_build_paths_last{0};

extern "C" int sba_debug_build_paths(int off)
{
    if (off < 0 || off > 7) return SBA_EINVAL;
    g_build_paths_off = off;
    return 0;
}

extern "C" int sba_debug_last_build_paths(void) { return g_build_paths_last.load(); }

int build_segments(const sba_polygons *polys, int64_t eps, hipStream_t st, sba_handle *h,
                   BuildState &B, bool need_boundary_cells)
{
    (void)need_boundary_cells;
    const int32_t np = polys->n_polys;
    // device scalars read back together (one copy per synchronisation):
    // [0] error bits (int), [1..2] ring and vertex counts, [3..6] union cell
    // box, [8..13] totals of the scans
    RC(B.alloc(&B.sc, SC_SLOTS));
    int *err = (int *)B.sc;
    int64_t *sizes = B.sc + 1, *dbox = B.sc + 3, *tot = B.sc + 8;
    int64_t hsc[SC_READ];
    auto fetch = [&]() -> int {
        RC(B.ws.read(hsc, B.sc, sizeof(hsc)));
        return B.ws.sync();
    };

    // validate the offsets on the device (each stage reads only what the
    // previous one validated) and read sizes and bounding boxes in one sync
    if (np <= CHECK_POLYS) {
        hipLaunchKernelGGL(k_check_offsets, dim3(1), dim3(1024), 0, st, polys->ring_off,
                           polys->vert_off, np, B.sc, SC_SLOTS);
    } else {
        HIP_OK(hipMemsetAsync(B.sc, 0, sizeof(int64_t) * SC_SLOTS, st));
        hipLaunchKernelGGL(k_check_rings, dim3(grid_for(np + 1)), dim3(256), 0, st,
                           polys->ring_off, np, sizes, err);
        hipLaunchKernelGGL(k_check_verts, dim3(1024), dim3(256), 0, st, polys->vert_off, sizes, err);
    }
    HIP_OK(hipGetLastError());
    int4 *bbox = nullptr;
    int32_t *part = nullptr;
    RC(B.alloc(&bbox, np));
    RC(B.alloc(&part, 4 * BOX_GRID));
    RC(B.ws.read(hsc, B.sc, sizeof(hsc)));
    hipLaunchKernelGGL(k_poly_bbox, dim3(box_grid(np)), dim3(BOX_BLOCK), 0, st,
                       polys->ring_off, polys->vert_off, polys->xy, np, h->s, bbox, part, err, dbox,
                       (unsigned long long *)(B.sc + SC_TICKET), B.ws.reads());
    HIP_OK(hipGetLastError());
    RC(B.ws.wait());
    int herr = (int)(uint32_t)hsc[0];
    if (herr & 2) return SBA_EINVAL;
    if (herr & 1) return SBA_ERANGE;
    const int32_t nr = (int32_t)hsc[1];
    const int64_t nv = hsc[2];
    if (nv > ((int64_t)1 << 31) - 1) return SBA_ELIMIT;
    const int64_t s = h->s;
    int64_t gi0 = hsc[3], gj0 = hsc[4], gi1 = hsc[5], gj1 = hsc[6];
    if (B.window) {
        gi0 = std::max(gi0, floordiv64(B.wx0, s));
        gj0 = std::max(gj0, floordiv64(B.wy0, s));
        gi1 = std::min(gi1, floordiv64(B.wx1 - 1, s));
        gj1 = std::min(gj1, floordiv64(B.wy1 - 1, s));
        if (gi0 > gi1 || gj0 > gj1) {  // nothing of any polygon inside the window
            h->gi0 = h->gj0 = 0;
            h->gw = h->gh = 0;
            B.empty = true;
            return 0;
        }
    }
    if (B.key_level > 0) {
        // a given key grid: cells outside it are cut off (at the grid's own
        // edges, which the curve never crosses, so no border keys are
        // needed), and the stored box starts at the grid's first cell
        const int64_t side = (int64_t)1 << B.key_level;
        gi0 = std::max(gi0, B.key_i0);
        gj0 = std::max(gj0, B.key_j0);
        gi1 = std::min(gi1, B.key_i0 + side - 1);
        gj1 = std::min(gj1, B.key_j0 + side - 1);
        if (gi0 > gi1 || gj0 > gj1) {
            h->gi0 = h->gj0 = 0;
            h->gw = h->gh = 0;
            B.empty = true;
            return 0;
        }
        gi0 = B.key_i0;
        gj0 = B.key_j0;
    }
    h->gi0 = gi0;
    h->gj0 = gj0;
    h->gw = gi1 - gi0 + 1;
    h->gh = gj1 - gj0 + 1;
    if (h->gw > MAX_GRID_SIDE || h->gh > MAX_GRID_SIDE) return SBA_ELIMIT;
    if (h->gw * s >= ((int64_t)1 << 31) || h->gh * s >= ((int64_t)1 << 31)) return SBA_ELIMIT;
    const int64_t gw = h->gw, gh = h->gh;
    B.xbits = bits_for((uint64_t)gw);
    B.rbits = bits_for((uint64_t)(gh - 1));
    if (B.rbits < 1) B.rbits = 1;
    const int pbits = bits_for((uint64_t)(np - 1)) < 1 ? 1 : bits_for((uint64_t)(np - 1));

    // 1-4 row by row in LDS (rows.hip) unless a row is too large for that
    const int paths_off = g_build_paths_off.load();
    g_build_paths_last = 0;
    if (!(paths_off & 1)) {
        bool taken = false, one = false;
        RC(rows_coverage(polys, bbox, nv, st, h, B, paths_off, &taken, &one));
        g_build_paths_last = 1 | (taken ? 2 : 0) | (one ? 4 : 0);
        if (taken) return h->n_sets >= (int64_t)(TILE_MIXED - CODE_SET_BASE) ? SBA_ELIMIT : 0;
    }
    B.n_edges = nv;
    RC(B.alloc(&B.edges, nv));
    RC(B.alloc(&B.epoly, nv));
    hipLaunchKernelGGL(k_edges, dim3(grid_for(nv)), dim3(256), 0, st, polys->ring_off, np,
                       polys->vert_off, nr, polys->xy, nv, B.edges, B.epoly);
    HIP_OK(hipGetLastError());

    // 1-2: boundary intervals and crossings per edge
    int64_t *nb = nullptr, *nc = nullptr;
    RC(B.alloc(&nb, nv + 1));
    RC(B.alloc(&nc, nv + 1));
    hipLaunchKernelGGL(k_edge_counts, dim3(grid_for(nv)), dim3(256), 0, st, B.edges, B.epoly, bbox,
                       nv, s, gi0, gj0, gi1, gj1, B.centre ? 1 : 0, nb, nc);
    HIP_OK(hipGetLastError());
    {
        const int64_t *in[2] = {nb, nc}, n[2] = {nv, nv};
        int64_t *out[2] = {nb, nc}, *sum[2] = {tot, tot + 1};
        RC(scan_exclusive_i64_multi(2, in, out, n, sum, st, &B.ws));
    }
    RC(fetch());
    // boundary-only approximations take no row-line crossings (no interior
    // spans); centre-sampled ones no boundary cells, except as the Hilbert
    // layout's candidate keys (where the cell sets can change along the curve)
    const bool need_b = !B.centre || B.on_boundary_events;
    const int64_t NB = need_b ? hsc[8] : 0, NC = B.boundary_only ? 0 : hsc[9];
    if (NC % 2) return SBA_EDEVICE;
    h->n_boundary = NB;
    B.NB = NB;
    const int64_t NB_cov = B.centre ? 0 : NB;  // boundary intervals in the coverage
    int64_t NE = 2 * NB + NC;
    if (NE >= ((int64_t)1 << 32)) return SBA_ELIMIT;
    RC(B.alloc(&B.evkey, NE));
    RC(B.alloc(&B.evpay, NE));
    uint64_t *ckey = B.evkey + 2 * NB;
    uint32_t *cpay = B.evpay + 2 * NB;
    if (B.centre && NB) {  // crossings in arrays of their own, coverage input alone
        RC(B.alloc(&ckey, std::max<int64_t>(NC, 1)));
        RC(B.alloc(&cpay, std::max<int64_t>(NC, 1)));
    }
    if (NB)
        hipLaunchKernelGGL(k_emit_boundary, dim3(grid_for(NB)), dim3(256), 0, st, B.edges, B.epoly,
                           nv, nb, NB, s, gi0, gj0, gi1, B.xbits, B.rbits, B.evkey, B.evpay);
    if (NC)
        hipLaunchKernelGGL(k_emit_cross, dim3(grid_for(NC)), dim3(256), 0, st, B.edges, B.epoly, nv,
                           nc, NC, s, gi0, gj0, gi1, B.centre ? 1 : 0, B.xbits, B.rbits, ckey,
                           cpay);
    HIP_OK(hipGetLastError());

    // the Hilbert layout needs the boundary cells before the events are sorted
    if (B.on_boundary_events) RC(B.on_boundary_events(B, h, st));
    if (B.centre && NB) {
        B.release(B.evkey);
        B.release(B.evpay);
        B.evkey = ckey;
        B.evpay = cpay;
    }
    NE = 2 * NB_cov + NC;
    // 3: coverage.  Events by (polygon, row, x); one scan gives every
    // polygon's coverage count at every event, whose changes (toggles) are
    // the maximal covered intervals of each polygon in each row.
    const int rxbits = B.rbits + B.xbits;
    int64_t NT = 0;
    uint64_t *tkey = nullptr, *E = nullptr;
    int32_t *tpoly = nullptr;
    int64_t *tf = nullptr;
    B.release(nb);
    B.release(nc);
    RC(radix_sort_u64_ws(&B.evkey, &B.evpay, NE, pbits + rxbits, B.ws));
    int64_t *cex = nullptr;
    RC(B.alloc(&cex, NE));
    RC(B.alloc(&tf, NE));
    hipLaunchKernelGGL(k_ev_values, dim3(grid_for(NE)), dim3(256), 0, st, B.evpay, NE, cex);
    HIP_OK(hipGetLastError());
    RC(scan_exclusive_i64(cex, cex, NE, tot, st, &B.ws));
    hipLaunchKernelGGL(k_toggle_flags, dim3(grid_for(NE)), dim3(256), 0, st, B.evkey,
                       B.evpay, cex, NE, B.xbits, tf, err);
    HIP_OK(hipGetLastError());
    RC(scan_exclusive_i64(tf, tf, NE, tot, st, &B.ws));
    RC(fetch());
    NT = hsc[8];
    herr = (int)(uint32_t)hsc[0];
    if (herr || (NT & 1)) return SBA_EDEVICE;
    B.release(cex);
    RC(B.alloc(&tkey, std::max<int64_t>(NT, 1)));
    RC(B.alloc(&tpoly, std::max<int64_t>(NT, 1)));
    hipLaunchKernelGGL(k_toggle_emit, dim3(grid_for(NE)), dim3(256), 0, st, B.evkey, tf, NE,
                       NT, rxbits, tkey, tpoly);
    HIP_OK(hipGetLastError());
    B.release(tf);
    B.release(B.evkey);
    B.evkey = nullptr;
    B.release(B.evpay);
    B.evpay = nullptr;

    // 4: elementary pieces between distinct toggle positions of a row, their
    // depth, and the polygons of each piece
    const int64_t NI = NT / 2;                     // covered intervals
    const int64_t NP = std::max<int64_t>(NT, 1);   // pieces (upper bound)
    int64_t *pos = nullptr, *ika = nullptr, *xoff = nullptr, *diff = nullptr, *dex = nullptr;
    int64_t *segc = nullptr, *mm = nullptr;
    RC(B.alloc(&E, NP));
    RC(B.alloc(&pos, NP));
    RC(B.alloc(&ika, std::max<int64_t>(NI, 1)));
    RC(B.alloc(&xoff, std::max<int64_t>(NI, 1)));
    RC(B.alloc(&diff, NP + 1));
    RC(B.alloc(&dex, NP));
    RC(B.alloc(&segc, NP));
    RC(B.alloc(&mm, NP));
    if (NT == 0) HIP_OK(hipMemsetAsync(diff, 0, sizeof(int64_t) * (NP + 1), st));
    if (NT) {
        if (NT >= ((int64_t)1 << 32)) return SBA_ELIMIT;
        // sorted with each toggle's slot as payload, so that every toggle
        // learns its index in E without a search (the toggle keys are not
        // needed in slot order afterwards)
        uint32_t *src = nullptr;
        int64_t *rank = nullptr;
        RC(B.alloc(&src, NT));
        RC(B.alloc(&rank, NT));
        hipLaunchKernelGGL(k_iota_u32, dim3(grid_for(NT)), dim3(256), 0, st, src, NT);
        HIP_OK(hipGetLastError());
        RC(radix_sort_u64_ws(&tkey, &src, NT, rxbits, B.ws));
        hipLaunchKernelGGL(k_flag_new, dim3(grid_for(NT)), dim3(256), 0, st, tkey, NT, pos);
        HIP_OK(hipGetLastError());
        RC(scan_exclusive_i64(pos, pos, NT, tot + 1, st, &B.ws));
        hipLaunchKernelGGL(k_unique_rank, dim3(grid_for(NT)), dim3(256), 0, st, tkey, NT, pos,
                           tot + 1, src, E, rank, diff);
        HIP_OK(hipGetLastError());
        B.release(src);
        hipLaunchKernelGGL(k_interval_span, dim3(grid_for(NI)), dim3(256), 0, st, rank, NI, ika,
                           xoff);
        HIP_OK(hipGetLastError());
        B.release(rank);
    }
    B.release(pos);
    RC(scan_exclusive_i64(diff, dex, NP, tot + 2, st, &B.ws));
    hipLaunchKernelGGL(k_piece_classify, dim3(grid_for(NP)), dim3(256), 0, st, dex, diff, NP, segc,
                       mm, err);
    HIP_OK(hipGetLastError());
    {
        const int64_t *in[3] = {segc, mm, xoff}, n[3] = {NP, NP, std::max<int64_t>(NI, 1)};
        int64_t *out[3] = {segc, mm, xoff}, *sum[3] = {tot + 3, tot + 4, tot + 5};
        RC(scan_exclusive_i64_multi(3, in, out, n, sum, st, &B.ws));
    }
    RC(fetch());
    const int64_t *h6 = hsc + 8;
    herr = (int)(uint32_t)hsc[0];
    if (herr & 8) return SBA_ELIMIT;
    if (herr) return SBA_EDEVICE;
    const int64_t NS = h6[3] >> 32, NM = h6[3] & 0xffffffffll, NMEM = h6[4];
    const int64_t NX = NI ? h6[5] : 0;
    if (NS >= ((int64_t)1 << 31)) return SBA_ELIMIT;
    h->n_segments = NS;
    B.NS = NS;
    int64_t *cs = nullptr;
    uint32_t *seg_row = nullptr;
    int32_t *sid = nullptr, *fill = nullptr;
    RC(B.alloc(&cs, gh + 1));
    RC(B.alloc(&B.seg_x0, std::max<int64_t>(NS, 1)));
    RC(B.alloc(&B.seg_x1, std::max<int64_t>(NS, 1)));
    RC(B.alloc(&B.seg_code, std::max<int64_t>(NS, 1)));
    RC(B.alloc(&seg_row, std::max<int64_t>(NS, 1)));
    RC(B.alloc(&sid, NP));
    RC(B.alloc(&fill, NP));
    int64_t *multi_seg = nullptr, *multi_mem = nullptr;
    int32_t *mem_ids = nullptr;
    RC(B.alloc(&multi_seg, std::max<int64_t>(NM, 1)));
    RC(B.alloc(&multi_mem, std::max<int64_t>(NM, 1)));
    RC(B.alloc(&mem_ids, std::max<int64_t>(NMEM, 1)));
    HIP_OK(hipMemsetAsync(fill, 0, sizeof(int32_t) * NP, st));
    if (NX)
        hipLaunchKernelGGL(k_piece_members, dim3(grid_for(NX)), dim3(256), 0, st, xoff, NI, NX,
                           ika, tpoly, dex, diff, mm, sid, fill, mem_ids);
    if (NT)
        hipLaunchKernelGGL(k_piece_emit, dim3(grid_for(NT)), dim3(256), 0, st, E, NT, dex, diff,
                           segc, mm, sid, B.xbits, B.seg_x0, B.seg_x1, B.seg_code, seg_row,
                           multi_seg, multi_mem, mem_ids);
    hipLaunchKernelGGL(k_seg_row_off, dim3(grid_for(gh + 1)), dim3(256), 0, st, seg_row, NS, gh,
                       cs);
    HIP_OK(hipGetLastError());
    B.seg_beg = cs;
    B.seg_end = cs + 1;
    for (void *p : {(void *)tkey, (void *)tpoly, (void *)E, (void *)ika, (void *)xoff,
                    (void *)diff, (void *)dex, (void *)segc, (void *)mm, (void *)seg_row,
                    (void *)sid, (void *)fill})
        B.release(p);

    // 5: the sets of multi-polygon segments
    if (NM > 0) {
        SetStage S{};
        uint64_t *mkey = nullptr;
        uint32_t *mval = nullptr;
        RC(B.alloc(&mkey, NM));
        RC(B.alloc(&mval, NM));
        RC(B.alloc(&S.memloc, NS));
        S.fb = std::min(pbits + 1, 21);  // ids + 1 < 2^21
        S.mem_ids = mem_ids;
        hipLaunchKernelGGL(k_multi_keys, dim3(grid_for(NM)), dim3(256), 0, st, multi_mem, multi_seg,
                           NM, NMEM, mem_ids, S.fb, mkey, mval, S.memloc);
        HIP_OK(hipGetLastError());
        bool done = false;
        if (!(paths_off & 4)) RC(sets_hash_list(S, B, h, mkey, mval, NM, NMEM, NS, st, &done));
        if (!done) RC(sets_from_list(S, B, h, mkey, mval, NM, NMEM, NS, st));
        if (S.one_workgroup) g_build_paths_last = g_build_paths_last.load() | 4;
        sets_release(S, B);
    }
    B.release(multi_seg);
    B.release(multi_mem);
    B.release(mem_ids);
    if (h->n_sets >= (int64_t)(TILE_MIXED - CODE_SET_BASE)) return SBA_ELIMIT;
    return 0;
}

// debug switch: store the grid in the 32-bit format even where the compact
// one would fit
bool g_build_wide = false;

template <int G>
static void launch_classify(const BuildState &B, const sba_handle *h, const int64_t *mt, int tl,
                            int sl, int64_t n_sq, uint32_t *code, int64_t *mixed, hipStream_t st)
{
    hipLaunchKernelGGL(k_square_classify<G>, dim3(xcd_grid(grid_for(n_sq * G))), dim3(256), 0, st,
                       B.seg_beg, B.seg_end, B.seg_x0, B.seg_x1, B.seg_code, h->gw, h->gh, mt, tl, sl,
                       h->tw, n_sq, code, mixed);
}

static void classify(const BuildState &B, const sba_handle *h, const int64_t *mt, int tl, int sl,
                     int64_t n_sq, uint32_t *code, int64_t *mixed, hipStream_t st)
{
    int side_log2 = mt ? sl : tl;
    const int qlog = mt ? tl - sl : 4;
    const int64_t nsq = (int64_t)(tl < 8 ? 256 >> tl : 1) << (mt ? 2 * qlog : qlog);
    if (tl >= 6 && qlog >= 2 && qlog <= 5 && nsq <= SQ_MAX) {
        const int64_t regions = mt ? n_sq >> (2 * qlog)
                                   : ((h->tw + SQ_Q - 1) / SQ_Q) * h->th;
        const SquareGeo G{B.seg_beg, B.seg_end, B.seg_x0, B.seg_x1, B.seg_code, h->gw, h->gh,
                          h->tw, h->th, mt, tl, sl, qlog, regions};
        const int rpb = tl < 8 ? 256 >> tl : 1;
        hipLaunchKernelGGL(k_squares, dim3(xcd_grid((unsigned)((regions + rpb - 1) / rpb))), dim3(256),
                           (size_t)nsq * 8, st, G, code, mixed);
        return;
    }
    if (side_log2 >= 6) launch_classify<64>(B, h, mt, tl, sl, n_sq, code, mixed, st);
    else if (side_log2 == 5) launch_classify<32>(B, h, mt, tl, sl, n_sq, code, mixed, st);
    else if (side_log2 == 4) launch_classify<16>(B, h, mt, tl, sl, n_sq, code, mixed, st);
    else if (side_log2 == 3) launch_classify<8>(B, h, mt, tl, sl, n_sq, code, mixed, st);
    else launch_classify<4>(B, h, mt, tl, sl, n_sq, code, mixed, st);
}

int build_grid(sba_handle *h, BuildState &B, int tile_log2, int sub_log2, hipStream_t st)
{
    int tl = tile_log2;
    if (tl == 0) {
        // the smallest tile whose 16-bit directory, with the probe's LDS bins
        // (12 B per polygon and per set), fits the LDS of a compute unit: the
        // finer the directory, the fewer points need a lookup in global memory
        auto tiles = [&](int t) {
            return ((h->gw + (1 << t) - 1) >> t) * ((h->gh + (1 << t) - 1) >> t);
        };
        auto fits = [&](int t, int64_t bins) {
            int64_t nt16 = (tiles(t) + 7) & ~(int64_t)7;
            return tiles(t) <= COMPACT_DIR_TILES_MAX && nt16 * 2 + bins * 12 <= PROBE_LDS_BYTES;
        };
        const int64_t all = (int64_t)h->n_polys + h->n_sets;
        tl = 2;
        while (tl < 10 && !fits(tl, all)) tl++;
        if (!fits(tl, all)) {  // set bins never fit: directory and polygon bins
            tl = 2;
            while (tl < 10 && !fits(tl, h->n_polys)) tl++;
            if (!fits(tl, h->n_polys)) {  // polygon bins do not fit either
                tl = 2;
                while (tl < 10 && tiles(tl) > COMPACT_DIR_TILES) tl++;
            }
        }
    }
    if (tl < 2 || tl > 10) return SBA_EINVAL;
    // sub-tiles of 16 x 16 cells under big tiles, of 8 x 8 under tiles of 32
    // (until the mixed tiles are known, see below)
    int sl = sub_log2 ? sub_log2 : (tl >= 6 ? 4 : (tl == 5 ? 3 : tl));
    if (sl < 1 || sl > tl) return SBA_EINVAL;
    h->tile_log2 = tl;
    h->sub_log2 = sl;
    h->tw = (h->gw + (1 << tl) - 1) >> tl;
    h->th = (h->gh + (1 << tl) - 1) >> tl;
    const int64_t nt = h->tw * h->th;
    if (nt >= ((int64_t)1 << 31)) return SBA_ELIMIT;
    const uint32_t np = (uint32_t)h->n_polys;
    uint32_t *tcode = nullptr;
    int64_t *tpos = nullptr, *tot = B.sc + 16;
    int64_t hsc[SC_READ];
    RC(B.alloc(&tcode, nt));
    RC(B.alloc(&tpos, nt + 1));
    classify(B, h, nullptr, tl, sl, nt, tcode, tpos, st);
    HIP_OK(hipGetLastError());
    // in one launch when the 16-bit directory is sure, or likely, to be taken
    const bool compact_nt = !g_build_wide && (int64_t)np + h->n_sets < 0x8000 &&
                            nt <= COMPACT_DIR_TILES_MAX;
    const int64_t nt16 = (nt + 7) & ~(int64_t)7;  // LDS copies move 16 bytes at a time
    int64_t *mt = nullptr;  // mixed tiles in order
    bool numbered = compact_nt && nt16 <= NUMBER_MAX;
    RC(B.ws.read(hsc, B.sc, sizeof(hsc)));
    if (numbered) {
        RC(B.alloc(&mt, nt));
        RC(handle_alloc(h, &h->dir16, nt16));
        hipLaunchKernelGGL(k_number, dim3(grid_for(nt16, NUMBER_TILE)), dim3(NUMBER_BLOCK), 0, st,
                           tcode, (int)nt, (int)nt16, np, 2, (uint32_t *)nullptr, h->dir16, mt,
                           tot, B.ws.reads());
        HIP_OK(hipGetLastError());
        RC(B.ws.wait());
        if (hsc[16] >= 0x8000) {  // too many mixed tiles for it after all
            handle_put_last(h, (size_t)nt16 * sizeof(*h->dir16));
            h->dir16 = nullptr;
            B.release(mt);
            mt = nullptr;
            numbered = false;
            RC(scan_exclusive_i64(tpos, tpos, nt, nullptr, st, &B.ws));
        }
    } else {
        RC(scan_exclusive_i64(tpos, tpos, nt, tot, st, &B.ws));
        RC(B.ws.sync());
    }
    const int64_t nblk = hsc[16];
    if (nblk >= (int64_t)TILE_MIXED) return SBA_ELIMIT;
    h->n_blocks = nblk;
    const bool compact = compact_nt && nblk < 0x8000;
    h->compact = compact;
    if (sub_log2 == 0 && compact && nblk > 0) {
        // the smallest sub-tile whose 16-bit sub-directory fits the LDS of a
        // compute unit beside the directory and the bins: the probe then
        // stages it there, and only points in mixed sub-tiles read a fine
        // block from global memory
        const int64_t dir = ((nt + 7) & ~(int64_t)7) * 2, bins = ((int64_t)np + h->n_sets) * 12;
        for (int t = 1; t < tl; t++) {
            const int64_t ne = ((nblk << (2 * (tl - t))) + 7) & ~(int64_t)7;
            if (dir + ne * 2 + bins <= PROBE_LDS_BYTES) {
                sl = t;
                break;
            }
        }
        h->sub_log2 = sl;
    }

    // directory
    if (numbered) {
    } else if (compact) {
        RC(handle_alloc(h, &h->dir16, nt16));
        hipLaunchKernelGGL(k_entries, dim3(grid_for(nt16)), dim3(256), 0, st, tcode, tpos, nt, nt16,
                           np, 2, (uint32_t *)nullptr, h->dir16);
    } else {
        RC(handle_alloc(h, &h->dir, nt));
        hipLaunchKernelGGL(k_entries, dim3(grid_for(nt)), dim3(256), 0, st, tcode, tpos, nt, nt, np,
                           0, h->dir, (uint16_t *)nullptr);
    }
    HIP_OK(hipGetLastError());
    if (nblk == 0) {
        // one-element placeholders: the batched lookups read element 0 of
        // the lower levels for points that need nothing from them
        if (sl < tl) {
            RC(handle_alloc(h, &h->sub, 1));
            HIP_OK(hipMemsetAsync(h->sub, 0, 4, st));
        }
        if (compact) {
            RC(handle_alloc(h, &h->blocks16, 1));
            HIP_OK(hipMemsetAsync(h->blocks16, 0, 2, st));
        } else {
            RC(handle_alloc(h, &h->blocks, 1));
            HIP_OK(hipMemsetAsync(h->blocks, 0, 4, st));
        }
        return 0;
    }
    if (!numbered) {
        RC(B.alloc(&mt, nblk));
        hipLaunchKernelGGL(k_flag_list, dim3(grid_for(nt)), dim3(256), 0, st, tpos, nt, nblk, mt);
        HIP_OK(hipGetLastError());
    }

    // sub-directories of the mixed tiles
    const int64_t *fine_sq = mt;        // squares stored as fine blocks
    const int64_t *fine_mt = nullptr;   // their tile list (sub-tiles) or NULL (tiles)
    int64_t nfine = nblk;
    int fine_log2 = tl;
    if (sl < tl) {
        const int64_t nq = nblk << (2 * (tl - sl));
        uint32_t *scode = nullptr;
        int64_t *spos = nullptr, *ms = nullptr;
        RC(B.alloc(&scode, nq));
        RC(B.alloc(&spos, nq + 1));
        classify(B, h, mt, tl, sl, nq, scode, spos, st);
        HIP_OK(hipGetLastError());
        RC(B.ws.read(hsc, B.sc, sizeof(hsc)));
        RC(handle_alloc(h, &h->sub, nq));
        if (nq <= NUMBER_MAX) {
            RC(B.alloc(&ms, nq));
            hipLaunchKernelGGL(k_number, dim3(grid_for(nq, NUMBER_TILE)), dim3(NUMBER_BLOCK), 0, st,
                               scode, (int)nq, (int)nq, np, compact ? 1 : 0, h->sub,
                               (uint16_t *)nullptr, ms, tot + 1, B.ws.reads());
            HIP_OK(hipGetLastError());
            RC(B.ws.wait());
        } else {
            RC(scan_exclusive_i64(spos, spos, nq, tot + 1, st, &B.ws));
            RC(B.ws.sync());
        }
        const int64_t nsub = hsc[17];
        if (nsub >= (int64_t)TILE_MIXED) return SBA_ELIMIT;
        h->n_sub = nsub;
        if (nq > NUMBER_MAX) {
            hipLaunchKernelGGL(k_entries, dim3(grid_for(nq)), dim3(256), 0, st, scode, spos, nq, nq,
                               np, compact ? 1 : 0, h->sub, (uint16_t *)nullptr);
            HIP_OK(hipGetLastError());
            RC(B.alloc(&ms, std::max<int64_t>(nsub, 1)));
            hipLaunchKernelGGL(k_flag_list, dim3(grid_for(nq)), dim3(256), 0, st, spos, nq, nsub,
                               ms);
            HIP_OK(hipGetLastError());
        }
        fine_sq = ms;
        fine_mt = mt;
        nfine = nsub;
        fine_log2 = sl;
    }

    // fine blocks
    const int64_t cells = nfine << (2 * fine_log2);
    const int side = 1 << fine_log2;
    const int64_t threads = nfine * side * (side > 16 ? side >> 4 : 1);
    if (compact) {
        RC(handle_alloc(h, &h->blocks16, std::max<int64_t>(cells, 1)));
        if (nfine)
            hipLaunchKernelGGL(k_block_fill<uint16_t>, dim3(xcd_grid(grid_for(threads))), dim3(256), 0, st,
                               B.seg_beg, B.seg_end, B.seg_x0, B.seg_x1, B.seg_code, h->gw, h->gh, fine_sq,
                               nfine, fine_mt, tl, sl, h->tw, fine_log2, np, h->blocks16);
    } else {
        RC(handle_alloc(h, &h->blocks, std::max<int64_t>(cells, 1)));
        if (nfine)
            hipLaunchKernelGGL(k_block_fill<uint32_t>, dim3(xcd_grid(grid_for(threads))), dim3(256), 0, st,
                               B.seg_beg, B.seg_end, B.seg_x0, B.seg_x1, B.seg_code, h->gw, h->gh, fine_sq,
                               nfine, fine_mt, tl, sl, h->tw, fine_log2, np, h->blocks);
    }
    HIP_OK(hipGetLastError());
    return 0;
}

int build_handle(const sba_polygons *polys, int64_t eps, const sba_build_opts *opts,
                 hipStream_t st, sba_handle *h)
{
    auto t0 = std::chrono::steady_clock::now();
    sba_build_opts o{};
    o.kind = SBA_KIND_GRID;
    o.search = SBA_SEARCH_BINARY;
    o.log2_leaves = 16;
    if (opts) o = *opts;
    if ((o.alloc == nullptr) != (o.release == nullptr)) return SBA_EINVAL;
    h->ua = UserAlloc{o.alloc, o.release, o.alloc_ctx};
    if (o.use_window && (o.win_x1 <= o.win_x0 || o.win_y1 <= o.win_y0)) return SBA_EINVAL;
    if (o.log2_leaves == 0) o.log2_leaves = 16;
    if (o.kind != SBA_KIND_GRID && o.kind != SBA_KIND_HILBERT) return SBA_EINVAL;
    if (o.search != SBA_SEARCH_BINARY && o.search != SBA_SEARCH_LEARNED) return SBA_EINVAL;
    if (o.log2_leaves < 1 || o.log2_leaves > 24) return SBA_EINVAL;
    if (o.key_level < 0 || o.key_level > 21 || (o.key_level > 0 && o.kind != SBA_KIND_HILBERT))
        return SBA_EINVAL;
    if (o.centre_sampled != 0 && o.centre_sampled != 1) return SBA_EINVAL;
    if (o.centre_sampled && o.boundary_only) return SBA_EINVAL;
    if (o.key_level > 0 && (o.key_i0 < -((int64_t)1 << 31) || o.key_i0 >= ((int64_t)1 << 31) ||
                            o.key_j0 < -((int64_t)1 << 31) || o.key_j0 >= ((int64_t)1 << 31)))
        return SBA_EINVAL;
    h->kind = o.kind;
    h->search = o.search;
    h->eps = eps;
    const int64_t s = cell_side(eps);
    h->s = s;
    magic_for(s, &h->mag, &h->shift);
    h->n_polys = polys->n_polys;
    if (polys->n_polys == 0) {
        h->gw = h->gh = 0;
        h->build_ms = 0;
        return 0;
    }
    BuildState B(st);
    B.ws.set_allocator(h->ua);
    B.boundary_only = o.boundary_only != 0;
    h->boundary_only = o.boundary_only != 0;
    B.centre = o.centre_sampled != 0;
    h->centre_sampled = o.centre_sampled != 0;
    B.window = o.use_window != 0;
    B.wx0 = o.win_x0;
    B.wy0 = o.win_y0;
    B.wx1 = o.win_x1;
    B.wy1 = o.win_y1;
    B.key_level = o.key_level;
    B.key_i0 = o.key_i0;
    B.key_j0 = o.key_j0;
    if (h->kind == SBA_KIND_HILBERT) RC(hilbert_prepare(B, h));
    RC(build_segments(polys, eps, st, h, B, h->kind == SBA_KIND_HILBERT));
    if (B.empty) {
        HIP_OK(hipStreamSynchronize(st));
        h->build_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0)
                          .count();
        return 0;
    }
    if (h->kind == SBA_KIND_GRID) {
        RC(build_grid(h, B, o.tile_log2, o.sub_log2, st));
    } else {
        RC(hilbert_finish(B, h, o, st));
    }
    HIP_OK(hipStreamSynchronize(st));
    auto t1 = std::chrono::steady_clock::now();
    h->build_ms = std::chrono::duration<double, std::milli>(t1 - t0).count();
    return 0;
}
