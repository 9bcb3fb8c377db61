// hilbert.hip -- the adaptive-quadtree layout: the approximation stored as
// the maximal runs of consecutive Hilbert keys whose cells carry the same
// polygon set (Sec. 3: cells linearised on a space-filling curve and kept in
// a sorted array; a run of the curve is a union of aligned quadtree blocks,
// so interior cells come out as large cells, Sec. 2.2), and the learned
// index that predicts a key's run (Sec. 3, learned index over the sorted
// cell array).
//
// The key grid is anchored at the first cell of the stored box (the union of
// the polygons' cell boxes), so every cell of every approximation has a key;
// or at a grid the caller gives (a point index's), the box cut to it.
//
// Runs are found without visiting interior cells.  Consecutive Hilbert cells
// share an edge; two edge-adjacent cells that are boundary cells of no
// polygon have the same polygon set (a polygon boundary separating them
// would touch both closed squares).  So the polygon set is constant on every
// gap between consecutive boundary keys, and one lookup at the gap's first
// cell gives it.
#include "sba_internal.h"
#include "build_state.h"

__device__ __forceinline__ int64_t ub_i64(const int64_t *a, int64_t n, int64_t v)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] <= v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// cells of boundary interval t (relative to the stored box, which is also
// the origin of the Hilbert key grid); event keys are (polygon, row, x)
__global__ void k_bcell_counts(const uint64_t *evkey, int64_t nb, int xbits, int64_t *cnt)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nb) return;
    uint64_t xm = (1ull << xbits) - 1;
    cnt[t] = (int64_t)(evkey[2 * t + 1] & xm) - (int64_t)(evkey[2 * t] & xm);
}

__global__ void k_bcell_keys(const uint64_t *evkey, int64_t nb, int xbits, int rbits,
                             const int64_t *off, int64_t ncells, int L, uint64_t *keys)
{
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncells) return;
    int64_t t = ub_i64(off, nb, c) - 1;
    uint64_t xm = (1ull << xbits) - 1;
    uint32_t j = (uint32_t)((evkey[2 * t] >> xbits) & ((1ull << rbits) - 1));
    uint32_t i = (uint32_t)((evkey[2 * t] & xm) + (uint64_t)(c - off[t]));
    keys[c] = hilbert_index(L, i, j);
}

// cells on the border of the stored box (used when a clip window cut the
// box through polygon interiors: a gap of the curve must not run from a cell
// inside the box to an empty cell outside it without a key in between)
__global__ void k_border_keys(int64_t gw, int64_t gh, int L, uint64_t *keys)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * (gw + gh)) return;
    uint32_t i, j;
    if (t < gw) { i = (uint32_t)t; j = 0; }
    else if (t < 2 * gw) { i = (uint32_t)(t - gw); j = (uint32_t)(gh - 1); }
    else if (t < 2 * gw + gh) { i = 0; j = (uint32_t)(t - 2 * gw); }
    else { i = (uint32_t)(gw - 1); j = (uint32_t)(t - 2 * gw - gh); }
    keys[t] = hilbert_index(L, i, j);
}

__global__ void k_flag_first(const uint64_t *keys, int64_t n, int64_t *flag)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    flag[t] = (t == 0 || keys[t] != keys[t - 1]) ? 1 : 0;
}

__global__ void k_compact_first(const uint64_t *keys, int64_t n, const int64_t *pos, uint64_t *out)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    if (t == 0 || keys[t] != keys[t - 1]) out[pos[t]] = keys[t];
}

static int hilbert_boundary_cells(BuildState &B, sba_handle *h, hipStream_t st)
{
    const int64_t NB = B.NB;
    if (NB == 0 && !B.window) return 0;
    int64_t *cnt = nullptr, *tot = nullptr;
    RC(B.alloc(&cnt, NB + 1));
    RC(B.alloc(&tot, 1));
    hipLaunchKernelGGL(k_bcell_counts, dim3(grid_for(NB)), dim3(256), 0, st, B.evkey, NB, B.xbits,
                       cnt);
    HIP_OK(hipGetLastError());
    RC(scan_exclusive_i64(cnt, cnt, NB, tot, st, &B.ws));
    int64_t ncb = 0;
    RC(B.ws.read(&ncb, tot, sizeof(int64_t)));
    RC(B.ws.sync());
    const int64_t nborder = B.window ? 2 * (h->gw + h->gh) : 0;
    const int64_t nc = ncb + nborder;
    if (nc == 0) return 0;
    uint64_t *keys = nullptr;
    RC(B.alloc(&keys, nc));
    if (ncb)
        hipLaunchKernelGGL(k_bcell_keys, dim3(grid_for(ncb)), dim3(256), 0, st, B.evkey, NB, B.xbits,
                           B.rbits, cnt, ncb, h->level, keys);
    if (nborder)
        hipLaunchKernelGGL(k_border_keys, dim3(grid_for(nborder)), dim3(256), 0, st, h->gw, h->gh,
                           h->level, keys + ncb);
    HIP_OK(hipGetLastError());
    B.release(cnt);
    RC(radix_sort_u64_ws(&keys, nullptr, nc, 2 * h->level, B.ws));
    int64_t *flag = nullptr;
    RC(B.alloc(&flag, nc + 1));
    hipLaunchKernelGGL(k_flag_first, dim3(grid_for(nc)), dim3(256), 0, st, keys, nc, flag);
    HIP_OK(hipGetLastError());
    RC(scan_exclusive_i64(flag, flag, nc, tot, st, &B.ws));
    int64_t nu = 0;
    RC(B.ws.read(&nu, tot, sizeof(int64_t)));
    RC(B.ws.sync());
    RC(B.alloc(&B.bkeys, nu));
    hipLaunchKernelGGL(k_compact_first, dim3(grid_for(nc)), dim3(256), 0, st, keys, nc, flag,
                       B.bkeys);
    HIP_OK(hipGetLastError());
    B.nbkeys = nu;
    B.release(keys);
    B.release(flag);
    return 0;
}

int hilbert_level(const BuildState &B, sba_handle *h)
{
    // key grid: the stored cell box, padded to 2^L x 2^L
    int L = 1;
    while (((int64_t)1 << L) < std::max(h->gw, h->gh)) L++;
    if (B.key_level > 0) L = B.key_level;  // the box was cut to fit it
    if (L > 21) return SBA_ELIMIT;
    h->level = L;
    return 0;
}

int hilbert_prepare(BuildState &B, sba_handle *h)
{
    (void)h;
    B.on_boundary_events = [](BuildState &b, sba_handle *hh, hipStream_t st) -> int {
        RC(hilbert_level(b, hh));
        return hilbert_boundary_cells(b, hh, st);
    };
    return 0;
}

// ---------------------------------------------------------------- runs

struct SegView {
    const int64_t *beg, *end;
    const int32_t *x0, *x1;
    const uint32_t *code;
    int64_t gw, gh;
};

// code of the cell with the key: the last segment of its row that starts at
// or before it, if it reaches it
__device__ __forceinline__ uint32_t code_of_key(const SegView &S, int L, uint64_t key)
{
    uint32_t x, r;
    hilbert_cell(L, key, &x, &r);
    if (x >= S.gw || r >= S.gh) return 0;
    const int64_t a = S.beg[r];
    int64_t lo = a, hi = S.end[r];
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (S.x0[mid] <= (int32_t)x) lo = mid + 1; else hi = mid;
    }
    return lo > a && (int32_t)x < S.x1[lo - 1] ? S.code[lo - 1] : 0;
}

// Candidate run starts: key 0, every boundary key, and the key after one
// when a gap follows.  A candidate whose code differs from the one before it
// starts a run.
#define RUN_BLOCK 256
#define NO_GAP 0xffffffffu

// codes of boundary key t and of the gap after it
template <typename K>
__device__ __forceinline__ uint32_t gap_code(const K *bk, int64_t nb, uint64_t total, int64_t t,
                                             const SegView &S, int L)
{
    const uint64_t next = t + 1 < nb ? (uint64_t)bk[t + 1] : total;
    return next > (uint64_t)bk[t] + 1 ? code_of_key(S, L, (uint64_t)bk[t] + 1) : NO_GAP;
}

template <typename K>
__device__ __forceinline__ uint32_t bkey_code(const K *bk, const uint32_t *bseg, int64_t t,
                                              const SegView &S, int L)
{
    if (!bseg) return code_of_key(S, L, (uint64_t)bk[t]);
    const uint32_t q = bseg[t];
    return q == 0xffffffffu ? 0u : S.code[q];
}

// bit 0: boundary key t starts a run, bit 1: the gap after it does
__device__ __forceinline__ uint32_t run_bits(uint32_t c, uint32_t g, uint32_t prev)
{
    return (c != prev ? 1u : 0u) | (g != NO_GAP && g != c ? 2u : 0u);
}

// codes, and the workgroup's number of run starts
template <typename K>
__global__ __launch_bounds__(RUN_BLOCK) void k_run_count(const K *bk, const uint32_t *bseg,
                                                         int64_t nb, uint64_t total, SegView S,
                                                         int L, uint32_t *ccode, uint32_t *gcode,
                                                         int64_t *cnt)
{
    __shared__ uint32_t last[RUN_BLOCK];
    __shared__ uint32_t sum;
    const int64_t t = (int64_t)blockIdx.x * RUN_BLOCK + threadIdx.x;
    uint32_t c = 0, g = NO_GAP;
    if (threadIdx.x == 0) sum = 0;
    if (t < nb) {
        c = bkey_code(bk, bseg, t, S, L);
        g = gap_code(bk, nb, total, t, S, L);
        ccode[t] = c;
        gcode[t] = g;
        last[threadIdx.x] = g != NO_GAP ? g : c;
    }
    __syncthreads();
    uint32_t m = 0;
    if (t < nb) {
        uint32_t prev;
        if (threadIdx.x) {
            prev = last[threadIdx.x - 1];
        } else if (t == 0) {
            prev = code_of_key(S, L, 0);
        } else {
            const uint32_t pg = gap_code(bk, nb, total, t - 1, S, L);
            prev = pg != NO_GAP ? pg : bkey_code(bk, bseg, t - 1, S, L);
        }
        m = (uint32_t)__popc(run_bits(c, g, prev));
    }
    for (int o = 32; o > 0; o >>= 1) m += (uint32_t)__shfl_xor((int)m, o, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(&sum, m);
    __syncthreads();
    if (threadIdx.x == 0) cnt[blockIdx.x] = sum;
}

// run 0 starts at key 0; off: exclusive scan of k_run_count's numbers
template <typename K>
__global__ __launch_bounds__(RUN_BLOCK) void k_run_write(const K *bk, int64_t nb, SegView S, int L,
                                                         const uint32_t *ccode,
                                                         const uint32_t *gcode, const int64_t *off,
                                                         uint64_t *starts, uint32_t *starts32,
                                                         uint32_t *rcode)
{
    __shared__ uint32_t wsum[RUN_BLOCK / 64];
    const int64_t t = (int64_t)blockIdx.x * RUN_BLOCK + threadIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t c = 0, g = NO_GAP, bits = 0;
    if (t < nb) {
        c = ccode[t];
        g = gcode[t];
        uint32_t prev;
        if (t == 0) {
            prev = code_of_key(S, L, 0);
        } else {
            const uint32_t pg = gcode[t - 1];
            prev = pg != NO_GAP ? pg : ccode[t - 1];
        }
        bits = run_bits(c, g, prev);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        starts[0] = 0;
        if (starts32) starts32[0] = 0;
        rcode[0] = code_of_key(S, L, 0);
    }
    const uint32_t m = (uint32_t)__popc(bits);
    uint32_t incl = m;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    if (!bits) return;
    int64_t o = 1 + off[blockIdx.x] + incl - m;
    for (int k = 0; k < w; k++) o += wsum[k];
    if (bits & 1u) {
        starts[o] = (uint64_t)bk[t];
        if (starts32) starts32[o] = (uint32_t)bk[t];
        rcode[o] = c;
        o++;
    }
    if (bits & 2u) {
        starts[o] = (uint64_t)bk[t] + 1;
        if (starts32) starts32[o] = (uint32_t)bk[t] + 1u;
        rcode[o] = g;
    }
}

template <typename K>
static int write_runs(BuildState &B, sba_handle *h, const K *bk, hipStream_t st)
{
    const int L = h->level;
    const uint64_t total = (uint64_t)1 << (2 * L);
    const int64_t nb = B.nbkeys, blocks = std::max<int64_t>((nb + RUN_BLOCK - 1) / RUN_BLOCK, 1);
    const SegView S{B.seg_beg, B.seg_end, B.seg_x0, B.seg_x1, B.seg_code, h->gw, h->gh};
    uint32_t *ccode = nullptr, *gcode = nullptr;
    int64_t *cnt = nullptr;
    RC(B.alloc(&ccode, nb));
    RC(B.alloc(&gcode, nb));
    RC(B.alloc(&cnt, blocks + 1));
    hipLaunchKernelGGL(k_run_count<K>, dim3((unsigned)blocks), dim3(RUN_BLOCK), 0, st, bk, B.bseg,
                       nb, total, S, L, ccode, gcode, cnt);
    HIP_OK(hipGetLastError());
    RC(scan_exclusive_i64(cnt, cnt, blocks, cnt + blocks, st, &B.ws));
    int64_t nr = 0;
    RC(B.ws.read(&nr, cnt + blocks, sizeof(int64_t)));
    RC(B.ws.sync());
    nr += 1;  // key 0's run
    if (nr >= ((int64_t)1 << 31)) return SBA_ELIMIT;
    h->n_runs = nr;
    RC(handle_alloc(h, &h->starts, nr));
    RC(handle_alloc(h, &h->run_code, nr));
    if (2 * L <= 32) RC(handle_alloc(h, &h->starts32, nr));
    hipLaunchKernelGGL(k_run_write<K>, dim3((unsigned)blocks), dim3(RUN_BLOCK), 0, st, bk, nb, S, L,
                       ccode, gcode, cnt, h->starts, h->starts32, h->run_code);
    HIP_OK(hipGetLastError());
    B.release(ccode);
    B.release(gcode);
    B.release(cnt);
    return 0;
}

// ---------------------------------------------------------------- block directory
//
// One entry per aligned square block of cells of the stored box (a stretch of
// consecutive keys): the code of the run that holds the whole block, or
// TILE_MIXED | the run that holds its first key, from which a search reaches
// any key of the block.  Most
// blocks of a partition lie in one run (91 % of the 16 x 16 blocks of 40,000
// polygons at 1 m), so most lookups are one 4-byte read, at an address that
// takes no Hilbert key, where a search over the runs takes 6 to 9 cache lines.
// Blocks as small as 4 to 8 of them a run allow, and at most 2^24.  Four times as
// many leave fewer mixed blocks but more lines: 2e7 points over 260 polygons at
// 10 m (230,000 runs) in no order, counts only, 141 us with up to 32 a run, 122 so,
// with values 183 and 173; in order 93 and 107.  (2^24 are 64 MB, which the
// memory-side cache holds; 2^22 and 2^23 made the probe of 2e7 points over 40,000
// polygons at 1 m in no order 9 and 4 % slower, by their mixed blocks.)  They cover the stored box
// only, not the whole key grid: on a grid much larger than the polygons (a
// point index's, or one for several sets) blocks of 4^-12 of it held all runs.
#define DIR_MAX ((int64_t)1 << 24)
// blocks of a workgroup: a square of 2^6 a side, or of down to 2^4 where that leaves
// fewer than DIR_WGS workgroups (500,000 blocks of 260 polygons at 10 m: 144 squares
// 22 us, 2,025 of 2^4 8.8, 7,921 of 2^3 20.4; 4.2M blocks under one large ring: 1,089
// squares 138, 4,225 80)
#define DIR_SQUARE 6
#define DIR_SQUARE_MIN 4
#define DIR_WGS 2048

struct DirGeo {
    int L, r;           // levels of the key grid; blocks of 2^r cells a side
    int q;              // workgroups' squares of 2^q blocks a side (at most the grid)
    uint32_t bw, bh;    // blocks of the box
    uint32_t sw;        // squares a row
    uint32_t cols;      // tiles of 8 blocks a row (block_index)
};

// The first run in (lo, hi] that starts at or after v (hi if none does); run lo
// starts before it.  All 64 lanes of the wavefront search together.
__device__ __forceinline__ int64_t first_at_least(const uint64_t *starts, int64_t lo, int64_t hi,
                                                  uint64_t v)
{
    const int lane = threadIdx.x & 63;
    while (hi - lo > 1) {
        // places lo + 1 .. hi - 1 in 64 steps
        const int64_t step = (hi - lo + 63) >> 6, at = lo + (lane + 1) * step;
        const uint64_t below = __ballot(at < hi && starts[at] < v);
        const int n = __popcll(below);  // starts ascend: the first n lanes
        const int64_t l = lo + (int64_t)n * step, h = lo + (int64_t)(n + 1) * step;
        lo = l;
        hi = h < hi ? h : hi;
    }
    return hi;
}

// A workgroup writes the entries of one square of blocks, a stretch of keys:
// each of its runs has the blocks whose first key it holds.  It takes 256 runs
// at a time, the next ones loaded meanwhile, and its lanes share their entries.
// (A wavefront for 64 runs and their entries: 182 us instead of 140 for 2^24
// entries of 28.9M runs, and 2.2 times as long for 230,000 runs of 260 polygons, some of
// hundreds of blocks.  One launch over all runs, with a
// list of those over more than 2,048 blocks that the whole grid then filled one
// after another: 800 us for a few hundred large polygons, which are mostly such
// runs.)
__global__ __launch_bounds__(256) void k_dir_fill(const uint64_t *__restrict__ starts,
                                                  const uint32_t *__restrict__ code, int64_t n,
                                                  DirGeo D, uint32_t *__restrict__ dir)
{
    __shared__ int64_t range[2];
    __shared__ uint32_t wsum[4];
    // of each run: entries up to its last one, its first block and the first block
    // it does not hold whole (in the square), its code
    __shared__ uint32_t s_incl[256], s_first[256], s_whole[256], s_code[256];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lv = D.L - D.r, rb = 2 * D.r;
    const uint32_t sj = blockIdx.x / D.sw, si = blockIdx.x - sj * D.sw;
    const int kb = rb + 2 * D.q;  // bits of a key inside the square
    const uint64_t k0 = hilbert_index(lv - D.q, si, sj) << kb, k1 = k0 + ((uint64_t)1 << kb);
    const uint64_t total = (uint64_t)1 << (2 * D.L), part = ((uint64_t)1 << rb) - 1;
    // the run that holds the first key, and the first past the last one
    if (w < 2) {
        const int64_t f = first_at_least(starts, 0, n, w ? k1 : k0 + 1);
        if (lane == 0) range[w] = w ? f : f - 1;
    }
    __syncthreads();
    const int64_t r0 = range[0], r1 = range[1];
    uint64_t at = 0, next = 0;
    uint32_t c = 0;
    auto load = [&](int64_t i) {
        if (i < r1) {
            at = starts[i];
            next = i + 1 < n ? starts[i + 1] : total;
            c = code[i];
        }
    };
    load(r0 + tid);
    for (int64_t base = r0; base < r1; base += 256) {
        uint32_t m = 0, first = 0, whole = 0;
        if (base + tid < r1) {
            const uint64_t a = (at > k0 ? at : k0) - k0, b = (next < k1 ? next : k1) - k0;
            first = (uint32_t)((a + part) >> rb);
            m = (uint32_t)((b + part) >> rb) - first;
            whole = (uint32_t)(b >> rb);
        }
        uint32_t incl = m;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
            if (lane >= o) incl += u;
        }
        if (lane == 63) wsum[w] = incl;
        s_first[tid] = first;
        s_whole[tid] = whole;
        s_code[tid] = c;
        __syncthreads();
        uint32_t all = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            if (k < w) incl += wsum[k];
            all += wsum[k];
        }
        s_incl[tid] = incl;
        load(base + 256 + tid);
        __syncthreads();
        for (uint32_t t = tid; t < all; t += 256) {
            // the entry's run: the first whose entries end past t
            int i = 0;
#pragma unroll
            for (int step = 128; step > 0; step >>= 1) i += s_incl[i + step - 1] <= t ? step : 0;
            const uint32_t q = s_first[i] + (t - (i ? s_incl[i - 1] : 0u));
            uint32_t ib, jb;
            hilbert_cell(lv, (k0 >> rb) + q, &ib, &jb);
            if (ib < D.bw && jb < D.bh)
                dir[block_index(ib, jb, D.cols)] =
                    q < s_whole[i] ? s_code[i] : (TILE_MIXED | (uint32_t)(base + i));
        }
        __syncthreads();
    }
}

static int build_directory(sba_handle *h, hipStream_t st)
{
    DirGeo D{};
    D.L = h->level;
    const int64_t most = std::min(
        DIR_MAX, std::max<int64_t>(1024, (int64_t)4 << bits_for((uint64_t)h->n_runs - 1)));
    int64_t entries = 0;
    for (D.r = 0;; D.r++) {
        D.bw = (uint32_t)(((h->gw - 1) >> D.r) + 1);
        D.bh = (uint32_t)(((h->gh - 1) >> D.r) + 1);
        D.cols = (D.bw + 7) >> 3;
        entries = (int64_t)D.cols * ((D.bh + 3) >> 2) * 32;
        if (entries <= most || D.r == D.L) break;
    }
    // smaller squares where there would be too few for the chip
    uint32_t sh = 0;
    for (D.q = std::min(DIR_SQUARE, D.L - D.r);; D.q--) {
        D.sw = ((D.bw - 1) >> D.q) + 1;
        sh = ((D.bh - 1) >> D.q) + 1;
        if (D.q <= DIR_SQUARE_MIN || D.sw * sh >= DIR_WGS) break;
    }
    h->dir_r = D.r;
    h->dir_cols = D.cols;
    RC(handle_alloc(h, &h->pdir, entries));
    hipLaunchKernelGGL(k_dir_fill, dim3(D.sw * sh), dim3(256), 0, st, h->starts, h->run_code,
                       h->n_runs, D, h->pdir);
    HIP_OK(hipGetLastError());
    return 0;
}

// ---------------------------------------------------------------- learned index
//
// Two-level piecewise-linear model over the sorted run starts (the idea of a
// learned index over a sorted cell array with a bounded last-mile search,
// Sec. 3).  Root: leaf = floor(key * a) in fp32, clamped, monotone in key.
// Leaf l covers the keys [K_l, K_{l+1}); it predicts the position of the run
// holding a key as floor(slope * (key - K_l) + icpt) in fp32 (no fused
// multiply-add, identical in the fit and in the probe), fitted by least
// squares on the leaf's run starts.  Its stored error bounds |prediction -
// answer| over EVERY key of [K_l, K_{l+1}), not only the stored ones: the
// answer is a step function of the key and the prediction is monotone, so the
// largest gap sits at an end of a step, and the fit evaluates exactly those
// keys.  A probe starts its search inside a mixed block of the directory at
// the model's position (clamped to the block) and goes on until two runs bracket
// the key, so it needs no bound; the stored errors are reported and tested.

// smallest key whose leaf is >= l (keys in [0, total])
__device__ uint64_t leaf_first_key(uint32_t l, float a, uint32_t nl, uint64_t total)
{
    if (l == 0) return 0;
    uint64_t lo = 0, hi = total;
    while (lo < hi) {
        uint64_t mid = lo + ((hi - lo) >> 1);
        if (root_leaf(mid, a, nl) >= l) hi = mid; else lo = mid + 1;
    }
    return lo;
}

__device__ __forceinline__ int64_t lower_bound_u64(const uint64_t *a, int64_t n, uint64_t v)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// first q >= from with a[q] >= v (a[from - 1] < v when from > 0): doubling
// steps from `from`, then a binary search in the last step (a leaf holds a
// few dozen runs, so this takes a few loads where a search over all runs
// would take about 25)
__device__ __forceinline__ int64_t lower_bound_from(const uint64_t *a, int64_t n, int64_t from,
                                                    uint64_t v)
{
    if (from >= n || a[from] >= v) return from;
    int64_t base = from, step = 1;  // a[base] < v
    while (base + step < n && a[base + step] < v) {
        base += step;
        step <<= 1;
    }
    int64_t lo = base + 1, hi = min(base + step, n);  // the answer is in [lo, hi]
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// The fit of leaf l over the run starts [lo, hi) of its keys [K0, K1) by one
// wavefront; returns its error bound (every lane).
__device__ int64_t leaf_fit_one(const uint64_t *starts, int64_t n, uint32_t nl, uint32_t l,
                                uint64_t K0, uint64_t K1, int64_t lo, int64_t hi, int lane,
                                int4 *leaves, int32_t *leaf_lo)
{
    // least squares of y = q - lo against x = starts[q] - K0 over q in [lo, hi)
    double sx = 0, sy = 0, sxx = 0, sxy = 0;
    for (int64_t q = lo + lane; q < hi; q += 64) {
        double x = (double)(starts[q] - K0), y = (double)(q - lo);
        sx += x; sy += y; sxx += x * x; sxy += x * y;
    }
    for (int o = 32; o > 0; o >>= 1) {
        sx += __shfl_xor(sx, o, 64);
        sy += __shfl_xor(sy, o, 64);
        sxx += __shfl_xor(sxx, o, 64);
        sxy += __shfl_xor(sxy, o, 64);
    }
    double cnt = (double)(hi - lo);
    float slope = 0.f, icpt;
    if (hi - lo >= 2) {
        double mx = sx / cnt, my = sy / cnt;
        double var = sxx / cnt - mx * mx, cov = sxy / cnt - mx * my;
        double sl = var > 0 ? cov / var : 0.0;
        if (sl < 0) sl = 0;
        slope = (float)sl;
        icpt = (float)(my - sl * mx + (double)lo);
    } else if (hi - lo == 1) {
        icpt = (float)lo;
    } else {
        icpt = (float)(lo - 1);
    }
    const int4 lf = make_int4((int)(uint32_t)K0, __float_as_int(slope), __float_as_int(icpt), 0);
    // error over every key of [K0, K1): the answer is q on [max(starts[q],K0),
    // min(starts[q+1],K1) - 1] for q in [lo-1, hi-1]; the clamped prediction is
    // monotone, so both ends of each step bound it
    int64_t err = 0;
    if (K1 > K0) {
        for (int64_t q = lo - 1 + lane; q <= hi - 1; q += 64) {
            if (q < 0) continue;  // keys before the first start do not occur (starts[0] = 0)
            uint64_t ka = starts[q] > K0 ? starts[q] : K0;
            uint64_t kb = (q + 1 < n && starts[q + 1] < K1) ? starts[q + 1] - 1 : K1 - 1;
            if (ka > kb) continue;
            int64_t pa = predict_in_leaf(lf, lo, hi, ka), pb = predict_in_leaf(lf, lo, hi, kb);
            int64_t e1 = pa > q ? pa - q : q - pa, e2 = pb > q ? pb - q : q - pb;
            err = max(err, max(e1, e2));
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        int64_t v = __shfl_xor(err, o, 64);
        err = max(err, v);
    }
    if (lane == 0) {
        leaves[l] = make_int4(lf.x, lf.y, lf.z, (int)err);
        leaf_lo[l] = (int32_t)lo;
        if (l == nl - 1) leaf_lo[nl] = (int32_t)n;
    }
    return err;
}

// Each wavefront fits a contiguous chunk of leaves: key range, least-squares
// fit, exact error bound.  A leaf's end (key and run position) is the next
// leaf's start, found from it by doubling steps, and the wave adds the
// largest and the summed error of its leaves to err_stats once.
__global__ void k_leaf_fit(const uint64_t *starts, int64_t n, float a, uint32_t nl, uint64_t total,
                           int4 *leaves, int32_t *leaf_lo, unsigned long long *err_stats)
{
    const int lane = threadIdx.x & 63;
    const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t chunk = ((int64_t)nl + waves - 1) / waves;
    const int64_t l0 = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * chunk;
    const int64_t l1 = min(l0 + chunk, (int64_t)nl);
    unsigned long long emax = 0, esum = 0;
    if (l0 < l1) {
        uint64_t K0 = leaf_first_key((uint32_t)l0, a, nl, total);
        int64_t lo = lower_bound_u64(starts, n, K0);
        for (int64_t l = l0; l < l1; l++) {
            const uint64_t K1 = (l + 1 < nl) ? leaf_first_key((uint32_t)l + 1, a, nl, total) : total;
            const int64_t hi = lower_bound_from(starts, n, lo, K1);
            const int64_t err =
                leaf_fit_one(starts, n, nl, (uint32_t)l, K0, K1, lo, hi, lane, leaves, leaf_lo);
            emax = max(emax, (unsigned long long)err);
            esum += (unsigned long long)err;
            K0 = K1;
            lo = hi;
        }
    }
    if (lane == 0 && esum + emax > 0) {
        atomicMax(&err_stats[0], emax);
        atomicAdd(&err_stats[1], esum);
    }
}


int hilbert_finish(BuildState &B, sba_handle *h, const sba_build_opts &o, hipStream_t st)
{
    const int L = h->level;
    const uint64_t total = (uint64_t)1 << (2 * L);
    if (B.bkeys32) RC(write_runs<uint32_t>(B, h, B.bkeys32, st));
    else RC(write_runs<uint64_t>(B, h, B.bkeys, st));
    const int64_t nr = h->n_runs;
    RC(build_directory(h, st));

    if (o.search == SBA_SEARCH_LEARNED) {
        if (2 * L > 32) return SBA_ELIMIT;  // leaves store 32-bit key bases
        const uint32_t nl = 1u << o.log2_leaves;
        h->log2_leaves = o.log2_leaves;
        uint64_t last = 0;
        RC(B.ws.read(&last, h->starts + (nr - 1), sizeof(uint64_t)));
        RC(B.ws.sync());
        h->root_k0 = 0;
        h->root_a = (float)nl / (float)(last + 1);
        unsigned long long *stats = nullptr;
        RC(B.alloc(&stats, 2));
        HIP_OK(hipMemsetAsync(stats, 0, 2 * sizeof(unsigned long long), st));
        RC(handle_alloc(h, &h->leaves, nl));
        RC(handle_alloc(h, &h->leaf_lo, (int64_t)nl + 1));
        const int64_t fit_blocks = std::min<int64_t>(grid_for((int64_t)nl * 64), 4096);
        hipLaunchKernelGGL(k_leaf_fit, dim3((unsigned)fit_blocks), dim3(256), 0, st, h->starts,
                           nr, h->root_a, nl, total, h->leaves, h->leaf_lo, stats);
        HIP_OK(hipGetLastError());
        unsigned long long hs[2];
        RC(B.ws.read(hs, stats, sizeof(hs)));
        RC(B.ws.sync());
        h->max_leaf_err = (int64_t)hs[0];
        h->mean_leaf_err = (double)hs[1] / (double)nl;
    }
    return 0;
}
