// sets.hip -- the polygon sets of multi-polygon segments: distinct keys,
// their numbers in key order, the handle's set table, and the segments' codes
// (step 5 of the build, see build.hip; keys: sets.h).
#include "sets.h"

#define SEG_BLOCK 1024
#define SEG_WAVES (SEG_BLOCK / 64)
#define SEG_DBITS 7
#define SEG_RADIX (1 << SEG_DBITS)
#define SEG_ROUNDS (SET_CAP / SEG_BLOCK)

// exclusive scan across a workgroup of SEG_BLOCK lanes (wsum: SEG_WAVES words)
__device__ __forceinline__ uint32_t seg_excl_scan(uint32_t v, uint32_t *wsum)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (int k = 0; k < w; k++) before += wsum[k];
    __syncthreads();
    return before + incl - v;
}

// Stable LSD radix sort, by one workgroup of SEG_BLOCK lanes, of n <= SET_CAP
// keys in LDS by their bits [0, kbits): 7-bit digits; wave w ranks its own
// rpw x 64 consecutive keys (rpw = the fewest rounds that spread the keys over
// every wave), 64 at a time, equal digits finding each other with SEG_DBITS
// ballots.  The keys end in *src (the two buffers swap once per pass); wcnt
// holds SEG_WAVES x SEG_RADIX counters.
__device__ __forceinline__ void lds_radix(uint64_t *&src, uint64_t *&dst, int n, int kbits,
                                          uint32_t *wcnt, uint32_t *doff, uint32_t *wtot)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int rpw = (n + SEG_BLOCK - 1) / SEG_BLOCK;  // <= SEG_ROUNDS
    const int wbase = w * 64 * rpw;
    for (int shift = 0; shift < kbits; shift += SEG_DBITS) {
        for (int k = threadIdx.x; k < SEG_WAVES * SEG_RADIX; k += SEG_BLOCK) wcnt[k] = 0;
        __syncthreads();
        uint64_t kk[SEG_ROUNDS];
        uint32_t loc[SEG_ROUNDS];
#pragma unroll
        for (int q = 0; q < SEG_ROUNDS; q++) {
            // rounds past the wave's share or past the keys are skipped
            // (uniform per wave)
            if (q >= rpw || wbase + q * 64 >= n) break;
            const int idx = wbase + q * 64 + lane;
            const bool valid = idx < n;
            const uint64_t key = valid ? src[idx] : 0ull;
            kk[q] = key;
            const uint32_t d = (uint32_t)(key >> shift) & (SEG_RADIX - 1);
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < SEG_DBITS; b++) {
                const uint64_t bal = __ballot((d >> b) & 1u);
                peers &= ((d >> b) & 1u) ? bal : ~bal;
            }
            const uint32_t old = wcnt[w * SEG_RADIX + d];
            loc[q] = old + (uint32_t)__popcll(peers & lt);
            __builtin_amdgcn_wave_barrier();
            if (valid && (peers & lt) == 0) wcnt[w * SEG_RADIX + d] = old + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // digit d = threadIdx.x: offsets of the waves within the digit, then
        // the digit's first slot
        uint32_t run = 0, incl = 0;
        if (threadIdx.x < SEG_RADIX) {
            const int d = threadIdx.x;
#pragma unroll
            for (int k = 0; k < SEG_WAVES; k++) {
                const uint32_t c = wcnt[k * SEG_RADIX + d];
                wcnt[k * SEG_RADIX + d] = run;
                run += c;
            }
            incl = run;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
                if (lane >= o) incl += u;
            }
            if (lane == 63) wtot[w] = incl;
        }
        __syncthreads();
        if (threadIdx.x < SEG_RADIX) {
            uint32_t before = 0;
            for (int k = 0; k < w; k++) before += wtot[k];
            doff[threadIdx.x] = before + incl - run;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < SEG_ROUNDS; q++) {
            const int idx = wbase + q * 64 + lane;
            if (q < rpw && idx < n) {
                const uint32_t d = (uint32_t)(kk[q] >> shift) & (SEG_RADIX - 1);
                dst[doff[d] + wcnt[w * SEG_RADIX + d] + loc[q]] = kk[q];
            }
        }
        __syncthreads();
        uint64_t *t = src;
        src = dst;
        dst = t;
    }
}

// number of members of the set with key k; *loc = -1 when they are the fields
// of the key, else where they are in mem_ids
__device__ __forceinline__ int set_members(uint64_t k, int fb, const uint64_t *memloc, int64_t *loc)
{
    if (k < (1ull << (3 * fb))) {
        const uint64_t fm = (1ull << fb) - 1;
        *loc = -1;
        return ((k & fm) != 0) + (((k >> fb) & fm) != 0) + (((k >> (2 * fb)) & fm) != 0);
    }
    const uint64_t m = memloc[k - (1ull << (3 * fb))];
    *loc = (int64_t)(m >> 6);
    return (int)(m & 63);
}

__device__ __forceinline__ void set_write(uint64_t k, int fb, int c, int64_t loc,
                                          const int32_t *mem_ids, int32_t *out)
{
    if (loc < 0) {
        const uint64_t fm = (1ull << fb) - 1;
        for (int t = 0; t < c; t++) out[t] = (int32_t)((k >> (fb * t)) & fm) - 1;
    } else {
        for (int t = 0; t < c; t++) out[t] = mem_ids[loc + t];
    }
}

__device__ __forceinline__ uint32_t set_find(const SetTab &T, uint64_t k)
{
    const uint32_t mask = (1u << T.hb) - 1u;
    uint32_t s = set_hash(k, T.hb);
    // every key asked for was inserted: it is ahead of any empty slot
    for (uint32_t q = 0; q <= mask && T.tab[s] != k; q++) s = (s + 1) & mask;
    return s;
}

// One workgroup, n <= SET_CAP distinct keys, the table's and the listed ones of
// larger sets (among nlist places): sorts them in LDS, numbers the sets in key
// order, lays out and fills the set table and leaves each key's number in rank,
// a larger set's as its segment's code.  Dynamic LDS: two buffers of `cap` keys (n rounded up) and
// the digit counters.
__global__ __launch_bounds__(SEG_BLOCK) void k_set_table(SetTab T, int ntab, int n, int nlist,
                                                         int cap, int kbits, int fb,
                                                         const uint64_t *memloc,
                                                         const int32_t *mem_ids, int64_t *set_off,
                                                         int32_t *set_ids, uint32_t *seg_code)
{
    extern __shared__ __align__(16) uint64_t set_lds[];
    uint64_t *src = set_lds, *dst = set_lds + cap;
    uint32_t *wcnt = (uint32_t *)(set_lds + 2 * cap);
    __shared__ uint32_t doff[SEG_RADIX];
    __shared__ uint32_t wtot[SEG_RADIX / 64];
    __shared__ uint32_t wsum[SEG_WAVES];
    __shared__ int at;
    if (threadIdx.x == 0) at = ntab;
    for (int i = threadIdx.x; i < ntab; i += SEG_BLOCK) src[i] = T.list[i];
    __syncthreads();
    for (int i = threadIdx.x; i < nlist; i += SEG_BLOCK) {
        const uint64_t k = T.large[i];
        if (k == SET_EMPTY) continue;
        const int to = atomicAdd(&at, 1);
        if (to < n) src[to] = k;
    }
    __syncthreads();
    lds_radix(src, dst, n, kbits, wcnt, doff, wtot);
    // set r = src[r]: sizes, offsets (each lane `per` consecutive sets)
    const int per = (n + SEG_BLOCK - 1) / SEG_BLOCK;
    const int i0 = threadIdx.x * per, i1 = min(i0 + per, n);
    uint32_t sum = 0;
    int64_t loc;
    for (int i = i0; i < i1; i++) sum += (uint32_t)set_members(src[i], fb, memloc, &loc);
    uint32_t off = seg_excl_scan(sum, wsum);
    for (int i = i0; i < i1; i++) {
        const uint64_t k = src[i];
        const int c = set_members(k, fb, memloc, &loc);
        set_off[i] = off;
        set_write(k, fb, c, loc, mem_ids, set_ids + off);
        if (nlist && loc >= 0) seg_code[k - (1ull << (3 * fb))] = CODE_SET_BASE + (uint32_t)i;
        else T.rank[set_find(T, k)] = (uint32_t)i;
        off += (uint32_t)c;
    }
    if (threadIdx.x == SEG_BLOCK - 1) set_off[n] = off;
}

// sorted distinct keys: sizes, and the number of each key's slot
__global__ void k_set_rank(const uint64_t *key, const uint32_t *slot, int64_t n, int fb,
                           const uint64_t *memloc, uint32_t *rank, int64_t *sz)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    int64_t loc;
    sz[t] = set_members(key[t], fb, memloc, &loc);
    rank[slot[t]] = (uint32_t)t;
}

__global__ void k_set_ids(const uint64_t *key, int64_t n, int fb, const uint64_t *memloc,
                          const int32_t *mem_ids, const int64_t *set_off, int32_t *set_ids)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    int64_t loc;
    const int c = set_members(key[t], fb, memloc, &loc);
    set_write(key[t], fb, c, loc, mem_ids, set_ids + set_off[t]);
}

// SEG_SLOT codes of the segments to set codes, a wavefront per row, which also
// lays out the row's larger sets
__global__ __launch_bounds__(256) void k_set_codes(const int64_t *seg_beg, const int64_t *seg_end,
                                                   int64_t gh, const uint32_t *rank,
                                                   uint32_t *seg_code, LargeSets G)
{
    const int lane = threadIdx.x & 63;
    const int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (r >= gh) return;
    const uint32_t ids = G.sets ? G.row_ids[r] : 0u;
    const int64_t first = ids ? G.first + G.sets[r] : 0, to = ids ? G.first_id + G.ids[r] : 0;
    int64_t from = -1;  // of the row's members in mem_ids
    for (int64_t q0 = seg_beg[r], e = seg_end[r]; q0 < e; q0 += 64) {
        const int64_t q = q0 + lane;
        const uint32_t c = q < e ? seg_code[q] : 0u;
        const bool large = ids && (c & SEG_SLOT) && (c & SEG_LARGE);
        const uint64_t any = __ballot(large);
        const int64_t loc = large ? (int64_t)(G.memloc[q] >> 6) : 0;
        if (any) {
            const int64_t least = __shfl((long long)loc, __ffsll((unsigned long long)any) - 1, 64);
            if (from < 0) from = least;
        }
        if (large) {
            const int64_t k = first + (c & (SEG_LARGE - 1));
            G.set_off[k] = to + (loc - from);
            seg_code[q] = CODE_SET_BASE + (uint32_t)k;
        } else if (c & SEG_SLOT) {
            seg_code[q] = CODE_SET_BASE + rank[c & ~SEG_SLOT];
        }
    }
    for (uint32_t t = lane; t < ids; t += 64) G.set_ids[to + t] = G.mem_ids[from + t];
}

__global__ void k_set_widen(const uint32_t *a, int64_t n, int64_t *b, int64_t *end, int64_t total)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) b[t] = a[t];
    if (t == 0) *end = total;
}

// the multi segments' keys through the table; neighbouring multi segments
// mostly share their set, which the table's read sees without an atomic
__global__ void k_set_insert(const uint64_t *key, const uint32_t *val, int64_t n, int fb,
                             const uint64_t *memloc, SetTab T, uint32_t *seg_code)
{
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n || set_full(T)) return;
    int64_t loc;
    const uint64_t k = key[m];
    seg_code[val[m]] = SEG_SLOT | set_insert(T, k, (uint32_t)set_members(k, fb, memloc, &loc));
}

// sorted multi segments: first segment of each key, sizes, the table, codes
__global__ void k_flag_first_key(const uint64_t *key, int64_t n, int64_t *flag)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) flag[t] = (t == 0 || key[t] != key[t - 1]) ? 1 : 0;
}

__global__ void k_set_sizes(const uint64_t *key, const int64_t *gexcl, int64_t n, int fb,
                            const uint64_t *memloc, int64_t *set_sz)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    int64_t loc;
    if (t == 0 || key[t] != key[t - 1]) set_sz[gexcl[t]] = set_members(key[t], fb, memloc, &loc);
}

__global__ void k_set_fill(const uint64_t *key, const uint32_t *val, const int64_t *gexcl,
                           int64_t n, int fb, const uint64_t *memloc, const int32_t *mem_ids,
                           const int64_t *set_off, int32_t *set_ids, uint32_t *seg_code)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const bool first = (t == 0 || key[t] != key[t - 1]);
    const int64_t g = gexcl[t] + (first ? 1 : 0) - 1;
    if (first) {
        int64_t loc;
        const int c = set_members(key[t], fb, memloc, &loc);
        set_write(key[t], fb, c, loc, mem_ids, set_ids + set_off[g]);
    }
    seg_code[val[t]] = CODE_SET_BASE + (uint32_t)g;
}

// ---------------------------------------------------------------- host

// A partition's distinct sets are its shared sides and corners, a few per
// polygon: 16 slots a polygon (at least 2^15, at most 2^22), a quarter of them
// usable, hold those; more (deep overlaps) go through the list.
int sets_table(SetStage &S, BuildState &B, int32_t np, bool fill)
{
    SetTab &T = S.tab;
    T.hb = 15;
    while (T.hb < 22 && ((int64_t)1 << T.hb) < (int64_t)16 * np) T.hb++;
    T.cap = 1u << (T.hb - 2);
    RC(B.alloc(&T.tab, set_tab_words(T)));
    T.large = T.tab + ((int64_t)1 << T.hb);
    RC(B.alloc(&T.rank, (int64_t)1 << T.hb));
    RC(B.alloc(&T.list, T.cap));
    RC(B.alloc(&T.lslot, T.cap));
    T.cnt = (unsigned long long *)(B.sc + SC_SET_N);
    if (fill) HIP_OK(hipMemsetAsync(T.tab, 0xff, sizeof(uint64_t) * set_tab_words(T), B.st));
    return 0;
}

void sets_release(SetStage &S, BuildState &B)
{
    for (void *p : {(void *)S.tab.tab, (void *)S.tab.rank, (void *)S.tab.list, (void *)S.tab.lslot,
                    (void *)S.memloc})
        B.release(p);
    S.tab = SetTab{};
    S.memloc = nullptr;
}

static int key_bits(const SetStage &S, int64_t slots)
{
    return bits_for(((uint64_t)1 << (3 * S.fb)) + (uint64_t)slots);
}

int sets_from_table(SetStage &S, BuildState &B, sba_handle *h, int64_t NM, int64_t NMEM,
                    int64_t nset, int64_t nids, int64_t slots, int64_t nlarge, int64_t nlargeids,
                    const uint32_t *row_large, hipStream_t st)
{
    SetTab &T = S.tab;
    const int kbits = key_bits(S, slots);
    RC(handle_alloc(h, &h->set_off, NM + 1));
    RC(handle_alloc(h, &h->set_ids, NMEM));
    S.one_workgroup = nset + nlarge <= SET_CAP;
    // all by one workgroup, or the larger sets row by row (three more launches)
    const bool listed = nlarge && S.one_workgroup && nlargeids <= 4 * LARGE_FEW;
    if (nset + (listed ? nlarge : 0) == 0) {
    } else if (nset <= SET_CAP) {
        const int64_t n = nset + (listed ? nlarge : 0);
        const int cap = (int)((n + 63) & ~(int64_t)63);
        constexpr int wc = SEG_WAVES * SEG_RADIX * (int)sizeof(uint32_t);
        (void)hipFuncSetAttribute((const void *)k_set_table,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 16 * SET_CAP + wc);
        (void)hipGetLastError();
        hipLaunchKernelGGL(k_set_table, dim3(1), dim3(SEG_BLOCK), 16 * cap + wc, st, T, (int)nset,
                           (int)n, listed ? (int)((nlargeids + 3) / 4) : 0, cap, kbits, S.fb,
                           S.memloc, S.mem_ids, h->set_off, h->set_ids, B.seg_code);
    } else {
        int64_t *sz = nullptr;
        RC(B.alloc(&sz, nset));
        RC(radix_sort_u64_ws(&T.list, &T.lslot, nset, kbits, B.ws));
        hipLaunchKernelGGL(k_set_rank, dim3(grid_for(nset)), dim3(256), 0, st, T.list, T.lslot,
                           nset, S.fb, S.memloc, T.rank, sz);
        HIP_OK(hipGetLastError());
        RC(scan_exclusive_i64(sz, h->set_off, nset, h->set_off + nset, st, &B.ws));
        hipLaunchKernelGGL(k_set_ids, dim3(grid_for(nset)), dim3(256), 0, st, T.list, nset, S.fb,
                           S.memloc, S.mem_ids, h->set_off, h->set_ids);
        B.release(sz);
    }
    LargeSets G{};
    int64_t *before = nullptr;
    if (nlarge && !listed) {
        const int64_t gh = h->gh;
        RC(B.alloc(&before, 2 * gh));
        hipLaunchKernelGGL(k_set_widen, dim3(grid_for(2 * gh)), dim3(256), 0, st, row_large, 2 * gh,
                           before, h->set_off + nset + nlarge, nids + nlargeids);
        HIP_OK(hipGetLastError());
        const int64_t *in[2] = {before, before + gh}, n[2] = {gh, gh};
        int64_t *out[2] = {before, before + gh}, *sum[2] = {nullptr, nullptr};
        RC(scan_exclusive_i64_multi(2, in, out, n, sum, st, &B.ws));
        G = LargeSets{before, before + gh, row_large + gh, S.memloc, S.mem_ids, h->set_off,
                      h->set_ids, nset, nids};
    }
    hipLaunchKernelGGL(k_set_codes, dim3(grid_for(h->gh * 64)), dim3(256), 0, st, B.seg_beg,
                       B.seg_end, h->gh, T.rank, B.seg_code, G);
    HIP_OK(hipGetLastError());
    B.release(before);
    h->n_sets = nset + nlarge;
    h->n_set_ids = nids + nlargeids;
    return 0;
}

int sets_hash_list(SetStage &S, BuildState &B, sba_handle *h, const uint64_t *mkey,
                   const uint32_t *mval, int64_t NM, int64_t NMEM, int64_t slots, hipStream_t st,
                   bool *done)
{
    *done = false;
    RC(sets_table(S, B, h->n_polys, true));
    hipLaunchKernelGGL(k_set_insert, dim3(grid_for(NM)), dim3(256), 0, st, mkey, mval, NM, S.fb,
                       S.memloc, S.tab, B.seg_code);
    HIP_OK(hipGetLastError());
    int64_t hsc[SC_READ];
    RC(B.ws.read(hsc, B.sc, sizeof(hsc)));
    RC(B.ws.sync());
    const int64_t nset = set_count(hsc[SC_SET_N]);
    if (nset > (int64_t)S.tab.cap) return 0;
    RC(sets_from_table(S, B, h, NM, NMEM, nset, set_ids_count(hsc[SC_SET_N]), slots, 0, 0, nullptr,
                       st));
    *done = true;
    return 0;
}

int sets_from_list(SetStage &S, BuildState &B, sba_handle *h, uint64_t *mkey, uint32_t *mval,
                   int64_t NM, int64_t NMEM, int64_t slots, hipStream_t st)
{
    const int kbits = key_bits(S, slots);
    int64_t *g = nullptr, *sz = nullptr, *tot = B.sc + 8;
    RC(handle_alloc(h, &h->set_off, NM + 1));
    RC(handle_alloc(h, &h->set_ids, NMEM));
    RC(B.alloc(&g, NM + 1));
    RC(radix_sort_u64_ws(&mkey, &mval, NM, kbits, B.ws));
    hipLaunchKernelGGL(k_flag_first_key, dim3(grid_for(NM)), dim3(256), 0, st, mkey, NM, g);
    HIP_OK(hipGetLastError());
    RC(scan_exclusive_i64(g, g, NM, tot, st, &B.ws));
    RC(B.alloc(&sz, NM + 1));
    HIP_OK(hipMemsetAsync(sz, 0, sizeof(int64_t) * (NM + 1), st));
    hipLaunchKernelGGL(k_set_sizes, dim3(grid_for(NM)), dim3(256), 0, st, mkey, g, NM, S.fb,
                       S.memloc, sz);
    HIP_OK(hipGetLastError());
    RC(scan_exclusive_i64(sz, h->set_off, NM, h->set_off + NM, st, &B.ws));
    hipLaunchKernelGGL(k_set_fill, dim3(grid_for(NM)), dim3(256), 0, st, mkey, mval, g, NM, S.fb,
                       S.memloc, S.mem_ids, h->set_off, h->set_ids, B.seg_code);
    HIP_OK(hipGetLastError());
    int64_t ns = 0, nids = 0;
    RC(B.ws.read(&ns, tot, sizeof(int64_t)));
    RC(B.ws.read(&nids, h->set_off + NM, sizeof(int64_t)));
    RC(B.ws.sync());
    h->n_sets = ns;
    h->n_set_ids = nids;
    B.release(g);
    B.release(sz);
    B.release(mkey);
    B.release(mval);
    return 0;
}
