// sets.h -- the polygon sets of multi-polygon segments (sets.hip), shared by
// the build's stages.  Not part of the public ABI.
#pragma once

#include "sba_internal.h"
#include "build_state.h"

// A multi-polygon segment's code until the sets are numbered: SEG_SLOT | the
// hash slot of its set key.
#define SEG_SLOT 0x80000000u
// From the row sweep, a larger set's (of more than three polygons, which is not
// shared): SEG_SLOT | SEG_LARGE | its number among its row's larger sets.
#define SEG_LARGE 0x40000000u

// The key of a set of two or three polygons holds its ids + 1, ascending, in
// fields of fb bits; a larger set is not shared and has the key 2^(3 fb) + the
// index of its segment (memloc[index]: where its members are in mem_ids << 6 |
// their number).
//
// Distinct keys: an open-addressing table of 2^hb keys, each first insert
// appending its key and slot to a list (cap entries).  *cnt holds the number
// of inserts above bit 32 and the sum of their sets' sizes below it (one
// addition for both).  More distinct keys than the list takes, or a run of
// SET_PROBES taken slots, leaves the number above cap.
struct SetTab {
    uint64_t *tab = nullptr;
    uint32_t *rank = nullptr;  // [2^hb] number of the slot's set
    uint64_t *list = nullptr;
    uint32_t *lslot = nullptr;
    unsigned long long *cnt = nullptr;
    uint64_t *large = nullptr;  // [LARGE_FEW] behind tab: keys of the row sweep's larger
                                // sets, at a quarter of their first member's place
    int hb = 0;
    uint32_t cap = 0;
};

// The row sweep's larger sets, numbered after the others in order of their
// segments, where they are too many for one workgroup (which then numbers all):
// of each row how many, and their members, which lie together in
// mem_ids in that order (memloc: of the first one's and the others' segments).
struct LargeSets {
    const int64_t *sets = nullptr, *ids = nullptr;  // [gh] numbers before each row
    const uint32_t *row_ids = nullptr;              // [gh]
    const uint64_t *memloc = nullptr;
    const int32_t *mem_ids = nullptr;
    int64_t *set_off = nullptr;                     // the handle's table
    int32_t *set_ids = nullptr;
    int64_t first = 0, first_id = 0;                // sets and members before all of them
};

struct SetStage {
    int fb = 0;
    uint64_t *memloc = nullptr;
    const int32_t *mem_ids = nullptr;
    SetTab tab;
    bool one_workgroup = false;  // the sets were numbered by one workgroup
};

#define SET_EMPTY (~(uint64_t)0)
#define SET_PROBES 64
#define SET_ASK 12
// distinct sets that one workgroup sorts in LDS
#define SET_CAP 8192
// quarters of the row sweep's larger sets' members up to which these are listed
// for it too
#define LARGE_FEW 4096

// words to empty (SET_EMPTY): the slots and the list of larger sets
inline int64_t set_tab_words(const SetTab &T) { return ((int64_t)1 << T.hb) + LARGE_FEW; }

__host__ __device__ inline int64_t set_count(int64_t cnt) { return (int64_t)((uint64_t)cnt >> 32); }
__host__ __device__ inline int64_t set_ids_count(int64_t cnt) { return cnt & 0xffffffffll; }

__device__ __forceinline__ bool set_full(const SetTab &T)
{
    return (*(const volatile unsigned long long *)T.cnt >> 32) > T.cap;
}

__device__ __forceinline__ uint32_t set_hash(uint64_t k, int hb)
{
    return (uint32_t)((k * 0x9e3779b97f4a7c15ull) >> (64 - hb));
}

// the key's slot (d: the size of its set).  Whether the table is full is asked
// only after a run of taken slots, as an overfull table has them: one read of
// the shared counter by every wavefront of a sweep, about 9 ns each, one after
// another, made 50,000 rows take 2.8 ms instead of 1.8.
__device__ __forceinline__ uint32_t set_insert(const SetTab &T, uint64_t key, uint32_t d)
{
    const uint32_t mask = (1u << T.hb) - 1u;
    uint32_t s = set_hash(key, T.hb);
    for (int probe = 0; probe < SET_PROBES; probe++) {
        if (probe == SET_ASK && set_full(T)) return 0;
        // a slot that already holds the key is seen without an atomic
        const uint64_t seen = *(const volatile uint64_t *)(T.tab + s);
        if (seen == key) return s;
        if (seen == SET_EMPTY) {
            const uint64_t prev = atomicCAS((unsigned long long *)(T.tab + s),
                                            (unsigned long long)SET_EMPTY, (unsigned long long)key);
            if (prev == SET_EMPTY) {
                const unsigned long long at = atomicAdd(T.cnt, (1ull << 32) | d) >> 32;
                if (at < T.cap) {
                    T.list[at] = key;
                    T.lslot[at] = s;
                }
                return s;
            }
            if (prev == key) return s;
        }
        s = (s + 1) & mask;
    }
    atomicMax(T.cnt, (unsigned long long)(T.cap + 1) << 32);
    return 0;
}

// an empty table for the sets of np polygons
int sets_table(SetStage &S, BuildState &B, int32_t np, bool fill);
// number the nset distinct sets (nids members) of the table in key order, lay
// out h's set table (NM multi segments with NMEM members bound its size) and
// replace the SEG_SLOT codes of B's segments; slots: segment indices.  The row
// sweep's larger sets: nlarge with nlargeids members, and per row ([gh] each, at
// row_large) how many of both.
int sets_from_table(SetStage &S, BuildState &B, sba_handle *h, int64_t NM, int64_t NMEM,
                    int64_t nset, int64_t nids, int64_t slots, int64_t nlarge, int64_t nlargeids,
                    const uint32_t *row_large, hipStream_t st);
// the same from the list of multi segments (key, segment), sorted as a whole;
// mkey and mval come from B.ws and go back to it
int sets_from_list(SetStage &S, BuildState &B, sba_handle *h, uint64_t *mkey, uint32_t *mval,
                   int64_t NM, int64_t NMEM, int64_t slots, hipStream_t st);
// the list through the table: *done when it held them all
int sets_hash_list(SetStage &S, BuildState &B, sba_handle *h, const uint64_t *mkey,
                   const uint32_t *mval, int64_t NM, int64_t NMEM, int64_t slots, hipStream_t st,
                   bool *done);
void sets_release(SetStage &S, BuildState &B);
