// build_state.h -- temporaries shared by the build stages (build.hip,
// hilbert.hip).  Not part of the public ABI.
#pragma once

#include <algorithm>
#include <vector>

#include "sba_internal.h"

#define SC_SLOTS 32
#define SC_READ 20
// slot of the set table's counter
#define SC_SET_N 18
#define SC_TICKET 20  // workgroups of k_poly_bbox that have ended

struct BuildState {
    explicit BuildState(hipStream_t s) : st(s), ws(s) {}
    hipStream_t st;
    Workspace ws;  // temporaries; returned (after a sync) when the build ends

    template <typename T>
    int alloc(T **p, int64_t n)
    {
        return ws.alloc(p, n);
    }
    void release(void *p) { ws.put(p); }

    // device scalars of the build (error bits, sizes, scan totals) that are
    // read back together: slots [0, SC_READ) in one copy
    int64_t *sc = nullptr;

    bool boundary_only = false;  // no interior spans: B(P) only
    bool centre = false;         // centre-sampled cells: crossings of the centre lines only

    // clip window in coordinates, [wx0, wx1) x [wy0, wy1)
    bool window = false;
    int64_t wx0 = 0, wy0 = 0, wx1 = 0, wy1 = 0;
    bool empty = false;  // the window holds no cell of any polygon
    // Hilbert key grid given by the caller (key_level 0: the stored box's own)
    int32_t key_level = 0;
    int64_t key_i0 = 0, key_j0 = 0;
    // edges: (x1,y1,x2,y2) and polygon id, one per vertex
    int4 *edges = nullptr;
    int32_t *epoly = nullptr;
    int64_t n_edges = 0;
    int xbits = 0, rbits = 0;    // event key fields: row << xbits | x
    int64_t NB = 0;              // boundary intervals (events [0, 2 NB) until sorted)
    uint64_t *evkey = nullptr;
    uint32_t *evpay = nullptr;
    // row segments of constant polygon set: row r's are [seg_beg[r], seg_end[r])
    int64_t NS = 0;
    int64_t *seg_beg = nullptr, *seg_end = nullptr;
    int32_t *seg_x0 = nullptr, *seg_x1 = nullptr;
    uint32_t *seg_code = nullptr;
    // Hilbert layout: unique keys of boundary cells, ascending (bkeys, or
    // bkeys32 with each cell's segment in bseg from the row sweep, which
    // takes 32-bit keys where they fit)
    int (*on_boundary_events)(BuildState &, sba_handle *, hipStream_t) = nullptr;
    uint64_t *bkeys = nullptr;
    uint32_t *bkeys32 = nullptr, *bseg = nullptr;
    int64_t nbkeys = 0;
};

int build_segments(const sba_polygons *polys, int64_t eps, hipStream_t st, sba_handle *h,
                   BuildState &B, bool need_boundary_cells);
// segments and sets row by row in LDS (rows.hip); *taken: done, else the
// caller takes the global sorts; *one: the sets were numbered by one workgroup
int rows_coverage(const sba_polygons *polys, const int4 *bbox, int64_t nv,
                  hipStream_t st, sba_handle *h, BuildState &B, int paths_off, bool *taken,
                  bool *one);
int hilbert_prepare(BuildState &B, sba_handle *h);
// the key grid's level (SBA_ELIMIT above 21)
int hilbert_level(const BuildState &B, sba_handle *h);
int hilbert_finish(BuildState &B, sba_handle *h, const sba_build_opts &o, hipStream_t st);
