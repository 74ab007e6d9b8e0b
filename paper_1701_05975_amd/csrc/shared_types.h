// shared_types.h -- plain data layouts shared by host code and kernels.
#pragma once

#include <stddef.h>
#include <stdint.h>

#define BC_INF 0x7fffffffu
#define WAVE 64
// Default degree thresholds (bc_options): more than BC_DEF_WAVE_DEG in-arcs take a
// wave in the plain form's counts; in the batched expansion more than BC_HUB_DEG
// arcs -> the whole workgroup (only graphs that have such a vertex pay for the step).
#define BC_DEF_LANE_DEG 8
#define BC_DEF_WAVE_DEG 64
#define BC_HUB_DEG 512
// Graphs of at most NARROW_DEG arcs a vertex (grids): short queues are expanded
// by groups of NARROW_VW lanes (k_batched)
#define NARROW_DEG 8
#define NARROW_VW 4
// Most buckets of the far-bucket ring (batched form).
#define BC_BUCKETS_MAX 128

// ---------------------------------------------------------------------------
// Graph as seen by the kernels.
//
// The arcs leaving v are row[v] .. row[v+1]-1 (CSR, Sec. 3.1).  When the
// head index and the weight fit together in 32 bits the arc is one word,
// head << wshift | (weight - 1); otherwise `arc` holds the heads and `wt`
// the weights.  trow/tarc/twt are the arcs entering each vertex (the same
// arrays as row/arc/wt for an undirected graph).
// ---------------------------------------------------------------------------
struct DevGraph {
    const uint32_t *row;
    const uint32_t *arc;
    const int32_t *wt;
    const uint32_t *trow;
    const uint32_t *tarc;
    const int32_t *twt;
    int32_t n;
    int32_t n_act; // vertices from n_act on have no in-arcs: no source reaches them
                   // (each is reached only as a source itself)
    uint32_t wshift;
    uint32_t wmask;
};

// ---------------------------------------------------------------------------
// Per-source state ("slab").  One slab per source in flight.
//
// Distances, the most often read field (every arc relaxation and every
// tightness test reads one at a random vertex), stay a dense array so that
// a cache line holds as many of them as possible.  The other per-vertex
// fields, which the count, dependency and split passes touch together,
// share one 32-byte record, so that such a visit of a random vertex fetches
// one line instead of one line per field.  Record layout:
// ---------------------------------------------------------------------------
#define VREC_BYTES 32
// (fields that one pass reads or writes together lie in one 16-byte half: a
// scattered access costs the same at 4 and at 16 bytes)
#define VREC_LEVEL 0  // i32 number of the count round the vertex became final in
#define VREC_PRED1 4  // i32 the only DAG predecessor, or -(m + 1): m of them in preds[]
#define VREC_SIGMA 8  // u64 shortest-path count (plain form: 0 = not yet final)
#define VREC_DELTA 16 // f64 dependency (plain form: negative = not yet final); before the
                      // vertex is counted its predecessor key (batched form)
#define VREC_FLAGS 24 // i32 flags, and the count of ties (VFLAG_*, TIE_SHIFT)
#define VREC_STAMP 28 // i32 tag of the latest near queue an improvement put the vertex in

// Byte offsets of the slab arrays inside one slot (all 256-byte aligned).
struct SlabLayout {
    size_t d, rec, bcp, order, qa, qb, fa, fb, bx, oa, ob, band_off, hdr, preds, stride;
};

// ---------------------------------------------------------------------------
// Error reporting shared by all kernels: err[0] is a bit set, err[1] the
// smallest source-list index whose path counts overflowed.
// ---------------------------------------------------------------------------
#define BC_ERRBIT_SIGMA 1
#define BC_ERRBIT_INTERNAL 2
#define BC_ERRBIT_SOURCE 4

struct DevStats {
    unsigned long long reached, arcs, dag, improvements, bands, iterations, sigma_rounds,
        delta_rounds;
    // device wall-clock ticks summed over workgroups: initialisation, frontier
    // expansion, count rounds, dependency rounds, far-pile splits
    unsigned long long ticks[5];
};

// Distance bounds of the team form (one byte each): steps above a base, or none
#define SEEN_NONE 0xffu
#define SEEN_WIN 254u
#define SEEN_REBASE 32u // re-base once the band threshold is this many steps above
