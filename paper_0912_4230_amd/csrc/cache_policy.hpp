// cache_policy.hpp -- which cache policy the populations take in a step.
// Host code without HIP: it also compiles alone.
#pragma once

#include <stddef.h>

#include "lbm.h"

namespace plbm {

inline size_t storage_bytes(int storage)
{
    switch (storage) {
    case LBM_F64: return 8;
    case LBM_F32: return 4;
    default: return 2;
    }
}

inline bool split_storage(int storage) { return storage == LBM_BF16_SPLIT || storage == LBM_F16_SPLIT; }

// Miscible lattices in 16-bit storage keep f and h in paired planes of
// 32-bit words (and split codecs their two masses as one 8-byte pair per
// cell); the planes are padded as planes of 4-byte elements.
inline bool paired_storage(int physics, int storage) { return physics == LBM_MISCIBLE && storage_bytes(storage) == 2; }

// Cache policy of the populations in a step.  Loads (NT): non-temporal, or plain.
// Stores (WT): non-temporal, or written through to the memory side at once (a
// relaxed store of agent scope), which leaves nothing dirty in the L2s for the
// end of the launch and the values in the memory-side cache (256 MB).  The
// launch chooses (cache_policy).
enum {
    CACHE_STREAM = 0,   // non-temporal loads and stores
    CACHE_REUSE = 1,    // plain loads, non-temporal stores
    CACHE_KEEP = 2      // plain loads, stores written through
};

// what the choice depends on, per lattice of a launch
struct CacheLattice {
    int physics, storage, nx;
    bool links, tensor;     // an obstacle mask; a full permeability tensor
    double cells, bytes;    // bytes: the populations (and split masses), both copies
};

// Cache policy of the populations in a step of these lattices (results are
// bitwise the same under all three).  us per step, FP32 miscible unless named,
// CACHE_STREAM / CACHE_REUSE / CACHE_KEEP:
//
// KEEP, when all the launch's populations (both copies) fit in the memory-side
// cache (256 MB): a step then reads what the last one left there, where
// non-temporal stores send it to memory.
//   61^3 (69 MB) 15.4 / 15.7 / 13.6, 83^3 (174 MB) 40 / 39 / 32.6, 94^3 (252 MB)
//   57 / 56 / 46, 98^3 (286 MB) 66 / 63 / 67; 70^3 BF16 (52 MB) 15.3 / 16.1 /
//   14.4, 110^3 BF16 (202 MB) 47 / 46 / 41, 120^3 BF16 (263 MB) 59 / 57 / 60;
//   two-fluid 80^3 36 / 37 / 30; channel FP64 64^3 17 / 18 / 14.
// Lattices that the L2s (32 MB) hold in part step as fast or faster under STREAM:
//   48^3 9.6 / 10.2 / 10.7, 58^3 12.0 / 13.4 / 12.6, 64^3 BF16 9.2 / 10.5 / 10.4;
// the line lies at 62 MB in the miscible model in FP32 and FP64 (96 MB with rows
// of whole lines: 64^3, 80 MB, 14.4 / 15.9 / 14.8), at 50 MB else.  The smallest
// gain again (32^3 FP64 channel, 10 MB, 6.6 / 6.6 / 6.0; 64^3 BF16 channel, 20
// MB, 8.0 / 7.3 / 7.0; miscible 32^3, 10 MB, 7.9 / 7.9 / 7.7, but 40^3, 20 MB,
// 8.3 / 8.9 / 9.0).
//
// REUSE, when lines are read by two waves: rows that are not whole lines put
// most lines across a wave boundary (243 x 251 x 238 970 / 935, tensor 1075 /
// 997; 250^3 988 / 936; 131^3 two-fluid 142 / 135, BF16 93 / 87; channel 150^3
// FP64 201 / 190; where rows are whole lines 256^3 945 / 970, 128^3 two-fluid
// 122 / 128); bounced links read a line once more (10% obstacles 256^3 1120 /
// 1035, BF16 567 / 553).  The paired 16-bit planes of the miscible model gain
// only where rows are not whole sectors of 32 bytes (tensor 243 x 251 x 238 BF16
// 562 / 546; 200^3 BF16 254 / 255), the split forms among them only in larger
// lattices (251^3 BF16 split 621 / 608, 101 x 310 x 299 FP16 split 372 / 365, 200^3
// with 10% obstacles 364 / 354, but 155 x 151 x 140 136.8 / 139.0: the line lies
// between, at 6M cells).  The FP32 tensor step gains with whole lines too where
// it is larger still (224^3 719 / 698, 256^3 1050 / 1025, 320 x 256 x 256 1343 /
// 1302, but 128 x 256 x 300 603 / 611, 192^3 417 / 439, 128^3 125 / 136: 10.5M
// cells).
//
// The free-surface step leaves the gas cells out; KEEP from 50 to 256 MB of
// populations there, STREAM else (us, whole step, STREAM / KEEP: 48^3 FP32 17 MB
// 24.8 / 25.2, 61 x 71 x 81 53 MB 30.0 / 29.4, 101 x 100 x 97 149 MB 34.8 / 32.9,
// FP16 split 82 MB 33.2 / 31.1, 110^3 202 MB 36.4 / 34.3, 128^3 BF16 159 MB 33.6 /
// 33.8; 128^3 319 MB 44.5 / 45.2, 200 x 190 x 180 1040 MB 130 / 139); plain loads
// alone gain nothing.
//
// The lattices of a batch share the launch: their bytes add up, and the larger
// part of their cells decides between REUSE and STREAM.
//
// lbm_step_batch advances groups of lattices one after the other, in launches of
// their own, and a group finds what its last step left only if the others have
// not pushed it out: KEEP is for groups that fit in the cache together (the bytes
// of those that would take it alone; streamed ones do not disturb them).  us per
// step of a batch, 20 miscible steps (first and third edge) and 10 two-fluid
// steps (second), every group by itself / together: 64^3 94^3 64^3 65.7 / 59.1,
// 80^3 80^3 51.7 / 49.2, 90^3 64^3 55.1 / 52.4, BF16 110^3 110^3 75.7 / 71.3.
// Streaming where only one of the two would keep loses: 64^3 90^3 35.6 / 40.0, 96^3
// 80^3 72.5 / 75.2.

constexpr double CACHE_MB = 1e6, CACHE_SIDE = 256 * CACHE_MB;

// the bytes of a launch, and from where on its step gains by KEEP or REUSE
struct CacheLaunch {
    double bytes, low;
};

inline CacheLaunch cache_launch(const CacheLattice *l, int n)
{
    CacheLaunch a = {0.0, 50 * CACHE_MB};
    bool whole_lines = true;
    for (int i = 0; i < n; ++i) {
        whole_lines = whole_lines && l[i].nx * storage_bytes(l[i].storage) % 128 == 0;
        a.bytes += l[i].bytes;
    }
    if (l->physics == LBM_MISCIBLE && !paired_storage(l->physics, l->storage)) a.low = (whole_lines ? 96 : 62) * CACHE_MB;
    return a;
}

// The bytes of a launch that steps fastest under KEEP when it has the cache to
// itself, else 0.
inline double keep_bytes(const CacheLattice *l, int n)
{
    const CacheLaunch a = cache_launch(l, n);
    const double tiny = (l->physics == LBM_FREESURF ? 0 : (l->physics == LBM_SINGLE ? 24 : 12)) * CACHE_MB;
    return a.bytes <= tiny || (a.bytes >= a.low && a.bytes <= CACHE_SIDE) ? a.bytes : 0.0;
}

// keep: keep_bytes of all the launches of the step, together
inline int cache_policy(const CacheLattice *l, int n, double keep)
{
    if (keep <= CACHE_SIDE && keep_bytes(l, n) > 0.0) return CACHE_KEEP;
    if (l->physics == LBM_FREESURF) return CACHE_STREAM;
    double cells = 0, reuse = 0;
    for (int i = 0; i < n; ++i) {
        const CacheLattice &c = l[i];
        const bool paired = paired_storage(c.physics, c.storage);
        const size_t row = c.nx * storage_bytes(c.storage) * (paired ? 2 : 1);
        const bool shared = row % (paired ? 32 : 128) != 0 || c.links;
        cells += c.cells;
        if (paired ? shared && (!split_storage(c.storage) || c.cells > 6e6)
                   : shared || (c.tensor && c.storage == LBM_F32 && c.cells > 10.5e6))
            reuse += c.cells;
    }
    const CacheLaunch a = cache_launch(l, n);
    return a.bytes > a.low && 2 * reuse > cells ? CACHE_REUSE : CACHE_STREAM;
}

}  // namespace plbm
