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
    int solutes;            // of the miscible model, else 1
    bool links, tensor;     // an obstacle mask; a full permeability tensor
    double cells, bytes;    // bytes: the populations (and split masses), both copies
    double medium;          // bytes of the other fields that a step reads
    double bounced;         // share of the cells that have a link cut by the mask
};

// Cache policy of the populations in a step of these lattices (results are
// bitwise the same under all three).  us per step, FP32 miscible unless named,
// CACHE_STREAM / CACHE_REUSE / CACHE_KEEP:
//
// KEEP, when all that the launch reads, the populations of both copies and the
// medium, fits in the memory-side cache (256 MiB): a step then reads what the last
// one left there, where non-temporal stores send it to memory.
//   61^3 (69 MB) 15.4 / 15.7 / 13.6, 83^3 (174 MB) 40 / 39 / 32.6, 94^3 (252 MB)
//   57 / 56 / 46, 98^3 (286 MB) 66 / 63 / 67; 70^3 BF16 (52 MB) 15.3 / 16.1 /
//   14.4, 110^3 BF16 (202 MB) 47 / 46 / 41, 120^3 BF16 (263 MB) 59 / 57 / 60;
//   two-fluid 80^3 36 / 37 / 30; channel FP64 64^3 17 / 18 / 14.
// The end is sharp.  As gain over STREAM in percent, at MB of populations and
// medium: BF16 deviations 243 16, 259 12, 265 -1, 271 -2; with a tensor 263 20, 268 0,
// 282 -5; obstacles 250 22, 265 -1; FP16 split 254 25, 265 17, 278 -6; tensor 258 14,
// 273 -3; obstacles 269 12, 284 -1; FP32 263 11, tensor 265 7, 274 3, obstacles and
// tensor 282 5 (REUSE 11); FP64 tensor 264 8, 275 6, 282 -1.  The line lies at 264 MB
// for the deviations, at 270 else, and at 256 of populations (BF16 channel without
// medium planes 269 MB: REUSE 23, KEEP 20 to 26, by the workspace's place in memory).
// Lattices that the L2s (32 MB) hold in part step as fast or faster under STREAM:
//   48^3 9.6 / 10.2 / 10.7, 58^3 12.0 / 13.4 / 12.6, 64^3 BF16 9.2 / 10.5 / 10.4;
// the line lies at 62 MB in the miscible model in FP32 and FP64 (96 MB with rows
// of whole lines: 64^3, 80 MB, 14.4 / 15.9 / 14.8), at 40 MB in its 16-bit forms
// (1024 blocks, four per CU; FP16 deviations 68 x 47 x 78, 38 MB, 9.6 / 10.5 / 9.9,
// 98 x 50 x 56, 42 MB, 12.7 / 13.5 / 11.3, 46 x 105 x 64, 47 MB, 13.5 / 14.2 / 11.8,
// tensor 61 x 58 x 76, 41 MB, 14.4 / 15.2 / 13.2, BF16 with obstacles 67 x 64 x 72, 47
// MB, 14.9 / 13.6 / 11.6), at 50 MB else.  The smallest gain again (32^3 FP64
// channel, 10 MB, 6.6 / 6.6 / 6.0; 64^3 BF16 channel, 20 MB, 8.0 / 7.3 / 7.0; miscible
// 32^3, 10 MB, 7.9 / 7.9 / 7.7, but 40^3, 20 MB, 8.3 / 8.9 / 9.0): up to 12 MB, the
// single-fluid step up to 24 MB, in FP64 to 15 MB (13 MB 6.3 / 6.2 / 6.0, 19 MB 6.9 / 6.9 /
// 7.3, 46 x 33 x 47, 22 MB, 7.1 / 7.2 / 7.9).
//
// REUSE, when lines are read by two waves: rows that are not whole lines put
// most lines across a wave boundary (FP32 243 x 251 x 238 970 / 935, 250^3 988 / 936;
// 131^3 two-fluid 142 / 135, BF16 93 / 87; channel 150^3 FP64 201 / 190; where rows
// are whole lines 256^3 945 / 970, 128^3 two-fluid 122 / 128); bounced links read a
// line once more (10% obstacles 256^3 1120 / 1035, BF16 567 / 553).  The single-fluid
// and two-fluid steps and the miscible one in FP32 and FP64 gain over the whole
// range; the others by size, as gain of REUSE over STREAM in percent:
//   deviations, rows not whole sectors of 32 bytes (whole ones: 200^3 254 / 255):
//     331 MB of populations 4.3, 454 MB 4.2, 551 MB 1.5, 603 MB 0, 630 MB -1.2, 0.7
//     to 1.2 GB -1 to -2, 1.6 GB (planes of 41 MB) 0, 2.2 GB 1.4, 4.2 GB 5.5
//   with a tensor: 307 MB 1, 415 MB -1.7, 0.54 to 0.95 GB -5, 1.3 GB (34 MB) -1.5,
//     1.4 GB (38 MB) 2.1, 2.0 GB 2.9; and obstacles: 367 MB 3.3, 522 MB -3.3, 0.9 GB
//     -3.7, 1.07 GB (28 MB) -2.7, 1.17 GB (31 MB) 4, 1.4 GB 5.9
//   split: 14 MB planes -2.4, 26 MB -2.7, 32 MB -2, 35 MB -0.4, 36.3 MB 2, 114 MB 2.3;
//     tensor: 8 to 16 MB -3 to -5, 25 MB -0.8, 26.5 MB 2.1, 33 MB 1.9; obstacles
//     from 23 MB 1.9; two solutes 16 MB -1.3, 24 MB 0.3, 42 MB 2.2
//   FP32 tensor: 0.35 GB 4.1, 0.58 GB 2 to 3, 0.62 GB -0.2 to -2.4, 0.71 GB -5 to 2.3, 0.89
//     GB -2.1, 1.2 GB -1.9, 1.6 GB -1.9, 2.3 GB (30 MB) 0.3, 2.4 GB (32 MB) 1.2, 4.2 GB (55
//     MB) 7.9; FP64 0.46 GB 2.4, 0.52 GB -0.4, 0.59 GB -1.7, 0.88 GB -4.9, 1.7 GB -2.6, 2.8 GB
//     (36 MB) 1.9; whole lines in FP32: 17 to 25 MB -5, 35 MB 0, 39 MB (128 x 256 x 300)
//     -1.3, 54 MB 2.5, 67 MB 3.1
// So it gains again where a plane no longer fits in the L2s (32 MB together), and
// up to two or three times the memory-side cache.  Between, with rows of whole lines,
// it depends on how many cells have a bounced link.  Mean gain in percent over
// planes of 12 to 36 MB (1,290 random boxes with 4^3 cubes of solid) at shares of
// 0 / 0.02 / 0.06 / 0.11 / 0.18 / 0.28: deviations -2.8 / -2 / -0.7 / 1 / 1.9 / 4.7, FP32 -4 /
// -3.6 / 0 / 2.7 / 5.5 / 10, its tensor step -5 / -4 / -2.5 / - / 2 / 6, FP64 -3.8 / -3.1 / -2.4 /
// -0.9 / 0.6 / 3.8, its tensor step -5 / -6 / -6 / -3.5 / -1.7 / 1, split -2.9 / -2.8 / -2 / -0.9 /
// 0 / 0; a mask taken for obstacles whatever it held lost up to 10 there (FP64 128^3
// 6, BF16 160^3 3.6, FP32 tensor 10).  The single-fluid and two-fluid steps gain 1 to 4 from
// the first obstacles on; with none they range from -4 (256^3 FP32) to 2.
//
// The free-surface step leaves the gas cells out; KEEP from 50 to 256 MB of
// populations there, STREAM else (us, whole step, STREAM / KEEP: 48^3 FP32 17 MB
// 24.8 / 25.2, 61 x 71 x 81 53 MB 30.0 / 29.4, 101 x 100 x 97 149 MB 34.8 / 32.9,
// FP16 split 82 MB 33.2 / 31.1, 110^3 202 MB 36.4 / 34.3, 128^3 BF16 159 MB 33.6 /
// 33.8; 128^3 319 MB 44.5 / 45.2, 200 x 190 x 180 1040 MB 130 / 139); plain loads
// alone gain nothing.  21 boxes of odd sizes from 55 to 256 MB: KEEP 2 to 14% faster
// in FP32 and BF16, 4 to 20% in FP16 split.
//
// The lattices of a batch share the launch: their bytes and planes add up (BF16,
// seven lattices with 12.7M miscible cells, the largest 6.5M, STREAM 588 / REUSE 559;
// 9.4M of 187^3, 75^3 and others 428 / 415), and the larger part of their cells decides
// between REUSE and STREAM.
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
// Plain loads do push kept lines out.  Beside kept groups the others stream, unless
// they have more than 4.5 times their bytes: then nothing is kept.  us per step, both /
// the others streamed / nothing kept, by that ratio: 2.1 BF16 98 95 56 106 60 (the
// second and fifth two-fluid) 120.2 / 116 / 117, 3.1 FP32 50 125 71 54 107.1 / 100.0 /
// 102.3, 4.3 BF16 100 161 119.4 / 115 / 117.5, 5 BF16 121 77 117 63 96 143 65 272.6 / 272.6 /
// 268, 8.6 BF16 120 104 63 126 64 112 190 424 / 435 / 422, 10 FP32 83 178 226.6 / 230.7 / 221,
// 18 FP32 180 72 95 126 55 108 626 / 660 / 622.

constexpr double CACHE_MB = 1e6, CACHE_SIDE = 270 * CACHE_MB;
constexpr double CACHE_BESIDE = 4.5;   // REUSE bytes beside a kept byte, from where on keeping loses

// the bytes of a launch's populations and of all that it reads (free surface: the
// populations, of which half or so are gas), and between which its step gains by KEEP
struct CacheLaunch {
    double bytes, all, low, end;
};

inline CacheLaunch cache_launch(const CacheLattice *l, int n)
{
    CacheLaunch a = {0.0, 0.0, 50 * CACHE_MB, CACHE_SIDE};
    bool whole_lines = true;
    for (int i = 0; i < n; ++i) {
        whole_lines = whole_lines && l[i].nx * storage_bytes(l[i].storage) % 128 == 0;
        a.bytes += l[i].bytes;
        a.all += l[i].bytes + (l->physics == LBM_FREESURF ? 0.0 : l[i].medium);
    }
    if (l->physics == LBM_MISCIBLE) {
        const bool paired = paired_storage(l->physics, l->storage);
        a.low = (paired ? 40 : (whole_lines ? 96 : 62)) * CACHE_MB;
        if (paired && !split_storage(l->storage)) a.end = 264 * CACHE_MB;
    }
    return a;
}

// The bytes of a launch that steps fastest under KEEP when it has the cache to
// itself, else 0.
inline double keep_bytes(const CacheLattice *l, int n)
{
    const CacheLaunch a = cache_launch(l, n);
    const double tiny = (l->physics == LBM_FREESURF ? 0 : (l->physics != LBM_SINGLE ? 12 : (l->storage == LBM_F64 ? 15 : 24))) *
                        CACHE_MB;
    return a.bytes <= tiny || (a.bytes >= a.low && a.bytes <= 256 * CACHE_MB && a.all <= a.end) ? a.all : 0.0;
}

// The same of a lattice with an obstacle mask, whatever its rows: do its bounced
// links pay for plain loads?
inline bool bounces_pay(const CacheLattice &c, double plane, double bytes)
{
    const bool f64 = c.storage == LBM_F64;
    const double b = c.bounced;
    if (c.physics != LBM_MISCIBLE) return b > 0.004;
    if (split_storage(c.storage)) {
        if (plane > 35 || (plane > 24 && (c.tensor || c.solutes > 1))) return true;
        return (plane > 30 && b > 0.05) || (plane > 24 && b > 0.12);
    }
    if (paired_storage(c.physics, c.storage)) {
        if (c.solutes > 1) return true;
        return c.tensor ? plane > 30 || bytes <= 400 : plane > 45 || bytes <= 450 || b > 0.09;
    }
    if (c.solutes > 1) return plane > 42 || b > (f64 ? 0.05 : 0.03);
    if (c.tensor) return plane > 30 || b > (f64 ? (bytes <= 500 ? 0.1 : 0.25) : (bytes <= 600 ? 0.015 : 0.12));
    return plane > (f64 ? 60 : 42) || b > (f64 ? (bytes <= 600 ? 0.05 : 0.15) : (bytes <= 600 ? 0.015 : 0.08));
}

// Does a lattice beyond the memory-side cache step faster under REUSE than under
// STREAM, in a launch of so many cells?
inline bool reuse_pays(const CacheLattice &c, double cells)
{
    const bool paired = paired_storage(c.physics, c.storage);
    const size_t word = storage_bytes(c.storage) * (paired ? 2 : 1);
    const bool shared = c.nx * word % (paired ? 32 : 128) != 0;
    const double plane = cells * double(word) / CACHE_MB, bytes = c.bytes / CACHE_MB;
    if (c.links && bounces_pay(c, plane, bytes)) return true;
    if (!shared) return c.tensor && c.storage == LBM_F32 && plane > 42;
    if (c.physics != LBM_MISCIBLE) return true;
    if (split_storage(c.storage)) return plane > (c.tensor || c.solutes > 1 ? 24 : 35);
    if (paired) return c.solutes > 1 || plane > 35 || bytes <= (c.tensor ? 400 : 600);
    return !c.tensor || c.solutes > 1 || plane > 29 || bytes <= (c.storage == LBM_F64 ? 500 : 600);
}

inline bool launch_reuses(const CacheLattice *l, int n)
{
    const CacheLaunch a = cache_launch(l, n);
    double cells = 0, reuse = 0;
    for (int i = 0; i < n; ++i) cells += l[i].cells;
    for (int i = 0; i < n; ++i)
        if (reuse_pays(l[i], cells)) reuse += l[i].cells;
    return l->physics != LBM_FREESURF && a.bytes > 50 * CACHE_MB && a.bytes > a.low && 2 * reuse > cells;
}

// What the launches of one step would keep and, the others, read by plain loads.
struct CacheStep {
    double keep, reuse;
};

inline void add_launch(CacheStep &s, const CacheLattice *l, int n)
{
    const double k = keep_bytes(l, n);
    s.keep += k;
    if (k == 0.0 && launch_reuses(l, n)) s.reuse += cache_launch(l, n).all;
}

// The policy of a launch in a step s (its own launch counted).
inline int cache_policy(const CacheLattice *l, int n, const CacheStep &s)
{
    const bool keeps = s.keep > 0.0 && s.keep <= CACHE_SIDE && s.reuse <= CACHE_BESIDE * s.keep;
    if (keeps && keep_bytes(l, n) > 0.0) return CACHE_KEEP;
    return !keeps && launch_reuses(l, n) ? CACHE_REUSE : CACHE_STREAM;
}

}  // namespace plbm
