// Launch shapes of the dslash: the one an untuned launch takes, and the ones the autotuner times.
// Host code without HIP, so that the rule can be checked where there is no GPU.
#pragma once

#include <stddef.h>

#include <vector>

#include "wdirac.h"

namespace wd {

// Launch shape of one kernel: workgroup size, XCD-aware block remap, and
// non-temporal (streaming) link loads.
struct TuneParam {
    int block = 64;
    int remap = 1;
    int nt = -1;  // non-temporal link loads (-1: by the rule in settle_shape)
    int pf = 1;   // software-pipelined directions
    int rhs_inner = 1;   // several rhs: interleave them with the site tiles
    int zb = 0;          // z-blocked site traversal depth (0: natural order)
    int mf = 0;          // 16-bit, 12-real, 16k rhs: colour multiply on the matrix cores
    int split = -1;      // four waves per 64 sites; block, pf and zb then do not matter
                         // (-1: by the rule in settle_shape)
};

// What the rule looks at.
struct ShapeCall {
    int prec = WD_F32;
    int recon = 12;
    int nrhs = 1;
    int uses = 4;          // the caller's launches that read these links one after another; 4: or more
    long long groups = 0;  // 64-site groups of all rhs
    size_t links = 0;      // bytes of the links (all directions, both parities)
    size_t half = 0;       // bytes of a half field of all rhs
};

// What an untuned launch shape leaves open.  Times in us per call on one MI355X, three sets of links
// and fields in turn; "before" is one wave per 64 sites with streamed links, what every untuned launch
// once took.  MB are of 2^20 bytes.
//
// Non-temporal link loads leave the 256 MB last-level cache to the spinors; ordinary ones pay where
// the links are still there when they are read again (kept / streamed / before):
// * Four launches or more on them (M^dagger M, solvers): kept up to 160 MB.  Mhat^dagger Mhat F32
//   20^3 x 40 (59 MB) 71.7 / 83.0 / 90.0, 28^3 x 40 (161) 208 / 210 / 215, 32^3 x 64 (384) 543 / 469 /
//   472; a launch on one set of links F32 24^3 x 48 (122) 35.3 / 40.8, F64 20^3 x 40 (117) 36.4 / 40.7.
// * One launch (a hop onto one parity): only where links and spinors come to less than 90 MB, so that
//   what a program works on besides leaves them room.  F32 20^3 x 40 (88 MB in all) 18.6 / 19.9 / 22.1,
//   24^3 x 32 (121) 27.4 / 25.6 / 27.9, 24^3 x 48 (182) 44.7 / 38.2 / 39.3; F64 18-real 20x12x18x28
//   (88) 18.1 / 18.9 / 18.9, 16^3 x 32 (96) 23.0 / 20.6 / 20.5.
// * Two (both parities, or a Schur operator): so too, but beyond 220 MB, with both launches' spinors,
//   they are gone by the next call either way and only the second launch counts.  Hop F32 24^3 x 32
//   (162) 54.5 / 51.3 / 56.0, 24^3 x 48 (243) 79.5 / 86.2 / 87.7; M F64 18-real 16^3 x 32 (120)
//   47.9 / 43.4 / 43.0.  F64 has nothing to gain there (20^3 x 40, 234 MB: hop 86.9 / 89.1 / 89.1, Schur
//   operator 89.8 / - / 86.9).
// * Several rhs read them again within a launch, and keep them (16 on 16^3 x 32: F32 90 / 110 a launch,
//   BF16 46 / 57), but for one launch of two or three between 110 and 220 MB: 2 F32 18-real rhs on
//   24^3 x 32 (202) 56.0 / 51.9 / 55.4, 24^3 x 48 (303) 84.9 / 85.8 / 92.5; 2 BF16 18-real on
//   28^3 x 40 (206) 60.4 / 55.0 / 58.6.  F64 keeps them (2 18-real on 22^4 64.4 / 66.0 / 66.3).
//
// Four waves per 64 sites (split) hide latency, at the price of a trip through LDS and of fewer bytes
// in flight per register: Mhat^dagger Mhat F32 8^3 x 16 18.3 / 22.0 with one wave, 16^3 x 32 32.7 / 33.9,
// 32^3 x 64 (16 384 groups) 482 / 469.  They are chosen up to
// * F64 512 groups (20x12x18x28, 945: 66.2 / 56.0); 18-real links kept over several launches gain again
//   from 1000 (16^3 x 32 80.3 / 89.4, 18x22x12x36 103.9 / 108.1; 20x12x18x28 74.0 / 69.8);
// * F32 12 288 (hop 28^3 x 56, 9604: 74.1 / 75.6), with 18-real links streamed 4096 (24^3 x 32, 3456:
//   32.6 / 33.5; 24^3 x 48, 5184: 50.4 / 49.7; 28^3 x 56 100.9 / 97.5);
// * 16 bits 12 288 (F16 18-real 30x32x34x40, 10 200: 49.6 / 50.5), 12-real 10 000 (the same lattice
//   43.2 / 42.2);
// * several rhs F32 32 768 (3 on 24^3 x 48, 15 552: 96.3 / 99.2), 16 bits, bound by their vector work
//   once the chip is full, 4096 (16 BF16 on 16^3 x 32, 52.6 / 46.5 a launch), but all that stream their
//   links (2 BF16 on 26x30x22x44, 11 796: 43.7 / 46.0) other than F16 with 12 reals (2 on 28^3 x 40:
//   53.9 / 53.2).
inline void settle_shape(const ShapeCall& c, TuneParam* t)
{
    const size_t MB = (size_t)1 << 20;
    const bool one = c.nrhs == 1, f64 = c.prec == WD_F64, f32 = c.prec == WD_F32, r12 = c.recon == 12;
    const size_t launch = c.links + 2 * c.half;   // what a launch reads and writes
    if (t->nt < 0) {
        if (one)
            t->nt = c.links > 160 * MB ||
                    (launch > 90 * MB && (c.uses == 1 || (c.uses == 2 && (f64 || launch + 2 * c.half < 220 * MB))));
        else
            t->nt = !f64 && c.uses == 1 && c.nrhs <= (f32 ? 2 : 3) && launch > 110 * MB && launch < 220 * MB;
    }
    if (t->split < 0) {
        if (f64) t->split = c.groups <= 512 || (one && !r12 && c.uses > 2 && !t->nt && c.groups > 1000);
        else if (one) t->split = c.groups <= (f32 ? (r12 || !t->nt ? 12288 : 4096) : r12 ? 10000 : 12288);
        else if (f32) t->split = c.groups <= 32768;
        else t->split = c.groups <= 4096 || (t->nt && !(c.prec == WD_F16 && r12));
    }
}

// The shapes the autotuner times for a launch on nrhs right-hand sides of a lattice of Z = z, groups as
// above.  matrix: the matrix-core kernel can run it.
inline std::vector<TuneParam> tune_candidates(int nrhs, int z, long long groups, bool matrix)
{
    std::vector<TuneParam> all;
    std::vector<int> zbs{0};
    for (int d = 2; d < z; d *= 2)
        if (z % d == 0) zbs.push_back(d);
    TuneParam tp;
    tp.split = 0;
    for (int zb : zbs)
        for (int block = 64; block <= 256; block += 64)
            for (int remap = 0; remap < 2; ++remap)
                for (int nt = 0; nt < 2; ++nt)
                    for (int pf = 0; pf < 2; ++pf)
                        for (int ri = (nrhs > 1 ? 0 : 1); ri < 2; ++ri) {
                            tp.block = block;
                            tp.remap = remap;
                            tp.nt = nt;
                            tp.pf = pf;
                            tp.rhs_inner = ri;
                            tp.zb = zb;
                            all.push_back(tp);
                        }
    tp = TuneParam();
    tp.split = 1;
    if (groups < 1ll << 24)   // 256 work-items a group, 2^32 a launch
        for (int remap = 0; remap < 2; ++remap)
            for (int nt = 0; nt < 2; ++nt)
                for (int ri = (nrhs > 1 ? 0 : 1); ri < 2; ++ri) {
                    tp.remap = remap;
                    tp.nt = nt;
                    tp.rhs_inner = ri;
                    all.push_back(tp);
                }
    if (matrix) {   // no launch-shape parameters
        tp = TuneParam();
        tp.nt = 1;
        tp.split = 0;
        tp.mf = 1;
        all.push_back(tp);
    }
    return all;
}

} // namespace wd
