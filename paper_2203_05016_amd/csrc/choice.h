// Which kernel a linear layer, a convolution in runs and a LayerNorm-side transposition take and how their work is cut, from sizes alone.
// Host code without HIP.
#pragma once

#include <cmath>

namespace shflbw {

// A workgroup's tiles: four of 64 or of 128 columns, one wavefront each; one of 128 columns whose k-steps 2 or 4 wavefronts
// share; one of 64 whose steps 2, 4 or 8 share; and the shared-slab kernel.
enum Cut { WHOLE_64, WHOLE_128, WIDE_BY_2, WIDE_BY_4, BY_2, BY_4, BY_8, SLAB };
constexpr int GATHER_CUTS = 7;

// The rows of X: whole 16-byte units, no particular alignment, or those of images (1x1 convolutions; short rows).
enum class Rows { ALIGNED, ANY, IMAGES };

struct CutSizes {
    int V;
    long G, N, steps;       // groups, output columns (whole slots of 8 where rows are not aligned), k-steps of all groups
    int K;
    Rows rows;
    bool uneven;            // groups of different numbers of steps
    bool f32;               // 32-bit results
    bool slab;              // the layout and the operands admit the slab kernel
    double kept;            // share of the weights that is kept

    long per;               // steps of a group, rounded down (a division: once)

    long tiles() const { return (N + 63) / 64 * G; }
    int v() const { return V == 16 ? 0 : V == 32 ? 1 : V == 64 ? 2 : 3; }
};

// Whole tiles take their weights by way of the LDS from 5 k-steps (V = 16 from 4, in 128 columns from 13): four fetches of them
// become one, at the price of a barrier every 4 or 8 steps.  Time shared / own, geometric mean over the products of
// profiles/cut_sweep.csv with 200 workgroups or more, by steps:
//                     up to 4   5-8    9-12   13-16   17-32   33-64   more
//   64 columns, V 16     .98    .96    .95    .91     .90     .90     .85
//               V 32     .99    .96    .94    .92     .90     .87     .81
//               V 64     .98    .96    .94    .93     .89     .86     .78
//               V 128    .99    .97    .96    .92     .94     .88     .82
//   128 columns, V 16   1.05   1.01   1.04    .96     .99    1.03    1.00
//               V 32    1.01    .99    .97    .97     .94     .91     .88
//               V 64    1.00    .98    .97    .97     .95     .92     .87
// (4 steps, the most frequent number below 5: V = 16 .975, 95 % of them below 1.0; V = 64 .97, but on unaligned rows and images 1.0, up to 1.17)
inline bool shares_weights(int V, bool wide, long per) { return per > (V != 16 ? 4 : wide ? 12 : 3); }

// Workgroups of the fullest of 256 CUs; beyond four rounds they even out.
inline double rounds_of(long workgroups) { return workgroups > 1024 ? (double)workgroups / 256 : (double)((workgroups + 255) / 256); }

// The slab kernel deals column tiles of 128 to the eight XCDs in turn, one workgroup of 12 (V = 64: 8, V = 128: 4) groups
// per CU: what counts is the XCD with most tiles.  (1152 columns are nine tiles, two of them on one XCD: 6624 x 4152 at
// 75 %, V = 32, 162 workgroups, 68 us where 36 would be a full round's.)
inline long slab_group_blocks(const CutSizes& s)
{
    const long per = s.V <= 32 ? 12 : s.V == 64 ? 8 : 4;
    return (s.G + per - 1) / per;
}
inline double slab_rounds(const CutSizes& s)
{
    const long on_xcd = ((s.N + 127) / 128 + 7) / 8 * slab_group_blocks(s);
    return on_xcd > 256 ? (double)on_xcd / 32 : (double)((on_xcd + 31) / 32);
}
// ... with enough groups to fill its compute wavefronts, a quarter of a round of workgroups, and more than very few tiles,
// which the gather kernel's split steps spread better
inline bool slab_considered(const CutSizes& s)
{
    return s.slab && s.G >= (s.V <= 32 ? 12 : s.V == 64 ? 8 : 4) && s.tiles() > 512 && (s.N + 127) / 128 * slab_group_blocks(s) >= 64;
}

// Estimated time of a cut, us.  A CU's first workgroup takes `start` plus `first` per k-step, each further one `step`
// per k-step (the memory pipeline is full by then), each `store` for its epilogue and stores (16-bit results).  From the
// times of 3740 products in every cut that they admit (profiles/cut_sweep.csv: V 16 to 128, 1 to 500 steps, 1 to
// 512 groups, 1 to 16384 columns, aligned, unaligned, images): the parameters that make the choice below lose least.
inline double cut_time(const CutSizes& s, Cut cut)
{
    struct Cost { double start, first, step, store; };
    static constexpr Cost NONE = {1e9, 0, 0, 0};   // four row blocks x four tiles of accumulators do not fit
    static constexpr Cost COSTS[4][GATHER_CUTS] = {
        {{2.91, .17, .188, .272}, {3.59, .29, .336, .369}, {3, .113, .089, .269}, {3.4, .078, .103, .381},
         {2.8, .097, .063, .111}, {2.81, .055, .066, .19}, {2.97, .054, .059, .597}},
        {{2.31, .129, .094, .688}, {2.84, .165, .164, 1.09}, {2.49, .083, .045, .66}, {2.99, .052, .06, .854},
         {2.18, .091, .038, .247}, {2.42, .054, .041, .315}, {2.38, .037, .042, .694}},
        {{2.22, .167, .111, 1.32}, {.75, .236, .16, 3.5}, {3.38, .106, .06, 1.06}, {3.57, .064, .093, 1.24},
         {2.8, .111, .056, .362}, {2.47, .066, .058, .541}, {2.75, .047, .064, 1.07}},
        {{2.37, .221, .176, 3.27}, NONE, NONE, NONE,
         {2.95, .14, .09, .906}, {2.94, .079, .109, 1.32}, {2.99, .06, .13, 2.98}}};
    // us per round of workgroups: per k-step, per chunk of 64 rows of X (all are streamed, kept or not), and for the stores
    struct SlabCost { double step, chunk, store, start; };
    static constexpr SlabCost SLAB_COSTS[4] = {{.298, .215, 2.83, 1.13}, {.198, .249, 4.47, .208}, {.262, .239, 5.49, 0}, {.271, .276, 4.88, 0}};
    const double per = (double)s.per;
    if (cut == SLAB) {
        const SlabCost& c = SLAB_COSTS[s.v()];
        return c.start + slab_rounds(s) * (per * c.step + s.K / 64. * c.chunk + c.store * (s.f32 ? 1.56 : 1));
    }
    const Cost& c = COSTS[s.v()][cut];
    const bool whole = cut == WHOLE_64 || cut == WHOLE_128;
    const long columns = cut == WHOLE_128 || cut == WIDE_BY_2 || cut == WIDE_BY_4 ? 128 : 64, tiles = (s.N + columns - 1) / columns;
    const double rounds = rounds_of(s.G * (whole ? (tiles + 3) / 4 : tiles));
    double steps = per, store = c.store;
    if (s.uneven) steps *= whole ? 1.47 : 1.09;   // a CU's workgroups wait for the longest group
    if (s.f32) {
        store *= !whole ? 1.18 : s.V == 64 && cut == WHOLE_128 ? 2.09 : 2.18;
        // two row blocks in wide tiles leave in bursts, which the next tile's loads wait for: whole tiles of 128 columns against 64, geometric
        // means, 8 steps 1.18, 24 1.13, 48 1.06, 96 1.02, more .97
        if (s.V == 64 && columns == 128) steps *= cut == WHOLE_128 && per < 96 ? 1.5 : 1.18;
    }
    // unaligned rows cost the address unit twice the accesses, and their stores two lines
    if (s.rows == Rows::ANY) { steps *= whole ? 1.21 : 1.16; store *= 1.44; }
    if (s.rows == Rows::IMAGES) { steps *= whole ? 1.23 : 1.03; store *= 1.45; }
    return c.start + steps * c.first + store + (rounds - 1) * (steps * c.step + store);
}

// By tiles of 64 columns x one group and k-steps of a group: fewer tiles than four to seven per CU (by V and steps) leave
// CUs idle or unevenly loaded, so the k-steps of a tile are shared by 2, 4 or 8 wavefronts.  WHOLE_64: they are not.
// Measured, us by whole tiles / split by 2 / 4 / 8 (the host's part is 3.1):
//   32 tiles of 2 k-steps (512 x 512 by 64 at 90 %, V = 16)         3.1 /  3.1 /  3.1 /  3.2
//   32 tiles of 4 k-steps (512 x 512 by 64 at 75 %, V = 16)         3.6 /  3.2 /  3.1 /  3.2
//   8 tiles of 2 k-steps (512 x 512 by 64 at 90 %, V = 64)          3.2 /  3.4 /  3.3 /  3.9
//   512 tiles of 2 k-steps (512 x 512 by 1024 at 90 %, V = 16)      3.1 /  3.2 /  3.4 /  4.3
//   1024 tiles of 2 k-steps (512 x 512 by 2048 at 90 %, V = 16)     3.0 /  3.5 /  4.2 /  6.2
//   128 tiles of 64 k-steps (4096 x 4096 by 64, V = 32)            14.0 /  9.1 /  6.2 /  5.1
//   128 tiles of 16 k-steps (1024 x 1024 by 512, V = 64)            5.6 /  4.5 /  4.0 /  4.4
//   448 tiles of 72 k-steps (3x3, 14x14x256 -> 256, V = 64)        36.5 / 18.0 / 13.3 / 13.6
//   512 tiles of 26 k-steps (2048 x 4096 by 1024, V = 64)          10.5 /  7.9 /  6.8 /  7.6
//   784 tiles of  5 k-steps (3x3, 28x28x64 -> 64, V = 16)           9.4 /  9.3 / 10.1 / 12.7
//   1200 tiles of  8 k-steps (1024 x 1024 by 9600 at 88 %, V = 128) 10.3 / 11.3 / 14.0 / 24.7
//   1408 tiles of 16 k-steps (1024 x 1024 by 2816, V = 32)          7.0 /  6.6 /  7.6 / 10.1
//   1536 tiles of  8 k-steps (1024 x 1024 by 1536, V = 16)          7.2 /  7.0 /  7.3 /  9.9
//   1568 tiles of 18 k-steps (3x3 / 2, 56x56x128 -> 128, V = 32)   10.3 / 10.3 / 11.0 / 13.7
//   1792 tiles of 32 k-steps (1x1, 7x7x512 -> 2048, V = 32)        20.8 / 18.9 / 19.3 / 21.0
//   1792 tiles of 32 k-steps (1024 x 2048 by 7168, V = 64)         13.9 / 14.5 / 15.9 / 19.5
// Convolutions take it as it is: over 132 of them, 3x3 and 5x5, it costs 1.025 of the best cut's time (geometric mean); what it misses is
// one to two thousand tiles of whole groups, which would do better split (25x25, 128 -> 416 channels at 90 %, 61 images, V = 32, 56 us, split by 2 32).
inline Cut cut_by_tiles(int V, long tiles, long per)
{
    if (tiles <= 256 && per >= 32) return BY_8;
    if ((tiles <= 256 && per >= 4) || (tiles <= 512 && per >= 32)) return BY_4;
    const bool by2 = tiles <= 1024 ? per >= (V == 16 && tiles > 512 ? 3 : 2) :
                     V <= 64 && (tiles <= 1360 ? per >= 8 : tiles <= 1600 ? per >= (V == 16 ? 8 : 16) : V == 32 && tiles <= 1800 && per >= 32);
    return by2 ? BY_2 : WHOLE_64;
}

// 128 columns fetch the weights half as often, which decides where there are thousands of tiles and many steps
inline bool wide_by_tiles(const CutSizes& s) { return s.V <= 64 && s.steps >= 20 * s.G && (s.N + 127) / 128 * s.G >= 2048; }

// The cut of a linear layer of four groups or more.  Numbers of tiles, steps and kept weights propose one, and the
// estimates overrule it where another is 10 % below: they are within 15 to 20 % of the times, and better between cuts
// of one product.  Over the sweep the choice takes 1.02 times the best cut's time (geometric mean; 95 % of the products within
// 1.12).  The proposal alone takes 1.05 (1.23), the least estimate alone 1.03 (1.15); cuts by time per k-step without a workgroup's
// own cost, and the slab kernel for V = 16 and 32 alone, took 1.05 (1.24).
// Slab against gather, us, 16-bit results: V = 16, 4096 x 1024 by 8192 at 83 % 54.2 / 49.0, 80 % 53.8 / 49.5, 75 % 56.1 / 68.6;
// V = 32, the same 83 % 34.0 / 27.5, 80 % 34.5 / 31.7, 75 % 34.9 / 33.7, 70 % 38.8 / 38.1, 60 % 43.6 / 48.4, 50 % 46.6 / 54.9;
// 4096 x 4096 by 8192 at 80 % 105 / 92, 75 % 109 / 108, 70 % 121 / 131, 50 % 160 / 203; V = 64, 4096 x 1024 by 8192 at 75 % 31.4 / 26.7,
// 50 % 42.9 / 42.7, 0 % 67.5 / 74.5; 8192 x 8192 by 16384 at 75 % 671 / 574, 50 % 1048 / 1083, 0 % 1937 / 2075; 2048 x 296 by
// 14216 at 50 % 29.5 / 31.4, with 32-bit results 44.4 / 53.4; V = 128, 4096 x 4096 by 8192 at 75 % 97 / 79, 50 % 140 / 140, 0 % 247 / 267.
// The proposal's limits are where the two cross; at 75 %, V = 32, they are within 8 % of each other.
inline Cut choose_cut(const CutSizes& s)
{
    Cut proposed = cut_by_tiles(s.V, s.tiles(), s.per);
    if (proposed == WHOLE_64 && wide_by_tiles(s)) proposed = WHOLE_128;
    const bool slab = slab_considered(s);
    if (slab) {
        const long workgroups = (s.N + 127) / 128 * slab_group_blocks(s);
        const double need = s.V == 16 ? (workgroups >= 128 ? .2 : .6) : workgroups < 128 ? 2 : workgroups < 256 ? .5 : s.V == 32 ? .25 : .4;
        if (s.kept >= need) proposed = SLAB;
    }
    Cut best = proposed;
    double least = .9 * cut_time(s, proposed);
    for (int c = 0; c <= SLAB; ++c) {
        if (c == SLAB && !slab) continue;
        const double t = cut_time(s, (Cut)c);
        if (t < least) { least = t; best = (Cut)c; }
    }
    return best;
}

// The slab kernel with a resident slab (resident_kernel.hip): 64 columns of X with all their rows stay in a workgroup's LDS,
// `parts` workgroups of `waves` wavefronts share a column tile, each with a share of the row groups.
struct ResidentPlan { int parts = 0, waves = 0; double time = 1e9; };

// K rows of 128 bytes, a row of zeros and a counter fill the LDS of a CU; half of it, and 8 wavefronts, leave room for a
// second workgroup, whose products hide the copy of this one's slab (K = 512, 4096 rows by 8192, V = 32: 18.1 us with 16
// wavefronts, 17.4 with 8; K = 256 16.8 and 15.1).  Two row blocks (V >= 64) need the registers of 16 wavefronts for 8.
constexpr int RESIDENT_K = 1278, RESIDENT_K_HALF = 638;
inline int resident_waves(int V, int K) { return V >= 64 || K <= RESIDENT_K_HALF ? 8 : 16; }

// Estimated time, us, in `parts` shares: a round of workgroups takes Cost::copy per row of the slab (`copy` times it for other
// than aligned rows), then per item (a group; V = 128: half of one) `step` per k-step and `store` for its results, or the time of one
// wavefront's items, `chain` per step, where there are few of them; `start` once, `round` per round.  k-steps come in fours.
// whole: results are rows of whole 64-byte blocks (else these are written in parts by two column tiles).
// Fitted to 11 000 times of 3200 random layers (V 16 to 128, K 64 to 1278, 256 to 16384 columns, unpruned to 95 %), which it meets within 12 %.
inline double resident_time(const CutSizes& s, bool whole, int parts, int waves, double copy)
{
    struct Cost { double start, copy, step, store, chain, round, parted; };
    static constexpr Cost COSTS[4] = {{2.32, .00182, .019, .0328, .108, .904, 1.99}, {2.26, .00156, .0159, .0796, .0828, 1.21, 1.53},
                                      {2.74, .00207, .0265, .228, .0961, 1.03, 1.32}, {3.02, .00225, .0277, .213, .103, .923, 1.32}};
    const Cost& c = COSTS[s.v()];
    const long items = s.G * (s.V == 128 ? 2 : 1), per = (items + parts - 1) / parts;
    const long workgroups = (s.N + 63) / 64 * ((items + per - 1) / per);
    const int at_once = waves == 8 && s.V < 64 ? 2 : 1;               // workgroups of a CU
    const long cus = 256 * at_once;
    const double rounds = workgroups > 4 * cus ? (double)workgroups / cus : (double)((workgroups + cus - 1) / cus);
    const double live = at_once == 2 && workgroups > 256 ? 2 : 1;
    const double steps = (double)((s.per + 3) / 4 * 4) * (s.uneven ? 1.09 : 1);
    const double work = per * (steps * c.step + c.store * (s.f32 ? 2.4 : 1) * (whole ? 1 : c.parted)) * live;
    const double chain = (double)((per + waves - 1) / waves) * steps * c.chain;
    const double longer = work > chain ? work : chain, ratio = (work + chain - longer) / longer, r2 = ratio * ratio;
    return c.start + rounds * (s.K * c.copy * copy * live + longer * std::sqrt(std::sqrt(1 + r2 * r2)) + c.round);
}

// The number of shares with the least estimate: whole rounds of 256 workgroups.  (Twice 128 shares of half a round each
// copy every slab twice; 4096 x 1024 by 8192, V = 32 at 75 %: 128 / 256 / 512 workgroups 35.7 / 26.8 / 30.2 us.)
inline ResidentPlan plan_resident(const CutSizes& s, bool whole, double copy)
{
    ResidentPlan best;
    const long tiles = (s.N + 63) / 64, items = s.G * (s.V == 128 ? 2 : 1);
    if (s.K > RESIDENT_K || s.G < 4 || tiles * (items < 1024 ? items : 1024) >= (1L << 19)) return best;
    const int waves = resident_waves(s.V, s.K);
    long last = 0;
    for (long rounds = 1; rounds <= 4; ++rounds) {
        long parts = 256 * rounds / tiles;
        parts = parts < 1 ? 1 : parts > items ? items : parts;
        if (parts == last) continue;
        last = parts;
        const double t = resident_time(s, whole, (int)parts, waves, copy);
        if (t < best.time) { best.time = t; best.parts = (int)parts; best.waves = waves; }
    }
    return best;
}

// Taken where its estimate is below the best cut's by a margin.  Both estimates are low, by 5 to 20 % by V and by how results lie, and neither
// is better than 13 to 20 %, worst where a group has few steps, or where there are few columns or little work: hence the
// margins, which are such that few layers get slower, at the price of some that would have gained.  Of 7363 random layers (half
// of them are profiles/resident_sweep.csv) 2882 take it, at .765 of the other kernels' time (geometric mean; over all .900, the best of both
// .877): 49 of these lose more than 4 %, 7 more than 10 %, the worst 14 %.  Two runs of one kernel differ by more than 4 % in .5 % of the layers, V = 64 in 2 %.
// Margins and limits are not fitted to these, but that few fetches count on images is what their worst showed.
// Wider ones (6163 layers of 1 to 1278 features, up to 16 384 rows and 200 000 columns), which the last limits below come from: 1771 take it, at .78, 33 lose more than 4 %, 8 more than 10 %, up to 20 %; of 5385 others
// of these sizes 1596, at .78, 33 and 6, up to 21 %.  With one margin for all images and the same for little work
// 6 % of those that took it lost more than 4 %, 3 % more than 10 %, and the gain over all was the same .900.
// 4096 x 1024, V = 32 at 75 %, us other
// kernels / resident: by 8192 34.9 / 26.8, with 32-bit results 52.6 / 35.0, by 8191 (rows of no alignment) 50.5 / 28.6, by 2047
// 16.3 / 12.0 to 15.2, by card; V = 16 by 8192 56.5 / 31.6, by 2047 33.1 / 14.6; not taken: V = 64 28.3 / 25.2 to 27.1, unpruned 82 / 76; 1024 x 1024 by 4096 6.8 / 7.5 and
// 2048 x 1024 by 2048 at 90 %, V = 16 6.0 / 6.9: few groups, or few steps, to share a copy.
constexpr double RESIDENT_COPY_UNALIGNED = 1.4;
// Fewer tiles than this gain little (of the layers below it a sixth would take it, and win 1 %), half of those that lose are among them,
// and the estimates cost a call of 3 us 0.1.
inline bool resident_worth_a_look(const CutSizes& s) { return s.K <= RESIDENT_K && s.tiles() >= 1024; }
inline bool resident_conv_worth_a_look(int V, int K, long tiles) { return V <= 32 && K <= RESIDENT_K && tiles >= 512; }
// cut: choose_cut(s)
inline bool resident_pays(const CutSizes& s, Cut cut, bool whole, const ResidentPlan& plan)
{
    if (plan.parts <= 0) return false;
    // rows of no whole 64-byte blocks, the same with few steps (4, V = 64 in whole blocks 12) or columns, rows of whole blocks, the same with few; then
    // the same of images.  0: never.
    static constexpr double MARGINS[4][8] = {{.98, .98, .9, .85, .99, 1.02, .87, .95}, {.98, .86, .85, .74, .94, .94, .87, 0},
                                             {1.01, .86, .95, .81, .88, .88, .74, 0}, {.93, .8, 1.05, .8, 0, 0, 0, 0}};
    const int few = s.per <= (s.V == 64 && whole ? 12 : 4) || s.N < 1024 ? 1 : 0;
    // not where few groups share a copy (512 x 353 by 73 664 at 50 %, V = 128 32.5 / 39.3; 64 x 55 by 146 488 at 96 %, V = 16 14.6 / 18.5), the slab is next to nothing
    // (11 904 x 23 by 11 088, V = 32 86 / 108; V = 16 gains there, .80 of 1043 layers' time, V = 32 with 32-bit results .83 of 107), nor many groups of few steps (16 288 x 299 by 6632 at 80 %, V = 32 78 / 98)
    if ((s.G < 6 && (s.V == 16 || s.V == 128)) || (s.K < 64 && s.V > 16 && !(s.V == 32 && s.f32)) || (few && s.V == 32 && s.G > 256)) return false;
    double margin = MARGINS[s.v()][(s.rows == Rows::IMAGES ? 4 : 0) + (whole ? 2 : 0) + few];
    const double work = (double)s.tiles() * s.per;
    if (few && s.V < 128 && work < 12000) margin *= std::sqrt(std::sqrt(work / 12000));
    // images whose rows less than one group fetches (98 of 31x31, 121 -> 64 channels at 90 %, V = 16 11.0 / 14.6)
    const double fetches = s.G * s.kept;
    if (s.rows == Rows::IMAGES && fetches < 1 && margin > std::sqrt(std::sqrt(fetches))) margin = std::sqrt(std::sqrt(fetches));
    return plan.time < margin * cut_time(s, cut);
}

// Convolutions in runs of 8 (GeomConvRuns): the rows of the unfolded matrix are gathered once per workgroup instead of once per
// group, or staged and read in single values.  What decides is how often a row is fetched, groups x kept share.  Estimates
// from 1900 convolutions (3x3, 32 to 128 channels, 7x7 to 56x56, stride 1 and 2, both layouts): 10 to 30 % off, the resident slab's
// with the copy at 2.1 (NCHW: at any alignment, moved in registers) and 1.6 times that of aligned rows 9 and 13 % (4.1 times with a stride along x).
// A gathered row that few groups fetch is where they err: there, and where the alternative to a stride along x is a well filled
// staged box, the margin is wider.  Of 3873 random ones without a
// stride along x in NCHW, which nothing was fitted to, 2578 take it, at .59 of the other kernels' time, and 30 of these lose more than 4 %, 13 more than 10 %, up to 45 %; of 1403 with one 571 at .45, 3 lose more than 4 %
// (profiles/resident_conv_sweep.csv).
// us before / resident: 55 images of 18x18, 128 -> 1024
// channels at 50 %, V = 16 147.5 / 55.5, 46 of 41x41, 112 -> 240 143.8 / 63.9, 32 of 28x28, 128 -> 512 at 75 %, V = 32 40.1 / 23.0.
// V >= 64 gains nothing, and 32-bit results were not measured: neither comes here.
// NCHW with a stride of two along x (GeomConvRuns2): two loads per run.
enum class Runs { NCHW, CHWN, NCHW_BY_2 };
constexpr double RESIDENT_COPY_RUNS[3] = {2.12, 1.61, 4.09};
inline bool resident_conv_pays(const CutSizes& s, Runs runs, bool gathered, const ResidentPlan& plan)
{
    if (plan.parts <= 0) return false;
    struct Cost { double start, step, item; };
    static constexpr Cost GATHERED[3][2] = {{{4.09, .127, .0913}, {4.06, .0728, .176}}, {{3.84, .114, .0264}, {3.55, .061, .206}},
                                            {{4.49, .25, .274}, {4.36, .153, .124}}};
    static constexpr Cost STAGED[2] = {{6.08, .141, 0}, {6.88, .0736, .00289}};   // item: per row of the unfolded matrix and tile
    const int v = s.V == 16 ? 0 : 1;
    const double tiles = (double)((s.N + 63) / 64) / 256;
    const Cost& g = GATHERED[(int)runs][v];
    const double other = gathered ? g.start + tiles * s.G * (s.per * g.step + g.item)
                                  : STAGED[v].start + tiles * (s.G * s.per * STAGED[v].step + s.K * STAGED[v].item);
    double margin = .9;
    if (runs == Runs::NCHW_BY_2) {
        margin = .8;
    } else if (gathered) {
        margin = runs == Runs::CHWN && s.V == 32 ? .8 : .85;
        const double fetches = s.G * s.kept;
        if (fetches < 2.5) margin *= std::sqrt(fetches / 2.5);
    }
    return plan.time < margin * other;
}

// NCHW convolutions with a stride of two along x are gathered but where a kernel larger than 1x1 has groups that fetch many rows, which
// staging reads once; work: tiles x k-steps, small where most CUs would idle on the staged kernel's boxes.  1x1 layers only go back where most
// is kept.  Of 4164 random ones (1x1 and 3x3, 8 to 60 columns, 16-bit results) that nothing was fitted to 2898 are gathered, at .57 of the staged kernel's time, and 20 of these lose
// more than 4 %, up to 36 %; of 2287 dear ones 857 at .65, 20 lose as much, up to 45 % (profiles/strided_sweep.csv holds those that the limits came from).
// Where it does not hold: 52 images of 35x35, 220 -> 896 channels at 50 %, V = 64 107 us staged, 289 gathered; 37 of 28x28, 256 -> 560,
// V = 16 106 and 429; 19 of 34x33, 231 -> 64 at 30 %, V = 16 19.3 and 37.8; where it does: 32 of 56x56, 128 -> 128 at 75 %,
// V = 32 22.6 and 19.1; 1x1, 6 of 19x19, 1968 -> 96 at 95 % 16.0 and 4.4.
inline bool strided_runs_pay(int V, long G, int taps, double kept, double work)
{
    const double fetches = G * kept;
    if (taps == 1) return V == 128 || kept < (V == 32 ? .81 : .61) || work < (V == 16 ? 6000 : V == 32 ? 8000 : 48000);
    if (V == 16) return fetches < 3 && (kept < .21 || work < 4000);
    if (V == 32) return fetches < (work < 8000 ? 3 : 1.5);
    if (V == 64) return fetches < 1.2 || work < 12000;
    return fetches < 2.5;
}

// The LayerNorm-side transposition's kernels (layernorm_transpose.hip).  FEW: blocks of 16 or 8 tokens whose features several workgroups share; RESIDENT: 32 or
// 64 tokens with all their features in the LDS; REGISTER: 32 tokens, 4096 features at a time in registers; STREAM: 64 tokens, any number of features.
enum class Ln { FEW, RESIDENT, REGISTER, STREAM };
struct LnChoice { Ln kernel; int tokens; };

// RESIDENT: bytes of LDS for `tokens` tokens, and their pitch in 16-bit units, (pitch / 2) mod 8 as the kernel wants it
inline long ln_resident_bytes(int tokens, int K, int& pitch)
{
    const int want = tokens == 32 ? 2 : 1;
    int pad = 0;
    while (((K + pad) / 2) % 8 != want) pad += 2;
    pitch = K + pad;
    return (long)tokens * pitch * 2 + 2L * tokens * 4 + 2L * K * 4;
}

// Few tokens: 16 at a time (up to 2048 features) or 8, the features shared by about 128 workgroups (up to 256 for more
// than 64 blocks of 8; twice as many cost what their reads of the same rows take).  us by the other kernels / this one: 64 tokens of
// 256 features 4.1 / 3.7, 1024 5.5 / 3.9, 2048 7.8 / 4.5, 4096 8.3 / 5.1, 16 384 16.5 / 9.4; 552 tokens of 1024
// 5.9 / 4.3, 2048 8.3 / 5.3, 3584 10.2 / 6.8, 8192 14.5 / 12.3, 16 384 25.0 / 19.5; 2048 of 1024 5.9 / 5.2, of 2048
// 8.3 / 7.3; 4096 of 1024 6.6 / 6.2; but 4096 of 1600 8.3 / 9.2, 1024 of 4096 8.7 / 9.3, of 8192 13.3 / 15.5, of 16 384 23.3 / 27.3.
// Blocks of 32 tokens (64-byte row segments, two workgroups per CU) are faster than of 64 while input
// and output together stay well inside the 256 MB memory-side cache, where the halves of a
// line still meet; beyond that the 128-byte segments of 64-token blocks win (measured:
// 26 against 27 us at 134 MB, 53 against 44 us at 201 MB).
inline LnChoice choose_layernorm(long N, int K, bool normalize)
{
    if (normalize && K <= 16384 && N <= (K <= 1024 ? 4096 : K <= 2048 ? 2048 : 768)) return {Ln::FEW, K <= 2048 ? 16 : 8};
    constexpr long LDS_CAP = 160 * 1024 - 256;
    int pitch = 0;
    if (4.0 * (double)N * (double)K > 160e6 && ln_resident_bytes(64, K, pitch) <= LDS_CAP) return {Ln::RESIDENT, 64};
    if (ln_resident_bytes(32, K, pitch) <= LDS_CAP) return {Ln::RESIDENT, 32};
    if (K <= 16384) return {Ln::REGISTER, 32};
    return {Ln::STREAM, 64};
}

// REGISTER: workgroups that share a token block.
// Few tokens: the 1024-feature slices of a token block are shared by several workgroups, each of which takes the
// statistics for itself (its reads of the other slices come from the L2), as long as there is at
// most one workgroup per CU.  One workgroup per 32 tokens leaves most CUs idle: 848 tokens of 5800
// features 22.5 -> 16.1 us, 1600 of 13 152 47.9 -> 37.0 us, 2048 of 4096
// 15.0 -> 10.1.  (Up to 768 tokens do not come here with a LayerNorm, above.)
// With a LayerNorm every share reads all slices first: worth it when that at least halves what is left to each
// (us one / shared: 4000 tokens of 3000 features, 2 of 3 slices each, 12.4 / 14.2; of 5120, 3 of 5, 24.2 / 24.8;
// 4096 of 4096, 2 of 4, 14.9 / 13.4).  Nor by two where a token has more than 8 slices and the output rows are
// whole 64-byte blocks (stream; 4096 tokens of 16 384 features 69.5 / 71.8, transposed only 45 / 48; of 8192, 33.6 / 34.0
// and 24.0 / 22.4)
inline int ln_register_shares(long N, int K, bool normalize, bool stream)
{
    const long blocks = (N + 31) / 32;
    const int slices = (K + 1023) / 1024;
    int shares = blocks > 0 && blocks < 256 ? (int)(256 / blocks) : 1;
    if (shares > slices) shares = slices;
    if ((normalize && 2 * ((slices + shares - 1) / shares) > slices) || (stream && slices > 8 && shares < 3)) shares = 1;
    return shares;
}

}  // namespace shflbw
