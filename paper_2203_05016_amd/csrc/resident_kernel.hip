// Slab kernel with the whole slab resident, for the Shfl-BW product on gfx950 (CDNA4): linear layers, 1x1
// convolutions and convolutions in runs whose reduction is short enough (K <= 1278) that 64 columns of X (of the unfolded matrix)
// fit the 160 KB LDS of a CU.
//
// A workgroup copies its 64 columns of X to the LDS once, every row, and its wavefronts then take row groups of the
// workgroup's share one after the other, each at its own pace: no ring, no hand-over, no barrier after the first.
// Section 4.3's stitching happens at LDS-read time, as in the ring kernel: the transposing read takes an address per
// lane, so a lane points at the rows that the step's column indices name.
//
// Against the ring kernel (12 groups x 128 columns) the bytes from the L2s into the CUs are the same, 321 MB at 4096 x 1024 by 8192,
// V = 32, 75 %: X 34 instead of 184, weights 290 instead of 146.  But they are loads into registers, which run at twice the rate of
// direct-to-LDS loads, nothing waits for another wavefront's pace, and stores leave all the time instead of in three bursts: 34.9 -> 26.8
// us; 32-bit results 52.6 -> 35.0; unpruned 82 -> 76.  Against the gather kernel a group of V rows does not fetch its own copy of X, which counts
// most where V is small, and rows of no alignment cost twice once per workgroup and not once per group: by 8191 50.5 -> 28.6;
// V = 16, 56.5 -> 31.6 and by 2047 33.1 -> 14.8.
//
// What bounds it (the launch above; parts taken out, one at a time): without the products 21.3 us, without the loads of weights 20.0, without
// stores 22.5, of X's copy 21.9; the copy alone 4 to 5 us from launch to barrier.  The return path of loads moves 64 bytes per clock and
// CU, and a step of 64 columns brings 1 KB of weights through it (16 clocks, all that a step can do about it with 64 columns resident), beside 16 clocks
// of the matrix cores; clocks are 1.5 to 1.7 GHz in it.  What else used that path was taken out: an index load of 4 bytes per lane costs what one of 16 does, so
// indices come 16 steps at a time (2 loads per 4 steps -> 1 per 16: 28.3 -> 26.9).  HBM sees 102 MB, 86 of them what it cannot do without.
// Tried without a gain: weights eight steps ahead instead of four (+-1 %, V = 16 +10 %: registers), rows three ahead instead of two (+1 %, V = 16 +7 %),
// groups in another order on every CU (+1 %, by 2047 +8 %).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "gather_kernel.hip"

namespace shflbw {

typedef __attribute__((address_space(3))) char* lds_char_ptr;

constexpr int RESIDENT_TN = 64;                              // columns of the slab
constexpr int RESIDENT_ROW = RESIDENT_TN * 2;                // bytes of a row of it

// LDS of a workgroup: the slab, an all-zero row for padded slots, the counter of groups
constexpr int resident_lds_bytes(int K) { return (K + 1) * RESIDENT_ROW + 16; }

struct ResidentArgs {
    PackedView A;
    int K, parts;             // rows of X; workgroups that share a column tile, each with a share of the groups
    int per_part;             // groups of a share (the last may have fewer)
    unsigned long long m_parts;   // ceil(2^40 / parts)
    int per_xcd, total;       // workgroups of an XCD, and with work (column tiles x parts, below 2^19)
    unsigned pitch, ybytes;   // bytes of a result row (below 2^24, as are the rows), and from Y's start to its end (below 2^32)
    int uniform_steps;        // k-steps of every group when they all have the same number, else -1
};

// Lanes whose numbers differ in bit BIT (0 or 1) trade: p is what lanes with the bit clear keep, q with it set; afterwards
// p is the lane's share of what the lane with the bit clear had, q of what the other had.
// FRESH: p and q come straight from the matrix cores, whose results other instructions may read 18 cycles after the product
// at the earliest; the compiler keeps that distance for its own instructions, and does not look into these.
template <int BIT, bool FRESH, class T>
__device__ __forceinline__ void trade(T& p, T& q)
{
    // in one instruction per register: a select whose first operand comes from the other lane.  VCC has lanes with the bit clear.
    const unsigned long long clear = BIT == 0 ? 0x5555555555555555ull : 0x3333333333333333ull;
    T a, b;
#define SHFLBW_TRADE(WAIT, PERM)                                                                             \
    asm volatile(WAIT "s_mov_b64 vcc, %16\n\ts_nop 1\n\t"                                                          \
        "v_cndmask_b32_dpp %0, %12, %8, vcc " PERM "\n\tv_cndmask_b32_dpp %1, %13, %9, vcc " PERM "\n\t"   \
        "v_cndmask_b32_dpp %2, %14, %10, vcc " PERM "\n\tv_cndmask_b32_dpp %3, %15, %11, vcc " PERM "\n\t" \
        "s_not_b64 vcc, vcc\n\t"                                                                       \
        "v_cndmask_b32_dpp %4, %8, %12, vcc " PERM "\n\tv_cndmask_b32_dpp %5, %9, %13, vcc " PERM "\n\t"   \
        "v_cndmask_b32_dpp %6, %10, %14, vcc " PERM "\n\tv_cndmask_b32_dpp %7, %11, %15, vcc " PERM          \
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])        \
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(q[0]), "v"(q[1]), "v"(q[2]), "v"(q[3]), "s"(clear)            \
        : "vcc", "scc")
#define SHFLBW_BIT0 "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
#define SHFLBW_BIT1 "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
#define SHFLBW_WAIT "s_nop 15\n\ts_nop 3\n\t"
    if constexpr (BIT == 0 && FRESH) SHFLBW_TRADE(SHFLBW_WAIT, SHFLBW_BIT0);
    else if constexpr (BIT == 0) SHFLBW_TRADE("", SHFLBW_BIT0);
    else if constexpr (FRESH) SHFLBW_TRADE(SHFLBW_WAIT, SHFLBW_BIT1);
    else SHFLBW_TRADE("", SHFLBW_BIT1);
#undef SHFLBW_WAIT
#undef SHFLBW_BIT1
#undef SHFLBW_BIT0
#undef SHFLBW_TRADE
    p = a;
    q = b;
}

template <int V, int WAVES, typename OutT, class Geom, bool BF>
__global__ __launch_bounds__(64 * WAVES, V >= 64 ? 2 : 4) void shflbw_slab_kernel_resident(ResidentArgs a, Geom geom)
{
    constexpr bool SMALL = V == 16;                          // 16x16x32 instruction
    constexpr int TK = SMALL ? 32 : 16;
    constexpr int IPG = V == 128 ? 2 : 1;                    // items of a group: a wavefront takes 64 of its rows at most
    constexpr int RBG = SMALL ? 1 : V / 32, RB = RBG / IPG;  // row blocks of a group, of an item
    constexpr int TILE_N = SMALL ? 16 : 32;
    constexpr int NT = RESIDENT_TN / TILE_N;
    constexpr bool F32 = sizeof(OutT) == 4;
    constexpr int ROWS_E = SMALL ? 16 : 32;                  // rows of a row block
    // (rows one step ahead instead of two: by 2047 15.0 us instead of 12.2, by 4096 16.6 instead of 14.8; three gained nothing)
    constexpr int QUAD = 4, BATCH = 16, AHEAD = 2;       // steps of a pass through the loop; whose indices are loaded at a time; that rows are read ahead
    extern __shared__ __attribute__((aligned(128))) char slab[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned w = (blockIdx.x & 7) * (unsigned)a.per_xcd + (blockIdx.x >> 3);
    const int tile = (int)(((unsigned long long)w * a.m_parts) >> 40), part = (int)w - tile * a.parts;
    const int g_lo = part * a.per_part, g_hi = g_lo + a.per_part < a.A.G * IPG ? g_lo + a.per_part : a.A.G * IPG;
    const long n0 = (long)tile * RESIDENT_TN;
    const int K = a.K;
    int* claimed = reinterpret_cast<int*>(slab + (K + 1) * RESIDENT_ROW);

    // ---- the slab: thread t takes 8 columns of rows t/8, t/8 + 8*WAVES, ...
    constexpr int STAGE_ROWS = 8 * WAVES, STAGES = V >= 64 ? 20 : 10;
    const int srow = tid >> 3, sunit = tid & 7;
    geom.init(n0 + sunit * 8);
    typename Geom::loaded_t staged[STAGES];
    int moved[Geom::FINISH ? STAGES : 1];                    // what geom.finish8 needs to know of them
#pragma unroll
    for (int i = 0; i < STAGES; ++i) {
        int shift = 0;
        const int r = srow + i * STAGE_ROWS;
        if (i * STAGE_ROWS + wave * 8 < K) staged[i] = geom.load8(geom.entry(r, r < K), shift);   // uniform for the wavefront
        if constexpr (Geom::FINISH) moved[i] = shift;
    }
    // (after the loads: before them it would be a wait for the arguments of its own; tiles beyond the last read nothing)
    if (w >= (unsigned)a.total) return;                      // uniform for the workgroup
    __builtin_amdgcn_sched_barrier(0);

    // ---- the stream of k-steps, four at a time, of this wavefront's groups
    // a lane addresses the row of slot 8 * (l/32) + l/4 % 4 (V = 16: 8 * (l/16) + ..) in its first transposed read of a step, of slot + 4 in its second
    const int bl = lane >> 4, il = lane & 15;
    auto bounds = [&](int g, int& beg, int& n) __attribute__((always_inline)) {
        typedef const __attribute__((address_space(4))) int32_t* uniform_ptr;   // scalar loads
        const uniform_ptr p = (uniform_ptr)(size_t)a.A.step_ptr;
        beg = a.uniform_steps >= 0 ? g / IPG * a.uniform_steps : p[g / IPG];
        n = a.uniform_steps >= 0 ? a.uniform_steps : p[g / IPG + 1] - beg;
    };
    half8 wt[QUAD][RB];
    __amdgpu_buffer_rsrc_t wd;
    auto load_w = [&](int u) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            wt[u][rb] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(wd, lane * 16 + (u * RBG + rb) * 1024, 0, 0));
    };
    // the four steps at `beg` for item i, of which `left` exist: the others read zeros
    auto aim = [&](int i, int beg, int left) __attribute__((always_inline)) {
        left = left < 0 ? 0 : left;
        const long half = IPG > 1 ? i % IPG * RB * 64 : 0;   // (the last step's end minus what lies before the item's rows)
        wd = __builtin_amdgcn_make_buffer_rsrc(const_cast<half8*>(a.A.values + (long)beg * RBG * 64 + half), 0,
                                               left ? left * RBG * 1024 - (int)half * 16 : 0, GATHER_BUFFER_FLAGS);
    };
    // Column indices come 16 steps at a time.  A lane wants its two slots of steps s, 4 + s, 8 + s and 12 + s, s = l % 4:
    // lanes that differ in e = l/4 % 4 load four slots each of step 4*e + s and trade until each has its one of four steps.
    // V >= 32: lanes 16 apart want the same; one loads the lower four slots and one the upper, and they exchange.
    constexpr int LOADS = SMALL ? 2 : 1;
    run_t raw[LOADS];
    int cols[2][BATCH / QUAD];
    auto fetch = [&](int beg, int left) __attribute__((always_inline)) {
        left = left < 0 ? 0 : left;
        const __amdgpu_buffer_rsrc_t cd =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.A.col_idx + (long)beg * TK), 0, left * TK * 4, GATHER_BUFFER_FLAGS);
        const int at = ((4 * (il >> 2) + (lane & 3)) * TK + (SMALL ? 8 * bl : 8 * (bl >> 1) + 4 * (bl & 1))) * 4;
        raw[0] = load_run(cd, (unsigned)at);
        if constexpr (SMALL) raw[1] = load_run(cd, (unsigned)at + 16);
    };
    auto deal = [&]() __attribute__((always_inline)) {
        auto trade4 = [&](unsigned& p, unsigned& q) __attribute__((always_inline)) {   // lane ^ 4
            const unsigned p0 = p;
            p = (unsigned)__builtin_amdgcn_update_dpp((int)p, (int)q, 0x114, 0xf, 0xa, false);
            q = (unsigned)__builtin_amdgcn_update_dpp((int)q, (int)p0, 0x104, 0xf, 0x5, false);
        };
        auto trade8 = [&](unsigned& p, unsigned& q) __attribute__((always_inline)) {   // lane ^ 8
            const unsigned p0 = p;
            p = (unsigned)__builtin_amdgcn_update_dpp((int)p, (int)q, 0x128, 0xf, 0xc, false);
            q = (unsigned)__builtin_amdgcn_update_dpp((int)q, (int)p0, 0x128, 0xf, 0x3, false);
        };
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            unsigned r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (SMALL) r[i] = raw[h][i];
                else r[i] = __builtin_amdgcn_permlane16_swap(raw[0][i], raw[0][i], false, false)[h];
            }
            trade8(r[0], r[2]);
            trade8(r[1], r[3]);
            trade4(r[0], r[1]);
            trade4(r[2], r[3]);
#pragma unroll
            for (int i = 0; i < 4; ++i) cols[h][i] = (int)r[i];
        }
    };
    // The wavefront's groups: the first two by its number, the others are claimed one ahead, so that nothing waits for a claim.
    int g = g_lo + wave, next = g + WAVES;
    int beg = 0, n = 0, next_beg = 0, next_n = 0;
    const bool any = g < g_hi;
    if (any) bounds(g, beg, n);
    if (next < g_hi) bounds(next, next_beg, next_n);
    if (any) {
        fetch(beg, n);
        aim(g, beg, n);
#pragma unroll
        for (int u = 0; u < QUAD; ++u) load_w(u);
    }
    __builtin_amdgcn_sched_barrier(0);

    // Where byte b of row r lies: r * 128 + (b ^ turn(r)).  A transposed read covers, per 32 lanes, four rows (V = 16: eight)
    // and a 64-byte (32-byte) window of each; turn() moves the windows of rows that differ in their low bits into
    // different banks.
    auto turn = [](int r) __attribute__((always_inline)) {
        if constexpr (SMALL) return F32 ? ((r << 2) & 8) | ((r << 4) & 64) : (r << 2) & 24;
        else return F32 ? (r << 5) & 64 : (r << 4) & 32;
    };
#pragma unroll
    for (int i = 0; i < STAGES; ++i) {
        const int r = srow + i * STAGE_ROWS;
        if (i * STAGE_ROWS + wave * 8 < K && r < K) {
            run_t v;
            if constexpr (Geom::FINISH) v = Geom::finish8(staged[i], moved[i]);
            else v = staged[i];
            const int t = turn(r);
            if constexpr (SMALL) {
                if (t & 8) v = run_t{v[2], v[3], v[0], v[1]};
            }
            *reinterpret_cast<run_t*>(slab + r * RESIDENT_ROW + ((sunit * 16) ^ (t & ~15))) = v;
        }
    }
    if (tid < 8) *reinterpret_cast<run_t*>(slab + K * RESIDENT_ROW + tid * 16) = run_t{0, 0, 0, 0};
    if (tid == 0) *claimed = g_lo + 2 * WAVES;
    // byte of the row that this lane addresses for instruction tile 0.  The operand's columns are any that
    // suit the write-back, in fours: an accumulator quad of a lane then continues the one before it.
    //   16-bit results: a lane's quads make one run of 32 (V = 16: 16) columns;
    //   32-bit: a run of 16 (8) columns in each half of the tile.
    const int pc = il & 3;                                   // the four columns that the lane addresses, of its block's 16
    int pos;
    if constexpr (SMALL) pos = F32 ? 16 * pc : 32 * pc;
    else pos = F32 ? 32 * (pc & 1) + 16 * (bl & 1) + 8 * (pc >> 1) : 64 * (pc & 1) + 16 * (bl & 1) + 8 * (pc >> 1);
    auto tile_bits = [](int t) __attribute__((always_inline)) {
        if constexpr (SMALL) return F32 ? 8 * (t & 1) + 64 * (t >> 1) : 8 * t;
        else return F32 ? 64 * t : 32 * t;
    };

    const int slab_at = (int)(size_t)(lds_char_ptr)slab;
    int offa = 0, offb = 0;                                  // where the rows of the next four steps' slots lie
    auto offsets = [&](int left) __attribute__((always_inline)) {
        const bool real = (lane & 3) < left;
        const int rowa = real && cols[0][0] >= 0 ? cols[0][0] : K, rowb = real && cols[1][0] >= 0 ? cols[1][0] : K;
        offa = slab_at + rowa * RESIDENT_ROW + turn(rowa);
        offb = slab_at + rowb * RESIDENT_ROW + turn(rowb);
    };
    half8 x[QUAD][NT];
    auto read_x = [&](int u, half8 (&xs)[NT]) __attribute__((always_inline)) {
        // lane l's rows of step u are with lane 4*(l/4) + u
        auto of_step = [&](int off) __attribute__((always_inline)) {
            return u == 0 ? __builtin_amdgcn_mov_dpp(off, 0x00, 0xf, 0xf, true) : u == 1 ? __builtin_amdgcn_mov_dpp(off, 0x55, 0xf, 0xf, true) :
                   u == 2 ? __builtin_amdgcn_mov_dpp(off, 0xaa, 0xf, 0xf, true) : __builtin_amdgcn_mov_dpp(off, 0xff, 0xf, 0xf, true);
        };
        const int a0 = of_step(offa) ^ pos, b0 = of_step(offb) ^ pos;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(size_t)(a0 ^ tile_bits(t)));
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(size_t)(b0 ^ tile_bits(t)));
            const half4 l4 = __builtin_bit_cast(half4, lo), h4 = __builtin_bit_cast(half4, hi);
            xs[t] = half8{l4[0], l4[1], l4[2], l4[3], h4[0], h4[1], h4[2], h4[3]};
        }
    };
    deal();
    offsets(n);

    // ---- for the write-back: where this lane's columns lie in a result row, bytes (PAST: beyond the last)
    typedef unsigned unit_t __attribute__((ext_vector_type(4)));
    constexpr int OPV = 16 / (int)sizeof(OutT);
    constexpr unsigned PAST = 0xffffffffu;
    unsigned col_at[F32 ? 2 : 1];
#pragma unroll
    for (int h = 0; h < (F32 ? 2 : 1); ++h) {
        const long c = n0 + 32 * h + (SMALL ? 2 * bl + (lane & 1) : 4 * (lane >> 5) + (lane & 3)) * OPV;
        col_at[h] = c < geom.N ? geom.out_col(c) * (unsigned)sizeof(OutT) : PAST;
    }
    const __amdgpu_buffer_rsrc_t yd = __builtin_amdgcn_make_buffer_rsrc(geom.Y, 0, (int)a.ybytes, GATHER_BUFFER_FLAGS);
    auto unit16 = [&](floatx4 lo, floatx4 hi) __attribute__((always_inline)) {
        typedef typename std::conditional<F32, _Float16, OutT>::type half_t;   // (32-bit results have no use for it)
        typedef half_t vec8 __attribute__((ext_vector_type(8)));
        return __builtin_bit_cast(unit_t, vec8{(half_t)lo[0], (half_t)lo[1], (half_t)lo[2], (half_t)lo[3],
                                               (half_t)hi[0], (half_t)hi[1], (half_t)hi[2], (half_t)hi[3]});
    };

    __syncthreads();
    if (!any) return;
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) read_x(u, x[u]);

    for (;;) {
        int claim = 0;
        if (lane == 0) claim = __hip_atomic_fetch_add(claimed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        int row_of[RB];                                      // this lane's stored rows among the results'
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) row_of[rb] = a.A.row_indices[(long)g * (V / IPG) + rb * 32 + (lane & (ROWS_E - 1))];
        floatx16 acc32[SMALL ? 1 : RB][SMALL ? 1 : NT];
        floatx4 acc16[SMALL ? NT : 1];
        int left = n, pass_of = 0;                           // of the passes that share a load of indices
        // the indices after those at hand: of the same group or of the next
        auto fetch_more = [&]() __attribute__((always_inline)) {
            if (left > BATCH) fetch(beg + BATCH, left - BATCH);
            else fetch(next_beg, next_n);
        };
        fetch_more();
        // a pass; the first of a group starts the sums.  False after the group's last.
        auto pass = [&](auto first_tag) __attribute__((always_inline)) {
            constexpr bool FIRST = decltype(first_tag)::value;
            const bool last = left <= QUAD;
            // the weights of the next pass: the next group's after the last of this
            const int pass_beg = last ? next_beg : beg + QUAD, pass_left = last ? next_n : left - QUAD;
            aim(last ? next : g, pass_beg, pass_left);
#pragma unroll
            for (int u = 0; u < QUAD; ++u) {
                // the rows of the step after the next before the products of this
                const int v = u + AHEAD;
                if (v % QUAD == 0) {
                    bool deal_now = false;
                    if (v == QUAD) deal_now = last || ++pass_of == BATCH / QUAD;
                    if (deal_now) {
                        deal();
                        pass_of = 0;
                    } else {
#pragma unroll
                        for (int i = 0; i + 1 < BATCH / QUAD; ++i) { cols[0][i] = cols[0][i + 1]; cols[1][i] = cols[1][i + 1]; }
                    }
                    offsets(v == QUAD ? pass_left : left - v);
                    if (v == QUAD) {
                        beg = pass_beg;
                        left = pass_left;
                        if (deal_now && !last) fetch_more();
                    }
                }
                read_x(v % QUAD, x[v % QUAD]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if constexpr (SMALL) {
                        acc16[t] = mma16<BF>(x[u % QUAD][t], wt[u][0], FIRST && u == 0 ? floatx4{} : acc16[t]);
                    } else {
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) acc32[rb][t] = mma32<BF>(x[u % QUAD][t], wt[u][rb], FIRST && u == 0 ? floatx16{} : acc32[rb][t]);
                    }
                }
                load_w(u);
                __builtin_amdgcn_sched_barrier(0);
            }
            return !last;
        };
        bool more = pass(std::true_type{});
        while (more) more = pass(std::false_type{});
        const int claimed_now = __builtin_amdgcn_readfirstlane(claim);
        int claimed_beg = 0, claimed_n = 0;
        if (claimed_now < g_hi) bounds(claimed_now, claimed_beg, claimed_n);
        unsigned row_at[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) row_at[rb] = __umul24((unsigned)row_of[rb], a.pitch);

        // ---- reordered write-back, in registers.  A lane holds one stored row and units of 16 bytes of it that follow each
        // other; lanes whose numbers differ in bit 0 (and bit 1) trade units until each has one unit of several rows, and
        // neighbouring lanes neighbouring units.
        constexpr int HALVES = F32 ? 2 : 1;
        // (trades and row offsets before the branch: lanes beyond the last column take part)
        auto store4 = [&](auto stream_tag) __attribute__((always_inline)) {
            constexpr int NT_BIT = decltype(stream_tag)::value ? 2 : 0;
            if constexpr (SMALL) {
                // result column 4 * (t-th quad): 16 bits 16*(l/16) + 4t, 32 bits 32*(t/2) + 8*(l/16) + 4*(t%2)
#pragma unroll
                for (int h = 0; h < HALVES; ++h) {
                    unit_t r[2];
                    if constexpr (F32) {
                        r[0] = __builtin_bit_cast(unit_t, acc16[2 * h]);
                        r[1] = __builtin_bit_cast(unit_t, acc16[2 * h + 1]);
                    } else {
                        r[0] = unit16(acc16[0], acc16[1]);
                        r[1] = unit16(acc16[2], acc16[3]);
                    }
                    trade<0, F32>(r[0], r[1]);
                    const unsigned at[2] = {(unsigned)__builtin_amdgcn_mov_dpp((int)row_at[0], 0xa0, 0xf, 0xf, true) + col_at[h],
                                            (unsigned)__builtin_amdgcn_mov_dpp((int)row_at[0], 0xf5, 0xf, 0xf, true) + col_at[h]};
                    if (col_at[h] != PAST) {
#pragma unroll
                        for (int i = 0; i < 2; ++i) __builtin_amdgcn_raw_buffer_store_b128(r[i], yd, (int)at[i], 0, NT_BIT);
                    }
                }
            } else {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    auto quad = [&](int t, int q) __attribute__((always_inline)) {
                        return floatx4{acc32[rb][t][4 * q], acc32[rb][t][4 * q + 1], acc32[rb][t][4 * q + 2], acc32[rb][t][4 * q + 3]};
                    };
#pragma unroll
                    for (int h = 0; h < HALVES; ++h) {
                        unit_t r[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if constexpr (F32) r[i] = __builtin_bit_cast(unit_t, quad(h, i));
                            else r[i] = unit16(quad(i / 2, 2 * (i % 2)), quad(i / 2, 2 * (i % 2) + 1));
                        }
                        trade<1, F32>(r[0], r[2]);
                        trade<1, F32>(r[1], r[3]);
                        trade<0, false>(r[0], r[1]);
                        trade<0, false>(r[2], r[3]);
                        const unsigned at[4] = {(unsigned)__builtin_amdgcn_mov_dpp((int)row_at[rb], 0x00, 0xf, 0xf, true) + col_at[h],
                                                (unsigned)__builtin_amdgcn_mov_dpp((int)row_at[rb], 0x55, 0xf, 0xf, true) + col_at[h],
                                                (unsigned)__builtin_amdgcn_mov_dpp((int)row_at[rb], 0xaa, 0xf, 0xf, true) + col_at[h],
                                                (unsigned)__builtin_amdgcn_mov_dpp((int)row_at[rb], 0xff, 0xf, 0xf, true) + col_at[h]};
                        if (col_at[h] != PAST) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) __builtin_amdgcn_raw_buffer_store_b128(r[i], yd, (int)at[i], 0, NT_BIT);
                        }
                    }
                }
            }
        };
        with_stores(geom, store4);

        if (next >= g_hi) break;
        g = next;
        n = next_n;
        next = claimed_now;
        next_beg = claimed_beg;
        next_n = claimed_n;
    }
}

}  // namespace shflbw
