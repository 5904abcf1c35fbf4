// Per-wavefront gather kernel for the Shfl-BW product on gfx950 (CDNA4).
//
// One wavefront owns one row group (V stored rows) x WN output columns and runs Algorithm 1's loop on its own
// (sharing weights with its workgroup's other wavefronts, or steps, where that pays: SHARES below):
//   BulkLoadMeta  - the column indices are fetched 64 at a time, one to two batches ahead, and become a list of
//                   row offsets in the LDS, private to the wavefront;
//   StitchTile    - the TK activation rows of a k-step are loaded (16 bytes per lane, coalesced along N) two steps
//                   ahead into registers and turned into matrix-core operands there: pairs of rows, then trades
//                   between the lanes that hold the other rows of the operand;
//   WarpMMA       - the operands are multiplied with the weight operand (16 bytes per lane from the packed array,
//                   already in operand order, straight from memory or by way of the LDS), fp32 accumulation;
//   ReorderedWriteBack - accumulators go through LDS so that every stored row leaves as full 16-byte-per-lane
//                   row segments, to the row named by row_indices.
//
// The product is computed as (X^T tile) x (W^T tile), i.e. the instruction's row dimension runs over output
// columns n and its column dimension over the group's rows: a lane's accumulators are columns of one row, and which
// columns is free (operands(), quad_col()): four neighbouring ones make one LDS write in the epilogue.
//
// What bounds it: a load of 16 bytes per lane takes the address unit 16 cycles where every four lanes stay inside a 64-byte
// block and about 32 where they do not (130 and 60 GB/s per CU, whatever the length of a row segment; 8 bytes per lane cost
// as much as 16), so a step of 64 columns costs a CU 32 cycles for X and 16 per row block for weights that are
// not shared, beside 8 matrix-core cycles per row block; and below 10 us the chain launch -> column indices -> rows ->
// products -> partial sums -> stores (1.2 us between launches, 0.9 to the first indices, 0.4 to the first rows, 0.5 to 1
// at the end).  Passing the rows through the LDS for the transposition, as this kernel did before, cost 36 LDS cycles per step
// and 64 columns and a write-read latency per step: 8192 x 8192 by 16384, V = 64 at 75 %, 713 -> 593 us with the weights
// shared; 4096 x 1024 by 2047 18.4 -> 16.4; 1024 x 1024 by 4096 7.15 -> 7.05.
//
// Operand and accumulator lane maps (checked on hardware):
//   v_mfma_f32_32x32x16_f16  A: lane l = row l%32, k = 8*(l/32)+e
//                            B: lane l = col l%32, k = 8*(l/32)+e
//                            D: lane l, reg r = row 8*(r/4)+4*(l/32)+r%4, col l%32
//   v_mfma_f32_16x16x32_f16  A: lane l = row l%16, k = 8*(l/16)+e; B alike;
//                            D: lane l, reg r = row 4*(l/16)+r, col l%16
//   ds_read_b64_tr_b16 (the slab kernel's): inside each block of 16 lanes, result element e of
//     lane i is element i%4 of the 8 bytes addressed by lane 4*e + i/4; with
//     lanes 4q..4q+3 pointing at 16 consecutive n of row k_q, lane i ends up
//     with column n_i of rows k_0..k_3.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "shflbw_internal.h"

namespace shflbw {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The matrix-core products.  Operands travel as 16-bit patterns in half8
// registers whatever their format; BF selects the bfloat16 instruction, whose
// operand and accumulator lane maps are those of the binary16 one.
template <bool BF>
__device__ __forceinline__ floatx16 mma32(half8 a, half8 b, floatx16 c)
{
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
template <bool BF>
__device__ __forceinline__ floatx4 mma16(half8 a, half8 b, floatx4 c)
{
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// Orders LDS traffic between the lanes of one wavefront.  The hardware runs a
// wavefront's LDS instructions in order; this only stops the compiler from
// moving accesses across the point.
#define SHFLBW_WAVE_LDS_SYNC()                                   \
    do {                                                         \
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   \
        __builtin_amdgcn_wave_barrier();                         \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");   \
    } while (0)

// 8 consecutive 16-bit values in registers, two to a register
typedef unsigned run_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ run_t load_run(__amdgpu_buffer_rsrc_t d, unsigned off)
{
    return __builtin_amdgcn_raw_buffer_load_b128(d, (int)off, 0, 0);
}

struct PackedView {
    const int32_t* row_indices;
    const int32_t* step_ptr;
    const int32_t* col_idx;
    const half8* values;  // 16-byte units
    int G;
};

// ---------------------------------------------------------------- geometry
// A geometry answers two questions: which 8 activation values sit at
// (reduction index k, output columns n..n+7), and where do output values
// (original row, columns n..n+cnt-1) go, with streaming stores or plain ones
// where it has the choice (CHOICE).  init(n) fixes the lane's columns; a reduction index comes as an
// entry of the wavefront's list, which entry() makes of the column index; FINISH: finish8() turns
// what load8() returned into the values.

// Linear layer: X[K][N] and Y[M][N] row-major.  ALIGNED: N, ldx, ldy are
// multiples of 8 and both bases are 16-byte aligned.
template <bool ALIGNED>
struct GeomLinear {
    const _Float16* X;
    void* Y;
    long ldx, ldy, N;
    long n0;                                // the lane's first column
    static constexpr bool FINISH = false, CONV = false, CHOICE = false;
    typedef int entry_t;
    typedef run_t loaded_t;

    __device__ __forceinline__ void init(long n) { n0 = n; }
    __device__ __forceinline__ entry_t entry(int col, bool exists) const { return exists ? col : -1; }
    __device__ __forceinline__ run_t load8(entry_t col, int&) const
    {
        half8 v = {};
        if (col < 0) return __builtin_bit_cast(run_t, v);
        const _Float16* p = X + (long)col * ldx + n0;
        if (ALIGNED) {
            if (n0 < N) v = *reinterpret_cast<const half8*>(p);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (n0 + e < N) v[e] = p[e];
        }
        return __builtin_bit_cast(run_t, v);
    }

    template <bool STREAM, int CNT, typename OutT>
    __device__ __forceinline__ void store(int row, long n, const OutT* vals) const
    {
        OutT* p = static_cast<OutT*>(Y) + (long)row * ldy + n;
        if (ALIGNED) {
            if (n < N) {
                typedef OutT vec_t __attribute__((ext_vector_type(CNT)));
                vec_t v;
#pragma unroll
                for (int e = 0; e < CNT; ++e) v[e] = vals[e];
                // the output is not read again by this kernel: keep it from displacing X and W in the L2
                __builtin_nontemporal_store(v, reinterpret_cast<vec_t*>(p));
            }
        } else {
#pragma unroll
            for (int e = 0; e < CNT; ++e)
                if (n + e < N) p[e] = vals[e];
        }
    }
};

// CNT consecutive values to p, at the alignment of one value.  STREAM: a streaming store, for an output that must
// not displace X and W in the L2.
template <bool STREAM, int CNT, typename OutT>
__device__ __forceinline__ void store_run(OutT* p, const OutT* vals)
{
    typedef OutT vec_t __attribute__((ext_vector_type(CNT)));
    typedef vec_t run_t __attribute__((aligned(sizeof(OutT))));
    vec_t v;
#pragma unroll
    for (int e = 0; e < CNT; ++e) v[e] = vals[e];
    if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<run_t*>(p));
    else *reinterpret_cast<run_t*>(p) = v;
}

// The aligned linear layer again, with X behind a buffer descriptor: a load's
// address is a saturating addition and a minimum in a vector register (byte offset of the
// row, one 24-bit multiplication per entry of the list, plus the lane's column offset) instead of 64-bit
// arithmetic, and the descriptor's range check stands in for the two conditions - a padded slot
// (column -1) and a lane beyond N get an offset past the end and read as zero.
// The host uses it when K and 2*ldx are below 2^24 and X spans less than 4 GiB.
constexpr int GATHER_BUFFER_FLAGS = 0x00020000;   // last word of a raw buffer descriptor: untyped 32-bit data
struct GeomLinearBuf {
    const _Float16* X;
    void* Y;
    long ldx, ldy, N;
    unsigned xbytes;          // (K-1)*ldx*2 + N*2: what the descriptor covers
    int stream;               // streaming stores (the host's stream_stores)
    __amdgpu_buffer_rsrc_t xd;
    unsigned ldx2, ln2;
    // beyond every descriptor the host admits, and 16 bytes from there do not wrap
    static constexpr unsigned PAST_END = 0xffffffe0u;
    static constexpr bool FINISH = false;   // load returns the values as they are used
    static constexpr bool CONV = false;     // the list's entries take divisions
    static constexpr bool CHOICE = true;    // of streaming and plain stores
    typedef run_t loaded_t;                 // what a load returns, in registers

    __device__ __forceinline__ void init(long n)
    {
        xd = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(X), 0, (int)xbytes, GATHER_BUFFER_FLAGS);
        ldx2 = (unsigned)ldx * 2u;
        ln2 = n < N ? (unsigned)n * 2u : PAST_END;
    }

    // row of X as the kernel's list holds it: its byte offset, past the end for one that does not exist
    typedef unsigned entry_t;
    __device__ __forceinline__ entry_t entry(int col, bool exists) const
    {
        return exists && col >= 0 ? __umul24((unsigned)col, ldx2) : PAST_END;
    }
    // a row or a lane past the end stays there: the sum saturates
    __device__ __forceinline__ run_t load8(entry_t e, int&) const
    {
        return load_run(xd, __builtin_elementwise_min(__builtin_elementwise_add_sat(e, ln2), PAST_END));
    }

    template <bool STREAM, int CNT, typename OutT>
    __device__ __forceinline__ void store(int row, long n, const OutT* vals) const
    {
        if (n < N) store_run<STREAM, CNT>(static_cast<OutT*>(Y) + (long)row * ldy + n, vals);
    }
    // where column n of a result row lies, elements from the row's start (n < N); elements between rows
    __device__ __forceinline__ unsigned out_col(long n) const { return (unsigned)n; }
    long out_pitch() const { return ldy; }
};

// Rows of P contiguous columns with no particular alignment, in `images` matrices (1 for a
// linear layer): X + img*x_image + k*ldx + c and Y + img*y_image + row*ldy + c, c = 0 .. P-1,
// P >= 8.  Linear layers whose N, leading dimensions or bases are not multiples of 16 bytes, and
// 1x1 convolutions with unit stride and no padding on NCHW tensors (Section 4.1's implicit GEMM
// with R = S = 1: image b is a row-major [K][H*W] matrix).
//
// The product's columns are cut into slots of 8 per image; the last slot of an image ends at its
// last column and so overlaps the one before it where 8 does not divide P.  Every load and
// store is then a whole 16 bytes inside one row (at the alignment of its elements, which the
// hardware takes), none is conditional, and the columns of an overlap are computed twice, with
// the same terms in the same order, and stored twice with the same bits.  Measured on 4096 x
// 1024 by 1024 x 2047 (V = 32, 75 %): 18.5 us against 65 us with element-wise loads and stores
// (12.6 us at N = 2048: a row segment of 128 bytes spans two lines when it is not aligned).
// What a load costs is set by whether it is aligned at all (58 to 72 GB/s per CU at any misalignment, 130 aligned), not by the
// address unit's accesses that the counters show, 62 for a load at an odd element, 20 at an even one: loading odd offsets one
// value early, with the missing last value from the next lane, gained nothing when rows went through the LDS (18.6 us; convolutions
// lost 1 us to the extra instructions).  It was not repeated with the rows in registers.
struct GeomRows : GeomLinearBuf {
    long x_image, y_image;   // element strides between images
    int P, slots;            // columns of an image, and ceil(P / 8)
    // min(2^32 / slots, 2^32 - 1), rounded down: quotients by it are at most one short.  (Divisions proper, one
    // before the first load and one before the stores: 24x24 images, 128 -> 384 channels, 50 %, V = 64 5.35 us
    // against 5.18, 56x56, 64 -> 256 channels 13.9 against 13.55.)
    unsigned m_slots;

    // slot of virtual column n -> image and first column
    __device__ __forceinline__ void place(long n, unsigned& img, unsigned& c) const
    {
        const unsigned slot = (unsigned)((unsigned long)n >> 3);
        img = __umulhi(slot, m_slots);
        c = slot - img * (unsigned)slots;
        if (c >= (unsigned)slots) { ++img; c -= (unsigned)slots; }
        c *= 8u;
        c = c < (unsigned)(P - 8) ? c : (unsigned)(P - 8);
    }
    __device__ __forceinline__ void init(long n)
    {
        xd = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(X), 0, (int)xbytes, GATHER_BUFFER_FLAGS);
        ldx2 = (unsigned)ldx * 2u;
        ln2 = PAST_END;
        if (n < N) {
            unsigned img, c;
            place(n, img, c);
            ln2 = (img * (unsigned)x_image + c) * 2u;
        }
    }
    template <bool STREAM, int CNT, typename OutT>
    __device__ __forceinline__ void store(int row, long n, const OutT* vals) const
    {
        if (n < N) {
            unsigned img, c;
            place(n, img, c);
            OutT* p = static_cast<OutT*>(Y) + (long)img * y_image + (long)row * ldy + c + ((unsigned)n & 7u);
            store_run<STREAM, CNT>(p, vals);
        }
    }
    __device__ __forceinline__ unsigned out_col(long n) const
    {
        unsigned img, c;
        place(n, img, c);
        return img * (unsigned)y_image + c + ((unsigned)n & 7u);
    }
};

// 1x1 convolutions with unit stride and no padding on NCHW images of four positions (2x2): a lane's 8 columns
// are two whole images, loaded and stored as two runs of 4.  64 images, 512 -> 512 channels, V = 32, 75 %:
// 7.3 us staged, 3.7 gathered (what is left is one launch and the chain index -> X -> result).
struct GeomQuads : GeomLinearBuf {
    unsigned x_image;        // bytes between images
    long y_image;            // elements between images
    unsigned ln2b;           // offset of the lane's second image
    static constexpr bool CHOICE = false;

    __device__ __forceinline__ void init(long n)
    {
        xd = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(X), 0, (int)xbytes, GATHER_BUFFER_FLAGS);
        ldx2 = 8;
        ln2 = n < N ? (unsigned)((unsigned long)n >> 2) * x_image : PAST_END;
        ln2b = n + 4 < N ? (unsigned)((unsigned long)n >> 2) * x_image + x_image : PAST_END;
    }
    __device__ __forceinline__ run_t load8(entry_t e, int&) const
    {
        const auto lo = __builtin_amdgcn_raw_buffer_load_b64(xd, (int)__builtin_elementwise_min(__builtin_elementwise_add_sat(e, ln2), PAST_END), 0, 0);
        const auto hi = __builtin_amdgcn_raw_buffer_load_b64(xd, (int)__builtin_elementwise_min(__builtin_elementwise_add_sat(e, ln2b), PAST_END), 0, 0);
        return run_t{lo[0], lo[1], hi[0], hi[1]};
    }
    template <bool STREAM, int CNT, typename OutT>
    __device__ __forceinline__ void store(int row, long n, const OutT* vals) const
    {
#pragma unroll
        for (int h = 0; h < CNT; h += 4)
            if (n + h < N)
                store_run<STREAM, 4>(static_cast<OutT*>(Y) + (long)((unsigned long)(n + h) >> 2) * y_image + (long)row * 4, vals + h);
    }
};

// Rows of fewer than 8 columns (one token, a few tokens).  The one lane of eight that has columns
// loads 16 bytes from the row's start, whatever follows the row (columns beyond N are neither stored
// nor mixed with others); where that would reach past the end of X it loads the last 16 bytes and
// moves the values down (finish8).  X must hold 8 values or more.  4096 x 4096 by 4096 x 1 (V = 32, 75 %): 38.3 us with element-wise loads, 6.3 us.
struct GeomNarrow : GeomLinearBuf {
    static constexpr bool FINISH = true, CHOICE = false;
    __device__ __forceinline__ run_t load8(entry_t e, int& shift) const
    {
        const unsigned off = __builtin_elementwise_add_sat(e, ln2), lim = xbytes - 16u;
        const unsigned at = off < lim ? off : lim;
        shift = (int)(off - at) >> 1;
        return load_run(xd, e == PAST_END || ln2 == PAST_END ? PAST_END : at);
    }
    // values shift .. 7 of v moved to 0 (shift 0 .. 7; only columns that exist are looked at afterwards)
    static __device__ __forceinline__ run_t finish8(run_t x, int shift)
    {
        if (shift & 4) { x[0] = x[2]; x[1] = x[3]; }
        if (shift & 2) {
#pragma unroll
            for (int i = 0; i + 1 < 4; ++i) x[i] = x[i + 1];
        }
        const unsigned bits = (shift & 1) * 16;
#pragma unroll
        for (int i = 0; i + 1 < 4; ++i) x[i] = __builtin_amdgcn_alignbit(x[i + 1], x[i], bits);
        x[3] >>= bits;
        return x;
    }
    template <bool STREAM, int CNT, typename OutT>
    __device__ __forceinline__ void store(int row, long n, const OutT* vals) const
    {
        OutT* p = static_cast<OutT*>(Y) + (long)row * ldy + n;
#pragma unroll
        for (int e = 0; e < CNT; ++e)
            if (n + e < N) p[e] = vals[e];
    }
};

// Convolution whose gathered values come in runs of 8 along the tensor's innermost dimension
// (Section 4.1's implicit GEMM, unfolded on the way into the registers): images for CHWN (any stride,
// 8 or more images), output columns of one row for NCHW (unit stride along x, 8 or more output
// columns, padding of at most one column).  As in GeomRows the innermost dimension is cut into slots
// of 8 of which the last may overlap the one before, so that every load is 16 bytes of one row of
// the input and every store 16 bytes of one row of the output.
//
// A row of the unfolded matrix, k = (c*R + r)*S + s, is an input row iy0 + r, shifted by s: outside
// the image it reads as zeros (the descriptor's range check, as for padded slots).  Along x a run
// may begin one column before the image or end one after it; it is then loaded one column over and
// moved back in registers, with a zero in the column that does not exist (finish8).
//
// Each gathered byte serves the V rows of one group, so the L2 moves N * kept * 2 bytes per group;
// staging a box of the input once (conv_kernel.hip) moves less but feeds the matrix cores with
// 2-byte LDS reads.
template <bool CHWN>
struct GeomConvRuns : GeomLinearBuf {
    unsigned m_RS, m_S;       // ceil(2^32 / (R*S)) and ceil(2^16 / S): exact quotients (the host checks the ranges)
    int RS, S, H, W, B, Ho, Wo, sh, sw, ph, pw;
    int slots;                // ceil(innermost output dimension / 8)
    unsigned cst, rst, sst;   // input bytes between channels, rows, columns (below 2^24)
    unsigned ist;             // input bytes between images (NCHW)
    long osM, osB;            // output elements between channels, and between images (NCHW)
    int iy0, ix0;             // this lane's window origin
    static constexpr bool FINISH = !CHWN, CONV = true;
    static constexpr unsigned NO_ROW = 0x7fff0000u;   // padded images have fewer than 32768 rows

    // slot of virtual column n: image (the first of 8 for CHWN), output row and column (the first of 8 for NCHW)
    __device__ __forceinline__ void place(long n, int& b, int& y, int& x) const
    {
        const unsigned slot = (unsigned)((unsigned long)n >> 3);
        const unsigned q = slot / (unsigned)slots;
        const int i = (int)(slot - q * (unsigned)slots) * 8;
        if (CHWN) {
            b = i < B - 8 ? i : B - 8;
            y = (int)(q / (unsigned)Wo);
            x = (int)q - y * Wo;
        } else {
            x = i < Wo - 8 ? i : Wo - 8;
            b = (int)(q / (unsigned)Ho);
            y = (int)q - b * Ho;
        }
    }
    __device__ __forceinline__ void init(long n)
    {
        xd = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(X), 0, (int)xbytes, GATHER_BUFFER_FLAGS);
        ln2 = 0;
        iy0 = 0x10000;   // a lane beyond N reads rows below every image
        ix0 = 0;
        if (n < N) {
            int b, y, x;
            place(n, b, y, x);
            iy0 = y * sh - ph;
            ix0 = x * sw - pw;
            ln2 = (unsigned)iy0 * rst + (CHWN ? (unsigned)ix0 * sst + (unsigned)b * 2u : (unsigned)b * ist);
        }
    }
    // Row k of the unfolded matrix as the kernel's list holds it: byte offset of (channel, kernel row,
    // kernel column for CHWN) and the kernel position, row in the high half.  A row that does not
    // exist gets a kernel row below every image.
    typedef unsigned entry_t __attribute__((ext_vector_type(2)));
    __device__ __forceinline__ entry_t entry(int col, bool exists) const
    {
        const unsigned k = (unsigned)col;
        const unsigned c = RS == 1 ? k : __umulhi(k, m_RS);
        const unsigned rs = k - __umul24(c, (unsigned)RS);
        const unsigned r = __umul24(rs, m_S) >> 16, s = rs - __umul24(r, (unsigned)S);
        unsigned off = __umul24(c, cst) + __umul24(r, rst);
        if (CHWN) off += __umul24(s, sst);
        return entry_t{off, exists && col >= 0 ? (r << 16) | s : NO_ROW};
    }
    // shift: by how many columns the run lies right of the one asked for (-1, 0 or 1; NCHW only)
    __device__ __forceinline__ run_t load8(entry_t e, int& shift) const
    {
        const int iy = iy0 + (int)(e[1] >> 16);
        const int ix = ix0 + (int)(e[1] & 0xffffu);
        bool ok = (unsigned)iy < (unsigned)H;
        unsigned off = e[0] + ln2;
        if (CHWN) {
            ok = ok && (unsigned)ix < (unsigned)W;
        } else {
            int ic = ix < 0 ? 0 : ix;
            ic = ic < W - 8 ? ic : W - 8;
            shift = ic - ix;
            off += (unsigned)ic * 2u;
        }
        return load_run(xd, ok ? off : PAST_END);
    }
    // the run that was asked for, from the one loaded `shift` columns over
    static __device__ __forceinline__ run_t finish8(run_t x, int shift)
    {
        const unsigned up = shift > 0 ? 0x05040302u : 0x07060504u, down = shift < 0 ? 0x05040302u : 0x03020100u;
        run_t y, z;
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = __builtin_amdgcn_perm(x[i], i ? x[i - 1] : 0u, up);
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = __builtin_amdgcn_perm(i + 1 < 4 ? y[i + 1] : 0u, y[i], down);
        return z;
    }
    template <bool STREAM, int CNT, typename OutT>
    __device__ __forceinline__ void store(int row, long n, const OutT* vals) const
    {
        if (n < N) {
            int b, y, x;
            place(n, b, y, x);
            const long pos = CHWN ? ((long)y * Wo + x) * B + b : (long)b * osB + (long)y * Wo + x;
            store_run<STREAM, CNT>(static_cast<OutT*>(Y) + (long)row * osM + pos + (n & 7), vals);
        }
    }
    __device__ __forceinline__ unsigned out_col(long n) const
    {
        int b, y, x;
        place(n, b, y, x);
        return (unsigned)(CHWN ? ((long)y * Wo + x) * B + b : (long)b * osB + (long)y * Wo + x) + ((unsigned)n & 7u);
    }
    long out_pitch() const { return osM; }
};

// The same for NCHW with a stride of two along x (images of 16 columns or more): the 8 values lie in 16 neighbouring ones, two
// loads, of which every other one is kept.  The 16 may begin one column before the image, or end up to two after it.
struct runs2_t { run_t a, b; };
struct GeomConvRuns2 : GeomConvRuns<false> {
    typedef runs2_t loaded_t;
    __device__ __forceinline__ runs2_t load8(entry_t e, int& shift) const
    {
        const int iy = iy0 + (int)(e[1] >> 16);
        const int ix = ix0 + (int)(e[1] & 0xffffu);
        int ic = ix < 0 ? 0 : ix;
        ic = ic < W - 16 ? ic : W - 16;
        shift = ic - ix;
        const unsigned off = (unsigned)iy < (unsigned)H ? e[0] + ln2 + (unsigned)ic * 2u : PAST_END - 16u;
        return runs2_t{load_run(xd, off), load_run(xd, off + 16u)};
    }
    // values 0, 2 .. 14 of those asked for, from the 16 loaded `shift` columns over (-2 .. 1)
    static __device__ __forceinline__ run_t finish8(const runs2_t& x, int shift)
    {
        const unsigned d[10] = {0, x.a[0], x.a[1], x.a[2], x.a[3], x.b[0], x.b[1], x.b[2], x.b[3], 0};
        const unsigned half = shift & 1 ? 0x07060302u : 0x05040100u;
        unsigned u[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            u[j] = shift > 0 ? d[j] : d[j + 1];
            u[j] = shift < -1 ? d[j + 2] : u[j];
        }
        return run_t{__builtin_amdgcn_perm(u[1], u[0], half), __builtin_amdgcn_perm(u[3], u[2], half),
                     __builtin_amdgcn_perm(u[5], u[4], half), __builtin_amdgcn_perm(u[7], u[6], half)};
    }
};

// Convolution as implicit GEMM (Section 4.1): k = (c*R + r)*S + s, and
// n = (b*Ho + y)*Wo + x for NCHW or n = (y*Wo + x)*B + b for CHWN.  This is
// the general element-wise form; the unfolded matrix never exists in memory.
struct GeomConv {
    const _Float16* in;
    void* out;
    int B, Cin, H, W, Cout, R, S, sh, sw, ph, pw, Ho, Wo;
    int chwn;
    long N;
    // per-lane decode of the 8 output positions this lane gathers for:
    // base[e] = offset of the window origin (may be negative), yx[e] = packed
    // (iy0, ix0) window origin; valid bit e of `live` = position exists
    int base[8];
    int yx[8];
    int live;
    static constexpr bool FINISH = false, CONV = false, CHOICE = false;
    typedef int entry_t;
    typedef run_t loaded_t;
    __device__ __forceinline__ entry_t entry(int col, bool exists) const { return exists ? col : -1; }

    __device__ __forceinline__ void split_n(long n, int& b, int& y, int& x) const
    {
        int q;
        if (chwn) {
            b = (int)(n % B);
            q = (int)(n / B);
        } else {
            q = (int)(n % ((long)Ho * Wo));
            b = (int)(n / ((long)Ho * Wo));
        }
        y = q / Wo;
        x = q % Wo;
    }

    __device__ __forceinline__ void init(long n)
    {
        live = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            base[e] = 0;
            yx[e] = 0;
            if (n + e >= N) continue;
            int b, y, x;
            split_n(n + e, b, y, x);
            const int iy0 = y * sh - ph, ix0 = x * sw - pw;
            yx[e] = (iy0 << 16) | (ix0 & 0xffff);
            base[e] = chwn ? (iy0 * W + ix0) * B + b : (b * Cin * H + iy0) * W + ix0;
            live |= 1 << e;
        }
    }

    __device__ __forceinline__ run_t load8(entry_t col, int&) const
    {
        half8 v = {};
        if (col < 0) return __builtin_bit_cast(run_t, v);
        const int c = col / (R * S);
        const int rs = col - c * (R * S);
        const int r = rs / S, s = rs - r * S;
        const int koff = ((c * H + r) * W + s) * (chwn ? B : 1);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int iy = (yx[e] >> 16) + r, ix = (int)(short)(yx[e] & 0xffff) + s;
            const bool ok = ((live >> e) & 1) && iy >= 0 && iy < H && ix >= 0 && ix < W;
            if (ok) v[e] = in[(long)base[e] + koff];
        }
        return __builtin_bit_cast(run_t, v);
    }

    template <bool STREAM, int CNT, typename OutT>
    __device__ __forceinline__ void store(int row, long n, const OutT* vals) const
    {
        OutT* o = static_cast<OutT*>(out);
#pragma unroll
        for (int e = 0; e < CNT; ++e) {
            if (n + e >= N) break;
            int b, y, x;
            split_n(n + e, b, y, x);
            const long idx = chwn ? (((long)row * Ho + y) * Wo + x) * B + b
                                  : (((long)b * Cout + row) * Ho + y) * Wo + x;
            o[idx] = vals[e];
        }
    }
};

// ---------------------------------------------------------------- kernel
template <int V, int WN>
struct GatherShape {
    static constexpr bool SMALL = (V == 16);          // 16x16x32 instruction
    static constexpr int TK = SMALL ? 32 : 16;        // columns per k-step
    static constexpr int RB = SMALL ? 1 : V / 32;     // row blocks per group
    static constexpr int TILE_N = SMALL ? 16 : 32;    // output columns per instruction
    static constexpr int NT = WN / TILE_N;
    static constexpr int LPR = WN / 8;                // lanes per activation row, 8 columns (16 B) each
    static constexpr int NLD = TK * LPR / 64;         // activation rows, and loads, of a lane per k-step
    static constexpr int ROWS_E = SMALL ? 16 : 32;    // rows per epilogue pass
    static constexpr int EPI = ROWS_E * (WN + 8);     // binary16 needed by one epilogue pass
};

// Which workgroup takes which block of column tiles and which group.  Workgroups are dealt to the eight
// XCDs in turn.  per_xcd = 0: blockIdx.x is the block of tiles, blockIdx.y the group.  Otherwise the grid is
// 8 x per_xcd and XCD x takes items x*per_xcd .. of the list that runs over all groups of one
// block of tiles before the next.
struct GatherOrder {
    int per_xcd, total;          // items of an XCD, and of the launch (tile blocks x groups, below 2^19)
    unsigned long long m_G;      // ceil(2^40 / G)
    int uniform_steps;           // k-steps of every group when they all have the same number, else -1
};

// f with std::true_type or std::false_type: streaming stores or not.  One choice for all the stores of a
// pass: taken at every store, it keeps the reads of the finished tile from running ahead of the stores (1x1 on
// 28x28 images, 64 -> 256 channels, V = 64 7.05 -> 6.78 us; 1024 x 1024 by 5632 at 90 %, V = 64 5.70 -> 5.47).
template <class Geom, class F>
__device__ __forceinline__ void with_stores(const Geom& geom, F&& f)
{
    if constexpr (Geom::CHOICE) {
        if (geom.stream) {
            asm volatile("");   // kept apart: merged with the other branch, the stores lose their hint
            f(std::true_type{});
            asm volatile("");
            return;
        }
    }
    f(std::false_type{});
}

// k-steps whose weights the wavefronts of a workgroup bring into the LDS at a time
template <int V, int WAVES>
constexpr int gather_chunk() { return V == 128 || (V == 64 && WAVES == 4) ? 4 : 8; }

// k-steps whose rows (and weights, unless shared) are on their way while a step multiplies (four gained nothing)
constexpr int GATHER_AHEAD = 2;

// k-steps of one pass through the loop where the weights are not shared.  Whole tiles of 128 columns, V = 32: two, which
// leaves three wavefronts per SIMD (136 to 159 registers; four steps took 202 to 223 of them, two wavefronts).  us by four /
// two steps, 3x3, V = 32: 64 images of 56x56, 64 -> 256 channels at 50 %, NCHW 124 / 112, CHWN 75.0 / 65.7; 64 of 28x28,
// 128 -> 512 at 50 %, CHWN 63.9 / 58.2; linear layers: 6272 x 65 by 2880 10.3 / 9.5, 2816 x 3200 by 12121 at 95 % 87.9 / 85.0.
// Shared steps run on one or two workgroups per CU either way: 608 x 240 by 14241 unpruned 19.2 / 20.0, 704 x 1568 by 2021
// at 85 % 8.1 / 7.7.
template <int V, int WN, int SHARES>
constexpr int gather_batch() { return V == 32 && WN == 128 && SHARES > 1 ? 4 : 2; }

// Wavefronts a SIMD must be able to hold (SPLIT: SHARES of the kernel).  Left alone, the compiler counts on one workgroup per CU: with four
// wavefronts or fewer in it, a SIMD to each, it keeps the accumulators in registers of their own (V = 128: 328
// registers, one wavefront per SIMD).  Two are asked for, and four (128 registers) for V = 64, which takes
// up to 132 otherwise, two workgroups of eight becoming one (not for the split by 8, of which there is no more
// than one workgroup per CU).  Us before -> after, splits by 2 and 4: 3x3, 56x56, 12 images, CHWN, 64 -> 128
// channels, dense, V = 128: 24.9 -> 15.7; 3x3 / 2, 56x56, CHWN, 128 channels, V = 128 at 50 %: 17.4 -> 11.6;
// 3x3, 56x56, 64 channels, V = 64 at 75 %: 12.8 -> 11.5; aligned products -1 to +2 %.
template <int V, int WN, class Geom, int SPLIT>
constexpr int gather_min_waves()
{
    return V == 64 && WN == 64 && SPLIT > 0 && SPLIT < 8 && !std::is_same<Geom, GeomConv>::value && !std::is_same<Geom, GeomConvRuns2>::value ? 4 : 2;
}

// SHARES = 1: the wavefronts of a workgroup own different column tiles of one group.
// SHARES = 0: the same, and they take the weights, which are the same for all, from the LDS, where each brings a part
// of them a chunk of k-steps ahead, with a barrier per chunk.
// SHARES > 1 (SPLIT; too few tiles to fill the chip): SHARES neighbouring wavefronts share one tile, each
// takes a contiguous share of the group's k-steps; the partial accumulators of a row block meet in
// the LDS, every wavefront of the tile adds up its share of them and stores its share of the rows.
template <int V, int WN, int WAVES, typename OutT, class Geom, bool BF, int SHARES>
__global__ __launch_bounds__(64 * WAVES, (gather_min_waves<V, WN, Geom, SHARES>()))
void shflbw_gather_kernel(PackedView A, Geom geom, int n_tiles, GatherOrder order)
{
    using S = GatherShape<V, WN>;
    constexpr int TK = S::TK, RB = S::RB, NT = S::NT, LPR = S::LPR, NLD = S::NLD, PD = GATHER_AHEAD;
    constexpr bool SHARE = SHARES == 0;
    constexpr int SPLIT = SHARE ? 1 : SHARES;
    constexpr int TILES = WAVES / SPLIT;                             // column tiles of a workgroup
    static_assert(TILES * SPLIT == WAVES, "whole tiles per workgroup");
    constexpr int QUADS = S::SMALL ? NT : NT * 4;                    // groups of 4 accumulators per lane and row block
    constexpr int EPS = WN + 16 / (int)sizeof(OutT);                 // row pitch of a finished tile (SPLIT > 1), in OutT units
    constexpr int RED_BYTES = WAVES * QUADS * 1024;
    constexpr int FIN_BYTES = TILES * S::ROWS_E * EPS * (int)sizeof(OutT);
    // the finished tile lies apart from the partial sums (over the lists, which are read by then), which saves two
    // barriers per row block, but where that would cost residency
    constexpr bool APART = sizeof(OutT) == 2 || SPLIT == 8;
    static_assert(SPLIT == 1 || APART || FIN_BYTES <= RED_BYTES, "the finished tile lies where the partial sums were");
    constexpr int TILE_BYTES = SPLIT == 1 ? WAVES * S::EPI * 2 : RED_BYTES;
    typedef typename Geom::entry_t entry_t;
    constexpr int LISTS = (int)sizeof(entry_t) * WAVES * 2 * 64;        // two batches of 64 entries per wavefront
    constexpr int LIST_BYTES = SPLIT > 1 && APART && FIN_BYTES > LISTS ? FIN_BYTES : LISTS;
    constexpr int CHUNK = gather_chunk<V, WAVES>();                         // SHARE: k-steps of a chunk of weights
    constexpr int CHUNK_BYTES = CHUNK * RB * 1024;
    constexpr int WPW = SHARE ? CHUNK * RB / WAVES : 1;              // kilobytes of it that a wavefront brings
    static_assert(!SHARE || WPW * WAVES == CHUNK * RB, "whole kilobytes per wavefront");
    __shared__ __attribute__((aligned(16))) char smem[TILE_BYTES + LIST_BYTES + (SHARE ? 2 * CHUNK_BYTES : 0)];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ti = wave / SPLIT, part = wave % SPLIT;
    int tblock = blockIdx.x, g = blockIdx.y;
    if (order.per_xcd) {
        const unsigned w = blockIdx.x * (unsigned)order.per_xcd + blockIdx.y;
        if (w >= (unsigned)order.total) return;   // uniform for the whole workgroup
        tblock = (int)(((unsigned long long)w * order.m_G) >> 40);
        g = (int)w - tblock * A.G;
    }
    const int tile = tblock * TILES + ti;
    // without SPLIT or SHARE a whole wavefront leaves and no workgroup barrier is used; with them one whose
    // tile does not exist stays for the barriers, with nothing to store
    if (SPLIT == 1 && !SHARE && tile >= n_tiles) return;
    const long n0 = (long)tile * WN;

    // without a memory access when every group has the same number of steps: the column indices can be
    // requested at once instead of after a dependent load (convolutions, which compute their list
    // first, lose 1 to 2 % by it: 3x3, 14x14x256 12.1 -> 12.3 us)
    const int uniform = Geom::CONV ? -1 : order.uniform_steps;
    int sbeg = uniform >= 0 ? g * uniform : A.step_ptr[g];
    int nsteps = uniform >= 0 ? uniform : A.step_ptr[g + 1] - sbeg;
    if (SPLIT > 1) {
        const int first = (int)((long)nsteps * part / SPLIT);
        const int end = (int)((long)nsteps * (part + 1) / SPLIT);
        sbeg += first;
        nsteps = tile < n_tiles ? end - first : 0;
    }

    // this lane's share of a step: rows lrow .. lrow+NLD-1, 8 columns
    const int lrow = lane / LPR * NLD;
    geom.init(n0 + lane % LPR * 8);

    floatx16 acc32[S::SMALL ? 1 : RB][S::SMALL ? 1 : NT];
    floatx4 acc16[S::SMALL ? NT : 1];
    if (S::SMALL) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc16[t] = floatx4{0, 0, 0, 0};
    } else {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc32[rb][t][r] = 0.f;
    }

    // Original rows for the write-back.  Those of the first EARLY row blocks are requested now, so that the
    // stores do not wait for them (with the step bounds that need no load: 1024 x 1024 by 4096 8.0 -> 7.4 us,
    // 4096 x 4096 by 64 6.35 -> 5.95), those of the second one of two after the last step.  Where registers
    // allow it: four row blocks have none to spare, nor have geometries that keep more than an offset per lane
    // (unaligned rows and convolutions lose 1 to 3 %).  Two row blocks early, V = 64 with 16-bit results, are
    // a wavefront less per SIMD, which costs more than the wait: 8192 x 2048 by 4096 at 90 % 31.6 us without,
    // 34.2 with both, 29.7 with one; 4096 x 1024 by 8192 20.7 / 21.5 / 18.0; 1024 x 1024 by 8192 9.1 / 8.5 / 8.4.
    // Two row blocks of 128 columns with 32-bit results take each row when it is stored: with the rows at hand the
    // streaming stores come faster than they drain (8192 x 8192 by 4096 at 95 % 58.3 us, 61.7 with the rows at hand,
    // 4096 x 4096 by 4096 at 90 % 29.1 and 30.9; but 8192 x 4096 by 8200, rows of no whole 64-byte blocks, 160 and 149).
    // V = 64 in 64 columns has registers for them in the loop only where the weights are shared (1024 x 4096 by 8192 at
    // 85 %, 32-bit results, 23.3 us without, 19.1 with them).  Wavefronts that share steps request theirs after the last
    // step, before the partial sums meet, whatever the geometry: at the stores, a row block after the other waited for them
    // (3968 x 7584 by 8, V = 128 13.4 -> 11.9 us, 576 x 632 by 64 and the like 4.5 -> 3.9).
    constexpr bool ROWS_AHEAD = RB <= 2 && std::is_same<Geom, GeomLinearBuf>::value && !(RB == 2 && WN == 128 && sizeof(OutT) == 4);
    constexpr int EARLY = !ROWS_AHEAD || (V == 64 && WN == 64 && !SHARE) ? 0 : RB == 2 && SPLIT == 1 && sizeof(OutT) == 2 ? 1 : RB;
    constexpr int OPV = 16 / (int)sizeof(OutT);                      // values per 16 bytes
    // a store instruction of 16 bytes per lane: lanes per row and rows, without and with SPLIT
    constexpr int LPR_S = SPLIT > 1 ? WN / OPV : WN / ((int)sizeof(OutT) / 2) / OPV, RPI_S = 64 / LPR_S;
    constexpr int STORES_S = SPLIT > 1 ? (S::ROWS_E / RPI_S + SPLIT - 1) / SPLIT : S::ROWS_E / RPI_S;
    constexpr bool ROWS_HELD = ROWS_AHEAD || SPLIT > 1;   // few per wavefront then, and requested before the partial sums meet
    int out_row[ROWS_HELD ? RB : 1][STORES_S];
    const int32_t* rows_g = A.row_indices + (long)g * V;
    auto row_of = [&](int i) __attribute__((always_inline)) {         // stored row of this lane in its i-th store of a row block
        return SPLIT > 1 ? (part + i * SPLIT) * RPI_S + lane / LPR_S : i * RPI_S + lane / LPR_S;
    };
    auto request_rows = [&](int rb) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < STORES_S; ++i) {
            const int r = row_of(i);
            out_row[rb][i] = rows_g[rb * 32 + (r < S::ROWS_E ? r : 0)];
        }
    };
    if constexpr (ROWS_AHEAD) {
#pragma unroll
        for (int rb = 0; rb < EARLY; ++rb) request_rows(rb);
    }

    // Column indices and weights of the wavefront's steps through buffer descriptors.  A buffer load checks
    // lane offset + immediate against the descriptor's size (not the scalar offset): the step goes into the
    // lane offset, so that a step beyond the wavefront's range reads zeros instead of memory past it.
    const __amdgpu_buffer_rsrc_t col_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t*>(A.col_idx + (long)sbeg * TK), 0, nsteps * TK * 4, GATHER_BUFFER_FLAGS);
    const __amdgpu_buffer_rsrc_t val_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<half8*>(A.values + (long)sbeg * RB * 64), 0, nsteps * RB * 1024, GATHER_BUFFER_FLAGS);

    // The rows a wavefront gathers are worked out 64 at a time (one per lane, U k-steps) and kept
    // in a private list in the LDS, two batches of it, so that the divisions by a convolution's kernel size are
    // paid once per 64 rows and not by every lane for each of its loads (32 images of 14x14,
    // 256 channels, 3x3, V = 32, 75 %: 12.6 -> 11.8 us), and an address is one addition.
    constexpr int U = 64 / TK;
    constexpr int AHEAD = (U + PD) / U;   // batches: the last step of a batch reads entries of the batch AHEAD further on
    static_assert(AHEAD <= 2, "the list holds two batches");
    entry_t* list = reinterpret_cast<entry_t*>(smem + TILE_BYTES) + wave * 128;
    auto fetch = [&](int q) __attribute__((always_inline)) {
        return (int)__builtin_amdgcn_raw_buffer_load_b32(col_rsrc, lane * 4 + q * 256, 0, 0);
    };
    auto work_out = [&](int q, int col) __attribute__((always_inline)) {
        list[(q & 1) * 64 + lane] = geom.entry(col, q * 64 + lane < nsteps * TK);
    };
    entry_t ent[NLD];
    auto look_up = [&](int step) __attribute__((always_inline)) {
        const entry_t* e = list + (step * TK & 127) + lrow;
#pragma unroll
        for (int i = 0; i < NLD; ++i) ent[i] = e[i];
    };
    typename Geom::loaded_t xr[PD][NLD];
    int xf[PD];   // what geom.finish8 needs to know of the loads, -8 .. 7 each
    auto request = [&](typename Geom::loaded_t (&x)[NLD], int& f) __attribute__((always_inline)) {
        f = 0;
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            int shift = 0;
            x[i] = geom.load8(ent[i], shift);
            if constexpr (Geom::FINISH) f |= (shift & 15) << (4 * i);
        }
    };

    // StitchTile in registers.  A lane has 8 columns of NLD neighbouring rows of the step; an operand wants 8 rows of one
    // column.  Rows are paired column by column (halves of two registers), and lanes that hold the other rows of
    // the operand trade columns with this one until each has all 8 rows of the columns it keeps: lanes 16 apart
    // in one instruction per pair of registers, lanes 8 apart (64-column tiles) through the lane shifter.  Operand
    // t of a lane is column
    //   128 columns, V >= 32: 8*(l % 16) + 2t + l/16 % 2             64: 8*(l % 8) + 4t + 2*(l/8 % 2) + l/16 % 2
    //   128 columns, V = 16:  8*(l % 16) + t                         64: 8*(l % 8) + 4*(l/8 % 2) + t
    // 6 vector instructions per operand (128 columns; V = 16: 4; 12 and 10 in 64 columns).
    constexpr int PAIRS = NLD / 2 * 8;
    // rows 2i, 2i+1 of column c at 8*i + c.  The rows' registers are free for the next request then.
    auto pairs = [&](const run_t (&x)[NLD], unsigned (&p)[PAIRS]) __attribute__((always_inline)) {
        constexpr unsigned LOW = 0x05040100u, HIGH = 0x07060302u;
#pragma unroll
        for (int i = 0; i < NLD / 2; ++i)
#pragma unroll
            for (int c = 0; c < 8; ++c) p[8 * i + c] = __builtin_amdgcn_perm(x[2 * i + 1][c / 2], x[2 * i][c / 2], c % 2 ? HIGH : LOW);
    };
    auto operands = [&](const unsigned (&p)[PAIRS], half8 (&o)[NT]) __attribute__((always_inline)) {
        // a: the own column's rows from the lane with the bit clear, b: from the one with it set
        auto trade16 = [&](unsigned& a, unsigned& b) __attribute__((always_inline)) {
            const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
            a = r[0];
            b = r[1];
        };
        auto trade8 = [&](unsigned& a, unsigned& b) __attribute__((always_inline)) {
            constexpr int ROR8 = 0x128;                                          // lane ^ 8
            const unsigned a0 = a;
            a = (unsigned)__builtin_amdgcn_update_dpp((int)a0, (int)b, ROR8, 0xf, 0xc, false);
            b = (unsigned)__builtin_amdgcn_update_dpp((int)b, (int)a0, ROR8, 0xf, 0x3, false);
        };
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            run_t v;
            if constexpr (S::SMALL && WN == 128) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = p[8 * i + t];
            } else if constexpr (S::SMALL) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    unsigned a = p[8 * i + t], b = p[8 * i + t + 4];
                    trade8(a, b);
                    v[i] = a;
                    v[2 + i] = b;
                }
            } else if constexpr (WN == 128) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    unsigned a = p[8 * i + 2 * t], b = p[8 * i + 2 * t + 1];
                    trade16(a, b);
                    v[i] = a;
                    v[2 + i] = b;
                }
            } else {
                unsigned a = p[4 * t], b = p[4 * t + 1], c = p[4 * t + 2], d = p[4 * t + 3];
                trade16(a, b);
                trade16(c, d);
                trade8(a, c);
                trade8(b, d);
                v = run_t{a, c, b, d};
            }
            o[t] = __builtin_bit_cast(half8, v);
        }
    };
    auto products = [&](const half8 (&x)[NT], const half8 (&w)[RB]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (S::SMALL) {
                acc16[t] = mma16<BF>(x[t], w[0], acc16[t]);
            } else {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) acc32[rb][t] = mma32<BF>(x[t], w[rb], acc32[rb][t]);
            }
        }
    };

    // weights: SHARE by way of the LDS, otherwise a wavefront loads them for itself PD steps ahead (one where
    // the registers of its share of a SIMD leave no room for more: with 64-bit addresses, V = 64, two steps spilled 2
    // registers of 128 in 64 columns and 11 of 256 in a convolution's 128)
    constexpr int WA = V == 64 && ((WN == 64 && Geom::FINISH) || !std::is_base_of<GeomLinearBuf, Geom>::value) ? 1 : PD;
    char* ring = smem + TILE_BYTES + LIST_BYTES;
    half8 ws[WPW], wr[SHARE ? 2 : WA][RB];
    auto bring = [&](int k) __attribute__((always_inline)) {          // a chunk from memory
#pragma unroll
        for (int j = 0; j < WPW; ++j)
            ws[j] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(
                val_rsrc, lane * 16 + (wave * WPW + j) * 1024 + k * CHUNK_BYTES, 0, 0));
    };
    auto deposit = [&](int k) __attribute__((always_inline)) {        // to the LDS
#pragma unroll
        for (int j = 0; j < WPW; ++j)
            *reinterpret_cast<half8*>(ring + (k & 1) * CHUNK_BYTES + (wave * WPW + j) * 1024 + lane * 16) = ws[j];
    };
    auto weights = [&](int k, int v, half8 (&w)[RB]) __attribute__((always_inline)) {   // of the v-th step of chunk k
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            w[rb] = *reinterpret_cast<const half8*>(ring + (k & 1) * CHUNK_BYTES + (v * RB + rb) * 1024 + lane * 16);
    };
    auto load_w = [&](int step, half8 (&w)[RB]) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            w[rb] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(val_rsrc, lane * 16 + (step * RB + rb) * 1024, 0, 0));
    };

    // The rows of the first PD steps do not wait for the list where an entry is one multiplication.
    int first[PD][NLD];
    if constexpr (!Geom::CONV) {
#pragma unroll
        for (int u = 0; u < PD; ++u) {
            const int at = (u * TK + lrow) * 4;
            if constexpr (NLD == 2) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(col_rsrc, at, 0, 0);
                first[u][0] = (int)v[0]; first[u][1] = (int)v[1];
            } else {
#pragma unroll
                for (int i = 0; i < NLD; i += 4) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(col_rsrc, at + 4 * i, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) first[u][i + e] = (int)v[e];
                }
            }
        }
    }
    int c[AHEAD];
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) c[q] = fetch(q);
    if constexpr (SHARE) bring(0);
    else {
#pragma unroll
        for (int u = 0; u < WA; ++u) load_w(u, wr[u]);
    }
    int cn = fetch(AHEAD);
    __builtin_amdgcn_sched_barrier(0);   // what the loop waits for first is requested first: its wait counts assume so
    if constexpr (!Geom::CONV) {
#pragma unroll
        for (int u = 0; u < PD; ++u) {
#pragma unroll
            for (int i = 0; i < NLD; ++i) ent[i] = geom.entry(first[u][i], u < nsteps);
            request(xr[u], xf[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) work_out(q, c[q]);
    SHFLBW_WAVE_LDS_SYNC();
    if constexpr (Geom::CONV) {
#pragma unroll
        for (int u = 0; u < PD; ++u) {
            look_up(u);
            request(xr[u], xf[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    SHFLBW_WAVE_LDS_SYNC();
    look_up(PD);
    if constexpr (SHARE) {
        deposit(0);
        bring(1);
        __syncthreads();
        weights(0, 0, wr[0]);
    }
    __builtin_amdgcn_sched_barrier(0);

    // Steps come in batches of ST that run without a test between their steps, which keeps the register sets static
    // and the wait counts exact.
    constexpr int ST = SHARE ? CHUNK : gather_batch<V, WN, SHARES>();
    static_assert(ST % PD == 0 && (!SHARE || (ST % U == 0 && ST % 2 == 0)), "register sets are static");
    // step s, the v-th of its batch
    auto one = [&](int s, int v) __attribute__((always_inline)) {
        if (U <= ST ? v % U == 0 : v == 0 && s % U == 0) {   // uniform
            work_out(s / U + AHEAD, cn);
            cn = fetch(s / U + AHEAD + 1);
            SHFLBW_WAVE_LDS_SYNC();
        }
        if constexpr (SHARE) {
            if (v == CHUNK - 2) { deposit(s / CHUNK + 1); bring(s / CHUNK + 2); }
        }
        __builtin_amdgcn_sched_barrier(0);   // steps stay in program order
        unsigned p[PAIRS];
        half8 o[NT];
        if constexpr (Geom::FINISH) {
            run_t x[NLD];
#pragma unroll
            for (int i = 0; i < NLD; ++i) x[i] = Geom::finish8(xr[v % PD][i], xf[v % PD] << (28 - 4 * i) >> 28);
            pairs(x, p);
        } else {
            pairs(xr[v % PD], p);
        }
        if constexpr (!SHARE && WA < PD) {
            operands(p, o);
            products(o, wr[0]);
            load_w(s + 1, wr[0]);   // before the rows that are waited for later
            request(xr[v % PD], xf[v % PD]);
            look_up(s + PD + 1);
        } else {
            request(xr[v % PD], xf[v % PD]);
            look_up(s + PD + 1);
            __builtin_amdgcn_sched_barrier(0);
            operands(p, o);
        }
        if constexpr (SHARE) {
            if (v != CHUNK - 1) weights(s / CHUNK, v + 1, wr[(v + 1) % 2]);
            products(o, wr[v % 2]);
            if (v == CHUNK - 1) {
                __syncthreads();
                weights(s / CHUNK + 1, 0, wr[0]);
            }
        } else if constexpr (WA == PD) {
            products(o, wr[v % PD]);
            load_w(s + PD, wr[v % PD]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = 0;
    for (; s + ST <= nsteps; s += ST) {
#pragma unroll
        for (int v = 0; v < ST; ++v) one(s + v, v);
    }
#pragma unroll
    for (int v = 0; v < ST - 1; ++v) {
        if (s + v >= nsteps) break;   // uniform
        one(s + v, v);
    }
    if constexpr (ROWS_HELD) {
#pragma unroll
        for (int rb = EARLY; rb < RB; ++rb) request_rows(rb);
    }
    SHFLBW_WAVE_LDS_SYNC();

    // accumulators in groups of four neighbouring columns: group q of row block rb, and its first column
    auto quad = [&](int rb, int q) __attribute__((always_inline)) {
        if constexpr (S::SMALL) {
            const int r = q / (NT / 4), t = q % (NT / 4) * 4;
            return floatx4{acc16[t][r], acc16[t + 1][r], acc16[t + 2][r], acc16[t + 3][r]};
        } else if constexpr (WN == 128) {
            const int r = q / 2, t = q % 2 * 2;
            return floatx4{acc32[rb][t][r], acc32[rb][t][r + 8], acc32[rb][t + 1][r], acc32[rb][t + 1][r + 8]};
        } else {
            const int r = q / 2, t = q % 2;
            return floatx4{acc32[rb][t][r], acc32[rb][t][r + 8], acc32[rb][t][r + 4], acc32[rb][t][r + 12]};
        }
    };
    auto quad_col = [&](int q) __attribute__((always_inline)) {
        if constexpr (S::SMALL) return WN == 128 ? 8 * (4 * (lane >> 4) + q / 2) + 4 * (q % 2) : 8 * (4 * (lane >> 4 & 1) + q) + 4 * (lane >> 5);
        else return WN == 128 ? 8 * (8 * (q / 8) + 4 * (lane >> 5) + q / 2 % 4) + 4 * (q % 2) : 8 * (4 * (lane >> 5) + q / 2) + 4 * (q % 2);
    };
    const int lane_row = lane & (S::ROWS_E - 1);   // this lane's row of a row block

    if constexpr (SPLIT > 1) {
        // quad q of wavefront w sits at float4 index (w*QUADS + q)*64 + lane, free of bank conflicts
        constexpr int OWN = (QUADS + SPLIT - 1) / SPLIT;           // quads a wavefront adds up
        floatx4* red = reinterpret_cast<floatx4*>(smem);
        OutT* fin = reinterpret_cast<OutT*>(smem + (APART ? RED_BYTES : 0)) + ti * S::ROWS_E * EPS;
        typedef OutT vec4 __attribute__((ext_vector_type(4)));
        typedef OutT vecw __attribute__((ext_vector_type(OPV)));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            // (APART: every wavefront has taken its sums of the row block before when its tile is finished)
            if (!APART && rb) __syncthreads();
#pragma unroll
            for (int q = 0; q < QUADS; ++q) red[(wave * QUADS + q) * 64 + lane] = quad(rb, q);
            __syncthreads();
            floatx4 sum[OWN];
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                const int q = part + i * SPLIT;
                if (QUADS % SPLIT == 0 || q < QUADS) {
                    sum[i] = red[(ti * SPLIT * QUADS + q) * 64 + lane];
#pragma unroll
                    for (int p = 1; p < SPLIT; ++p) sum[i] += red[((ti * SPLIT + p) * QUADS + q) * 64 + lane];
                }
            }
            if (!APART) __syncthreads();
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                const int q = part + i * SPLIT;
                if (QUADS % SPLIT == 0 || q < QUADS) {
                    // (the tile before was read before the barrier above)
                    *reinterpret_cast<vec4*>(fin + lane_row * EPS + quad_col(q)) = vec4{(OutT)sum[i][0], (OutT)sum[i][1], (OutT)sum[i][2], (OutT)sum[i][3]};
                }
            }
            __syncthreads();
            vecw v[STORES_S];
#pragma unroll
            for (int i = 0; i < STORES_S; ++i) {
                const int row = row_of(i);
                if ((S::ROWS_E / RPI_S) % SPLIT == 0 || row < S::ROWS_E)
                    v[i] = *reinterpret_cast<const vecw*>(fin + row * EPS + lane % LPR_S * OPV);
            }
            with_stores(geom, [&](auto stream_tag) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < STORES_S; ++i) {
                    const int row = row_of(i);
                    if ((S::ROWS_E / RPI_S) % SPLIT == 0 || row < S::ROWS_E) {
                        OutT tmp[OPV];
#pragma unroll
                        for (int e = 0; e < OPV; ++e) tmp[e] = v[i][e];
                        const int orig = ROWS_HELD ? out_row[ROWS_HELD ? rb : 0][i] : rows_g[rb * 32 + row];
                        geom.template store<decltype(stream_tag)::value, OPV>(orig, n0 + lane % LPR_S * OPV, tmp);
                    }
                }
            });
        }
        return;
    }

    // ---- reordered write-back
    // Each pass moves ROWS_E stored rows x CW columns through LDS.  A lane
    // holds 4 consecutive n of one row per accumulator quad.
    constexpr int PASSES = (int)sizeof(OutT) / 2;                   // column halves per row block
    constexpr int CW = WN / PASSES;                                  // columns per pass
    constexpr int EP = CW + 16 / (int)sizeof(OutT);                 // pitch in OutT units
    static_assert(S::ROWS_E * EP * (int)sizeof(OutT) <= S::EPI * 2, "epilogue tile must fit");
    OutT* ep = reinterpret_cast<OutT*>(smem + wave * S::EPI * 2);
    static_assert(SPLIT > 1 || CW / OPV == LPR_S, "lanes per row at readback");
    const int echunk = lane % LPR_S;

#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            // the columns of a pass are half of every lane's groups, or all groups of half of the lanes
            constexpr bool BY_GROUP = PASSES > 1 && !S::SMALL && WN == 128;
            if (PASSES == 1 || BY_GROUP || (WN == 128 || !S::SMALL ? lane >> 5 : lane >> 4 & 1) == pass) {
#pragma unroll
                for (int i = 0; i < (BY_GROUP ? QUADS / PASSES : QUADS); ++i) {
                    const int q = BY_GROUP ? pass * (QUADS / PASSES) + i : i;
                    const floatx4 a = quad(rb, q);
                    typedef OutT vec4 __attribute__((ext_vector_type(4)));
                    *reinterpret_cast<vec4*>(ep + lane_row * EP + quad_col(q) - pass * CW) = vec4{(OutT)a[0], (OutT)a[1], (OutT)a[2], (OutT)a[3]};
                }
            }
            SHFLBW_WAVE_LDS_SYNC();
            typedef OutT vecw __attribute__((ext_vector_type(OPV)));
            vecw v[STORES_S];
#pragma unroll
            for (int i = 0; i < STORES_S; ++i) v[i] = *reinterpret_cast<const vecw*>(ep + row_of(i) * EP + echunk * OPV);
            with_stores(geom, [&](auto stream_tag) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < STORES_S; ++i) {
                    OutT tmp[OPV];
#pragma unroll
                    for (int e = 0; e < OPV; ++e) tmp[e] = v[i][e];
                    const int orig = ROWS_HELD ? out_row[ROWS_HELD ? rb : 0][i] : rows_g[rb * 32 + row_of(i)];
                    geom.template store<decltype(stream_tag)::value, OPV>(orig, n0 + pass * CW + echunk * OPV, tmp);
                }
            });
            SHFLBW_WAVE_LDS_SYNC();
        }
    }
}

}  // namespace shflbw
