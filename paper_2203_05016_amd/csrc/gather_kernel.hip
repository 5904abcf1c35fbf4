// Per-wavefront gather kernel for the Shfl-BW product on gfx950 (CDNA4).
//
// One wavefront owns one row group (V stored rows) x WN output columns and
// runs Algorithm 1's loop on its own, with no workgroup barrier:
//   BulkLoadMeta  - the column indices of a k-step are fetched 2*PD steps
//                   ahead of their use, one 16-byte load per lane;
//   StitchTile    - the TK activation rows named by those indices are loaded
//                   (16 bytes per lane, coalesced along N) PD steps ahead into
//                   registers, then written to the wavefront's private LDS
//                   tile; the weight tile is one 16-byte load per lane from
//                   the packed array, already in operand order;
//   WarpMMA       - the activation tile is read back transposed
//                   (ds_read_b64_tr_b16) as the first matrix-core operand and
//                   multiplied with the weight operand, fp32 accumulation;
//   ReorderedWriteBack - accumulators go through LDS so that every stored
//                   row leaves as full 16-byte-per-lane row segments, to the
//                   row named by row_indices.
//
// The product is computed as (X^T tile) x (W^T tile), i.e. the instruction's
// row dimension runs over output columns n and its column dimension over the
// group's rows: each lane then holds 4 consecutive n of one row, which packs
// into one 8-byte LDS write in the epilogue.
//
// Operand and accumulator lane maps (checked on hardware):
//   v_mfma_f32_32x32x16_f16  A: lane l = row l%32, k = 8*(l/32)+e
//                            B: lane l = col l%32, k = 8*(l/32)+e
//                            D: lane l, reg r = row 8*(r/4)+4*(l/32)+r%4, col l%32
//   v_mfma_f32_16x16x32_f16  A: lane l = row l%16, k = 8*(l/16)+e; B alike;
//                            D: lane l, reg r = row 4*(l/16)+r, col l%16
//   ds_read_b64_tr_b16: inside each block of 16 lanes, result element e of
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
// where it has the choice (CHOICE).

// Linear layer: X[K][N] and Y[M][N] row-major.  ALIGNED: N, ldx, ldy are
// multiples of 8 and both bases are 16-byte aligned.
template <bool ALIGNED>
struct GeomLinear {
    const _Float16* X;
    void* Y;
    long ldx, ldy, N;

    __device__ __forceinline__ void init(long) {}

    __device__ __forceinline__ half8 load8(int col, long n) const
    {
        half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (col < 0) return v;
        const _Float16* p = X + (long)col * ldx + n;
        if (ALIGNED) {
            if (n < N) v = *reinterpret_cast<const half8*>(p);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (n + e < N) v[e] = p[e];
        }
        return v;
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
// address is one 24-bit multiply-add in a vector register (byte offset of the
// row plus the lane's column offset) instead of 64-bit arithmetic, and the
// descriptor's range check stands in for the two conditions - a padded slot
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
    static constexpr bool FINISH = false;   // load8 returns the values as they are used
    static constexpr bool LIST = false;     // load8 takes column indices as they are stored
    static constexpr bool CHOICE = true;    // of streaming and plain stores

    __device__ __forceinline__ void init(long n)
    {
        xd = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(X), 0, (int)xbytes, GATHER_BUFFER_FLAGS);
        ldx2 = (unsigned)ldx * 2u;
        ln2 = n < N ? (unsigned)n * 2u : PAST_END;
    }

    // zero (the same for the whole wavefront): read zeros whatever the column, at the price of
    // scalar instructions only
    __device__ __forceinline__ half8 load8(int col, bool zero, int&) const
    {
        // a lane beyond N keeps its offset past the end whatever the column
        unsigned off = __umul24((unsigned)col, ldx2) + ln2;
        off = (col < 0 || ln2 == PAST_END || zero) ? PAST_END : off;
        return __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(xd, (int)off, 0, 0));
    }

    template <bool STREAM, int CNT, typename OutT>
    __device__ __forceinline__ void store(int row, long n, const OutT* vals) const
    {
        if (n < N) store_run<STREAM, CNT>(static_cast<OutT*>(Y) + (long)row * ldy + n, vals);
    }
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
// Loading odd offsets one value early, with the missing last value from the next lane, takes the
// address unit's accesses from 62 to 20 per load and gains nothing (18.6 us; convolutions lose 1 us
// to the extra instructions).
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
        ln2 = n < N ? (unsigned)((unsigned long)n >> 2) * x_image : PAST_END;
        ln2b = n + 4 < N ? (unsigned)((unsigned long)n >> 2) * x_image + x_image : PAST_END;
    }
    __device__ __forceinline__ half8 load8(int col, bool zero, int&) const
    {
        typedef unsigned uint2v __attribute__((ext_vector_type(2)));
        typedef unsigned uint4v __attribute__((ext_vector_type(4)));
        const unsigned o = (unsigned)col * 8u;
        const bool none = col < 0 || zero;
        const uint2v lo = __builtin_amdgcn_raw_buffer_load_b64(xd, (int)(none || ln2 == PAST_END ? PAST_END : ln2 + o), 0, 0);
        const uint2v hi = __builtin_amdgcn_raw_buffer_load_b64(xd, (int)(none || ln2b == PAST_END ? PAST_END : ln2b + o), 0, 0);
        return __builtin_bit_cast(half8, uint4v{lo[0], lo[1], hi[0], hi[1]});
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
// moves the values down (finish8).  X must hold 8 values or more.  4096 x 4096 by 4096 x 1 (V = 32,
// 75 %): 38.3 us with element-wise loads, 6.3 us.
struct GeomNarrow : GeomLinearBuf {
    static constexpr bool FINISH = true, CHOICE = false;
    __device__ __forceinline__ half8 load8(int col, bool zero, int& shift) const
    {
        unsigned off = __umul24((unsigned)col, ldx2) + ln2;
        const unsigned lim = xbytes - 16u;
        const unsigned at = off < lim ? off : lim;
        shift = (int)(off - at) >> 1;
        off = (col < 0 || ln2 == PAST_END || zero) ? PAST_END : at;
        return __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(xd, (int)off, 0, 0));
    }
    // values shift .. 7 of v moved to 0 (shift 0 .. 7; only columns that exist are looked at afterwards)
    static __device__ __forceinline__ half8 finish8(half8 v, int shift)
    {
        typedef unsigned uint4v __attribute__((ext_vector_type(4)));
        uint4v x = __builtin_bit_cast(uint4v, v);
        if (shift & 4) { x[0] = x[2]; x[1] = x[3]; }
        if (shift & 2) { x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; }
        const unsigned bits = (shift & 1) * 16;
        x[0] = __builtin_amdgcn_alignbit(x[1], x[0], bits);
        x[1] = __builtin_amdgcn_alignbit(x[2], x[1], bits);
        x[2] = __builtin_amdgcn_alignbit(x[3], x[2], bits);
        x[3] >>= bits;
        return __builtin_bit_cast(half8, x);
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
// (Section 4.1's implicit GEMM, unfolded on the way into the LDS): images for CHWN (any stride,
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
    static constexpr bool FINISH = !CHWN, LIST = true;
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
    __device__ __forceinline__ half8 load8(entry_t e, int& shift) const
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
        off = ok ? off : PAST_END;
        return __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(xd, (int)off, 0, 0));
    }
    // the run that was asked for, from the one loaded `shift` columns over
    static __device__ __forceinline__ half8 finish8(half8 v, int shift)
    {
        typedef unsigned uint4v __attribute__((ext_vector_type(4)));
        const uint4v x = __builtin_bit_cast(uint4v, v);
        const unsigned up = shift > 0 ? 0x05040302u : 0x07060504u, down = shift < 0 ? 0x05040302u : 0x03020100u;
        uint4v y, z;
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = __builtin_amdgcn_perm(x[i], i ? x[i - 1] : 0u, up);
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = __builtin_amdgcn_perm(i < 3 ? y[i + 1] : 0u, y[i], down);
        return __builtin_bit_cast(half8, z);
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

    __device__ __forceinline__ half8 load8(int col, long) const
    {
        half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (col < 0) return v;
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
        return v;
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
    static constexpr int LPR = WN / 8;                // lanes per activation row (16 B each)
    static constexpr int RPI = 64 / LPR;              // rows per load instruction
    static constexpr int NLD = TK / RPI;              // loads per lane per k-step
    static constexpr int PITCH = WN + 8;              // LDS row pitch in binary16
    static constexpr int STAGE = TK * PITCH;          // binary16 per staged tile
    static constexpr int ROWS_E = SMALL ? 16 : 32;    // rows per epilogue pass
    static constexpr int EPI = ROWS_E * PITCH;        // binary16 needed by one epilogue pass
    static constexpr int REGION = (2 * STAGE > EPI) ? 2 * STAGE : EPI;
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

template <class Geom>
constexpr bool uses_list()
{
    if constexpr (std::is_base_of<GeomLinearBuf, Geom>::value) return Geom::LIST;
    else return false;
}

// f with std::true_type or std::false_type: streaming stores or not.  One choice for all the stores of a
// pass: taken at every store, it keeps the reads of the finished tile from running ahead of the stores (1x1 on
// 28x28 images, 64 -> 256 channels, V = 64 7.05 -> 6.78 us; 1024 x 1024 by 5632 at 90 %, V = 64 5.70 -> 5.47).
template <class Geom, class F>
__device__ __forceinline__ void with_stores(const Geom& geom, F&& f)
{
    if constexpr (std::is_base_of<GeomLinearBuf, Geom>::value) {
        if constexpr (Geom::CHOICE) {
            if (geom.stream) {
                asm volatile("");   // kept apart: merged with the other branch, the stores lose their hint
                f(std::true_type{});
                asm volatile("");
                return;
            }
        }
    }
    f(std::false_type{});
}

// Wavefronts a SIMD must be able to hold.  Left alone, the compiler counts on one workgroup per CU: with four
// wavefronts or fewer in it, a SIMD to each, it keeps the accumulators in registers of their own (V = 128: 328
// registers, one wavefront per SIMD).  Two are asked for, and four (128 registers) for V = 64, which takes
// up to 132 otherwise, two workgroups of eight becoming one (not for the split by 8, of which there is no more
// than one workgroup per CU).  Us before -> after, splits by 2 and 4: 3x3, 56x56, 12 images, CHWN, 64 -> 128
// channels, dense, V = 128: 24.9 -> 15.7; 3x3 / 2, 56x56, CHWN, 128 channels, V = 128 at 50 %: 17.4 -> 11.6;
// 3x3, 56x56, 64 channels, V = 64 at 75 %: 12.8 -> 11.5; aligned products -1 to +2 %.
template <int V, int WN, class Geom, int SPLIT>
constexpr int gather_min_waves()
{
    return V == 64 && WN == 64 && SPLIT < 8 && !std::is_same<Geom, GeomConv>::value ? 4 : 2;
}

// SPLIT = 1: the wavefronts of a workgroup own different column tiles of one group.
// SPLIT > 1 (too few tiles to fill the chip): SPLIT neighbouring wavefronts share one tile, each
// takes a contiguous share of the group's k-steps; the partial accumulators of a row block meet in
// the LDS, every wavefront of the tile adds up its share of them and stores its share of the rows.
template <int V, int WN, int WAVES, int PD, typename OutT, class Geom, bool BF, int SPLIT>
__global__ __launch_bounds__(64 * WAVES, (gather_min_waves<V, WN, Geom, SPLIT>()))
void shflbw_gather_kernel(PackedView A, Geom geom, int n_tiles, GatherOrder order)
{
    using S = GatherShape<V, WN>;
    constexpr int TK = S::TK, RB = S::RB, NT = S::NT, LPR = S::LPR, NLD = S::NLD;
    constexpr int PITCH = S::PITCH;
    constexpr bool BUF = std::is_base_of<GeomLinearBuf, Geom>::value;
    constexpr bool LIST = uses_list<Geom>();
    constexpr int TILES = WAVES / SPLIT;                             // column tiles of a workgroup
    static_assert(TILES * SPLIT == WAVES, "whole tiles per workgroup");
    constexpr int QUADS = S::SMALL ? NT : NT * 4;                    // groups of 4 accumulators per lane and row block
    constexpr int EPS = WN + 16 / (int)sizeof(OutT);                 // row pitch of a finished tile (SPLIT > 1), in OutT units
    constexpr int RED_BYTES = SPLIT > 1 ? WAVES * QUADS * 1024 : 0;
    constexpr int FIN_BYTES = SPLIT > 1 ? TILES * S::ROWS_E * EPS * (int)sizeof(OutT) : 0;
    constexpr int TILE_BYTES = WAVES * S::REGION * 2 > RED_BYTES ? (WAVES * S::REGION * 2 > FIN_BYTES ? WAVES * S::REGION * 2 : FIN_BYTES)
                                                                  : (RED_BYTES > FIN_BYTES ? RED_BYTES : FIN_BYTES);
    constexpr int LIST_BYTES = LIST ? WAVES * 2 * 64 * 8 : 0;        // two batches of 64 entries per wavefront
    __shared__ __attribute__((aligned(16))) _Float16 smem[(TILE_BYTES + LIST_BYTES) / 2];

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
    // without SPLIT a whole wavefront leaves and no workgroup barrier is used; with SPLIT one whose
    // tile does not exist stays for the barriers, with no steps and nothing to store
    if (SPLIT == 1 && tile >= n_tiles) return;
    const long n0 = (long)tile * WN;
    _Float16* my = smem + wave * S::REGION;

    // without a memory access when every group has the same number of steps: the column indices can be
    // requested at once instead of after a dependent load (convolutions, which compute their list
    // first, lose 1 to 2 % by it: 3x3, 14x14x256 12.1 -> 12.3 us)
    const int uniform = LIST ? -1 : order.uniform_steps;
    int sbeg = uniform >= 0 ? g * uniform : A.step_ptr[g];
    int nsteps = uniform >= 0 ? uniform : A.step_ptr[g + 1] - sbeg;
    if (SPLIT > 1) {
        const int first = (int)((long)nsteps * part / SPLIT);
        const int end = (int)((long)nsteps * (part + 1) / SPLIT);
        sbeg += first;
        nsteps = tile < n_tiles ? end - first : 0;
    }

    // this lane's share of a staged tile: rows lrow..lrow+NLD-1, 8 columns at lcol
    const int lrow = (lane / LPR) * NLD;
    const int lcol = (lane % LPR) * 8;
    const long ln = n0 + lcol;
    geom.init(ln);

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
    constexpr bool ROWS_AHEAD = RB <= 2 && std::is_same<Geom, GeomLinearBuf>::value && !(RB == 2 && WN == 128 && sizeof(OutT) == 4);
    constexpr int EARLY = !ROWS_AHEAD ? 0 : RB == 2 && SPLIT == 1 && sizeof(OutT) == 2 ? 1 : RB;
    constexpr int OPV = 16 / (int)sizeof(OutT);                      // values per 16 bytes
    // a store instruction of 16 bytes per lane: lanes per row and rows, without and with SPLIT
    constexpr int LPR_S = SPLIT > 1 ? WN / OPV : WN / ((int)sizeof(OutT) / 2) / OPV, RPI_S = 64 / LPR_S;
    constexpr int STORES_S = SPLIT > 1 ? (S::ROWS_E / RPI_S + SPLIT - 1) / SPLIT : S::ROWS_E / RPI_S;
    int out_row[ROWS_AHEAD ? RB : 1][STORES_S];
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

    // ---- pipeline registers
    int cols[PD][NLD];
    half8 xr[PD][NLD];
    int xf[PD][NLD];   // what geom.finish8 needs to know of a load
    half8 wr[PD][RB];

    // Column indices and weights of the wavefront's steps through buffer descriptors: the
    // step's offset is a scalar register, the lane's a constant vector register.
    typedef unsigned uint2v __attribute__((ext_vector_type(2)));
    typedef unsigned uint4v __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t col_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t*>(A.col_idx + (long)sbeg * TK), 0, nsteps * TK * 4, GATHER_BUFFER_FLAGS);
    const __amdgpu_buffer_rsrc_t val_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<half8*>(A.values + (long)sbeg * RB * 64), 0, nsteps * RB * 1024, GATHER_BUFFER_FLAGS);
    // A buffer load checks lane offset + immediate against the descriptor's size, NOT the
    // scalar offset.  CHECKED puts the step into the lane offset, so that a step beyond the
    // wavefront's range reads zeros instead of memory past it; the steady-state batches,
    // whose steps all exist, keep the step in the scalar offset (no vector arithmetic).
    auto load_cols = [&](int step, int (&c)[NLD], auto checked_tag) {
        constexpr bool CHECKED = decltype(checked_tag)::value;
        const int vo = CHECKED ? lrow * 4 + step * TK * 4 : lrow * 4;
        const int so = CHECKED ? 0 : step * TK * 4;
        if constexpr (NLD == 4) {
            uint4v v = __builtin_amdgcn_raw_buffer_load_b128(col_rsrc, vo, so, 0);
            c[0] = (int)v[0]; c[1] = (int)v[1]; c[2] = (int)v[2]; c[3] = (int)v[3];
        } else if constexpr (NLD == 2) {
            uint2v v = __builtin_amdgcn_raw_buffer_load_b64(col_rsrc, vo, so, 0);
            c[0] = (int)v[0]; c[1] = (int)v[1];
        } else {
#pragma unroll
            for (int i = 0; i < NLD; ++i)
                c[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(col_rsrc, vo + i * 4, so, 0);
        }
    };
    // in_range false: the step lies beyond the wavefront's range and gets zeros, like a padded slot
    auto load_x = [&](const int (&c)[NLD], half8 (&x)[NLD], int (&f)[NLD], bool in_range) {
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            if constexpr (LIST) x[i] = half8{0, 0, 0, 0, 0, 0, 0, 0};   // not reached
            else if constexpr (BUF) x[i] = geom.load8(c[i], !in_range, f[i]);
            else x[i] = geom.load8(in_range ? c[i] : -1, ln);
        }
    };
    auto arrived = [&](half8 x, int f) __attribute__((always_inline)) {
        if constexpr (BUF) {
            if constexpr (Geom::FINISH) return Geom::finish8(x, f);
        }
        return x;
    };
    auto load_w = [&](int step, half8 (&w)[RB], auto checked_tag) {
        constexpr bool CHECKED = decltype(checked_tag)::value;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int off = (step * RB + rb) * 1024;
            w[rb] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(
                val_rsrc, CHECKED ? lane * 16 + off : lane * 16, CHECKED ? 0 : off, 0));
        }
    };

    // The loop below is straight-line code over whole batches of PD steps, so that the
    // register sets stay static and the compiler's wait counts exact (a conditional refill
    // turns into a copy behind a full wait).  A step beyond the wavefront's range multiplies
    // zero weights (range-checked loads) with gathered zeros.
    const int nsteps_r = (nsteps + PD - 1) / PD * PD;
    if constexpr (!LIST) {
#pragma unroll
    for (int u = 0; u < PD; ++u) {
        int c0[NLD];
        load_cols(u, c0, std::true_type{});
        load_x(c0, xr[u], xf[u], u < nsteps);
        load_cols(u + PD, cols[u], std::true_type{});
        load_w(u, wr[u], std::true_type{});
        // sets in the order the loop issues them: its wait counts assume set 0 is the oldest
        __builtin_amdgcn_sched_barrier(0);
    }
    }

    // transposed-read addresses (in binary16 units inside a staged tile)
    // 32-wide: block b = lane/16 covers n = 16*(b%2)+0..15, k = 8*(b/2)+4h+0..3
    // 16-wide: block b covers n = 0..15,                k = 8*b+4h+0..3
    const int bl = lane >> 4, il = lane & 15;
    const int tr_row = S::SMALL ? (8 * bl + (il >> 2)) : (8 * (bl >> 1) + (il >> 2));
    const int tr_col = S::SMALL ? (4 * (il & 3)) : (16 * (bl & 1) + 4 * (il & 3));
    const int tr_off = tr_row * PITCH + tr_col;

    // the products of one step from its staged tile
    auto multiply = [&](const _Float16* buf, const half8 (&w)[RB]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const _Float16* base = buf + tr_off + t * S::TILE_N;
            short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(base));
            short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(base + 4 * PITCH));
            half4 l4 = __builtin_bit_cast(half4, lo), h4 = __builtin_bit_cast(half4, hi);
            half8 a = {l4[0], l4[1], l4[2], l4[3], h4[0], h4[1], h4[2], h4[3]};
            if (S::SMALL) {
                acc16[t] = mma16<BF>(a, w[0], acc16[t]);
            } else {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    acc32[rb][t] = mma32<BF>(a, w[rb], acc32[rb][t]);
            }
        }
    };

    if constexpr (LIST) {
        // The rows a wavefront gathers are worked out 64 at a time (one per lane, U k-steps) and kept
        // in a private list in the LDS, two batches of it, so that the divisions by the kernel's size are
        // paid once per 64 rows and not by every lane for each of its loads (32 images of 14x14,
        // 256 channels, 3x3, V = 32, 75 %: 12.6 -> 11.8 us).
        constexpr int U = 64 / TK;
        static_assert(PD == 2 && U % PD == 0, "loads of a step go out two steps ahead, from this batch's entries or the next one's");
        typedef typename Geom::entry_t entry_t;
        entry_t* list = reinterpret_cast<entry_t*>(reinterpret_cast<char*>(smem) + TILE_BYTES) + wave * 128;
        auto fetch = [&](int q) __attribute__((always_inline)) {
            return (int)__builtin_amdgcn_raw_buffer_load_b32(col_rsrc, lane * 4 + q * 256, 0, 0);
        };
        auto work_out = [&](int q, int col) __attribute__((always_inline)) {
            list[(q & 1) * 64 + lane] = geom.entry(col, q * 64 + lane < nsteps * TK);
        };
        // s: k-step; q: its batch
        auto request = [&](int s, int q, half8 (&x)[NLD], int (&f)[NLD]) __attribute__((always_inline)) {
            const entry_t* e = list + (q & 1) * 64 + (s - q * U) * TK + lrow;
#pragma unroll
            for (int i = 0; i < NLD; ++i) x[i] = geom.load8(e[i], f[i]);
        };
        int c = fetch(0);
#pragma unroll
        for (int u = 0; u < PD; ++u) load_w(u, wr[u], std::true_type{});
        work_out(0, c);
        c = fetch(1);
        SHFLBW_WAVE_LDS_SYNC();
#pragma unroll
        for (int u = 0; u < PD; ++u) {
            request(u, u / U, xr[u], xf[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int q = 0; q * U < nsteps; ++q) {
            work_out(q + 1, c);
            c = fetch(q + 2);
            SHFLBW_WAVE_LDS_SYNC();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s = q * U + u;
                if (u && u % PD == 0 && s >= nsteps) break;   // uniform
                _Float16* buf = my + (u & 1) * S::STAGE;
#pragma unroll
                for (int i = 0; i < NLD; ++i)
                    *reinterpret_cast<half8*>(buf + (lrow + i) * PITCH + lcol) = arrived(xr[u % PD][i], xf[u % PD][i]);
                SHFLBW_WAVE_LDS_SYNC();
                request(s + PD, u + PD < U ? q : q + 1, xr[u % PD], xf[u % PD]);
                multiply(buf, wr[u % PD]);
                load_w(s + PD, wr[u % PD], std::true_type{});
                __builtin_amdgcn_sched_barrier(0);   // steps stay in program order, see below
            }
        }
    } else {
    // One batch.  NEXT: the batch after this one exists, its X rows and weights are
    // requested; AFTER: so does the one after that, whose column indices are requested.
    // The last two batches therefore issue no loads that nobody waits for.
    auto batch = [&](int s0, auto next_tag, auto after_tag) __attribute__((always_inline)) {
        constexpr bool NEXT = decltype(next_tag)::value, AFTER = decltype(after_tag)::value;
#pragma unroll
        for (int u = 0; u < PD; ++u) {
            const int s = s0 + u;
            _Float16* buf = my + (s & 1) * S::STAGE;
#pragma unroll
            for (int i = 0; i < NLD; ++i)
                *reinterpret_cast<half8*>(buf + (lrow + i) * PITCH + lcol) = arrived(xr[u][i], xf[u][i]);
            SHFLBW_WAVE_LDS_SYNC();

            if (NEXT) load_x(cols[u], xr[u], xf[u], AFTER || s + PD < nsteps);
            // may name up to PD - 1 steps past the range: those indices (whatever follows in the
            // packed matrix) are never turned into addresses
            if (AFTER) load_cols(s + 2 * PD, cols[u], std::false_type{});

            multiply(buf, wr[u]);
            // refilled after its last use, so the load lands in the set's own registers
            // the last loading batch may reach past the range: checked there
            if (NEXT) load_w(s + PD, wr[u], std::integral_constant<bool, !AFTER>{});
            // steps stay in program order: hoisting the next step's LDS writes above this
            // step's products would make them wait for the loads issued just above
            __builtin_amdgcn_sched_barrier(0);
            // no second sync: the next step writes the other buffer, and its own
            // sync separates these reads from the writes of the step after it
        }
    };
    int s0 = 0;
    for (; s0 + 2 * PD < nsteps_r; s0 += PD) batch(s0, std::true_type{}, std::true_type{});
    if (s0 + PD < nsteps_r) {
        batch(s0, std::true_type{}, std::false_type{});
        s0 += PD;
    }
    if (s0 < nsteps_r) batch(s0, std::false_type{}, std::false_type{});
    }
    if constexpr (ROWS_AHEAD) {
#pragma unroll
        for (int rb = EARLY; rb < RB; ++rb) request_rows(rb);
    }
    SHFLBW_WAVE_LDS_SYNC();

    if constexpr (SPLIT > 1) {
        // quad q of wavefront w sits at float4 index (w*QUADS + q)*64 + lane, free of bank conflicts
        constexpr int SHARE = (QUADS + SPLIT - 1) / SPLIT;           // quads a wavefront adds up
        floatx4* red = reinterpret_cast<floatx4*>(smem);
        OutT* fin = reinterpret_cast<OutT*>(smem) + ti * S::ROWS_E * EPS;
        typedef OutT vec4 __attribute__((ext_vector_type(4)));
        typedef OutT vecw __attribute__((ext_vector_type(OPV)));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            __syncthreads();   // the staged tiles, or the finished tile of the row block before, are read
#pragma unroll
            for (int q = 0; q < QUADS; ++q) {
                floatx4 v;
                if (S::SMALL) v = acc16[q];
                else
                    v = floatx4{acc32[rb][q / 4][4 * (q % 4)], acc32[rb][q / 4][4 * (q % 4) + 1],
                                acc32[rb][q / 4][4 * (q % 4) + 2], acc32[rb][q / 4][4 * (q % 4) + 3]};
                red[(wave * QUADS + q) * 64 + lane] = v;
            }
            __syncthreads();
            floatx4 sum[SHARE];
#pragma unroll
            for (int i = 0; i < SHARE; ++i) {
                const int q = part + i * SPLIT;
                if (QUADS % SPLIT == 0 || q < QUADS) {
                    sum[i] = red[(ti * SPLIT * QUADS + q) * 64 + lane];
#pragma unroll
                    for (int p = 1; p < SPLIT; ++p) sum[i] += red[((ti * SPLIT + p) * QUADS + q) * 64 + lane];
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < SHARE; ++i) {
                const int q = part + i * SPLIT;
                if (QUADS % SPLIT == 0 || q < QUADS) {
                    OutT* d = S::SMALL ? fin + (lane & 15) * EPS + 16 * q + 4 * (lane >> 4)
                                       : fin + (lane & 31) * EPS + 32 * (q / 4) + 8 * (q % 4) + 4 * (lane >> 5);
                    *reinterpret_cast<vec4*>(d) = vec4{(OutT)sum[i][0], (OutT)sum[i][1], (OutT)sum[i][2], (OutT)sum[i][3]};
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
                        const int orig = ROWS_AHEAD ? out_row[ROWS_AHEAD ? rb : 0][i] : rows_g[rb * 32 + row];
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
    static_assert(S::ROWS_E * EP * (int)sizeof(OutT) <= S::REGION * 2, "epilogue tile must fit");
    OutT* ep = reinterpret_cast<OutT*>(my);
    static_assert(SPLIT > 1 || CW / OPV == LPR_S, "lanes per row at readback");
    const int echunk = lane % LPR_S;

#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            constexpr int TPP = NT / PASSES;  // instruction tiles per pass
#pragma unroll
            for (int tt = 0; tt < TPP; ++tt) {
                const int t = pass * TPP + tt;
                if (S::SMALL) {
                    // lane: row l%16, n = 16*tt + 4*(l/16) + 0..3
                    OutT* d = ep + (lane & 15) * EP + 16 * tt + 4 * (lane >> 4);
                    typedef OutT vec4 __attribute__((ext_vector_type(4)));
                    vec4 v = {(OutT)acc16[t][0], (OutT)acc16[t][1], (OutT)acc16[t][2], (OutT)acc16[t][3]};
                    *reinterpret_cast<vec4*>(d) = v;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        OutT* d = ep + (lane & 31) * EP + 32 * tt + 8 * q + 4 * (lane >> 5);
                        typedef OutT vec4 __attribute__((ext_vector_type(4)));
                        vec4 v = {(OutT)acc32[rb][t][4 * q + 0], (OutT)acc32[rb][t][4 * q + 1],
                                  (OutT)acc32[rb][t][4 * q + 2], (OutT)acc32[rb][t][4 * q + 3]};
                        *reinterpret_cast<vec4*>(d) = v;
                    }
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
                    const int orig = ROWS_AHEAD ? out_row[ROWS_AHEAD ? rb : 0][i] : rows_g[rb * 32 + row_of(i)];
                    geom.template store<decltype(stream_tag)::value, OPV>(orig, n0 + pass * CW + echunk * OPV, tmp);
                }
            });
            SHFLBW_WAVE_LDS_SYNC();
        }
    }
}

}  // namespace shflbw
