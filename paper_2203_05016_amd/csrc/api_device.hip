// Device-facing entry points of the C ABI: binding the packed matrix to a
// caller-owned device buffer, and the launchers of the SpMM / conv2d kernels.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <mutex>

#include "gather_kernel.hip"
#include "slab_kernel.hip"
#include "conv_kernel.hip"
#include "shflbw_internal.h"
#include "launch_gather.h"

namespace shflbw {
namespace {

// Device image of one packed matrix for shflbw_spmm_unbound: the library's own memory,
// one copy per GPU, held until the process ends.
constexpr size_t STATIC_IMAGE_BYTES = SHFLBW_UNBOUND_MAX_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_IMAGE_BYTES];
constexpr int MAX_DEVICES = 64;
void* g_scratch_ptr[MAX_DEVICES];          // address of `scratch` on each device, resolved on first use
std::mutex g_scratch_mutex;

__global__ void clear_status_kernel(int* word)
{
    if (threadIdx.x < 64) word[threadIdx.x] = 0;
}

int hip_fail(hipError_t e, const char* what)
{
    return fail(SHFLBW_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// "name<V,second,operand format,output format and more>" for shflbw_last_kernel
KernelName kernel_name(const char* base, int V, int second, bool f32_out, bool bf, const char* more = "")
{
    return KernelName("%s<%d,%d,%s,%s%s>", base, V, second, bf ? "bf16" : "f16", f32_out ? "f32 out" : bf ? "bf16 out" : "f16 out",
                      more);
}

PackedView view_of(const shflbw_matrix* A)
{
    const char* b = static_cast<const char*>(device_base(A));
    PackedView v;
    v.row_indices = reinterpret_cast<const int32_t*>(b + A->off_rows);
    v.step_ptr = reinterpret_cast<const int32_t*>(b + A->off_steps);
    v.col_idx = reinterpret_cast<const int32_t*>(b + A->off_cols);
    v.values = reinterpret_cast<const half8*>(b + A->off_vals);
    v.G = A->G;
    return v;
}

template <int V, int GW, typename OutT, bool BF>
int launch_slab(const shflbw_matrix* A, const void* X, long ldx, void* Y, long ldy, long N,
                hipStream_t stream)
{
    SlabArgs a;
    a.A = view_of(A);
    char* base = static_cast<char*>(const_cast<void*>(device_base(A)));
    a.table = reinterpret_cast<const uint32_t*>(base + A->off_table);
    a.first_chunk = reinterpret_cast<const int32_t*>(base + A->off_iter);
    a.status = reinterpret_cast<int*>(base + A->off_status);
    a.spin_limit = A->wait_limit;
    a.X = static_cast<const _Float16*>(X);
    a.Y = Y;
    a.ldx = ldx; a.ldy = ldy; a.N = N;
    // 4096 x 1024 by 8200 (rows of 16 400 bytes): 67 us streaming, 59 plain; 8192 x 8192 by 16376, V = 64: 784 and
    // 754; by 8224 (a multiple of 64 bytes): 48 and 54
    a.stream = (ldy * (long)sizeof(OutT) | (long)reinterpret_cast<uintptr_t>(Y)) % 64 == 0;
    a.K = A->K; a.C = A->slab_chunks;
    const long n_tiles = (N + SLAB_TN - 1) / SLAB_TN;
    a.n_tiles = (int)n_tiles;
    constexpr int GROUPS = V == 128 ? GW / 2 : GW;   // row groups per workgroup
    a.gblocks = (A->G + GROUPS - 1) / GROUPS;
    long wgs = ((n_tiles + 7) / 8) * 8 * a.gblocks;
    // packed weights well beyond an L2: blocks of 8 group blocks x 4 column tiles per XCD
    // (fabric traffic of 8192 x 8192 x 16384 at 75 %: 2.7 -> 1.6 GB); the column tiles of an
    // XCD are rounded up to whole blocks
    a.uniform_steps = A->uniform_steps;
    a.gb_side = 0;
    if (a.gblocks % 8 == 0 && A->values.size() * sizeof(uint16_t) > (size_t)(16 << 20)) {
        a.gb_side = 8;
        const long per_xcd = (n_tiles + 7) / 8;                 // column tiles of one XCD
        wgs = (per_xcd + 3) / 4 * 4 * 8 * a.gblocks;
    }
    if (wgs > 0x7fffffffL) return fail(SHFLBW_ERR_BAD_SHAPE, "grid too large");
    hipLaunchKernelGGL((shflbw_slab_kernel<V, GW, OutT, BF>), dim3((unsigned)wgs), dim3(64 * (GW + SLAB_LOADERS)), 0,
                       stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
    static const KernelName name = kernel_name("shflbw_slab_kernel", V, GW, sizeof(OutT) == 4, BF);
    note_kernel(name.text);
    return SHFLBW_OK;
}

template <typename OutT, bool BF>
int dispatch_slab(const shflbw_matrix* A, const void* X, long ldx, void* Y, long ldy, long N,
                  hipStream_t stream)
{
    switch (A->V) {
        case 16: return launch_slab<16, 12, OutT, BF>(A, X, ldx, Y, ldy, N, stream);
        case 32: return launch_slab<32, 12, OutT, BF>(A, X, ldx, Y, ldy, N, stream);
        case 64: return launch_slab<64, 8, OutT, BF>(A, X, ldx, Y, ldy, N, stream);
        case 128: return launch_slab<128, 8, OutT, BF>(A, X, ldx, Y, ldy, N, stream);
    }
    return fail(SHFLBW_ERR_BAD_OPTION, "the slab kernel supports V = 16, 32, 64, 128");
}

// The gather kernel's instantiations live in their own translation units, one per
// operand format (launch_gather_f16.hip, launch_gather_bf16.hip).
template <class Geom>
int dispatch_out(const shflbw_matrix* A, const Geom& geom, long N, shflbw_dtype ydtype,
                 hipStream_t stream)
{
    if (A->dtype == SHFLBW_BF16) return run_gather_bf16(A, geom, N, ydtype, stream);
    return run_gather_f16(A, geom, N, ydtype, stream);
}

// The same for linear layers' geometries; cut: their choose_cut where it is known already, else -1.
template <class Geom>
int dispatch_linear(const shflbw_matrix* A, const Geom& geom, long N, shflbw_dtype ydtype, hipStream_t stream, int cut)
{
    if (A->dtype == SHFLBW_BF16) return run_gather_bf16(A, geom, N, ydtype, stream, cut);
    return run_gather_f16(A, geom, N, ydtype, stream, cut);
}

// what stream_stores calls reads
double reads_of(const shflbw_matrix* A) { return (double)A->nnz / ((double)A->M * A->V); }

// Why set_tuning(4, ..) cannot be followed
int no_resident()
{
    return fail(SHFLBW_ERR_BAD_OPTION, "the resident slab needs K <= %d and four groups or more, few enough column tiles, results within 4 GiB; convolutions other "
                "than 1x1 also V = 16 or 32, runs of 8 and 16-bit results", RESIDENT_K);
}

// The slab kernel with a resident slab, where it applies, and pays or is forced: rc is the launch's status.  yelems: from Y's start to
// its end, in elements.  cut: the best cut of the other kernels where it was looked for, else untouched.
template <class Geom>
bool try_resident(const shflbw_matrix* A, const Geom& geom, long N, Rows rows, int64_t yelems, shflbw_dtype ydtype, hipStream_t stream, int* rc, int* cut)
{
    const bool forced = A->tune_kernel == 4;
    if (!forced && (A->tune_kernel != 0 || A->tune_tile_n != 0 || A->K > RESIDENT_K)) return false;
    const int ob = ydtype == SHFLBW_F32 ? 4 : 2;
    const int64_t pitch = geom.out_pitch() * ob, ybytes = yelems * ob;
    // results' offsets: 24-bit products in 32 bits
    if (pitch >= (1 << 24) || A->M >= (1 << 24) || ybytes >= ((int64_t)1 << 32) - 64) return false;
    // Streaming stores where results are rows of whole 64-byte blocks.  Else two column tiles write a block's parts, which meet
    // in the L2 only if the stores stay there: 4096 x 1024 by 2047 16.6 us streaming, 13.8 plain, by 8191 51 and 29; with 32-bit
    // results by 2047 30 and 17; 1x1, 512 -> 1024 channels of 14x14 10.6 and 9.5.
    const bool whole = (pitch | (int64_t)reinterpret_cast<uintptr_t>(geom.Y)) % 64 == 0;
    const CutSizes sizes = cut_sizes(A, N, rows, ydtype == SHFLBW_F32);
    if (!forced && !resident_worth_a_look(sizes)) return false;
    const ResidentPlan plan = plan_resident(sizes, whole, rows == Rows::ALIGNED ? 1 : RESIDENT_COPY_UNALIGNED);
    if (plan.parts <= 0) return false;
    if (!forced) {
        *cut = choose_cut(sizes);
        if (!resident_pays(sizes, (Cut)*cut, whole, plan)) return false;
    }
    Geom g = geom;
    g.stream = whole;
    *rc = A->dtype == SHFLBW_BF16 ? run_resident_bf16(A, g, N, plan, (unsigned)ybytes, ydtype, stream)
                                  : run_resident_f16(A, g, N, plan, (unsigned)ybytes, ydtype, stream);
    return true;
}

// `images` products over rows of P columns each (GeomRows)
int run_rows(const shflbw_matrix* A, const void* X, int64_t ldx, int64_t x_image, void* Y, int64_t ldy,
             int64_t y_image, int P, int images, int64_t xbytes, shflbw_dtype ydtype, hipStream_t stream)
{
    GeomRows g;
    g.X = static_cast<const _Float16*>(X);
    g.Y = Y;
    g.ldx = (long)ldx; g.ldy = (long)ldy;
    g.xbytes = (unsigned)xbytes;
    g.x_image = (long)x_image; g.y_image = (long)y_image;
    g.P = P; g.slots = (P + 7) / 8;
    g.m_slots = g.slots == 1 ? 0xffffffffu : (unsigned)(((uint64_t)1 << 32) / (unsigned)g.slots);
    const int ob = ydtype == SHFLBW_F32 ? 4 : 2;
    g.stream = stream_stores(Y, ldy * ob, ob, (double)xbytes, (double)A->M * P * images * ob, reads_of(A), images > 1);
    g.N = (long)images * g.slots * 8;
    int rc = SHFLBW_OK, cut = -1;
    if (try_resident(A, g, g.N, images > 1 ? Rows::IMAGES : Rows::ANY, (images - 1) * y_image + (A->M - 1) * ldy + P, ydtype, stream, &rc, &cut))
        return rc;
    if (A->tune_kernel == 4) return no_resident();
    return dispatch_linear(A, g, g.N, ydtype, stream, cut);
}

// ydtype must be the operand format of the matrix or fp32
int check_ydtype(const shflbw_matrix* A, shflbw_dtype ydtype)
{
    if (ydtype == SHFLBW_F32 || (int)ydtype == A->dtype) return SHFLBW_OK;
    return fail(SHFLBW_ERR_BAD_DTYPE, A->dtype == SHFLBW_BF16
                    ? "ydtype must be SHFLBW_BF16 or SHFLBW_F32 for a bfloat16 matrix"
                    : "ydtype must be SHFLBW_F16 or SHFLBW_F32 for a binary16 matrix");
}

// Up to which kept share a convolution is gathered in runs of 8 (below) rather than staged, by the length of
// the innermost dimension (Wo of NCHW results, the batch of CHWN): every kept row of the unfolded matrix is
// fetched once per group, in whole runs, and staging costs 2-byte LDS reads whatever is kept.  What decides is
// how full the last run is and how many groups fetch.  us staged / gathered, 3x3, by kept share:
//   V = 32, 128 -> 128 channels, 16x16 (full runs)        1: 15.9 / 12.8
//   V = 32, 256 -> 256, 9x9 (one of 8 in the last run)    .5: 16.5 / 17.5   .35: 13.4 / 13.4
//   V = 32, 256 -> 256, 12x12                             .5: 17.3 / 14.8   .25: 12.2 / 9.3
//   V = 32, 256 -> 256, 14x14 (six of 8)                  .5: 17.4 / 18.0   .25: 12.3 / 11.0
//   V = 32, 128 -> 128, 28x28 (4 groups)                  .5: 18.8 / 17.7   1: 28.0 / 30.0
//   V = 32, 128 -> 256, 28x28 (8 groups)                  .5: 26.1 / 32.8   .15: 17.1 / 14.2
//   V = 16, 256 -> 256, 9x9                               .25: 11.8 / 15.2   .1: 8.8 / 8.5
//   V = 16, 256 -> 256, 14x14                             .25: 17.8 / 18.5   .15: 14.5 / 12.7
//   V = 16, 128 -> 128, 17x17                             .25: 12.7 / 14.0   .15: 10.9 / 9.4
//   V = 16, 128 -> 128, 28x28 (8 groups)                  1: 47.4 / 56.5   .5: 32.7 / 32.4
//   V = 16, 128 -> 256, 28x28 (16 groups)                 .5: 51.0 / 61.8   .35: 44.9 / 37.1
//   CHWN, V = 16, 128 -> 128, 28x28, batch 9              .5: 17.5 / 19.4   .35: 15.8 / 15.3
//   CHWN, V = 16, 128 -> 128, 28x28, batch 10             1: 26.8 / 16.6
//   CHWN, V = 32, 256 -> 256, 14x14, batch 25             .5: 19.9 / 20.9   .35: 16.9 / 16.0
// V >= 64 fetches rows for so many results that gathering won everywhere but at 9x9 unpruned (4 %).
double runs_limit(int V, int groups, bool chwn, int innermost)
{
    const int last = innermost % 8;
    if (V >= 64) return 1;
    if (chwn) return last != 1 ? 1 : V == 16 && innermost > 16 ? 0.6 : 0.45;
    if (last == 0) return V == 32 ? 1 : 0.85;
    if (V == 32) {
        if (last == 1) return 0.4;
        if (groups <= 4) return 0.65;
        return innermost > 16 ? 0.22 : last <= 4 ? 0.65 : 0.45;
    }
    if (innermost < 16) return last <= 2 ? 0.12 : 0.22;
    return last == 1 && innermost < 24 ? 0.22 : innermost >= 24 && groups <= 8 ? 0.6 : 0.4;
}

// The convolution as gathers of runs of 8 (GeomConvRuns).  False when the tensor has no such
// runs or is beyond the kernel's 24-bit and 32-bit offset arithmetic.  step: the stride along x that the NCHW geometry takes.
template <bool CHWN>
bool fill_conv_runs(const shflbw_matrix* A, GeomConvRuns<CHWN>& g, const void* in, void* out, int B, int C, int H, int W,
                    int R, int S, int sh, int sw, int ph, int pw, int Ho, int Wo, int64_t in_total, int out_bytes, int step = 1)
{
    if (CHWN ? B < 8 : (sw != step || Wo < 8 || W < 8 * step || pw > 1)) return false;
    const int64_t RS = (int64_t)R * S;
    const int64_t sst = CHWN ? 2 * (int64_t)B : 2, rst = W * sst, cst = H * rst;
    // k / (R*S) by the high half of a product, the remainder / S by 16 bits of one: exact in these ranges
    if (RS * A->K >= ((int64_t)1 << 32) || RS * S > 65536) return false;
    if (cst >= (1 << 24) || C >= (1 << 24) || in_total >= ((int64_t)1 << 32) - 64) return false;
    g.X = static_cast<const _Float16*>(in);
    g.Y = out;
    g.ldx = g.ldy = 0;
    g.xbytes = (unsigned)in_total;
    g.RS = (int)RS; g.S = S; g.H = H; g.W = W; g.B = B; g.Ho = Ho; g.Wo = Wo;
    g.sh = sh; g.sw = sw; g.ph = ph; g.pw = pw;
    g.m_RS = RS == 1 ? 0 : (unsigned)((((uint64_t)1 << 32) + RS - 1) / RS);
    g.m_S = (unsigned)((65536 + S - 1) / S);
    g.cst = (unsigned)cst; g.rst = (unsigned)rst; g.sst = (unsigned)sst;
    g.ist = CHWN ? 0 : (unsigned)(C * cst);
    // NCHW rows are short and follow each other: streaming whatever their length (64 images of 56x56, 64 ->
    // 256 channels: 55 us against 72).  CHWN: by the bytes of a position's images (50 of them, 30x30, 64 -> 256
    // channels: 17.0 streaming, 15.0 plain; 32 of them, 56x56 / 2: 11.1 and 11.6)
    g.stream = !CHWN || stream_stores(out, (int64_t)B * out_bytes, out_bytes, (double)in_total,
                                      (double)A->M * Ho * Wo * B * out_bytes, reads_of(A));
    g.osM = CHWN ? (long)Ho * Wo * B : (long)Ho * Wo;
    g.osB = CHWN ? 0 : (long)A->M * Ho * Wo;
    g.slots = ((CHWN ? B : Wo) + 7) / 8;
    g.N = (CHWN ? (long)Ho * Wo : (long)B * Ho) * g.slots * 8;
    return true;
}

// Picks the box of output positions one workgroup of the staged convolution
// kernel owns, and fills the geometry part of its arguments.  Returns false
// when no box fits (too many channels for the LDS, or a V the kernel does not
// cover); the caller then takes the gather kernel.
bool plan_conv(const shflbw_matrix* A, int B, int C, int H, int W, int R, int S, int sh, int sw,
               int ph, int pw, int Ho, int Wo, bool chwn, ConvArgs& a, size_t& lds_bytes)
{
    if (A->V != 16 && A->V != 32 && A->V != 64 && A->V != 128) return false;
    if (A->K >= (1 << 20) || (long)R * S >= (1 << 20)) return false;   // exact division by multiplication
    // the kernel addresses the input through a buffer descriptor with 32-bit byte offsets
    const unsigned long long in_total = 2ULL * (unsigned long long)B * C * H * W;
    if (in_total >= 0xffffff00ULL) return false;
    // up to four groups: the wavefronts left over share a group's instruction tiles
    const int gpb = A->G <= 4 ? (A->G > 0 ? A->G : 1) : CONV_GW;
    const int gblocks = (A->G + gpb - 1) / gpb;
    const size_t list_bytes = CONV_LIST_BYTES;   // per-wavefront lists of LDS offsets
    const size_t lds_cap = 160 * 1024 - 512;
    const double kg_avg = A->G > 0 ? (double)A->nnz / ((double)A->V * A->G) : 0.0;
    const double groups_per_box = A->G < CONV_GW ? A->G : CONV_GW;
    // Staging with 4-byte loads wants pairs of elements that are neighbours in memory, 4-byte
    // aligned, and inside or outside the image together.  NCHW: pairs along x - an even image
    // width, boxes that start at even x (tw * sw even), the staged box widened by one column on the
    // left when the padding is odd, and an even staged row pitch.  CHWN: pairs along the batch - an
    // even batch and an even number of images per box.
    // It is asked for when it needs at most 0.7 of the load instructions of 2-byte staging (a
    // wavefront covers 64 elements of a channel per instruction there; with pairs it covers 64
    // pairs, or several channels when a channel has 32 pairs or fewer).
    auto pair_cols = [&](int tw) {
        size_t cols = (size_t)(tw - 1) * sw + S;
        if (!chwn) cols = (cols + (pw & 1) + 1) / 2 * 2;
        return cols;
    };
    auto pairs_ok = [&](int th, int tw, int tb) {
        if (!(chwn ? (B % 2 == 0 && tb % 2 == 0) : (W % 2 == 0 && (tw * sw) % 2 == 0))) return false;
        const size_t rows = (size_t)(th - 1) * sh + R;
        const size_t plane1 = rows * ((size_t)(tw - 1) * sw + S) * tb, plane2 = rows * pair_cols(tw) * tb / 2;
        const size_t lpp = plane2 <= 8 ? 8 : plane2 <= 16 ? 16 : plane2 <= 32 ? 32 : 64;
        const double n1 = (double)((plane1 + 63) / 64), n2 = (double)((plane2 + lpp - 1) / lpp) * (double)lpp / 64.0;
        return n2 <= 0.7 * n1;
    };
    auto staged_cols = [&](int th, int tw, int tb) {
        return pairs_ok(th, tw, tb) ? pair_cols(tw) : (size_t)(tw - 1) * sw + S;
    };
    auto staged_elems = [&](int th, int tw, int tb) {
        return ((size_t)C + 1) * ((size_t)(th - 1) * sh + R) * staged_cols(th, tw, tb) * tb;
    };
    auto fits = [&](int th, int tw, int tb) {
        const size_t e = staged_elems(th, tw, tb);
        return e * 2 + 16 + list_bytes <= lds_cap;   // the staged box and the wavefronts' lists share the LDS
    };
    // Candidate boxes: every split of at most `target` positions into images x rows x
    // columns whose innermost-running dimension keeps runs of 8 where the tensor allows
    // it.  The cost of a split is what all its boxes together read: the staged input
    // (global loads, weighted 4x; the halo of a small box is read again by its
    // neighbours) plus the LDS gathers of every 32-position instruction tile, ragged
    // edge tiles included.
    int th = 1, tw = 1, tb = 1;
    long boxes = 0;
    bool found = false;
    const int targets[3] = {CONV_TN, 64, 32};
    for (int target : targets) {
        if (A->V == 128 && target > 64) continue;   // four row blocks: accumulators for two instruction tiles at most
        double best_cost = 0;
        int bh = 0, bw = 0, bb = 0;
        for (int b = 1; b <= B && b <= target; b = (b < B && 2 * b > B) ? B : 2 * b) {
            if (chwn && b < 8 && b < B) continue;
            for (int w = 1; w <= Wo && b * w <= target; ++w) {
                if (!chwn && w < 8 && w < Wo) continue;
                int h = target / (b * w);
                if (h > Ho) h = Ho;
                if (h < 1) continue;
                while (h > 1 && !fits(h, w, b)) --h;
                if (!fits(h, w, b)) continue;
                const int npos = b * w * h;
                const double nboxes = (double)((B + b - 1) / b) * ((Ho + h - 1) / h) * ((Wo + w - 1) / w);
                const double cost = nboxes * (4.0 * staged_elems(h, w, b) +
                                              (double)((npos + 31) / 32) * 32.0 * kg_avg * groups_per_box);
                if (bh == 0 || cost < best_cost * (1 - 1e-9) ||
                    (cost < best_cost * (1 + 1e-9) && npos > bb * bw * bh)) {
                    best_cost = cost; bh = h; bw = w; bb = b;
                }
            }
            if (b == B) break;
        }
        if (bh == 0) continue;
        th = bh; tw = bw; tb = bb; found = true;
        boxes = (long)((B + tb - 1) / tb) * ((Ho + th - 1) / th) * ((Wo + tw - 1) / tw);
        if (boxes * gblocks >= 256) break;   // enough workgroups to fill the chip
    }
    if (!found || boxes * gblocks > 0x7fffffffL) return false;
    a.B = B; a.C = C; a.H = H; a.W = W; a.R = R; a.S = S; a.sh = sh; a.sw = sw; a.ph = ph; a.pw = pw;
    a.Ho = Ho; a.Wo = Wo; a.K = A->K;
    if (chwn) {
        a.isB = 1; a.isW = B; a.isH = (long)W * B; a.isC = (long)H * W * B;
        a.osB = 1; a.osW = B; a.osH = (long)Wo * B; a.osM = (long)Ho * Wo * B;
    } else {
        a.isW = 1; a.isH = W; a.isC = (long)H * W; a.isB = (long)C * H * W;
        a.osW = 1; a.osH = Wo; a.osM = (long)Ho * Wo; a.osB = (long)A->M * Ho * Wo;
    }
    a.th = th; a.tw = tw; a.tb = tb;
    a.ny = (Ho + th - 1) / th; a.nx = (Wo + tw - 1) / tw; a.nb = (B + tb - 1) / tb;
    a.rows_in = (th - 1) * sh + R; a.cols_in = (int)staged_cols(th, tw, tb);
    a.stage_pairs = pairs_ok(th, tw, tb) ? 1 : 0;
    a.dx = (!chwn && a.stage_pairs) ? (pw & 1) : 0;
    a.b_fast = chwn ? 1 : 0;
    a.gblocks = gblocks;
    a.in_bytes_total = (unsigned)in_total;
    a.gpb = gpb;
    {
        const int tiles = (th * tw * tb + 31) / 32;
        const int spare = CONV_GW / gpb;   // wavefronts per group
        a.tsplit = spare < tiles ? spare : tiles;
        if (a.tsplit == 3) a.tsplit = 2;   // tiles per wavefront come as 1, 2 or 4
    }
    auto magic = [](int d) { return (((unsigned long long)1 << 40) + d - 1) / (unsigned long long)d; };
    a.m_RS = magic(R * S); a.m_S = magic(S); a.m_tb = magic(tb); a.m_cols_in = magic(a.cols_in);
    a.m_tw = magic(tw); a.m_th = magic(th);
    a.m_cols2 = magic(a.cols_in / 2 > 0 ? a.cols_in / 2 : 1); a.m_tb2 = magic(tb / 2 > 0 ? tb / 2 : 1);
    size_t in_bytes = (staged_elems(th, tw, tb) * 2 + 15) / 16 * 16;
    const size_t scratch = (size_t)CONV_GW * CONV_SCRATCH;
    if (in_bytes < scratch) in_bytes = scratch;
    a.in_bytes = (int)in_bytes;
    lds_bytes = in_bytes + list_bytes;
    return true;
}

template <int V, int NT, typename OutT, bool BF, bool SP = false>
int launch_conv_nt(const shflbw_matrix* A, ConvArgs& a, size_t lds_bytes, hipStream_t stream)
{
    if constexpr (!SP)
        if (a.stage_pairs == 1) return launch_conv_nt<V, NT, OutT, BF, true>(A, a, lds_bytes, stream);
    // what belongs to the matrix itself and not to its sizes, for which alone a plan is kept
    a.A = view_of(A);
    a.uniform_steps = A->uniform_steps;
    // the attribute is raised once per kernel and device, to the most any box can ask for
    static thread_local int raised_on = -1;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (raised_on != dev) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&shflbw_conv_kernel<V, NT, OutT, BF, SP>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute");
        raised_on = dev;
    }
    const long wgs = (long)a.nb * a.ny * a.nx * a.gblocks;
    hipLaunchKernelGGL((shflbw_conv_kernel<V, NT, OutT, BF, SP>), dim3((unsigned)wgs), dim3(64 * CONV_GW), lds_bytes,
                       stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
    static const KernelName name = kernel_name("shflbw_conv_kernel", V, NT, sizeof(OutT) == 4, BF, SP ? ",4-byte staging" : "");
    note_kernel(name.text);
    return SHFLBW_OK;
}

template <int V, typename OutT, bool BF>
int launch_conv(const shflbw_matrix* A, ConvArgs& a, size_t lds_bytes, hipStream_t stream)
{
    const int tiles = (a.tb * a.th * a.tw + 31) / 32;
    const int npos = (tiles + a.tsplit - 1) / a.tsplit * 32;   // positions one wavefront covers
    if (npos <= 32) return launch_conv_nt<V, 1, OutT, BF>(A, a, lds_bytes, stream);
    if (npos <= 64) return launch_conv_nt<V, 2, OutT, BF>(A, a, lds_bytes, stream);
    if constexpr (V <= 64) return launch_conv_nt<V, 4, OutT, BF>(A, a, lds_bytes, stream);
    else return fail(SHFLBW_ERR_BAD_SHAPE, "box too large for V = 128");   // plan_conv never asks for it
}

template <int V>
int dispatch_conv_v(const shflbw_matrix* A, ConvArgs& a, size_t lds_bytes, shflbw_dtype ydtype,
                    hipStream_t stream)
{
    if (A->dtype == SHFLBW_BF16) {
        if (ydtype == SHFLBW_BF16) return launch_conv<V, __bf16, true>(A, a, lds_bytes, stream);
        return launch_conv<V, float, true>(A, a, lds_bytes, stream);
    }
    if (ydtype == SHFLBW_F16) return launch_conv<V, _Float16, false>(A, a, lds_bytes, stream);
    return launch_conv<V, float, false>(A, a, lds_bytes, stream);
}

int dispatch_conv(const shflbw_matrix* A, ConvArgs& a, size_t lds_bytes, shflbw_dtype ydtype,
                  hipStream_t stream)
{
    if (A->V == 16) return dispatch_conv_v<16>(A, a, lds_bytes, ydtype, stream);
    if (A->V == 32) return dispatch_conv_v<32>(A, a, lds_bytes, ydtype, stream);
    if (A->V == 64) return dispatch_conv_v<64>(A, a, lds_bytes, ydtype, stream);
    return dispatch_conv_v<128>(A, a, lds_bytes, ydtype, stream);
}

int check_bound(const shflbw_matrix* A)
{
    if (!device_base(A)) return fail(SHFLBW_ERR_NOT_ON_DEVICE, "call shflbw_bind_device first");
    return SHFLBW_OK;
}

}  // namespace
}  // namespace shflbw

extern "C" {

int shflbw_bind_device(shflbw_matrix* A, void* dev_buf, void* stream)
{
    using namespace shflbw;
    if (!A || !dev_buf) return fail(SHFLBW_ERR_NULL_ARG, "NULL argument");
    if (reinterpret_cast<uintptr_t>(dev_buf) % 256)
        return fail(SHFLBW_ERR_BAD_SHAPE, "dev_buf must be 256-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* b = static_cast<char*>(dev_buf);
    struct Part { size_t off; const void* src; size_t bytes; };
    const Part parts[] = {
        {A->off_rows, A->row_indices.data(), A->row_indices.size() * sizeof(int32_t)},
        {A->off_steps, A->step_ptr.data(), A->step_ptr.size() * sizeof(int32_t)},
        {A->off_iter, A->first_chunk.data(), A->first_chunk.size() * sizeof(int32_t)},
        {A->off_cols, A->col_idx.data(), A->col_idx.size() * sizeof(int32_t)},
        {A->off_table, A->slab_table.data(), A->slab_table.size() * sizeof(uint32_t)},
        {A->off_vals, A->values.data(), A->values.size() * sizeof(uint16_t)},
    };
    for (const Part& p : parts) {
        if (!p.bytes) continue;
        hipError_t e = hipMemcpyAsync(b + p.off, p.src, p.bytes, hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
    }
    hipError_t e = hipMemsetAsync(b + A->off_status, 0, 256, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemsetAsync");
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    A->dev_base = dev_buf;
    return SHFLBW_OK;
}

int shflbw_device_status(shflbw_matrix* A, void* stream)
{
    using namespace shflbw;
    if (!A) return fail(SHFLBW_ERR_NULL_ARG, "A is NULL");
    int rc = check_bound(A);
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* word = static_cast<char*>(A->dev_base) + A->off_status;
    int seen = 0;
    hipError_t e = hipMemcpyAsync(&seen, word, sizeof seen, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    if (seen == 0) return SHFLBW_OK;
    e = hipMemsetAsync(word, 0, sizeof seen, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemsetAsync");
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    return fail(SHFLBW_ERR_HANDOVER,
                seen == 1 ? "a compute wavefront of the slab kernel gave up waiting for a chunk of X"
                : seen == 2 ? "a loader wavefront of the slab kernel gave up waiting for a free stage"
                            : "compute and loader wavefronts of the slab kernel gave up waiting");
}

int shflbw_spmm(const shflbw_matrix* A, const void* X, int64_t ldx, void* Y, int64_t ldy,
                int64_t N, shflbw_dtype ydtype, void* stream)
{
    using namespace shflbw;
    if (!A) return fail(SHFLBW_ERR_NULL_ARG, "A is NULL");
    if (int rcd = check_ydtype(A, ydtype)) return rcd;
    if (N < 0) return fail(SHFLBW_ERR_BAD_SHAPE, "N < 0");
    if (N == 0) return SHFLBW_OK;
    if (!X || !Y) return fail(SHFLBW_ERR_NULL_ARG, "X and Y must not be NULL");
    if (ldx < N || ldy < N) return fail(SHFLBW_ERR_BAD_SHAPE, "leading dimension smaller than N");
    if (N > (int64_t)1 << 40) return fail(SHFLBW_ERR_BAD_SHAPE, "N too large");
    int rc = check_bound(A);
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool aligned = (N % 8 == 0) && (ldx % 8 == 0) && (ldy % 8 == 0) &&
                         (reinterpret_cast<uintptr_t>(X) % 16 == 0) &&
                         (reinterpret_cast<uintptr_t>(Y) % 16 == 0);
    const bool slab_possible = aligned && A->slab_ok;
    if (A->tune_kernel == 2 && !slab_possible)
        return fail(SHFLBW_ERR_BAD_OPTION, "slab kernel needs the windowed layout and aligned operands");
    // X behind a buffer descriptor where 24-bit offset arithmetic and a 32-bit range cover it
    const int64_t xbytes = ((int64_t)A->K - 1) * ldx * 2 + N * 2;
    const bool described = A->K < (1 << 24) && ldx * 2 < (1 << 24) && xbytes + 2 * ldx * 2 < ((int64_t)1 << 32) - 64;
    int cut = -1;   // choose_cut's answer, once it is known
    GeomLinearBuf g;
    if (aligned && described) {
        g.X = static_cast<const _Float16*>(X);
        g.Y = Y;
        g.ldx = (long)ldx; g.ldy = (long)ldy; g.N = (long)N;
        g.xbytes = (unsigned)xbytes;
        if (try_resident(A, g, (long)N, Rows::ALIGNED, (A->M - 1) * ldy + N, ydtype, st, &rc, &cut)) return rc;
    }
    if (A->tune_kernel == 4 && (aligned || !described || N < 8)) return no_resident();   // (the others: run_rows)
    bool use_slab = A->tune_kernel == 2;
    if (A->tune_kernel == 0 && slab_possible) {
        // the slab kernel streams all of X whatever the sparsity and its workgroup's groups share it: it pays where
        // enough of each chunk is used, sooner where a gathered byte serves few rows (V = 16, 32)
        if (cut < 0) {
            const CutSizes sizes = cut_sizes(A, (long)N, Rows::ALIGNED, ydtype == SHFLBW_F32);
            if (slab_considered(sizes)) cut = choose_cut(sizes);
        }
        use_slab = cut == SLAB;
    }
    if (use_slab) {
        if (A->dtype == SHFLBW_BF16) {
            if (ydtype == SHFLBW_BF16)
                return dispatch_slab<__bf16, true>(A, X, (long)ldx, Y, (long)ldy, (long)N, st);
            return dispatch_slab<float, true>(A, X, (long)ldx, Y, (long)ldy, (long)N, st);
        }
        if (ydtype == SHFLBW_F16)
            return dispatch_slab<_Float16, false>(A, X, (long)ldx, Y, (long)ldy, (long)N, st);
        return dispatch_slab<float, false>(A, X, (long)ldx, Y, (long)ldy, (long)N, st);
    }
    if (aligned) {
        if (described) {
            const int ob = ydtype == SHFLBW_F32 ? 4 : 2;
            g.stream = stream_stores(Y, ldy * ob, ob, 2.0 * A->K * N, (double)ob * A->M * N, reads_of(A));
            return dispatch_linear(A, g, (long)N, ydtype, st, cut);
        }
        GeomLinear<true> wide{static_cast<const _Float16*>(X), Y, (long)ldx, (long)ldy, (long)N};
        return dispatch_out(A, wide, (long)N, ydtype, st);
    }
    // rows of no particular alignment: whole 16-byte accesses where 24-bit offset arithmetic and a
    // 32-bit range cover X
    if (described) {
        if (N >= 8) return run_rows(A, X, ldx, 0, Y, ldy, 0, (int)N, 1, xbytes, ydtype, st);
        if (xbytes >= 16) {
            GeomNarrow narrow;
            narrow.X = static_cast<const _Float16*>(X);
            narrow.Y = Y;
            narrow.ldx = (long)ldx; narrow.ldy = (long)ldy; narrow.N = (long)N;
            narrow.xbytes = (unsigned)xbytes;
            narrow.stream = 0;
            return dispatch_out(A, narrow, (long)N, ydtype, st);
        }
    }
    GeomLinear<false> any{static_cast<const _Float16*>(X), Y, (long)ldx, (long)ldy, (long)N};
    return dispatch_out(A, any, (long)N, ydtype, st);
}

int shflbw_spmm_unbound(const shflbw_matrix* A, const void* X, int64_t ldx, void* Y, int64_t ldy,
                        int64_t N, shflbw_dtype ydtype, void* stream)
{
    using namespace shflbw;
    if (!A) return fail(SHFLBW_ERR_NULL_ARG, "A is NULL");
    if (A->dev_bytes > STATIC_IMAGE_BYTES)
        return fail(SHFLBW_ERR_BAD_SHAPE, "packed matrix of %zu bytes exceeds the library's static device image of %zu "
                    "bytes (SHFLBW_UNBOUND_MAX_BYTES): bind it to a buffer of your own and call shflbw_spmm",
                    A->dev_bytes, STATIC_IMAGE_BYTES);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= MAX_DEVICES) return fail(SHFLBW_ERR_HIP, "device ordinal out of range");
    char* base;
    {
        // the array's name is a host-side stand-in: its device address comes from the runtime, per device
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void* p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p) return hip_fail(e, "hipGetSymbolAddress(scratch)");
            g_scratch_ptr[dev] = p;
        }
        base = static_cast<char*>(g_scratch_ptr[dev]);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    struct Part { size_t off; const void* src; size_t bytes; };
    const Part parts[] = {
        {A->off_rows, A->row_indices.data(), A->row_indices.size() * sizeof(int32_t)},
        {A->off_steps, A->step_ptr.data(), A->step_ptr.size() * sizeof(int32_t)},
        {A->off_iter, A->first_chunk.data(), A->first_chunk.size() * sizeof(int32_t)},
        {A->off_cols, A->col_idx.data(), A->col_idx.size() * sizeof(int32_t)},
        {A->off_table, A->slab_table.data(), A->slab_table.size() * sizeof(uint32_t)},
        {A->off_vals, A->values.data(), A->values.size() * sizeof(uint16_t)},
    };
    for (const Part& p : parts) {
        if (!p.bytes) continue;
        e = hipMemcpyAsync(base + p.off, p.src, p.bytes, hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
    }
    // the status block keeps the last call's contents: it must start at zero (a kernel, not a
    // memset node, so that the call can also be recorded into a graph)
    hipLaunchKernelGGL(clear_status_kernel, dim3(1), dim3(64), 0, st, reinterpret_cast<int*>(base + A->off_status));
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
    set_device_base_override(base);
    const int rc = shflbw_spmm(A, X, ldx, Y, ldy, N, ydtype, stream);
    set_device_base_override(nullptr);
    return rc;
}

int shflbw_conv2d(const shflbw_matrix* A, const void* in, void* out, int batch, int C_in, int H,
                  int W, int R, int S, int stride_h, int stride_w, int pad_h, int pad_w,
                  shflbw_layout layout, shflbw_dtype ydtype, void* stream)
{
    using namespace shflbw;
    if (!A) return fail(SHFLBW_ERR_NULL_ARG, "A is NULL");
    if (int rcd = check_ydtype(A, ydtype)) return rcd;
    if (layout != SHFLBW_NCHW && layout != SHFLBW_CHWN)
        return fail(SHFLBW_ERR_BAD_SHAPE, "unknown layout");
    if (batch < 0 || C_in <= 0 || H <= 0 || W <= 0 || R <= 0 || S <= 0 || stride_h <= 0 ||
        stride_w <= 0 || pad_h < 0 || pad_w < 0)
        return fail(SHFLBW_ERR_BAD_SHAPE, "non-positive convolution dimension");
    if ((int64_t)C_in * R * S != A->K)
        return fail(SHFLBW_ERR_BAD_SHAPE, "C_in*R*S does not match the packed matrix's K");
    if (H + 2 * pad_h < R || W + 2 * pad_w < S)
        return fail(SHFLBW_ERR_BAD_SHAPE, "kernel larger than the padded input");
    if (H + 2 * pad_h > 32767 || W + 2 * pad_w > 32767)
        return fail(SHFLBW_ERR_BAD_SHAPE, "padded image side above 32767");
    const int Ho = (H + 2 * pad_h - R) / stride_h + 1;
    const int Wo = (W + 2 * pad_w - S) / stride_w + 1;
    const int64_t N = (int64_t)batch * Ho * Wo;
    if (N == 0) return SHFLBW_OK;
    if (!in || !out) return fail(SHFLBW_ERR_NULL_ARG, "in and out must not be NULL");
    const int64_t lim = (int64_t)1 << 31;
    // 32-bit element offsets inside the kernel, including the padded halo
    if ((int64_t)batch * C_in * (H + 2 * pad_h) * (W + 2 * pad_w) >= lim ||
        (int64_t)A->M * N >= lim)
        return fail(SHFLBW_ERR_BAD_SHAPE, "tensor above 2^31 elements");
    int rc = check_bound(A);
    if (rc) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // A 1x1 convolution with unit stride and no padding on a batch-innermost tensor IS the
    // linear-layer product: [C_in][H*W*batch] in, [C_out][H*W*batch] out, both row-major.
    const bool resident_only = A->tune_kernel == 4;
    if ((A->tune_kernel == 0 || resident_only) && layout == SHFLBW_CHWN && R == 1 && S == 1 && stride_h == 1 &&
        stride_w == 1 && pad_h == 0 && pad_w == 0)
        return shflbw_spmm(A, in, N, out, N, N, ydtype, stream);
    // The same on NCHW tensors is one such product per image; the gather kernel takes all images
    // in one launch, reading only the channels a group keeps instead of staging every channel of
    // a box (32 images of 7x7, 2048 -> 512 channels: 22.4 us staged, 8.5 us gathered).
    {
        const int64_t HW = (int64_t)H * W;
        const int64_t in_total = 2 * (int64_t)batch * C_in * HW;
        // Images of four positions, us staged / gathered: 64 images, 512 -> 512 channels, V = 32: 10.3 / 6.6
        // unpruned, 7.3 / 3.7 at 75 %.  Tiles enough for every CU gain nothing from being split, and then
        // groups that keep many rows are staged: 256 images, 1024 -> 2048, 50 %, V = 32 13.1 / 19.0; 1024 of
        // 512 -> 512, 50 %, V = 32 9.1 / 11.1; 1024 of 256 -> 1024, V = 64 11.8 / 13.2 unpruned, 10.3 / 9.1 at
        // 50 %, V = 16 23.8 / 19.0 at 50 %.
        const bool dense_quads = A->V <= 64 && (N + 63) / 64 * A->G >= 1024 && 2.5 * A->nnz > (double)A->M * A->K &&
                                 A->nnz >= (int64_t)160 * A->M;
        if ((A->tune_kernel == 0 || resident_only) && layout == SHFLBW_NCHW && R == 1 && S == 1 && stride_h == 1 &&
            stride_w == 1 && pad_h == 0 && pad_w == 0 && (HW >= 8 || (HW == 4 && !dense_quads && !resident_only)) && HW * 2 < (1 << 24) &&
            C_in < (1 << 24) && in_total < ((int64_t)1 << 32) - 64) {
            if (HW >= 8)
                return run_rows(A, in, HW, (long)C_in * HW, out, HW, (long)A->M * HW, (int)HW, batch, in_total, ydtype, st);
            GeomQuads g;
            g.X = static_cast<const _Float16*>(in);
            g.Y = out;
            g.ldx = g.ldy = HW;
            g.N = (long)N;
            g.xbytes = (unsigned)in_total;
            g.stream = 0;
            g.x_image = (unsigned)(2 * (int64_t)C_in * HW);
            g.y_image = (long)A->M * HW;
            return dispatch_out(A, g, g.N, ydtype, st);
        }
    }
    // Convolutions gathered in runs of 8 along the innermost dimension: forced, chosen by runs_limit, or
    // the choice left when the staged kernel's input box does not fit the LDS.
    const double kept = (double)A->nnz / ((double)A->M * A->K);
    const bool runs_pay = kept <= runs_limit(A->V, A->G, layout == SHFLBW_CHWN, layout == SHFLBW_CHWN ? batch : Wo);
    const auto gather_runs = [&](auto& g, int* status) {
        if (!fill_conv_runs(A, g, in, out, batch, C_in, H, W, R, S, stride_h, stride_w, pad_h, pad_w, Ho, Wo,
                            2 * (int64_t)batch * C_in * H * W, ydtype == SHFLBW_F32 ? 4 : 2))
            return false;
        *status = dispatch_out(A, g, g.N, ydtype, st);
        return true;
    };
    const auto try_runs = [&](int* status) {
        GeomConvRuns<true> chwn;
        GeomConvRuns<false> nchw;
        return layout == SHFLBW_CHWN ? gather_runs(chwn, status) : gather_runs(nchw, status);
    };
    int status = SHFLBW_OK;
    // the unfolded matrix resident in the LDS, 64 columns of it per workgroup
    const auto try_resident_runs = [&](auto& g, Runs runs) {
        const int64_t ybytes = 2 * (int64_t)A->M * N;
        if (!resident_only && !resident_conv_worth_a_look(A->V, A->K, (g.N + 63) / 64 * A->G)) return false;
        if (A->V > 32 || g.out_pitch() * 2 >= (1 << 24) || A->M >= (1 << 24) || ybytes >= ((int64_t)1 << 32) - 64) return false;
        // (stores: 4 to 7 % either way, as for linear layers)
        const bool whole = ((runs == Runs::CHWN ? batch : Wo) * 2 | (int64_t)reinterpret_cast<uintptr_t>(out)) % 64 == 0;
        const CutSizes sizes = cut_sizes(A, g.N, Rows::ANY, false);
        const ResidentPlan plan = plan_resident(sizes, whole, RESIDENT_COPY_RUNS[(int)runs]);
        if (plan.parts <= 0 || (!resident_only && !resident_conv_pays(sizes, runs, runs_pay || runs == Runs::NCHW_BY_2, plan))) return false;
        const int streams = g.stream;
        g.stream = whole;
        status = A->dtype == SHFLBW_BF16 ? run_resident_bf16(A, g, g.N, plan, (unsigned)ybytes, ydtype, st)
                                         : run_resident_f16(A, g, g.N, plan, (unsigned)ybytes, ydtype, st);
        g.stream = streams;
        return true;
    };
    GeomConvRuns2 by2;
    bool strided = false;   // by2 holds the convolution, of no more groups than the gather kernel's grid has rows (the staged kernel takes more)
    const auto gather_strided = [&] { return A->dtype == SHFLBW_BF16 ? run_gather_bf16(A, by2, by2.N, st) : run_gather_f16(A, by2, by2.N, st); };
    if (((A->tune_kernel == 0 && A->tune_tile_n == 0) || resident_only) && ydtype != SHFLBW_F32) {
        const auto fill = [&](auto& g, int step) {
            return fill_conv_runs(A, g, in, out, batch, C_in, H, W, R, S, stride_h, stride_w, pad_h, pad_w, Ho, Wo, 2 * (int64_t)batch * C_in * H * W, 2, step);
        };
        GeomConvRuns<true> chwn;
        GeomConvRuns<false> nchw;
        // (before the geometry is worked out: runs fill at most twice the columns)
        const bool look = resident_only || resident_conv_worth_a_look(A->V, A->K, (N / 32 + 1) * A->G);
        if (layout == SHFLBW_CHWN) {
            if (look && fill(chwn, 1) && try_resident_runs(chwn, Runs::CHWN)) return status;
        } else if (stride_w == 2) {
            if (fill(static_cast<GeomConvRuns<false>&>(by2), 2)) {
                if (try_resident_runs(by2, Runs::NCHW_BY_2)) return status;
                strided = A->G <= GATHER_MAX_GROUPS;
                if (!resident_only && strided && strided_runs_pay(A->V, A->G, R * S, kept, (double)((by2.N + 63) / 64) * A->total_steps()))
                    return gather_strided();
            }
        } else if (look && fill(nchw, 1) && try_resident_runs(nchw, Runs::NCHW)) {
            return status;
        }
    }
    if (resident_only) return no_resident();
    if ((A->tune_kernel == 1 || A->tune_kernel == 3 || (A->tune_kernel == 0 && runs_pay)) && try_runs(&status))
        return status;
    if (A->tune_kernel != 1 && A->tune_kernel != 3) {
        // the plan depends on the sizes below only (not on which matrix has them): keep the last one
        struct PlanKey {
            int64_t nnz;
            int K, V, M, batch, C, H, W, R, S, sh, sw, ph, pw, layout;   // no padding: compared as bytes
        };
        static_assert(sizeof(PlanKey) == 8 + 14 * 4, "compared as bytes");
        static thread_local PlanKey last_key = {};
        static thread_local bool last_ok = false;
        static thread_local ConvArgs last_args;
        static thread_local size_t last_lds = 0;
        const PlanKey key = {A->nnz, A->K, A->V, A->M, batch, C_in, H, W, R, S, stride_h, stride_w, pad_h, pad_w, (int)layout};
        if (memcmp(&key, &last_key, sizeof key) != 0) {
            last_ok = plan_conv(A, batch, C_in, H, W, R, S, stride_h, stride_w, pad_h, pad_w, Ho, Wo,
                                layout == SHFLBW_CHWN, last_args, last_lds);
            last_key = key;
        }
        if (last_ok) {
            ConvArgs ca = last_args;
            const size_t lds_bytes = last_lds;
            ca.in = static_cast<const _Float16*>(in);
            ca.out = out;
            if (reinterpret_cast<uintptr_t>(in) % 4) ca.stage_pairs = 2;   // laid out for pairs, staged with 2-byte loads
            return dispatch_conv(A, ca, lds_bytes, ydtype, st);
        }
        if (A->tune_kernel == 2)
            return fail(SHFLBW_ERR_BAD_OPTION,
                        "staged convolution kernel needs an input box that fits the LDS");
        // beyond the LDS the element-wise geometry is hundreds of times dearer than the runs (8 images of 14x14,
        // 2048 -> 128 channels, 3x3, unpruned, V = 32: 3400 us / 64)
        if (!runs_pay && try_runs(&status)) return status;
        if (strided) return gather_strided();
    }
    GeomConv g;
    g.in = static_cast<const _Float16*>(in);
    g.out = out;
    g.B = batch; g.Cin = C_in; g.H = H; g.W = W; g.Cout = A->M; g.R = R; g.S = S;
    g.sh = stride_h; g.sw = stride_w; g.ph = pad_h; g.pw = pad_w; g.Ho = Ho; g.Wo = Wo;
    g.chwn = (layout == SHFLBW_CHWN);
    g.N = N;
    return dispatch_out(A, g, (long)N, ydtype, st);
}

}  // extern "C"
