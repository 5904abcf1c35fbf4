// Launchers of the per-wavefront gather kernel, one set per operand format,
// compiled in translation units of their own so that the library builds in
// parallel.  ydtype has been checked by the caller.
#pragma once
#include <hip/hip_runtime.h>

#include "choice.h"
#include "gather_kernel.hip"
#include "shflbw_internal.h"

namespace shflbw {

constexpr int GATHER_MAX_GROUPS = 65535;   // rows of a launch's grid

// what the choice of a cut looks at
inline CutSizes cut_sizes(const shflbw_matrix* A, long N, Rows rows, bool f32)
{
    CutSizes s;
    s.V = A->V; s.G = A->G; s.N = N; s.K = A->K;
    s.steps = A->step_ptr.empty() ? 0 : A->step_ptr.back();
    s.per = s.steps / (s.G > 0 ? s.G : 1);
    s.rows = rows;
    s.uneven = A->uniform_steps < 0;
    s.f32 = f32;
    s.slab = rows == Rows::ALIGNED && A->slab_ok;
    s.kept = (double)A->nnz / ((double)A->M * A->K);
    return s;
}

int run_gather_f16(const shflbw_matrix* A, const GeomLinear<true>& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_f16(const shflbw_matrix* A, const GeomLinearBuf& g, long N, shflbw_dtype ydtype, hipStream_t stream, int cut);
int run_gather_f16(const shflbw_matrix* A, const GeomLinear<false>& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_f16(const shflbw_matrix* A, const GeomConv& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_f16(const shflbw_matrix* A, const GeomRows& g, long N, shflbw_dtype ydtype, hipStream_t stream, int cut);
int run_gather_f16(const shflbw_matrix* A, const GeomNarrow& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_f16(const shflbw_matrix* A, const GeomQuads& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_f16(const shflbw_matrix* A, const GeomConvRuns<false>& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_f16(const shflbw_matrix* A, const GeomConvRuns<true>& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_bf16(const shflbw_matrix* A, const GeomLinear<true>& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_bf16(const shflbw_matrix* A, const GeomLinearBuf& g, long N, shflbw_dtype ydtype, hipStream_t stream, int cut);
int run_gather_bf16(const shflbw_matrix* A, const GeomLinear<false>& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_bf16(const shflbw_matrix* A, const GeomConv& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_bf16(const shflbw_matrix* A, const GeomRows& g, long N, shflbw_dtype ydtype, hipStream_t stream, int cut);
int run_gather_bf16(const shflbw_matrix* A, const GeomNarrow& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_bf16(const shflbw_matrix* A, const GeomQuads& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_bf16(const shflbw_matrix* A, const GeomConvRuns<false>& g, long N, shflbw_dtype ydtype, hipStream_t stream);
int run_gather_bf16(const shflbw_matrix* A, const GeomConvRuns<true>& g, long N, shflbw_dtype ydtype, hipStream_t stream);

// 16-bit results only
int run_gather_f16(const shflbw_matrix* A, const GeomConvRuns2& g, long N, hipStream_t stream);
int run_gather_bf16(const shflbw_matrix* A, const GeomConvRuns2& g, long N, hipStream_t stream);
// the slab kernel with a resident slab (resident_kernel.hip).  ybytes: from g.Y to the end of the results
int run_resident_f16(const shflbw_matrix* A, const GeomLinearBuf& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_f16(const shflbw_matrix* A, const GeomRows& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_f16(const shflbw_matrix* A, const GeomConvRuns<false>& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_f16(const shflbw_matrix* A, const GeomConvRuns<true>& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_f16(const shflbw_matrix* A, const GeomConvRuns2& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_bf16(const shflbw_matrix* A, const GeomLinearBuf& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_bf16(const shflbw_matrix* A, const GeomRows& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_bf16(const shflbw_matrix* A, const GeomConvRuns<false>& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_bf16(const shflbw_matrix* A, const GeomConvRuns<true>& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);
int run_resident_bf16(const shflbw_matrix* A, const GeomConvRuns2& g, long N, const ResidentPlan& plan, unsigned ybytes, shflbw_dtype ydtype, hipStream_t stream);

}  // namespace shflbw
