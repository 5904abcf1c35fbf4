// The choice of a kernel and a cut, for tests/test_choice.py.
#include "choice.h"

using namespace shflbw;

namespace {
CutSizes sizes_of(int V, long G, long N, long steps, int K, int rows, int uneven, int f32, int slab, double kept)
{
    CutSizes s;
    s.V = V; s.G = G; s.N = N; s.steps = steps; s.K = K;
    s.per = steps / (G > 0 ? G : 1);
    s.rows = rows == 0 ? Rows::ALIGNED : rows == 1 ? Rows::ANY : Rows::IMAGES;
    s.uneven = uneven; s.f32 = f32; s.slab = slab; s.kept = kept;
    return s;
}
}  // namespace

extern "C" int probe_choice(int V, long G, long N, long steps, int K, int rows, int uneven, int f32, int slab, double kept, int what)
{
    const CutSizes s = sizes_of(V, G, N, steps, K, rows, uneven, f32, slab, kept);
    if (what == 1) return shares_weights(V, false, s.per);
    if (what == 2) return shares_weights(V, true, s.per);
    return choose_cut(s);
}

// A linear layer (rows: as above) on the resident slab: whether it is taken; its plan and both estimates.
extern "C" int probe_resident(int V, long G, long N, long steps, int K, int rows, int uneven, int f32, int slab, double kept, int whole,
                              int* parts, int* waves, double* time, double* other)
{
    const CutSizes s = sizes_of(V, G, N, steps, K, rows, uneven, f32, slab, kept);
    const ResidentPlan plan = plan_resident(s, whole, rows == 0 ? 1 : RESIDENT_COPY_UNALIGNED);
    const Cut cut = choose_cut(s);
    *parts = plan.parts; *waves = plan.waves; *time = plan.time; *other = cut_time(s, cut);
    return resident_worth_a_look(s) && resident_pays(s, cut, whole, plan);
}

// A convolution in runs (0: NCHW, 1: CHWN, 2: NCHW with a stride of two) likewise; gathered: what it would be otherwise.
extern "C" int probe_resident_conv(int V, long G, long N, long steps, int K, int uneven, double kept, int whole, int runs, int gathered,
                                   int* parts, int* waves, double* time)
{
    const CutSizes s = sizes_of(V, G, N, steps, K, 1, uneven, 0, 0, kept);
    const ResidentPlan plan = plan_resident(s, whole, RESIDENT_COPY_RUNS[runs]);
    *parts = plan.parts; *waves = plan.waves; *time = plan.time;
    return resident_conv_worth_a_look(V, K, s.tiles()) && resident_conv_pays(s, (Runs)runs, gathered, plan);
}

// Whether a strided convolution in NCHW is gathered.
extern "C" int probe_strided(int V, long G, int taps, double kept, double work) { return strided_runs_pay(V, G, taps, kept, work); }

// The LayerNorm-side transposition: its kernel; the tokens of a workgroup, the workgroups that share them (register kernel), bytes of LDS (resident kernel).
extern "C" int probe_layernorm(long N, int K, int normalize, int stream, int* tokens, int* shares, long* bytes)
{
    const LnChoice c = choose_layernorm(N, K, normalize);
    int pitch = 0;
    *tokens = c.tokens;
    *shares = c.kernel == Ln::REGISTER ? ln_register_shares(N, K, normalize, stream) : 1;
    *bytes = c.kernel == Ln::RESIDENT ? ln_resident_bytes(c.tokens, K, pitch) : 0;
    return (int)c.kernel;
}
