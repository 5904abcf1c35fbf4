// The choice of a kernel and a cut, for tests/test_choice.py.
#include "choice.h"

using namespace shflbw;

extern "C" int probe_choice(int V, long G, long N, long steps, int K, int rows, int uneven, int f32, int slab, double kept, int what)
{
    CutSizes s;
    s.V = V; s.G = G; s.N = N; s.steps = steps; s.K = K;
    s.per = steps / (G > 0 ? G : 1);
    s.rows = rows == 0 ? Rows::ALIGNED : rows == 1 ? Rows::ANY : Rows::IMAGES;
    s.uneven = uneven; s.f32 = f32; s.slab = slab; s.kept = kept;
    if (what == 1) return shares_weights(V, false, s.per);
    if (what == 2) return shares_weights(V, true, s.per);
    return choose_cut(s);
}
