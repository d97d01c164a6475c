// Arithmetic that the kernels share, compiled for the host from the kernels' own headers:
// each function returns what a kernel's lanes would compute.
#include "twiddle.h"

using namespace purify;

namespace {
// the twiddles of every butterfly k of one radix-R pass over blocks of NS: out[k][r - 1]
template <int LOGN, int R, int NS>
void pass(const cpx<float>* W, cpx<float>* out) {
    for (int k = 0; k < NS; ++k)
        twiddles<float, LOGN, R, (1 << LOGN) / (NS * R)>(W, k, [&](int r, cpx<float> w) { out[k * (R - 1) + r - 1] = w; });
}
template <int LOGN>
void stage(const cpx<float>* tw, cpx<float>* W) {
    for (int i = 0; i < twiddle_entries<float, LOGN>(); ++i) W[i] = tw[twiddle_entry<float, LOGN>(i)];
}
}  // namespace

extern "C" {

// tw: the n-entry table; out: passes of the FP32 line's plan after the first, one after another
void line_twiddles_1024(const cpx<float>* tw, cpx<float>* out) {
    static cpx<float> W[1024];
    stage<10>(tw, W);
    pass<10, 8, 8>(W, out);
    pass<10, 16, 64>(W, out + 7 * 8);
}
void line_twiddles_2048(const cpx<float>* tw, cpx<float>* out) {
    static cpx<float> W[2048];
    stage<11>(tw, W);
    pass<11, 16, 32>(W, out);
    pass<11, 4, 512>(W, out + 15 * 32);
}
void line_twiddles_4096(const cpx<float>* tw, cpx<float>* out) {
    static cpx<float> W[4096];
    stage<12>(tw, W);
    pass<12, 8, 8>(W, out);
    pass<12, 8, 64>(W, out + 7 * 8);
    pass<12, 8, 512>(W, out + 7 * 72);
}

}  // extern "C"
