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
// out[i][a]: tap a at fraction f[i], from coefficients c[a][k]
template <int J>
void taps(const float* c, const float* f, int count, float* out) {
    for (int i = 0; i < count; ++i) kb_weights<float, J>(c, f[i], out + i * J);
}
}  // namespace

extern "C" {

void kb_taps(int J, const float* c, const float* f, int count, float* out) {
    switch (J) {
        case 4: taps<4>(c, f, count, out); break;
        case 5: taps<5>(c, f, count, out); break;
        case 6: taps<6>(c, f, count, out); break;
        case 7: taps<7>(c, f, count, out); break;
        default: taps<8>(c, f, count, out); break;
    }
}
// the same taps, two at a time
void kb_tap_pairs(int J, const float* c, const float* f, int count, float* out) {
    for (int i = 0; i < count; ++i)
        for (int q = 0; q < (J + 1) / 2; ++q) {
            float l, h;
            kb_pair<float>(c + q * (KBDeg<float>::value + 1), f[i] - 0.5f, l, h);
            out[i * J + J - 1 - q] = h;
            out[i * J + q] = l;
        }
}

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
