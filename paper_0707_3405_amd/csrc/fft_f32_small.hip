// H.X passes, float, the small FFT sizes.
#include "fft_apply.h"

namespace pw {

bool run_apply_small(const ApplyItems<float> &items, int nk, const float *v, int nb, hipStream_t st) {
    switch (items.it[0].sp.n) {
#define PW_CASE(NN)                                 \
    case NN:                                        \
        run_apply<NN, float>(items, nk, v, nb, st); \
        return true;
        PW_FFT_SIZES_SMALL(PW_CASE)
#undef PW_CASE
        default:
            return false;
    }
}

}  // namespace pw
