// Instantiations of the FFT line kernel: MN_T, MN_V (values per thread) and
// MN_TAB (a batch's table of passes), in the three forms of a pass.
#include "fft_kernels.h"

namespace mn {
namespace fft {

template <typename T, int V, bool TAB>
hipError_t launch(int form, const FftPass &p, const FftPass *tab, int ntab, long long tiles, int threads,
                  int lds, const void *src, void *dst, hipStream_t s)
{
    using C = typename Cplx<T>::type;
    auto k = form == kWhole ? k_fft_lines<T, V, kWhole, TAB>
             : form == kCutOut ? k_fft_lines<T, V, kCutOut, TAB>
                               : k_fft_lines<T, V, kPadIn, TAB>;
    if (lds > 65536)
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    hipLaunchKernelGGL(k, dim3((unsigned)tiles), dim3(threads), lds, s, p, tab, ntab,
                       (const C *)src, (C *)dst);
    return hipGetLastError();
}

template hipError_t launch<MN_T, MN_V, MN_TAB>(int, const FftPass &, const FftPass *, int, long long,
                                               int, int, const void *, void *, hipStream_t);

}  // namespace fft
}  // namespace mn
