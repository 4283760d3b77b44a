// fft_f64.hip - the FFT and pair kernels of one precision.
#define LACE_FFT_T double
#include "fft_kernels.hip"
