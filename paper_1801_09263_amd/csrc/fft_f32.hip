// fft_f32.hip - the FFT and pair kernels of one precision.
#define LACE_FFT_T float
#include "fft_kernels.hip"
