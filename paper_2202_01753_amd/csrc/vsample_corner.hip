// Sampling-kernel instantiations for integrand id 2 (corner).
#include "vsample.hpp"

namespace mcubes {

const void *sample_kernel_f2(int dim, int kind, bool fp32) {
    switch (dim) {
    case 1: return sample_kernel_fd<2, 1>(kind, fp32);
    case 2: return sample_kernel_fd<2, 2>(kind, fp32);
    case 3: return sample_kernel_fd<2, 3>(kind, fp32);
    case 4: return sample_kernel_fd<2, 4>(kind, fp32);
    case 5: return sample_kernel_fd<2, 5>(kind, fp32);
    case 6: return sample_kernel_fd<2, 6>(kind, fp32);
    case 7: return sample_kernel_fd<2, 7>(kind, fp32);
    case 8: return sample_kernel_fd<2, 8>(kind, fp32);
    case 9: return sample_kernel_fd<2, 9>(kind, fp32);
    case 10: return sample_kernel_fd<2, 10>(kind, fp32);
    case 11: return sample_kernel_fd<2, 11>(kind, fp32);
    case 12: return sample_kernel_fd<2, 12>(kind, fp32);
    case 13: return sample_kernel_fd<2, 13>(kind, fp32);
    case 14: return sample_kernel_fd<2, 14>(kind, fp32);
    case 15: return sample_kernel_fd<2, 15>(kind, fp32);
    case 16: return sample_kernel_fd<2, 16>(kind, fp32);
    default: return nullptr;
    }
}

}  // namespace mcubes
