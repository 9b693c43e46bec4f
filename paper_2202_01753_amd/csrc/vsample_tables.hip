// Sampling-kernel instantiations for integrand id 3 (tables).
#include "vsample.hpp"

namespace mcubes {

const void *sample_kernel_f3(int dim, int kind, bool fp32) {
    switch (dim) {
    case 4: return sample_kernel_fd<3, 4>(kind, fp32);
    case 5: return sample_kernel_fd<3, 5>(kind, fp32);
    case 6: return sample_kernel_fd<3, 6>(kind, fp32);
    case 7: return sample_kernel_fd<3, 7>(kind, fp32);
    case 8: return sample_kernel_fd<3, 8>(kind, fp32);
    case 9: return sample_kernel_fd<3, 9>(kind, fp32);
    case 10: return sample_kernel_fd<3, 10>(kind, fp32);
    case 11: return sample_kernel_fd<3, 11>(kind, fp32);
    case 12: return sample_kernel_fd<3, 12>(kind, fp32);
    case 13: return sample_kernel_fd<3, 13>(kind, fp32);
    case 14: return sample_kernel_fd<3, 14>(kind, fp32);
    case 15: return sample_kernel_fd<3, 15>(kind, fp32);
    case 16: return sample_kernel_fd<3, 16>(kind, fp32);
    default: return nullptr;
    }
}

}  // namespace mcubes
