// Some 64 to 1000 rows on the packed weight in one launch: the kernel (gemm_mid_kernel.h) at its taller tiles.
#include "gemm_mid_kernel.h"

namespace marlaas {

hipError_t launch_gemm_tall(const GemmArgs& a, const MidPlan& p, int cu_count, hipStream_t stream) {
  return p.rb == 6 ? launch_mid<6, 4>(a, cu_count, stream) : p.rb == 8 ? launch_mid<8, 4>(a, cu_count, stream) : p.rb == 16 ? launch_mid<16, 4>(a, cu_count, stream) : launch_mid<10, 4>(a, cu_count, stream);
}

}  // namespace marlaas
