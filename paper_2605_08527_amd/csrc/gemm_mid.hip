// Some 64 to 1000 rows on the packed weight in one launch: the kernel (gemm_mid_kernel.h) at its four smaller tiles.
#include "gemm_mid_kernel.h"

namespace marlaas {

hipError_t launch_gemm_mid(GemmArgs a, const MidPlan& p, int cu_count, hipStream_t stream) {
  // How far apart neighbouring column tiles start (see MD_T): eight of them over the whole contraction, as long
  // as the part of x between the first and the last stays in an XCD's L2 (256 rows, 14336 x 4096 in one
  // split: 81 us over 1.4 MB of x, 91 over all of it).
  const int64_t kt = 32 * (MD_WAVES / p.wn), nt = ((a.Kc + kt - 1) / kt + p.ksplit - 1) / p.ksplit, window = (1400 << 10) / (a.T * kt * 2);
  a.rot = (int)((nt < window ? nt : window) / 8);
  a.ksplit = p.ksplit;
  a.tiles_m = p.tiles_m;
  a.tiles_n = 0;
  for (int q = 0; q < a.n_proj; ++q) {
    a.proj[q].tile0 = a.tiles_n;
    a.tiles_n += (int)((a.proj[q].Nout + 32 * p.wn - 1) / (32 * p.wn));
  }
  const int64_t consumers = (int64_t)p.tiles_m * a.tiles_n * p.ksplit, jobs = (int64_t)a.n_proj * a.proj_jobs;
  a.n_split = mid_u_splits(a.Kc, a.T * a.r_stride * a.n_proj, MID_U_FLOATS, consumers, jobs, cu_count, p.rb);
  a.n_prod = (int)((jobs * a.n_split + 7) / 8 * 8);
  if (p.rb > 5) return launch_gemm_tall(a, p, cu_count, stream);
  if (p.wn == 4) return p.rb == 4 ? launch_mid<4, 4>(a, cu_count, stream) : launch_mid<5, 4>(a, cu_count, stream);
  return p.rb == 4 ? launch_mid<4, 2>(a, cu_count, stream) : launch_mid<5, 2>(a, cu_count, stream);
}

}  // namespace marlaas
