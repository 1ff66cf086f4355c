// gemm_panel_kernel for tiles of up to 64 rows.
#include "gemm_panel.h"

template <>
void qdp::launch_panel<1>(const GemmArgs &p, int epi, const PnDeal &deal, int grid,
                          int ns, int dense, int lds, hipStream_t s) {
  if (epi == QD_EPI_SWIGLU) launch_panel_epi<1, QD_EPI_SWIGLU>(p, deal, grid, ns, dense, lds, s);
  else launch_panel_epi<1, QD_EPI_NONE>(p, deal, grid, ns, dense, lds, s);
}
