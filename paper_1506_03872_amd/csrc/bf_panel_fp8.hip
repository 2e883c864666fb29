// bf_panel_fp8.hip -- fp8 instances of the register-panel GEMM, one per even
// step count (K rounded up to 64).
#include "bf_panel.hpp"

namespace mad {

hipError_t launch_panel_fp8(const PanelArgs& a, int ns, bool hist,
                            int64_t grid, hipStream_t st) {
  switch (ns) {
#define MAD_PANEL_CASE(N) \
  case N:                 \
    return launch_panel_ns<kFP8, N>(a, hist, grid, st);
    MAD_PANEL_CASE(2) MAD_PANEL_CASE(4) MAD_PANEL_CASE(6) MAD_PANEL_CASE(8)
    MAD_PANEL_CASE(10) MAD_PANEL_CASE(12) MAD_PANEL_CASE(14)
    MAD_PANEL_CASE(16)
#undef MAD_PANEL_CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace mad
