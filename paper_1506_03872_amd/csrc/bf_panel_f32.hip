// bf_panel_f32.hip -- fp32 instances of the register-panel GEMM, one per step
// count (K rounded up to 8, above 160 to 16).
#include "bf_panel.hpp"

namespace mad {

hipError_t launch_panel_f32(const PanelArgs& a, int ns, bool hist,
                            int64_t grid, hipStream_t st) {
  switch (ns) {
#define MAD_PANEL_CASE(N) \
  case N:                 \
    return launch_panel_ns<kF32, N>(a, hist, grid, st);
    MAD_PANEL_CASE(1) MAD_PANEL_CASE(2) MAD_PANEL_CASE(3) MAD_PANEL_CASE(4)
    MAD_PANEL_CASE(5) MAD_PANEL_CASE(6) MAD_PANEL_CASE(7) MAD_PANEL_CASE(8)
    MAD_PANEL_CASE(9) MAD_PANEL_CASE(10) MAD_PANEL_CASE(11)
    MAD_PANEL_CASE(12) MAD_PANEL_CASE(13) MAD_PANEL_CASE(14)
    MAD_PANEL_CASE(15) MAD_PANEL_CASE(16) MAD_PANEL_CASE(17)
    MAD_PANEL_CASE(18) MAD_PANEL_CASE(19) MAD_PANEL_CASE(20)
    MAD_PANEL_CASE(22) MAD_PANEL_CASE(24) MAD_PANEL_CASE(26)
    MAD_PANEL_CASE(28) MAD_PANEL_CASE(30) MAD_PANEL_CASE(32)
#undef MAD_PANEL_CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace mad
