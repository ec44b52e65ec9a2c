// Beam kernels for float32 logits (beam_list.hpp, beam_rows.hpp).
#include "beam_rows.hpp"

namespace tbias {
namespace blist {

RowsLaunch rows_launcher_f32(int32_t V1) { return rows_launcher_t<LoadF32>(V1); }
StepLaunch step_launcher_f32(int32_t K, bool stream, bool rows) {
  return stream ? step_launcher_s<LoadF32, true>(K, rows) : step_launcher_s<LoadF32, false>(K, rows);
}

}  // namespace blist
}  // namespace tbias
