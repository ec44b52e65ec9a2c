// Beam kernels for bfloat16 logits (beam_list.hpp, beam_rows.hpp).
#include "beam_rows.hpp"

namespace tbias {
namespace blist {

RowsLaunch rows_launcher_bf16(int32_t V1) { return rows_launcher_t<LoadBF16>(V1); }
StepLaunch step_launcher_bf16(int32_t K, bool stream, bool rows) {
  return stream ? step_launcher_s<LoadBF16, true>(K, rows) : step_launcher_s<LoadBF16, false>(K, rows);
}

}  // namespace blist
}  // namespace tbias
