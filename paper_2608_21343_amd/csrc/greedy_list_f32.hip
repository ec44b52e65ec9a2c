// Greedy kernels from row summaries for float32 logits (greedy_list.hpp).
#include "greedy_list.hpp"

namespace tbias {
namespace glist {

Launch launcher_f32(int32_t V1) { return launcher_t<LoadF32>(V1); }

}  // namespace glist
}  // namespace tbias
