// Greedy kernels from row summaries for bfloat16 logits (greedy_list.hpp).
#include "greedy_list.hpp"

namespace tbias {
namespace glist {

Launch launcher_bf16(int32_t V1) { return launcher_t<LoadBF16>(V1); }

}  // namespace glist
}  // namespace tbias
