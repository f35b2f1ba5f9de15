// Fused decode kernel instances: bf16 weights, head_dim 128, 8 query heads per kv head.
#include "ff_fused.h"
namespace ff {
hipError_t launch_solo_bf16_hd128_g8(const FusedLaunch& a, const char** what) { return launch_solo_instance<W_BF16, 128, 8>(a, what); }
}  // namespace ff
