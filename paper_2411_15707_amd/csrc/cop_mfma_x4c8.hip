// the tile kernel's instances for four share planes and eight ciphertext planes
#include "cop_mfma_kernel.hpp"

namespace nimbus {

template hipError_t mfma_impl<4, 8>(const Problem &, int, const void *const *, const void *const *,
                                    const uint64_t *const *, const uint64_t *, uint64_t *const *, hipStream_t);

}  // namespace nimbus
