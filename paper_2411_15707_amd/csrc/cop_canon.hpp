// Shared by the two kernels on the canonical layout (cop_canon.hip, cop_canon32.hip).
#pragma once
#include "cop_mfma_common.hpp"

namespace nimbus {

struct CanonArgs {
    MfmaArgs e;               // sizes, tile mapping, OFFX and the epilogue's constants
    const uint64_t *X;        // [m][k]
    const uint64_t *ctW;      // [k][C]
    int k;
    LimbTable limbs;          // reduction of the column sums
};

// the kernel with 32 k a stage (cop_canon32.hip)
template <int DX, int DQ>
hipError_t launch_cop_canon32(const Problem &p, const CanonArgs &ca, bool centre, hipStream_t stream);

}  // namespace nimbus
