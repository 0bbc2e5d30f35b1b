// Lane exchanges on the vector ALU (device code for gfx950 only: the host build of
// the rotation kernel's emulation includes dev.h, not this).
#pragma once

#include "dev.h"

namespace fmm {

// Lane exchanges inside a row of 16 lanes by DPP.
constexpr int DPP_ROW_ROR = 0x120;      // + n: rotate the row right by n lanes
constexpr int DPP_ROW_SHR = 0x110;      // + n: from n lanes below in the row
constexpr int DPP_BCAST15 = 0x142;      // the last lane of a row to the next row
constexpr int DPP_BCAST31 = 0x143;      // lane 31 to lanes 32 .. 63

template <int CTRL>
__device__ __forceinline__ int dpp_int(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}

template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
    return __hiloint2double(dpp_int<CTRL>(__double2hiint(v)), dpp_int<CTRL>(__double2loint(v)));
}

}  // namespace fmm
