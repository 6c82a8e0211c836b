// Launcher of the decode for few runs (few.hip).
#pragma once

#include "decode.hpp"

namespace recoil {

struct FewShape {
    uint32_t cus;             // the device's compute units (set by the caller)
    uint32_t blocks, waves;   // workgroups, decoding waves of each
};

// True if p's runs are few enough for that kernel and fit the chip's LDS all at once, in
// workgroups of `waves` decoding waves (0: any), at most blocks_per_cu of them per CU (0: no
// cap); with launch set it is launched, and *e receives the launch error. shape receives the
// grid.
bool decode_few(const DecodeParams &p, uint32_t lanes, uint32_t symbol_bytes, uint32_t waves, uint32_t blocks_per_cu,
                FewShape &shape, bool launch, hipStream_t stream, hipError_t *e);

}  // namespace recoil
