// Launcher of the decode for few runs (few.hip).
#pragma once

#include "decode.hpp"

namespace recoil {

// True if a decode of p's runs (one per workgroup, all resident at once) fits the chip's
// LDS; with launch set it is launched, and *e receives the launch error.
bool decode_few(const DecodeParams &p, uint32_t lanes, uint32_t symbol_bytes, bool launch, hipStream_t stream,
                hipError_t *e);

}  // namespace recoil
