// Split-point metadata unpacking on the device (Sec. 4.3). The two series have
// fixed-width entries, so split point k's entries sit at a computable bit
// position. The blocks have data-dependent widths, so each block's bit offset is
// handed in (recorded when the section is packed or checked on the host). W lanes
// per output unit (two units per wave at W = 32): lane j reads lane j's state and
// group difference, the lanes reduce the differences to the unit's synchronisation
// group, which also gives the lowest group of the unit above, so every split point
// is read once.
//
// Bound by latency: three dependent rounds of reads (block offset, width, differences)
// and a launch. Each field is one unaligned 8-byte load. 16384 units at W = 32: 13.7 us
// with a wave per unit, five byte loads per field and every split point read twice, now
// 6.6 us.
#include "unpack.hpp"

namespace recoil {
namespace {

constexpr uint32_t kThreads = 256;

// `w` (1..33) bits at bit position `pos`, most significant bit first (reads 8 bytes).
__device__ inline uint64_t bits_at(const uint8_t *p, uint64_t pos, uint32_t w) {
    uint64_t v;
    __builtin_memcpy(&v, p + (pos >> 3), 8);
    v = __builtin_bswap64(v);
    return (v >> (64u - (uint32_t)(pos & 7) - w)) & ((1ull << w) - 1);
}

// Entry k of a signed series of magnitude width w whose entries start at bit `at`.
__device__ inline int64_t series_entry(const uint8_t *p, uint64_t at, uint32_t w, uint64_t k) {
    const uint64_t v = bits_at(p, at + k * (1 + w), 1 + w);
    const int64_t m = (int64_t)(v & ((1ull << w) - 1));
    return v >> w ? -m : m;
}

template <uint32_t W>
__global__ __launch_bounds__(kThreads) void unpack_units(UnpackParams p) {
    const uint32_t u = blockIdx.x * (kThreads / W) + threadIdx.x / W;
    const uint32_t j = threadIdx.x % W;
    if (u >= p.units) return;                      // all lanes of a unit leave together
    const uint64_t gtop = p.groups ? p.groups - 1 : 0;
    uint32_t next, top, ghi, word;
    if (u + 1 == p.units) {
        next = (uint32_t)p.words;
        top = (uint32_t)gtop;
        ghi = top;
        word = p.final_states[j];
    } else {
        const uint64_t k = (uint64_t)(u + 1) * p.step - 1;
        const uint64_t bb = p.block_bit[k];
        const int64_t o = (int64_t)((k + 1) * p.eb) + series_entry(p.bits, p.offset_at, p.offset_width, k);
        const int64_t x = (int64_t)((k + 1) * p.eg) + series_entry(p.bits, p.group_at, p.group_width, k) - 1;
        const uint32_t wd = (uint32_t)bits_at(p.bits, bb + 16ull * W, 4) + 1;
        const uint32_t state = (uint32_t)bits_at(p.bits, bb + 16ull * j, 16);
        const uint32_t d = (uint32_t)bits_at(p.bits, bb + 16ull * W + 4 + (uint64_t)j * wd, wd);
        uint32_t most = d;
#pragma unroll
        for (int i = W / 2; i > 0; i >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, i, 64));
        // Anchor group, clamped to the stream, and the group at which all lanes are on.
        next = (uint32_t)min<int64_t>(max<int64_t>(o, 0), (int64_t)p.words);
        top = (uint32_t)min<int64_t>(max<int64_t>(x, 0), (int64_t)gtop);
        ghi = top - min(most, top);
        word = state | (d << 16);
    }
    p.lanes[(uint64_t)u * W + j] = word;
    if (j == 0) {
        UnitMeta *m = p.meta + u;
        m->next = next;
        m->top = top;
        m->ghi = ghi;
        if (u == 0) m->glo = 0;
        if (u + 1 < p.units) m[1].glo = ghi + 1;
    }
}

}  // namespace

hipError_t launch_unpack(const UnpackParams &p, hipStream_t stream) {
    if (p.units == 0) return hipSuccess;
    const uint32_t per_block = kThreads / p.lanes_per_unit;
    const dim3 blocks((p.units + per_block - 1) / per_block), threads(kThreads);
    if (p.lanes_per_unit == 32) hipLaunchKernelGGL(unpack_units<32>, blocks, threads, 0, stream, p);
    else hipLaunchKernelGGL(unpack_units<64>, blocks, threads, 0, stream, p);
    return hipGetLastError();
}

}  // namespace recoil
