// Decode launches of few runs: one run per workgroup, decoded by its first wave (see
// few_core.hpp); the other waves only stage the decode table, while the first one
// fetches its records and its first words.
#include "few.hpp"

#include "few_core.hpp"

namespace recoil {

namespace {

using namespace dev;

constexpr uint32_t kThreads = 256;
constexpr uint32_t kLdsBytes = 160u << 10;   // per CU
// Groups of a run from which super-steps of 16 groups pay: 8-group ones round a run up by
// less and start sooner (1 MiB at W = 32 in 256 units, 128 groups each: 12.9 against
// 14.4 us), 16-group ones cost less per group (64 MiB in 256 units, 8192 groups each: 547
// against 614 us).
constexpr uint32_t kLongRun = 256;

template <typename Sym, bool WIDE>
__device__ inline void stage_table(const DecodeParams &p, uint32_t lut, uint32_t tid) {
    constexpr uint32_t kStagers = kThreads - 64;
    const u32x4 *src = static_cast<const u32x4 *>(p.lut);
    const uint32_t chunks = p.lut_bytes / 16;
#pragma unroll 6
    for (uint32_t i = tid; i < chunks; i += kStagers) {
        const u32x4 v = src[i];
        if constexpr (sizeof(Sym) == 1 && !WIDE) {
            // symbol | f << 8 | (slot - F) << 20  ->  {f | symbol << 24, slot - F}
            const u32x4 lo = {((v.x >> 8) & 0xFFFu) | (v.x << 24), v.x >> 20, ((v.y >> 8) & 0xFFFu) | (v.y << 24), v.y >> 20};
            const u32x4 hi = {((v.z >> 8) & 0xFFFu) | (v.z << 24), v.z >> 20, ((v.w >> 8) & 0xFFFu) | (v.w << 24), v.w >> 20};
            lds_st<u32x4>(lut + 32 * i, lo);
            lds_st<u32x4>(lut + 32 * i + 16, hi);
        } else {
            lds_st<u32x4>(lut + 16 * i, v);
        }
    }
}

template <typename Sym, bool WIDE>
__host__ __device__ inline uint32_t table_bytes(uint32_t lut_bytes) {
    return sizeof(Sym) == 1 && !WIDE ? 2 * lut_bytes : lut_bytes;
}

template <int W, typename Sym, int K, int NCH, bool WIDE, bool COUNT>
__global__ __launch_bounds__(kThreads) void decode_few_runs(DecodeParams p) {
    using D = FewDecoder<W, Sym, K, NCH, WIDE, COUNT>;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lut = lds_addr(smem);
    D d(p, lut, lut + table_bytes<Sym, WIDE>(p.lut_bytes), threadIdx.x & (W - 1u));
    uint32_t v[D::FILL][D::D];
    const uint32_t wave = uni(threadIdx.x >> 6);
    if (wave == 0) {
        d.records(blockIdx.x);
        d.fill_request(v);
    } else {
        stage_table<Sym, WIDE>(p, lut, threadIdx.x - 64);
    }
    __syncthreads();
    if (wave != 0) return;                              // the stagers
    if (W < 64 && (threadIdx.x & 63u) >= W) return;     // lanes without a coder
    d.fill_put(v);
    d.run();
}

template <int W, typename Sym, int K, int NCH, bool WIDE, bool COUNT>
bool try_launch(const DecodeParams &p, bool launch, hipStream_t stream, hipError_t *e) {
    const uint32_t lds = table_bytes<Sym, WIDE>(p.lut_bytes) + FewDecoder<W, Sym, K, NCH, WIDE, COUNT>::RING_BYTES;
    const uint32_t cus = (uint32_t)device_cus(), per_cu = (p.runs + cus - 1) / cus;
    if (lds * per_cu > kLdsBytes) return false;
    if (launch) {
        hipLaunchKernelGGL((decode_few_runs<W, Sym, K, NCH, WIDE, COUNT>), dim3(p.runs), dim3(kThreads), lds, stream, p);
        *e = hipGetLastError();
    }
    return true;
}

// The largest rings that leave every run resident (a run that has to wait for another
// doubles the launch): with 32 KiB of table (8-byte entries at n = 12) four runs per CU
// have 8 KiB each, the 4-group rings.
template <int W, typename Sym, bool WIDE, bool COUNT>
bool pick(const DecodeParams &p, bool launch, hipStream_t stream, hipError_t *e) {
    const uint64_t groups = p.n_symbols / W / p.runs;   // of a run
    if (groups >= kLongRun && try_launch<W, Sym, 16, 3, WIDE, COUNT>(p, launch, stream, e)) return true;
    return try_launch<W, Sym, 8, 3, WIDE, COUNT>(p, launch, stream, e) ||
           try_launch<W, Sym, 4, 3, WIDE, COUNT>(p, launch, stream, e);
}

template <int W, typename Sym>
bool pick_variant(const DecodeParams &p, bool launch, hipStream_t stream, hipError_t *e) {
    if (p.quant_bits > 12) return !p.counts && pick<W, Sym, true, false>(p, launch, stream, e);
    return p.counts ? pick<W, Sym, false, true>(p, launch, stream, e) : pick<W, Sym, false, false>(p, launch, stream, e);
}

}  // namespace

bool decode_few(const DecodeParams &p, uint32_t lanes, uint32_t symbol_bytes, bool launch, hipStream_t stream,
                hipError_t *e) {
    if (p.tidx || p.runs == 0) return false;
    if (lanes == 32) return symbol_bytes == 1 ? pick_variant<32, uint8_t>(p, launch, stream, e)
                                              : pick_variant<32, uint16_t>(p, launch, stream, e);
    if (lanes == 64) return symbol_bytes == 1 ? pick_variant<64, uint8_t>(p, launch, stream, e)
                                              : pick_variant<64, uint16_t>(p, launch, stream, e);
    return false;
}

}  // namespace recoil
