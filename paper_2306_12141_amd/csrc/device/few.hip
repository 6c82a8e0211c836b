// Decode launches of few runs (see few_core.hpp). Up to one run per SIMD: a workgroup per
// run, decoded by its first wave and supplied with looked-up words by its second; all but
// the first stage the decode table, while the first one fetches its records and its first
// words. Up to two per SIMD: a workgroup per CU, whose waves share one table.
//
// The decoding wave has the higher priority: with four runs on a CU its SIMD also runs
// another run's helper, which has time (n = 16, 64 MiB at W = 32 in 1024 units: 189 us
// without, 176 us with; in 512 units at n = 12 210 and 201 us). A run's first wave decodes:
// on a CU the first waves of workgroups start on different SIMDs; decoding waves chosen by
// block number met on one (64 MiB at W = 32 in 1024 units: 236 us).
#include "few.hpp"

#include "few_core.hpp"

namespace recoil {

namespace {

using namespace dev;

constexpr uint32_t kLdsBytes = 160u << 10;   // per CU
constexpr uint32_t kSimds = 4;               // per CU
// Groups of a run from which super-steps of 16 groups pay: 8-group ones round a run up by
// less and start sooner, 16-group ones cost less per group. 256 runs of bytes at W = 32 with
// 8- and 16-group super-steps: of 128 groups 10.7 and 11.4 us, 192 14.1 and 13.8, 256 17.2
// and 16.5, 512 30.4 and 28.3; at n = 16, where a super-step does more, of 128 groups 15.8 and
// 16.4, 192 21.1 and 21.4, 256 26.6 and 26.6, 512 48.4 and 47.2. One line for both, at what the
// second needs: one-level tables lose 1 to 4 % between 160 and 255 groups.
constexpr uint32_t kLongRun = 256;
constexpr int kRing = 3;                     // chunks of a ring

// Decoding waves of a workgroup, whether each has a helper, and its threads. In shared
// workgroups the waves of all runs meet at once, the helpers of 32-lane runs keep half
// their lanes idle and those of wide tables take two reads per word, so that only 64-lane
// runs on one-level tables gain (without and with helpers, 64 MiB of bytes or 32 Mi 16-bit
// symbols, four streams in turn: W = 64, 2048 units 56.3 and 52.2 us, 16-bit 39.4 and 38.4 us,
// 1100 units 86.3 and 76.0 us; one stream: W = 64, n = 16, 2048 units 80.4 and 83.2 us;
// W = 32, 2048 units 81.5 and 86.5 us, n = 16 131.5 and 134.6 us). A stream that the caches
// still hold loses a little at the far end: one of 64 MiB in 2048 units 48.0 and 49.9 us.
constexpr int kShared = 8;
template <int W, bool WIDE, int WAVES>
constexpr bool kHelp = WAVES == 1 || (W == 64 && !WIDE);
template <int W, bool WIDE, int WAVES>
constexpr uint32_t kThreads = WAVES == 1 ? 256 : 64 * WAVES * (kHelp<W, WIDE, WAVES> ? 2 : 1);

template <typename Sym, bool WIDE>
__device__ inline void stage_table(const DecodeParams &p, uint32_t lut, uint32_t tid, uint32_t threads) {
    const u32x4 *src = static_cast<const u32x4 *>(p.lut);
    const uint32_t chunks = p.lut_bytes / 16;
#pragma unroll 6
    for (uint32_t i = tid; i < chunks; i += threads) {
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

template <int W, typename Sym, int K, bool WIDE, bool COUNT, int WAVES>
__global__ __launch_bounds__((kThreads<W, WIDE, WAVES>)) void decode_few_runs(DecodeParams p) {
    constexpr bool HELP = kHelp<W, WIDE, WAVES>;
    using D = FewDecoder<W, Sym, K, kRing, WIDE, COUNT, HELP>;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lut = lds_addr(smem);
    const uint32_t wave = uni(threadIdx.x >> 6);
    const bool helps = HELP && wave >= WAVES;
    const uint32_t slot = helps ? wave - WAVES : wave;
    const uint32_t run = blockIdx.x + slot * gridDim.x;
    const bool works = slot < WAVES && run < p.runs;
    D d(p, lut, lut + table_bytes<Sym, WIDE>(p.lut_bytes) + slot * D::RING_BYTES, threadIdx.x & (W - 1u));
    uint32_t v[D::FILL][D::D];
    if (works) {
        d.records(run);
        d.fill_request(v, helps);
    }
    if (WAVES > 1) stage_table<Sym, WIDE>(p, lut, threadIdx.x, kThreads<W, WIDE, WAVES>);
    else if (wave > 0) stage_table<Sym, WIDE>(p, lut, threadIdx.x - 64, kThreads<W, WIDE, WAVES> - 64);
    __syncthreads();
    if (!works) return;     // (s_barrier does not wait for waves that have ended)
    if (W < 64 && (threadIdx.x & 63u) >= W) return;     // lanes without a coder
    d.fill_put(v, helps);
    if (helps) {
        d.supply();
    } else {
        if (HELP) __builtin_amdgcn_s_setprio(3);
        d.run();
    }
}

template <int W, typename Sym, int K, bool WIDE, bool COUNT, int WAVES>
bool try_launch(const DecodeParams &p, const FewShape &shape, bool launch, hipStream_t stream, hipError_t *e) {
    const uint32_t lds = table_bytes<Sym, WIDE>(p.lut_bytes) + WAVES * FewDecoder<W, Sym, K, kRing, WIDE, COUNT, kHelp<W, WIDE, WAVES>>::RING_BYTES;
    const uint32_t per_cu = (shape.blocks + shape.cus - 1) / shape.cus;
    if (lds * per_cu > kLdsBytes) return false;
    if (launch) {
        hipLaunchKernelGGL((decode_few_runs<W, Sym, K, WIDE, COUNT, WAVES>), dim3(shape.blocks), dim3((kThreads<W, WIDE, WAVES>)), lds,
                           stream, p);
        *e = hipGetLastError();
    }
    return true;
}

// The largest rings that leave every run resident (a run that has to wait for another
// doubles the launch): with 32 KiB of table (8-byte entries at n = 12) four runs per CU in
// workgroups of their own have 8 KiB each, the 4-group rings.
template <int W, typename Sym, bool WIDE, bool COUNT, int WAVES>
bool pick(const DecodeParams &p, const FewShape &shape, bool launch, hipStream_t stream, hipError_t *e) {
    const uint64_t groups = p.n_symbols / W / p.runs;   // of a run
    if (groups >= kLongRun && try_launch<W, Sym, 16, WIDE, COUNT, WAVES>(p, shape, launch, stream, e)) return true;
    return try_launch<W, Sym, 8, WIDE, COUNT, WAVES>(p, shape, launch, stream, e) ||
           try_launch<W, Sym, 4, WIDE, COUNT, WAVES>(p, shape, launch, stream, e);
}

template <int W, typename Sym, bool WIDE, bool COUNT>
bool pick_waves(const DecodeParams &p, const FewShape &shape, bool launch, hipStream_t stream, hipError_t *e) {
    return shape.waves == 1 ? pick<W, Sym, WIDE, COUNT, 1>(p, shape, launch, stream, e)
                            : pick<W, Sym, WIDE, COUNT, kShared>(p, shape, launch, stream, e);
}

template <int W, typename Sym>
bool pick_variant(const DecodeParams &p, const FewShape &shape, bool launch, hipStream_t stream, hipError_t *e) {
    if (p.quant_bits > 12) return !p.counts && pick_waves<W, Sym, true, false>(p, shape, launch, stream, e);
    return p.counts ? pick_waves<W, Sym, false, true>(p, shape, launch, stream, e)
                    : pick_waves<W, Sym, false, false>(p, shape, launch, stream, e);
}

// Groups of a run from which shared workgroups pay where the shape is left open: a CU's eight
// rings and its table are filled before the first group, so a short run is faster on the
// throughput kernel. Time against that kernel's (replayed graphs, streams in turn):
//   bytes, W = 64     2048 runs of 24, 48, 72, 128 groups 1.21, 1.07, 0.99, 0.93; 1500 runs 1.09,
//                     1.02, 0.95, 0.87; 1100 runs 1.00, 0.94, 0.90, 0.84
//   16-bit, W = 64    2048 runs 1.23, 1.03, 0.99, 0.95; 1100 runs 1.11, 0.98, 0.91, 0.86
//   16-bit, W = 32    2048 runs 1.13, 1.09, 1.01, 0.99; 1100 runs 1.05, 0.99, 0.98, 0.97
//   n = 16, W = 32    2048 runs of 24, 72, 112, 160 groups 1.17, 1.08, 1.03, 0.97; 1100 runs 1.07,
//                     1.01, 0.98, 0.95
//   n = 16, bytes, W = 64  2048 runs 1.30, 1.09, 1.01, 0.98; 1100 runs 1.10, 1.05, 1.00, 0.95
//   n = 16, 16-bit, W = 64 2048 runs of 24, 56, 72 groups 1.07, 0.99, 0.99; 1100 runs 0.97 to 1.02
// Bytes at W = 32 gain or break even (2048 runs of 10 groups 1.03, of 72 0.97, 1100 runs 0.97 and
// 0.88). few_more: at most an eighth more runs than SIMDs.
uint32_t shared_from(uint32_t lanes, uint32_t symbol_bytes, bool wide, bool few_more) {
    if (wide && lanes == 32) return few_more ? 88 : 112;
    if (wide) return symbol_bytes == 1 ? (few_more ? 56 : 112) : few_more ? 0 : 56;
    if (symbol_bytes == 1) return lanes == 32 ? (few_more ? 0 : 16) : few_more ? 24 : 64;
    return lanes == 32 ? (few_more ? 72 : 88) : few_more ? 48 : 64;
}

}  // namespace

bool decode_few(const DecodeParams &p, uint32_t lanes, uint32_t symbol_bytes, uint32_t waves, uint32_t blocks_per_cu,
                FewShape &shape, bool launch, hipStream_t stream, hipError_t *e) {
    const uint32_t cus = shape.cus;
    // Two runs per SIMD still run at almost the pace of one (64 MiB at W = 32 in 2048 units:
    // 117 us with the throughput kernel, 82 us here); four do not (4096 units: 70 against
    // 73 us, the rings are then down to 4 groups).
    if (p.tidx || p.runs == 0 || p.runs > 2 * kSimds * cus) return false;
    shape = p.runs <= kSimds * cus ? FewShape{cus, p.runs, 1} : FewShape{cus, cus, (uint32_t)kShared};
    if (waves && waves != shape.waves) return false;
    // Every run is resident from the start, so a cap below that is left to the throughput
    // kernel, whose workgroups decode one run after another.
    if (blocks_per_cu && (shape.blocks + cus - 1) / cus > blocks_per_cu) return false;
    if (waves == 0 && shape.waves > 1 &&
        p.n_symbols / lanes / p.runs < shared_from(lanes, symbol_bytes, p.quant_bits > 12, p.runs <= kSimds * cus * 9 / 8))
        return false;
    static_assert(kShared == 2 * kSimds, "a workgroup per CU holds two runs per SIMD");
    if (lanes == 32) return symbol_bytes == 1 ? pick_variant<32, uint8_t>(p, shape, launch, stream, e)
                                              : pick_variant<32, uint16_t>(p, shape, launch, stream, e);
    if (lanes == 64) return symbol_bytes == 1 ? pick_variant<64, uint8_t>(p, shape, launch, stream, e)
                                              : pick_variant<64, uint16_t>(p, shape, launch, stream, e);
    return false;
}

}  // namespace recoil
