// Device core of the decode for launches of few runs: one unit per wave, at most
// about one wave per SIMD, where nothing but the unit's own dependent chain from one
// symbol group to the next sets the pace (Lin et al., ICPP 2023, Sec. 4.1; Eq. 2, Eq. 4).
//
// The chain of the throughput kernel (decode_core.hpp) has two LDS round trips per
// group: a lane that renormalises reads its 16-bit word w from the ring and then, like
// every other lane, its table entry. But the slot of a lane that has just read w is
// w mod 2^n, whatever its state was (b >= n). So the ring here holds words that are
// already looked up: for a reader
//     x' = f ((x << 16 | w) >> n) + slot - F = f (x << (16 - n)) + c(w),
//     c(w) = f (w >> n) + (w mod 2^n) - F  < 2^16,
// with f, F and the symbol those of w's slot; for any other lane
//     x' = f (x >> n) + slot - F.
// Ring and table entries have one form {f, addend, symbol} of 8 bytes, so a lane selects
// an address (ring or table) and a factor (x << (16 - n) or x >> n) while the offset of
// its word is being counted, and a group needs one LDS read and one multiply-add after
// it. The look-up of the words (one table read per word, 0.3-0.7 words per symbol) runs
// off the chain, when a chunk is put into the ring: up to one run per SIMD on another
// wave (HELP), which costs the decoding wave one meeting per super-step.
//
// What bounds it: the chain, 45.8 ns per group in long runs, 105 to 110 cycles at 2.28 to
// 2.4 GHz. A lone wave issues in order, a vector instruction 8 cycles after one whose result it
// takes and about 4 after any other. Eight stand before the LDS read (multiply-add, compare,
// the table address's two, a wait state, count, word address, select): about 52 cycles; the
// read takes 44, bank conflicts at most 3 (256 runs of 8192 groups: 6.9 M conflict cycles for 2.1 M
// groups), the store and the super-step's account and meeting the rest. Without a helper the
// look-ups come on top, 18 ns per group at 0.36 words per symbol.
// Measured with the throughput kernel of one wave per workgroup, this one without a helper
// and with it: 64 MiB of bytes at W = 32 in 256 units 885, 524, 376 us, in 1024 units 225,
// 133, 112 us; at W = 64 in 256 units 405, 236, 201 us; n = 16 at W = 32 in 256 units 1353,
// 923, 665 us, in 1024 units 330, 211, 174 us; four streams in turn, 1 MiB at W = 32 in 256
// units 19.2, 12.8, 10.6 us, 1.5 M 16-bit symbols at W = 64 in 367 units 14.9, 9.3, 8.7 us.
#pragma once

#include "decode_core.hpp"

namespace recoil {
namespace dev {

// Entry forms. u8: .x = f | symbol << 24, .y = addend (a 24-bit multiply ignores the
// symbol). u16: .x = f | addend << 16, .y = symbol. Wide tables (13 <= n <= 16), rank
// entries as in decode.hpp: .x = f, .y = symbol | F << 16, with
// x' = .x * factor + base - (.y >> 16): base = slot for a table entry; ring entries hold
// 0xFFFF - c(w) in place of F and use base = 0xFFFF.
// The table address of a state is address(x, first(x)): first() is the bucket read of a
// wide table and nothing otherwise. word() makes the ring entry of word w from its slot's
// table entry.
template <typename Sym, bool WIDE>
struct FewTable {
    static constexpr uint32_t kSymShift = sizeof(Sym) == 1 ? 24 : 0;
    __device__ static __forceinline__ uint32_t first(uint32_t, uint32_t, uint32_t) { return 0; }
    __device__ static __forceinline__ uint32_t address(uint32_t lut, uint32_t x, uint32_t mask, uint32_t) {
        return lut + ((x & mask) << 3);
    }
    __device__ static __forceinline__ uint32_t next(u32x2 e, uint32_t factor, uint32_t) {
        if constexpr (sizeof(Sym) == 1) return __umul24(e.x, factor) + e.y;
        return __umul24(e.x & 0xFFFFu, factor) + (e.x >> 16);
    }
    __device__ static __forceinline__ uint32_t base(bool, uint32_t, uint32_t) { return 0; }
    __device__ static __forceinline__ u32x2 word(u32x2 e, uint32_t w, uint32_t n, uint32_t) {
        if constexpr (sizeof(Sym) == 1) return u32x2{e.x, __umul24(e.x, w >> n) + e.y};
        const uint32_t f = e.x & 0xFFFFu;
        return u32x2{f | ((__umul24(f, w >> n) + (e.x >> 16)) << 16), e.y};
    }
    __device__ static __forceinline__ uint32_t symbol(u32x2 e) { return sizeof(Sym) == 1 ? e.x : e.y; }
};

template <typename Sym>
struct FewTable<Sym, true> {
    static constexpr uint32_t kSymShift = 0;
    __device__ static __forceinline__ uint32_t first(uint32_t lut, uint32_t x, uint32_t mask) {
        return lds_ld<uint32_t>(lut + (((x & mask) >> 4) << 2));
    }
    __device__ static __forceinline__ uint32_t address(uint32_t lut, uint32_t x, uint32_t mask, uint32_t c) {
        const uint32_t r = (c >> 16) + __builtin_popcount(__builtin_amdgcn_ubfe(c, 0, x & 15u));
        return lut + ((mask + 1u) >> 2) + (r << 3);
    }
    __device__ static __forceinline__ uint32_t next(u32x2 e, uint32_t factor, uint32_t base) {
        return __umul24(e.x, factor) + base - (e.y >> 16);
    }
    __device__ static __forceinline__ uint32_t base(bool need, uint32_t x, uint32_t mask) {
        return need ? 0xFFFFu : x & mask;
    }
    __device__ static __forceinline__ u32x2 word(u32x2 e, uint32_t w, uint32_t n, uint32_t mask) {
        const uint32_t c = __umul24(e.x, w >> n) + (w & mask) - (e.y >> 16);
        return u32x2{e.x, (e.y & 0xFFFFu) | ((0xFFFFu - c) << 16)};
    }
    __device__ static __forceinline__ uint32_t symbol(u32x2 e) { return e.y; }
};

// K groups per super-step, ring of NCH chunks of C = K*W entries plus a C-entry mirror
// of its top chunk below slot 0 (as in decode_core.hpp, high to low).
//
// HELP: a second wave of the workgroup looks the words up and fills the ring (supply()),
// in step with the decoding one: see super_step.
template <int W, typename Sym, int K, int NCH, bool WIDE, bool COUNT, bool HELP>
struct FewDecoder {
    using T = FewTable<Sym, WIDE>;
    static constexpr uint32_t C = K * W, R = NCH * C, E = 8;
    static constexpr uint32_t RING_BYTES = E * (R + C);
    static constexpr uint32_t MSG = RING_BYTES - E;   // HELP: two words, in place of the mirror's
                                                      // last entry, which no super-step reaches
    static constexpr uint32_t D = K / 2;      // dwords of a chunk per lane
    static constexpr int32_t FILL = 2;        // chunks looked up before the first group
    static_assert(K % 2 == 0 && NCH >= 3, "ring shape");

    const DecodeParams &p;
    uint32_t lut, ring, lane, coder, n, mask;
    uint32_t top, ghi, steps, presync;
    bool full;
    uint32_t rec, act, lim, x;
    bool active;
    uint32_t a, a0;         // LDS address of the unit's next entry, and at the super-step's start
    int32_t res;            // words in the ring: (next word + 1) - fq * C
    int32_t fq;             // lowest chunk in the ring
    bool pend;              // chunk fq - 1 has been requested into pre (there is one)
    uint32_t age;           // super-steps since
    uint32_t turn;          // HELP: which word of MSG is next, 0 or 4
    uint32_t pre[D];
    uint32_t lane_off;

    __device__ FewDecoder(const DecodeParams &p_, uint32_t lut_, uint32_t ring_, uint32_t lane_)
        : p(p_), lut(lut_), ring(ring_), lane(lane_) {
        coder = W - 1 - lane;
        n = p.quant_bits;
        mask = (1u << n) - 1u;
    }

    __device__ __forceinline__ uint32_t slot_addr(int32_t s) const { return ring + E * (uint32_t)((int32_t)R - 1 - s); }

    // Dword i of this lane's share of chunk q: words 2d and 2d + 1, d = lane + W i.
    __device__ __forceinline__ void fetch(int32_t q, uint32_t (&v)[D]) const {
        const uint32_t *src = reinterpret_cast<const uint32_t *>(p.words) + (uint64_t)(uint32_t)q * (C / 2);
#pragma unroll
        for (uint32_t i = 0; i < D; ++i) v[i] = src[lane + W * i];
    }

    // Word g of this lane's share of a chunk.
    __device__ static __forceinline__ uint32_t word_of(const uint32_t (&v)[D], uint32_t g) {
        return g & 1u ? v[g / 2] >> 16 : v[g / 2] & 0xFFFFu;
    }

    // Looks chunk q's words up and writes them to its place in the ring, all reads of one
    // kind in flight together. (Spread over the groups instead, under the latency of their
    // entry reads, the same work cost four times as much: a lone wave pays 8 cycles for each
    // dependent instruction, and there is nothing to put between them.)
    __device__ __forceinline__ void put(int32_t q, const uint32_t (&v)[D]) const {
        const uint32_t pos = uni((uint32_t)q % NCH);
        u32x2 e[K];
        uint32_t c[K] = {};
        if constexpr (WIDE) {
#pragma unroll
            for (uint32_t g = 0; g < K; ++g) c[g] = T::first(lut, word_of(v, g), mask);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (uint32_t g = 0; g < K; ++g) e[g] = lds_ld<u32x2>(T::address(lut, word_of(v, g), mask, c[g]));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (uint32_t g = 0; g < K; ++g) e[g] = T::word(e[g], word_of(v, g), n, mask);
        const uint32_t at = ring + E * (R - 2u - pos * C) - 2u * E * lane;
#pragma unroll
        for (uint32_t i = 0; i < D; ++i)
            lds_st<u32x4>(at - 2u * E * W * i, u32x4{e[2 * i + 1].x, e[2 * i + 1].y, e[2 * i].x, e[2 * i].y});
        if (pos == NCH - 1) {
#pragma unroll
            for (uint32_t i = 0; i < D; ++i) {
                const uint32_t to = at + E * R - 2u * E * W * i;
                if (HELP && i == 0) {
                    lds_st<u32x2>(to, e[1]);
                    if (lane != 0) lds_st<u32x2>(to + E, e[0]);   // (lane 0's is MSG)
                } else {
                    lds_st<u32x4>(to, u32x4{e[2 * i + 1].x, e[2 * i + 1].y, e[2 * i].x, e[2 * i].y});
                }
            }
        }
    }

    // The run's records; touches no LDS, so that it can run before the table is staged.
    __device__ __forceinline__ void records(uint32_t run) {
        const uint32_t lo = run * p.run, hi = min(lo + p.run, p.units) - 1u;
        const bool last = hi + 1 == p.units;
        full = last || p.partitioned;              // starts from 32-bit final states
        const UnitMeta m = p.meta[hi];
        const uint32_t glo = uni(p.meta[lo].glo), next = uni(m.next);
        top = uni(m.top);
        ghi = uni(m.ghi);
        rec = p.lanes[(uint64_t)hi * W + coder];
        steps = top + 1 > glo ? top + 1 - glo : 0u;
        presync = full ? ((last && (p.n_symbols % W)) ? 1u : 0u) : top - ghi + 1;
        x = full ? rec : 0u;
        active = full;
        act = full ? 0u : (rec >> 16);
        lane_off = coder * (uint32_t)sizeof(Sym);
        const int32_t cur = (int32_t)next, q0 = cur > 0 ? (cur - 1) / (int32_t)C : -1;
        fq = q0 >= FILL - 1 ? q0 - (FILL - 1) : 0;
        res = cur - fq * (int32_t)C;
        a = uni(slot_addr(cur > 0 ? (cur - 1) % (int32_t)R : 0));
    }

    // First chunks of the run, and the one after them: all requested, then looked up. HELP:
    // the decoding wave takes the highest, its helper the others.
    __device__ __forceinline__ void fill_request(uint32_t (&v)[FILL][D], bool helper) {
#pragma unroll
        for (int32_t i = FILL - 1; i >= 0; --i)
            if (res > i * (int32_t)C && (!HELP || helper == (i < FILL - 1))) fetch(fq + i, v[i]);
        pend = fq > 0;
        age = 0;
        if (pend && (!HELP || helper)) fetch(fq - 1, pre);
    }
    __device__ __forceinline__ void fill_put(const uint32_t (&v)[FILL][D], bool helper) {
#pragma unroll
        for (int32_t i = FILL - 1; i >= 0; --i)
            if (res > i * (int32_t)C && (!HELP || helper == (i < FILL - 1))) put(fq + i, v[i]);
        if constexpr (HELP) {
            turn = 0;
            meet();
        }
    }

    // HELP. The two waves meet once before the first super-step and once after each, where the
    // decoding wave says how many words are left in the ring. From that number both decide
    // alike whether the next chunk goes in (claim), and the helper puts it there while the
    // next super-step runs.
    //   Supply: more than C words are in the ring at the start of a super-step, or all that
    // are left, as a super-step takes at most C and a chunk is claimed at up to 2C: before
    // the first one res > C, and after one that starts with r > 2C still r - C > C, after
    // one that starts with less r - C + C, the chunk claimed at its start.
    //   Overwriting: with at most R - C words left, those that the chunk's place held before
    // have all been read.
    //   MSG has two words, so that one is not written again before the helper has read it; the
    // last report ends the helper, so both waves meet the same number of times.
    static constexpr int32_t kDone = INT32_MIN;
    __device__ static __forceinline__ void meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
    __device__ __forceinline__ void report(int32_t left) {
        lds_st<uint32_t>(ring + MSG + turn, (uint32_t)left);
        turn ^= 4u;
    }
    __device__ __forceinline__ bool claim() {
        if (!pend || res > (int32_t)(R - C)) return false;
        fq -= 1;
        res += (int32_t)C;
        pend = fq > 0;
        return true;
    }
    __device__ __forceinline__ void supply() {
        res = (int32_t)uni((uint32_t)res), fq = (int32_t)uni((uint32_t)fq);
        for (;;) {
            if (claim()) {
                put(fq, pre);
                if (pend) fetch(fq - 1, pre);
            }
            meet();
            res = (int32_t)uni(lds_ld<uint32_t>(ring + MSG + turn));
            turn ^= 4u;
            if (res == kDone) return;
        }
    }

    // Read and decode step of one group for this lane (need: x < L and on), in three parts.
    // A wave alone on its SIMD issues in order and waits for each result, so the order is
    // part of the design: request() is the chain up to the LDS read and nothing else, work
    // that the chain does not wait for goes between it and next(), under the read's latency.
    // SCALAR keeps the unit's address an opaque scalar operand of one v_lshl_add (not in the
    // predicated body, where the compiler may move it).
    struct Read {
        u32x2 e;
        uint64_t bal;
        bool need;
    };
    template <bool SCALAR = true>
    __device__ __forceinline__ Read request(bool need) {
        Read r;
        r.need = need;
        r.bal = __ballot(need);
        const uint32_t taddr = T::address(lut, x, mask, T::first(lut, x, mask));
        uint32_t m = __builtin_amdgcn_mbcnt_lo((uint32_t)r.bal, 0u);
        if constexpr (W == 64) m = __builtin_amdgcn_mbcnt_hi((uint32_t)(r.bal >> 32), m);
        if constexpr (SCALAR) {
            a = uni(a);
            asm volatile("" : "+s"(a));
        }
        const uint32_t raddr = (m << 3) + a;
        r.e = lds_ld<u32x2>(need ? raddr : taddr);
        __builtin_amdgcn_sched_barrier(0);
        return r;
    }
    __device__ __forceinline__ uint32_t factor_of(const Read &r) const { return r.need ? x << (16u - n) : x >> n; }
    __device__ __forceinline__ void advance(const Read &r) {
        a += (uint32_t)(W == 64 ? __builtin_popcountll(r.bal) : __builtin_popcount((uint32_t)r.bal)) << 3;
    }
    template <bool SCALAR = true>
    __device__ __forceinline__ u32x2 step(bool need, uint32_t &y) {
        const Read r = request<SCALAR>(need);
        const uint32_t f = factor_of(r), base = T::base(need, x, mask);
        advance(r);
        __builtin_amdgcn_sched_barrier(0);
        y = T::next(r.e, f, base);
        return r.e;
    }

    __device__ __forceinline__ void count_store(uint64_t i) const { atomicAdd(p.counts + i, 1u); }
    __device__ __forceinline__ void store(uint64_t i, u32x2 e) const {
        static_cast<Sym *>(p.out)[i] = (Sym)(T::symbol(e) >> T::kSymShift);
        if constexpr (COUNT) count_store(i);
    }

    // A group of the unpredicated body. Under the latency of its entry read: the factor, the
    // address of the next word and the store of the group before.
    template <uint32_t G>
    __device__ __forceinline__ void group_fast(unsigned char *outh, uint32_t &sym) {
        const Read r = request(x < kL);
        const uint32_t f = factor_of(r), base = T::base(r.need, x, mask);
        advance(r);
        if constexpr (G > 0) emit<G - 1u>(outh, sym);
        if constexpr (HELP && G == K - 1u) account();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (HELP && G == K - 1u) meet();
        x = T::next(r.e, f, base);
        sym = T::symbol(r.e);
    }
    template <uint32_t G>
    __device__ __forceinline__ void emit(unsigned char *outh, uint32_t sym) const {
        unsigned char *dst = outh + lane_off - G * W * sizeof(Sym);
        *reinterpret_cast<Sym *>(dst) = (Sym)(sym >> T::kSymShift);
        if constexpr (COUNT) count_store((uint64_t)(dst - static_cast<unsigned char *>(p.out)) / sizeof(Sym));
    }

    // Synchronisation, every lane inside the unit's own groups (see PairDecoder::group_sync).
    __device__ __forceinline__ void group_sync(uint32_t k) {
        const bool on = k == act;
        x = on ? (rec & 0xFFFFu) : x;
        lim = on ? kL : lim;
        uint32_t y;
        const u32x2 e = step(x < lim, y);
        x = y;
        const uint32_t h = top - k;
        if (h <= ghi) store((uint64_t)h * W + coder, e);
    }

    // Fully predicated: synchronisation near the stream's ends, the ragged last group and
    // a unit's last groups. (A lane without a symbol in the ragged group holds a final
    // state, at least L: it reads nothing.)
    __device__ __forceinline__ void group_pred(uint32_t k) {
        const bool live = k < steps;
        if (live && !active && k == act) {
            active = true;
            x = rec & 0xFFFFu;
        }
        const bool on = live && active;
        const uint64_t i = (uint64_t)(top - k) * W + coder;
        uint32_t y;
        const u32x2 e = step<false>(on && x < kL, y);
        if (on && i < p.n_symbols) {
            x = y;
            if (top - k <= ghi) store(i, e);
        }
    }

    // The super-step's words, off the ring.
    __device__ __forceinline__ void consumed() {
        res -= (int32_t)((a - a0) >> 3);
        a = a >= slot_addr(-1) ? a - E * R : a;
    }
    // HELP: all that the decoding wave does about the ring after a super-step.
    __device__ __forceinline__ void account() {
        consumed();
        report(res);
        claim();
    }

    static constexpr int kFast = 0, kSync = 1, kPred = 2;

    template <int MODE, uint32_t... G>
    __device__ __forceinline__ void groups(std::integer_sequence<uint32_t, G...>, uint32_t k) {
        if constexpr (MODE == kPred) {
            (group_pred(k + G), ...);
        } else if constexpr (MODE == kSync) {
            (group_sync(k + G), ...);
        } else {
            unsigned char *outh = static_cast<unsigned char *>(p.out) + (uint64_t)(top - k) * W * sizeof(Sym);
            uint32_t sym;
            (group_fast<G>(outh, sym), ...);
            emit<K - 1u>(outh, sym);
        }
    }

    // KK <= K groups, then the look-up of the next chunk, which was requested after the one
    // before it. At the start at least C words are resident, or all that are left: a
    // super-step consumes at most C. So the chunk has to be put with fewer than C left after
    // it and can be when its place is free; in between it waits until AGE super-steps (a
    // group takes about 50 ns) have covered the latency of its request. Returns false if the
    // unit read past its first word (corrupt split data).
    static constexpr uint32_t AGE = K >= 16 ? 1 : 16 / K;
    template <int MODE, uint32_t KK = K>
    __device__ __forceinline__ bool super_step(uint32_t k) {
        a0 = a;
        groups<MODE>(std::make_integer_sequence<uint32_t, KK>{}, k);
        if constexpr (HELP) {
            if constexpr (MODE != kFast) {
                account();
                meet();
            }
            return res >= 0;
        }
        consumed();
        ++age;
        if (pend && (res < (int32_t)C || (res <= (int32_t)(R - C) && age >= AGE))) {
            fq -= 1;
            put(fq, pre);
            res += (int32_t)C;
            pend = fq > 0;
            age = 0;
            if (pend) fetch(fq - 1, pre);
        }
        return res >= 0;
    }

    __device__ __forceinline__ void run() {
        decode();
        if constexpr (HELP) {
            report(kDone);
            meet();
        }
    }

    // Decodes the run: the same phases and run-on rule as PairDecoder::run with one unit.
    __device__ __forceinline__ void decode() {
        top = uni(top), ghi = uni(ghi), steps = uni(steps), presync = uni(presync);
        a = uni(a), res = (int32_t)uni((uint32_t)res), fq = (int32_t)uni((uint32_t)fq);
        if constexpr (HELP) claim();
        if (steps == 0) return;
        bool ok = true;
        uint32_t k = 0;
        const uint32_t lead = (presync + K / 2 - 1) / (K / 2) * (K / 2);
        if (!full && lead <= steps) {
            lim = 0;
            for (; ok && k < presync; k += K / 2) ok = super_step<kSync, K / 2>(k);
            active = true;
        } else {
            for (; ok && k < steps && k < presync; k += K / 2) ok = super_step<kPred, K / 2>(k);
        }
        const uint32_t kend = k < steps ? k + (steps - k + K - 1) / K * K : k;
        const bool run_on = !p.partitioned && k <= steps && top + 1 >= kend &&
                            res + fq * (int32_t)C >= (int32_t)((kend - k) * W);
        const uint32_t fast_end = run_on ? steps : steps - min(steps, K - 1u);   // last start, plus one
        for (; ok && k < fast_end; k += K) ok = super_step<kFast>(k);
        for (; ok && k < steps; k += K) ok = super_step<kPred>(k);
        if (!ok && lane == 0) atomicOr(p.err, kDevErrUnderflow);
    }
};

}  // namespace dev
}  // namespace recoil
