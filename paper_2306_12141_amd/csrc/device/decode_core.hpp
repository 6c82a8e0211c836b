// Device core of the Recoil decoder, shared by the single-stream and batched
// kernels (Lin et al., ICPP 2023, Sec. 4.1; Eq. 2 and Eq. 4).
//
// A decode unit is W interleaved rANS lanes; a 64-lane wavefront runs one unit
// (W = 64) or two (W = 32, one per half-wave). Coder j of a unit lives in wave
// lane W-1-j of its half, so that "reading lanes with a higher coder index",
// the words a lane must skip because the decoder consumes words in decreasing
// coder order (Sec. 2.2), are exactly the reading lanes below it in the wave:
// its offset is one mbcnt of the read ballot, independent of how many lanes
// read in total.
//
// Bitstream ring (per unit, in LDS). Words are fetched from HBM in chunks of
// C = K*W words, the most a unit can consume in a super-step of K groups (one
// word per symbol at most, since b >= n). A chunk is requested into registers when
// the one above it is written to the ring, and written when fewer than C words are
// left. The ring has 3C slots plus a C-word mirror of
// its top chunk placed below slot 0, so reads never wrap inside a super-step:
// word w lives at slot w mod 3C, and positions down to -C read the mirror.
//
// Per group the scalar unit only advances the LDS address of the unit's next
// word by twice the number of reading lanes (one s_bcnt1 and one s_lshl1_add;
// a pair of W = 32 units keeps each unit's address, in words, in its half-wave's
// lanes instead); the per-group store offsets are immediates of the unrolled
// super-step.
//
// Synchronisation (Sec. 4.1.1): lane j is switched on with its recorded 16-bit
// state at the read step of the group its recorded symbol belongs to, just
// before its first read; groups above the unit's range only advance states.
// The synchronisation lead-in runs a predicated body (a lean one when no unit
// of the pair is the stream's last), and so do a ragged last group and units
// that end near group 0 or word 0; all other super-steps run the unpredicated
// body. A run of consecutive units is decoded as one unit from its highest
// unit's split point (Sec. 3.3).
#pragma once

#include <type_traits>

#include "decode.hpp"

namespace recoil {
namespace dev {

constexpr uint32_t kL = 1u << 16;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kDevErrUnderflow = 1u;

// LDS is addressed with plain 32-bit LDS addresses (address space 3), so that
// uniform parts of an address stay in SGPRs and constants fold into the
// instructions' immediate offsets.
template <typename V>
__device__ inline V lds_ld(uint32_t a) {
    return *reinterpret_cast<const __attribute__((address_space(3))) V *>((size_t)a);
}
template <typename V>
__device__ inline void lds_st(uint32_t a, const V &v) {
    *reinterpret_cast<__attribute__((address_space(3))) V *>((size_t)a) = v;
}
__device__ inline uint32_t lds_addr(unsigned char *generic) {
    return (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)generic;
}

template <typename Sym>
struct Table;

template <>
struct Table<uint8_t> {
    using Entry = uint32_t;   // symbol | f << 8 | (slot - F) << 20
    __device__ static inline uint32_t step(uint32_t &x, uint32_t n, uint32_t mask) {
        const Entry e = lds_ld<Entry>((x & mask) << 2);
        const uint32_t f = (e >> 8) & 0xFFFu;
        x = __umul24(f, x >> n) + (e >> 20);
        return e;             // the low byte is the symbol
    }
    // Adaptive coding: the symbol's own table at LDS address t of the tables laid end to end.
    __device__ static inline uint32_t step_t(uint32_t &x, uint32_t n, uint32_t mask, uint32_t t) {
        const Entry e = lds_ld<Entry>(((x & mask) << 2) + t);
        const uint32_t f = (e >> 8) & 0xFFFu;
        x = __umul24(f, x >> n) + (e >> 20);
        return e;
    }
};

template <>
struct Table<uint16_t> {
    using Entry = u32x2;      // .x = f | (slot - F) << 16, .y = symbol
    __device__ static inline uint32_t step(uint32_t &x, uint32_t n, uint32_t mask) {
        const Entry e = lds_ld<Entry>((x & mask) << 3);
        x = __umul24(e.x & 0xFFFFu, x >> n) + (e.x >> 16);
        return e.y;
    }
};

// Wide tables (13 <= n <= 16): the two-level layout of decode.hpp. The symbol's
// rank is the bucket's first rank plus the range starts between the bucket's first
// slot and this one (a popcount of the low p start bits, p = slot mod 16).
template <typename Sym>
struct WideTable {
    using Entry = u32x2;
    __device__ static inline uint32_t step(uint32_t &x, uint32_t n, uint32_t mask) {
        const uint32_t slot = x & mask;
        const uint32_t c = lds_ld<uint32_t>((slot >> 4) << 2);
        const uint32_t r = (c >> 16) + __builtin_popcount(__builtin_amdgcn_ubfe(c, 0, slot & 15u));
        const Entry e = lds_ld<Entry>(((mask + 1u) >> 2) + (r << 3));
        x = __umul24(e.x, x >> n) + slot - (e.y >> 16);
        return e.y;
    }
};

template <int W, int K, int SS = 64 / W>
struct Geo {
    static constexpr uint32_t S = SS;                 // units per wave (W = 32: one per half-wave, or one)
    static constexpr uint32_t C = K * W;              // chunk words
    static constexpr uint32_t R = 3 * C;              // ring slots
    static constexpr uint32_t UNIT = 2 * (C + R);     // LDS bytes per unit: mirror + ring
    static constexpr uint32_t WAVE_LDS = S * UNIT;
    static constexpr uint32_t LANE_BYTES = 2 * K;     // chunk bytes per lane of a unit
    using Chunk = typename std::conditional<LANE_BYTES == 16, u32x4, u32x2>::type;
    static_assert(sizeof(Chunk) == LANE_BYTES, "chunk slice must be 8 or 16 bytes");
};

// LDS layout of a workgroup: [decode table][pad][rings of every wave]. The table is at
// LDS address 0 (the kernels have no other shared memory), so that an entry's address is
// its slot shifted. The pad is a 16-byte slot the batched kernel uses to broadcast its
// work item.
template <int PADB, int K, int WAVES>
struct Lds {
    static constexpr uint32_t PAD = PADB;
    static constexpr uint32_t WAVE_LDS = Geo<32, K>::WAVE_LDS > Geo<64, K>::WAVE_LDS ? Geo<32, K>::WAVE_LDS
                                                                                     : Geo<64, K>::WAVE_LDS;
    static constexpr uint32_t RINGS = PAD + WAVES * WAVE_LDS;   // bytes after the table
};

__device__ inline uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Wave issue priority 0..3 (larger values go first; the level is clamped).
__device__ inline void set_priority(uint32_t level) {
    if (level >= 3) __builtin_amdgcn_s_setprio(3);
    else if (level == 2) __builtin_amdgcn_s_setprio(2);
    else if (level == 1) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// A wave-uniform record read from global memory: every dword through
// readfirstlane, so its fields live in SGPRs rather than in VGPR copies.
template <typename T>
__device__ inline T uni_load(const T *src) {
    static_assert(sizeof(T) % 4 == 0, "record of whole dwords");
    uint32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, src, sizeof(T));
#pragma unroll
    for (uint32_t i = 0; i < sizeof(T) / 4; ++i) w[i] = uni(w[i]);
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

// Scalar registers per wave for the decode kernels. A SIMD held eight waves of
// a kernel using 62 of them but only seven at 76 (measured per-wave start
// times), and the decode loop needs every wave it can get to hide its LDS
// latency, so the kernels are compiled to this budget (the values that do not
// fit are kept in VGPR lanes and mostly reloaded outside the group loops).
#define RECOIL_SGPR_BUDGET 64

// The read step after the compare has left the reading lanes in VCC (two wait states
// before a vector instruction reads VCC as a scalar operand: the move and the count).
#define RECOIL_READ_TAIL                 \
    "s_and_saveexec_b64 %[sv], vcc\n\t"  \
    "ds_read_u16 %[w], %[t]\n\t"         \
    "v_lshlrev_b32 %[x], 16, %[x]\n\t"   \
    "s_mov_b64 exec, %[sv]\n\t"
#define RECOIL_READ_64                             \
    "v_mov_b32 %[w], 0\n\t"                        \
    "s_bcnt1_i32_b64 %[c], vcc\n\t"                \
    "v_mbcnt_lo_u32_b32 %[t], vcc_lo, 0\n\t"       \
    "v_mbcnt_hi_u32_b32 %[t], vcc_hi, %[t]\n\t"    \
    "v_lshl_add_u32 %[t], %[t], 1, %[a]\n\t"       \
    RECOIL_READ_TAIL                               \
    "s_lshl1_add_u32 %[a], %[c], %[a]\n\t"         \
    "s_waitcnt lgkmcnt(0)\n\t"                     \
    "v_or_b32 %[x], %[x], %[w]"
#define RECOIL_READ_32                             \
    "v_mov_b32 %[w], 0\n\t"                        \
    "s_bcnt1_i32_b32 %[c], vcc_lo\n\t"             \
    "v_mbcnt_lo_u32_b32 %[t], vcc_lo, 0\n\t"       \
    "v_lshl_add_u32 %[t], %[t], 1, %[a]\n\t"       \
    RECOIL_READ_TAIL                               \
    "s_lshl1_add_u32 %[a], %[c], %[a]\n\t"         \
    "s_waitcnt lgkmcnt(0)\n\t"                     \
    "v_or_b32 %[x], %[x], %[w]"
// Pairs: readers below the lane in its own half-wave (the lower half's are masked off for
// upper lanes), counted onto the unit's address; each unit's address then advances by its
// own readers, e += pl + upper * (ph - pl) (a vector instruction reads at most one scalar
// operand, so the two counts cannot be selected per lane in one).
#define RECOIL_READ_PAIR                           \
    "v_mov_b32 %[w], 0\n\t"                        \
    "s_bcnt1_i32_b32 %[c], vcc_lo\n\t"             \
    "v_and_b32 %[t], vcc_lo, %[low]\n\t"           \
    "s_bcnt1_i32_b32 %[d], vcc_hi\n\t"             \
    "v_mbcnt_lo_u32_b32 %[t], %[t], %[e]\n\t"      \
    "v_mbcnt_hi_u32_b32 %[t], vcc_hi, %[t]\n\t"    \
    "s_sub_i32 %[d], %[d], %[c]\n\t"               \
    "v_lshlrev_b32 %[t], 1, %[t]\n\t"              \
    RECOIL_READ_TAIL                               \
    "v_mad_i32_i24 %[e], %[up], %[d], %[e]\n\t"    \
    "v_add_u32 %[e], %[c], %[e]\n\t"               \
    "s_waitcnt lgkmcnt(0)\n\t"                     \
    "v_or_b32 %[x], %[x], %[w]"

struct ScalarLim {
    uint32_t v;
};

// Kernel variants: kCount also adds 1 to counts[i] for every store of symbol i (a
// checking launch); kAdaptive codes symbol i with decode table tidx[i] (adaptive
// coding, uint8 symbols); kWide reads the two-level table of 13 <= n <= 16.
constexpr int kPlain = 0, kCount = 1, kAdaptive = 2, kWide = 3;

template <int W, typename Sym, int K, int SS = 64 / W, int VAR = kPlain>
struct PairDecoder {
    using G = Geo<W, K, SS>;
    using T = typename std::conditional<VAR == kWide, WideTable<Sym>, Table<Sym>>::type;
    using Chunk = typename G::Chunk;
    static constexpr uint32_t S = G::S, C = G::C, R = G::R;
    static constexpr bool COUNT = VAR == kCount, ADAPT = VAR == kAdaptive;
    // Fast-body stores of byte symbols four groups at a time (see store_quad), for
    // 32-lane units: there a byte store writes only 32 bytes per unit, and one
    // dword store per four groups decoded W = 32 streams 13-16 % faster, while at
    // W = 64 the transpose's seven VALU per four groups cost more than the three
    // stores they save (1 % slower).
    static constexpr bool QUAD = W == 32 && sizeof(Sym) == 1 && K % 4 == 0;
    static_assert(!ADAPT || (sizeof(Sym) == 1 && K == 4), "adaptive decoding reads the table indices at the symbols' byte offsets, four groups at a time");

    const DecodeParams &p;
    uint32_t ring0;        // LDS address of this wave's first unit
    uint32_t lane, col, upper, coder;
    uint32_t lane_ring;    // this lane's chunk-slice address in the top third of its unit's ring
    // In vector registers, all lanes alike: an and or a shift of vector registers only
    // issues every two cycles, one with a scalar operand every four.
    uint32_t n, mask;

    // Per unit of the pair (wave-uniform). Kept few: the register file holds
    // eight waves per SIMD only while a wave needs at most 64 scalar registers.
    uint32_t top0;         // unit 0's first group (the fast body's store base)
    uint32_t top_min;      // smallest first group of the pair's units
    uint32_t steps[S];     // groups the unit decodes
    uint32_t ua[S];        // LDS byte address of the unit's next word in its ring
    uint32_t presync;      // leading groups of the pair that need the predicated body
    bool sync_lean;        // no unit of the pair is the stream's last (ragged top group, 32-bit states)
    // Per lane, for the unit of the lane's half-wave: its ring bookkeeping lives in
    // vector registers, so one instruction keeps both units of a pair up to date and
    // the scalar registers hold only what the group loop needs.
    int32_t vres;          // words of the unit still in the ring: (next word + 1) - vfq * C
    int32_t vfq;           // lowest chunk held in the ring (the next fetch is vfq - 1)
    uint32_t vpo;          // byte offset from the top third of the third that chunk vfq - 1 goes to
    // Pairs (S == 2): the LDS address (in words) of the next word of the lane's unit, the
    // address at which it wraps, and a mask that confines a read ballot to the
    // lane's own half-wave.
    uint32_t vb, vlim, lowmask;
    // Adaptive coding: the LDS addresses of the super-step's tables.
    uint32_t tcur[K];
    uint32_t x, rec, act, lim;
    uint32_t my_top, my_ghi, my_steps, lane_off;
    uint32_t quad_off;     // QUAD: this lane's dword offset from the fast body's group pointer, plus 3W
    bool active;

    __device__ PairDecoder(const DecodeParams &p_, uint32_t ring0_, uint32_t lane_)
        : p(p_), ring0(ring0_), lane(lane_) {
        col = lane & (W - 1);
        upper = (S == 2) ? (lane >> 5) : 0u;
        coder = W - 1 - col;
        n = p.quant_bits;
        mask = (1u << n) - 1u;
        asm volatile("" : "+v"(n), "+v"(mask));
        lane_ring = lane_ring_addr();
    }

    // LDS byte address of ring position s (s in [-C, R)) of unit h. The ring is
    // stored in descending order (slot R-1 lowest, the mirror of slots 2C..3C-1
    // above slot 0), so consecutive reads of a group go upwards in LDS.
    __device__ inline uint32_t ring_addr(uint32_t h, int32_t s) const {
        return ring0 + h * G::UNIT + 2u * (uint32_t)((int32_t)R - 1 - s);
    }

    // Byte offset, from the top third, of the third holding chunk q.
    __device__ static inline uint32_t third_off(int32_t q) { return 2u * C * (uint32_t)(2 - q % 3); }

    // This lane's slice of chunk q, by a 32-bit byte offset from the scalar bitstream base.
    __device__ inline Chunk fetch(int32_t q) const {
        const uint32_t off = (uint32_t)q * (2 * C) + col * (uint32_t)sizeof(Chunk);
        return *reinterpret_cast<const Chunk *>(reinterpret_cast<const unsigned char *>(p.words) + off);
    }

    // This lane's slice (K words, ascending) of a chunk into the ring third at
    // byte offset off from the top third, words reversed; the top third is also
    // written to the mirror below slot 0.
    __device__ inline void put_chunk(uint32_t off, const Chunk &v) {
        Chunk r16;
        if constexpr (K == 4) {
            r16.x = __builtin_amdgcn_alignbit(v.y, v.y, 16);
            r16.y = __builtin_amdgcn_alignbit(v.x, v.x, 16);
        } else {
            r16.x = __builtin_amdgcn_alignbit(v.w, v.w, 16);
            r16.y = __builtin_amdgcn_alignbit(v.z, v.z, 16);
            r16.z = __builtin_amdgcn_alignbit(v.y, v.y, 16);
            r16.w = __builtin_amdgcn_alignbit(v.x, v.x, 16);
        }
        lds_st<Chunk>(lane_ring + off, r16);
        if (off == 0) lds_st<Chunk>(lane_ring + 6 * C, r16);
    }

    // Stores to the ring stay on their side of this, with respect to the read steps: those
    // are assembly that says nothing of memory. (A clobber on the read step itself would also
    // hold back the symbols' stores and the table reads: 60 streams of 4 KiB .. 16 MiB in one
    // batch 96.7 us, 104.8 with it.)
    __device__ static inline void order() { asm volatile("" ::: "memory"); }

    // Lane slice address for chunks in the top third of the ring.
    __device__ inline uint32_t lane_ring_addr() const { return ring_addr(upper, 2 * (int32_t)C + (int32_t)(K * col + K - 1)); }

    // A run of consecutive units decodes as one unit: it starts from its
    // highest unit's split point (records, first word, first group, completion
    // point) and ends at its lowest unit's last group; the split points in
    // between are not used (Sec. 3.3).
    //
    // request() reads the records and requests the first chunks, fill() writes them to
    // the ring: two rounds of memory latency, with the loads of both units of a pair and
    // of all chunks in flight together. request() touches no LDS, so the decode table is
    // staged under the second. A launch's last pair may have one run: both half-waves read
    // its records, and request() is true for the lanes of the lower one only, which decode it
    // alone (beside a partner without groups it ran predicated to its end: 4099 units of 300
    // groups 60.1 us, now 40.9; 4098 units 41.2). Two chunks: the least that leaves C words resident whatever
    // the first word's place in its chunk (every wave of the launch asks for them at once,
    // and a third one delays the first group by its share of the bandwidth).
    // Before (a chunk at a time, the units of a pair one after the other, the table
    // first) a 64 MiB stream at W = 32 in 16384 units took 43.1 us, now 41.0.
    static constexpr int32_t kFill = 2;
    struct First {
        Chunk c[kFill];
        int32_t q0;            // the lane's unit's highest chunk (-1: none)
    };
    __device__ inline bool request(uint32_t pair, First &f) {
        const bool valid = S == 1 || pair * S + upper < p.runs;
        const uint32_t mine = valid ? pair * S + upper : pair * S;
        const uint32_t lo = mine * p.run, hi = min(lo + p.run, p.units) - 1u;
        const bool last = hi + 1 == p.units;
        const bool full = last || p.partitioned;   // starts from 32-bit final states
        UnitMeta m = p.meta[hi];
        m.glo = p.meta[lo].glo;
        rec = p.lanes[(uint64_t)hi * W + coder];
        my_top = m.top;
        my_ghi = m.ghi;
        my_steps = m.top + 1 > m.glo ? m.top + 1 - m.glo : 0u;
        uint32_t sync = m.top - m.ghi + 1;
        if (full) sync = (last && (p.n_symbols % W)) ? 1u : 0u;   // only the stream's last group is ragged
        x = full ? rec : 0u;
        active = full;
        act = full ? 0u : (rec >> 16);
        sync_lean = __ballot(full) == 0;
        top0 = uni(my_top);
        steps[0] = uni(my_steps);
        presync = uni(sync);
        top_min = top0;
        if constexpr (S == 2) {
            const uint32_t t1 = __builtin_amdgcn_readlane(my_top, 32), s1 = __builtin_amdgcn_readlane(sync, 32);
            steps[1] = __builtin_amdgcn_readlane(my_steps, 32);
            top_min = min(top0, t1);
            presync = max(presync, s1);
        }
        // Fast-body store offset of this lane from unit 0's group pointer.
        lane_off = (coder + (S == 2 ? upper * W * (my_top - top0) : 0u)) * (uint32_t)sizeof(Sym);
        // Lane 4a + b of a quad writes group b of a block of four, at the column of
        // the quad's highest lane (its lowest coder): 3 - b columns below its own.
        quad_off = lane_off - 3u + (lane & 3u) + (3u - (lane & 3u)) * W;
        const int32_t cur = (int32_t)m.next;
        f.q0 = cur > 0 ? (cur - 1) / (int32_t)C : -1;
        vfq = max(f.q0 - (kFill - 1), 0);
        vres = cur - vfq * (int32_t)C;
        vpo = third_off(vfq + 2);      // chunk vfq - 1 shares a third with vfq + 2
        const uint32_t at = ring_addr(upper, cur > 0 ? (cur - 1) % (int32_t)R : 0);
        if constexpr (S == 2) {
            vb = at >> 1;
            vlim = ring_addr(upper, -1) >> 1;
            lowmask = upper ? 0u : 0xFFFFFFFFu;
        } else {
            ua[0] = uni(at);
            vfq = (int32_t)uni((uint32_t)vfq);
            vres = (int32_t)uni((uint32_t)vres);
            vpo = uni(vpo);
        }
#pragma unroll
        for (int32_t i = 0; i < kFill; ++i) f.c[i] = fetch(max(f.q0 - i, 0));
        return valid && (steps[0] > 0 || (S == 2 && steps[S - 1] > 0));
    }
    __device__ inline void fill(First &f) {
#pragma unroll
        for (int32_t i = 0; i < kFill; ++i) {
            // Both loads are waited for here, also where a chunk is not used: a load that
            // may still be in flight in the loops costs them a wait for every store.
            asm volatile("" : "+v"(f.c[i]));
            if (f.q0 >= i) put_chunk(third_off(f.q0 - i), f.c[i]);
        }
        order();
    }

    // One group's read step: the lanes with x < lim take a word each. For one unit per wave,
    // a is the unit's scalar LDS address of its next word; for a pair, e is the address of
    // the lane's own unit in words (a vector register), so that the address chain of a group
    // (compare, count, address, LDS read) has no scalar step.
    //
    // Written out because the issue of vector instructions bounds the decode (a wave64 add,
    // and, or, shift or move of vector registers takes two cycles of its SIMD, every other
    // instruction used here four): a lane that reads nothing adds a zero word to its
    // unshifted state, so the renormalisation is a masked shift and an or instead of a
    // shift-or and a select; what the address and the read do not wait for stands under
    // their latency. The wait for the read is in here with it. Against the compiler's form
    // (unmasked read, shift-or, select, scalar operands): 64 MiB at W = 32 in 16384 units
    // 44.3 -> 43.1 us, at n = 16 57.5 -> 52.1; 256 MiB at W = 32 144 -> 141; at W = 64
    // 117.4 -> 116.5, within the runs' spread.
    template <typename Lim>
    __device__ inline void read_step(Lim lim_, uint32_t &a, uint32_t &e) {
        uint32_t w, t, c, d;
        uint64_t sv;
        if constexpr (S == 2) {
            if constexpr (std::is_same<Lim, ScalarLim>::value)
                asm volatile("v_cmp_gt_u32 vcc, %[lim], %[x]\n\t" RECOIL_READ_PAIR
                             : [x] "+v"(x), [e] "+v"(e), [w] "=&v"(w), [t] "=&v"(t), [c] "=&s"(c), [d] "=&s"(d), [sv] "=&s"(sv)
                             : [lim] "s"(lim_.v), [low] "v"(lowmask), [up] "v"(upper) : "vcc", "scc");
            else
                asm volatile("v_cmp_gt_u32 vcc, %[lim], %[x]\n\t" RECOIL_READ_PAIR
                             : [x] "+v"(x), [e] "+v"(e), [w] "=&v"(w), [t] "=&v"(t), [c] "=&s"(c), [d] "=&s"(d), [sv] "=&s"(sv)
                             : [lim] "v"(lim_), [low] "v"(lowmask), [up] "v"(upper) : "vcc", "scc");
        } else if constexpr (W == 64) {
            if constexpr (std::is_same<Lim, ScalarLim>::value)
                asm volatile("v_cmp_gt_u32 vcc, %[lim], %[x]\n\t" RECOIL_READ_64
                             : [x] "+v"(x), [a] "+s"(a), [w] "=&v"(w), [t] "=&v"(t), [c] "=&s"(c), [sv] "=&s"(sv)
                             : [lim] "s"(lim_.v) : "vcc", "scc");
            else
                asm volatile("v_cmp_gt_u32 vcc, %[lim], %[x]\n\t" RECOIL_READ_64
                             : [x] "+v"(x), [a] "+s"(a), [w] "=&v"(w), [t] "=&v"(t), [c] "=&s"(c), [sv] "=&s"(sv)
                             : [lim] "v"(lim_) : "vcc", "scc");
        } else {
            if constexpr (std::is_same<Lim, ScalarLim>::value)
                asm volatile("v_cmp_gt_u32 vcc, %[lim], %[x]\n\t" RECOIL_READ_32
                             : [x] "+v"(x), [a] "+s"(a), [w] "=&v"(w), [t] "=&v"(t), [c] "=&s"(c), [sv] "=&s"(sv)
                             : [lim] "s"(lim_.v) : "vcc", "scc");
            else
                asm volatile("v_cmp_gt_u32 vcc, %[lim], %[x]\n\t" RECOIL_READ_32
                             : [x] "+v"(x), [a] "+s"(a), [w] "=&v"(w), [t] "=&v"(t), [c] "=&s"(c), [sv] "=&s"(sv)
                             : [lim] "v"(lim_) : "vcc", "scc");
        }
        if constexpr (S == 1) a = uni(a);   // no instruction: tells the compiler that the sum is uniform
    }

    // The table indices of the four groups of fast super-step k (groups inside the stream):
    // one dword per lane, lane 4a + b of a quad group b's four of the quad's coders, as
    // store_quad writes symbols. A super-step's dword is requested two super-steps ahead
    // (before: a byte per lane and group, one super-step ahead and moved from register to
    // register at its end, which waited for it and for all stores: 32 Mi symbols 46.0 us,
    // now 39.4).
    __device__ inline uint32_t load_tidx(uint32_t k) const {
        const uint8_t *b = p.tidx + (uint64_t)(top0 - k) * W;
        uint32_t v;
        __builtin_memcpy(&v, b + quad_off - 3 * W, 4);
        return v;
    }
    // Byte g of the result: this lane's index of group g (a 4 x 4 byte transpose across the
    // quad, its columns from the highest coder down).
    __device__ inline uint32_t spread_tidx(uint32_t v) const {
        const uint32_t b = lane & 3u;
        const uint32_t p2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);
        const uint32_t h = __builtin_amdgcn_perm(p2, v, (b & 2u) ? 0x00010405u : 0x06070203u);
        const uint32_t p1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)h, 0xB1, 0xF, 0xF, false);
        return __builtin_amdgcn_perm(p1, h, (b & 1u) ? 0x03070105u : 0x06020400u);
    }

    // The tables of KK groups of a predicated or synchronisation super-step, where a
    // lane's group may lie outside its unit or the stream: those lanes load nothing.
    template <uint32_t KK>
    __device__ inline void load_tidx_checked(uint32_t k) {
#pragma unroll
        for (uint32_t g = 0; g < KK; ++g) {
            const uint32_t kk = k + g;
            const uint64_t i = (uint64_t)(my_top - kk) * W + coder;
            tcur[g] = ((kk <= my_top && i < p.n_symbols) ? (uint32_t)p.tidx[i] : 0u) << (n + 2u);
        }
    }

    // Byte symbols of groups G0 .. G0 + 3 (the low bytes of v[0..3]) written as one
    // dword per lane: the four lanes of a quad hold four adjacent coders, so a 4 x 4
    // byte transpose across the quad (two DPP swaps, each followed by a byte
    // permute) leaves in lane 4a + b the four symbols of group G0 + b for coders
    // W-4-4a .. W-1-4a, in address order. One store per four groups replaces four
    // byte stores; the bytes written are the same.
    template <uint32_t G0>
    __device__ inline void store_quad(unsigned char *outh, const uint32_t (&v)[4]) const {
        const uint32_t b = lane & 3u;
        // d: byte j = this lane's symbol of group G0 + j.
        const uint32_t d = __builtin_amdgcn_perm(__builtin_amdgcn_perm(v[3], v[2], 0x00000400u),
                                                 __builtin_amdgcn_perm(v[1], v[0], 0x00000400u), 0x05040100u);
        // Swap 16-bit halves with lane b ^ 2: lanes 0, 1 keep groups 0-1, lanes 2, 3 groups 2-3.
        const uint32_t p2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)d, 0x4E, 0xF, 0xF, false);
        const uint32_t h = __builtin_amdgcn_perm(p2, d, (b & 2u) ? 0x03020706u : 0x05040100u);
        // Swap bytes with lane b ^ 1 and order the coders upwards in address.
        const uint32_t p1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)h, 0xB1, 0xF, 0xF, false);
        const uint32_t t = __builtin_amdgcn_perm(p1, h, (b & 1u) ? 0x05010703u : 0x00040206u);
        unsigned char *dst = outh + quad_off - (G0 + 3) * W;
        *reinterpret_cast<uint32_t *>(dst) = t;
        if constexpr (COUNT) {
            const uint64_t i = (uint64_t)(dst - static_cast<unsigned char *>(p.out));
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) count_store(i + j);
        }
    }

    template <uint32_t G_IDX>
    __device__ inline void group_fast(uint32_t &a, uint32_t &e, unsigned char *outh, uint32_t (&held)[4]) {
        read_step(ScalarLim{kL}, a, e);
        uint32_t s;
        if constexpr (ADAPT) s = T::step_t(x, n, mask, tcur[G_IDX]);
        else s = T::step(x, n, mask);
        if constexpr (QUAD) {
            held[G_IDX & 3u] = s;
            if constexpr ((G_IDX & 3u) == 3u) store_quad<G_IDX - 3u>(outh, held);
        } else {
            unsigned char *dst = outh + lane_off - G_IDX * W * sizeof(Sym);
            *reinterpret_cast<Sym *>(dst) = (Sym)s;
            if constexpr (COUNT) count_store((uint64_t)(dst - static_cast<unsigned char *>(p.out)) / sizeof(Sym));
        }
    }

    __device__ inline void count_store(uint64_t i) const { atomicAdd(p.counts + i, 1u); }

    template <uint32_t G_IDX>
    __device__ inline void group_pred(uint32_t k, uint32_t &a, uint32_t &e) {
        const bool live = k < my_steps;
        if (live && !active && k == act) {
            active = true;
            x = rec & 0xFFFFu;
        }
        read_step(live && active ? kL : 0u, a, e);
        const uint32_t h = my_top - k;
        const uint64_t i = (uint64_t)h * W + coder;
        if (live && active && i < p.n_symbols) {
            uint32_t s;
            if constexpr (ADAPT) s = T::step_t(x, n, mask, tcur[G_IDX]);
            else s = T::step(x, n, mask);
            if (h <= my_ghi) {
                static_cast<Sym *>(p.out)[i] = (Sym)s;
                if constexpr (COUNT) count_store(i);
            }
        }
    }

    // Synchronisation group of a pair whose units are all within their own
    // groups and below the stream's last group: only the switching-on of lanes
    // and the stores of groups above a unit's completion point are predicated.
    // Lanes not yet on decode garbage that is dropped when they switch on.
    // A lane reads while x < lim, and lim turns from 0 to L when the lane is
    // switched on, so the read predicate stays a single compare.
    template <uint32_t G_IDX>
    __device__ inline void group_sync(uint32_t k, uint32_t &a, uint32_t &e) {
        const bool on = k == act;
        x = on ? (rec & 0xFFFFu) : x;
        lim = on ? kL : lim;
        read_step(lim, a, e);
        const uint32_t h = my_top - k;
        uint32_t s;
        if constexpr (ADAPT) s = T::step_t(x, n, mask, tcur[G_IDX]);
        else s = T::step(x, n, mask);
        if (h <= my_ghi) {
            static_cast<Sym *>(p.out)[(uint64_t)h * W + coder] = (Sym)s;
            if constexpr (COUNT) count_store((uint64_t)h * W + coder);
        }
    }

    // Eighths of the share below which priority level L (1..3) ends.
    __device__ static inline uint32_t prio_cut(uint32_t L) { return L == 3 ? 4u : L == 2 ? 2u : 1u; }

    // Bodies of a super-step: unpredicated, synchronisation, fully predicated.
    static constexpr int kFast = 0, kSync = 1, kPred = 2;

    template <int MODE, uint32_t... G_IDX>
    __device__ inline void groups(std::integer_sequence<uint32_t, G_IDX...>, uint32_t k, uint32_t &a, uint32_t &e) {
        if constexpr (MODE == kPred) {
            (group_pred<G_IDX>(k + G_IDX, a, e), ...);
        } else if constexpr (MODE == kSync) {
            (group_sync<G_IDX>(k + G_IDX, a, e), ...);
        } else {
            unsigned char *outh = static_cast<unsigned char *>(p.out) + (uint64_t)(top0 - k) * W * sizeof(Sym);
            uint32_t held[4];
            (group_fast<G_IDX>(a, e, outh, held), ...);
        }
    }

    // K groups. Every step consumes at most C words and starts with at least C resident, so
    // reads stay within the ring plus its mirror.
    // Fast super-steps: the units left with fewer than C words write the chunk they
    // requested when they wrote the one above it (pre) to the ring, and request the next.
    // A request is then in flight for as long as a chunk lasts, one to three super-steps and
    // more; one super-step does not cover the latency of a cold read (before, adaptive
    // decoding of 32 Mi symbols took 53.5 us in pairs, now 47.0; n = 16, 64 MiB, 48.2 and
    // 46.8). At most 2C words are left when a chunk is written, so its third is free.
    // The others: every unit with fewer than 2C words requests its next chunk at the start
    // and writes it at the end.
    // Returns false if a unit read past its first word (corrupt split data).
    // fend: fast super-steps of the current loop are those at k' with k' + K <= fend.
    template <int MODE, uint32_t KK = K>
    __device__ inline bool super_step(uint32_t k, Chunk &pre, uint32_t fend, uint32_t &tq) {
        if constexpr (ADAPT && MODE == kFast) {
            // tq: this super-step's table indices; the next but one's are requested into it
            // when that is also fast (its groups are then inside the stream).
            const uint32_t t = spread_tidx(tq);
            if (k + 3 * K <= fend) tq = load_tidx(k + 2 * K);
#pragma unroll
            for (uint32_t g = 0; g < K; ++g) tcur[g] = ((t >> (8 * g)) & 0xFFu) << (n + 2u);
        } else if constexpr (ADAPT) {
            load_tidx_checked<KK>(k);
        }
        uint32_t a = ua[0], e = S == 2 ? vb : 0u;
        bool need = false;
        if constexpr (MODE != kFast) {
            // (Lanes of a unit that does not fetch load an in-range chunk and drop it; the
            // empty asm below keeps the chunk's use, and its wait, out of the groups.)
            need = (MODE != kPred || my_steps > k) && vfq > 0 && vres < 2 * (int32_t)C;
            pre = fetch(max(vfq - 1, 0));
        }
        groups<MODE>(std::make_integer_sequence<uint32_t, KK>{}, k, a, e);
        order();
        // Words the lane's unit consumed, from its address advance; an address that
        // moved into the mirror (below slot 0) wraps to the ring's top.
        if constexpr (S == 1) {
            vres -= (int32_t)((a - ua[0]) >> 1);
            ua[0] = a >= ring_addr(0, -1) ? a - 2 * R : a;
        } else {
            vres -= (int32_t)(e - vb);
            vb = e >= vlim ? e - R : e;
        }
        // Per lane: does this lane's unit put a chunk? (Uniform within each half-wave.)
        if constexpr (MODE == kFast) need = vfq > 0 && vres < (int32_t)C;
        else asm volatile("" : "+v"(pre));
        if (S == 1 ? need : __ballot(need) != 0) {
            if (need) {
                put_chunk(vpo, pre);
                vfq -= 1;
                vres += (int32_t)C;
                vpo = vpo == 4 * C ? 0u : vpo + 2 * C;
                if constexpr (MODE == kFast) pre = fetch(max(vfq - 1, 0));
            }
        }
        order();
        return __ballot(vres < 0) == 0;   // read below the first word: corrupt split data
    }

    // Decodes one pair whose first words have been requested. left: pairs of the wave's share
    // after this one.
    // The wave's issue priority follows the part of its share still to be
    // decoded (counted in groups with every pair as long as this one, updated
    // every super-step): 3 above one half, 2 above a quarter, 1 above an eighth,
    // else 0. The issue arbiter favours older waves; waves that fall behind are
    // given precedence so that all end together, and the last level, in which
    // the oldest wave goes first again, is kept short.
    __device__ void run(First &f, uint32_t left, uint32_t share) {
        fill(f);
        uint32_t kmax = 0, kmin = 0xFFFFFFFFu;
#pragma unroll
        for (uint32_t h = 0; h < S; ++h) {
            kmax = max(kmax, steps[h]);
            kmin = min(kmin, steps[h]);
        }
        // With rem = (left + 1) kmax - k and q = share kmax, level L > 0 holds while
        // 8 rem >= cut(L) q, i.e. until 8 k exceeds thr = 8 (left + 1) kmax - cut(L) q.
        const uint32_t q = share * kmax;
        const uint32_t r8 = 8 * (left + 1);
        uint32_t level = r8 > 4 * share ? 3u : r8 > 2 * share ? 2u : r8 > share ? 1u : 0u;
        uint32_t thr = level ? r8 * kmax - prio_cut(level) * q : 0xFFFFFFFFu;
        set_priority(level);
        // Synchronisation runs predicated, in half super-steps so that little
        // of the pair does.
        bool ok = true;
        uint32_t k = 0;
        Chunk pre;
        uint32_t tq0 = 0, tq1 = 0;   // adaptive coding only
        // The lean body needs every unit within its own groups for the whole
        // lead-in; it does not track which lanes are on, so afterwards (when all
        // are) the flag is set for the predicated body of the end.
        const uint32_t lead = (presync + K / 2 - 1) / (K / 2) * (K / 2);
        if (sync_lean && lead <= kmin) {
            lim = 0;
            for (; ok && k < presync; k += K / 2) ok = super_step<kSync, K / 2>(k, pre, 0u, tq0);
            active = true;
        } else {
            for (; ok && k < kmax && k < presync; k += K / 2) ok = super_step<kPred, K / 2>(k, pre, 0u, tq0);
        }
        // From here every state of every unit is exact, so a unit that has
        // decoded its own groups may run on into the groups below: it stores
        // there the symbols the unit below stores too, and reads that unit's
        // words. The rest of the pair then runs unpredicated in whole super-steps,
        // provided every unit is still within its own groups here (a unit that
        // ended during synchronisation stopped advancing) and running on reaches
        // neither below group 0 nor below word 0 (the first units of the stream);
        // otherwise the end runs predicated.
        const uint32_t kend = k < kmax ? k + (kmax - k + K - 1) / K * K : k;
        // Independent sub-sequences (Sec. 2.3) never run on: the states do not carry
        // over into the sub-sequence below.
        bool run_on = !p.partitioned && k <= kmin && top_min + 1 >= kend;
        run_on = run_on && __ballot(vres + vfq * (int32_t)C < (int32_t)((kend - k) * W)) == 0;
        const uint32_t fend = run_on ? kend : kmin;
        const uint32_t fast_end = run_on ? kmax : kmin - min(kmin, K - 1u);   // last start, plus one
        pre = fetch(max(vfq - 1, 0));
        auto lower_priority = [&]() {
            if (8 * k > thr) {
                --level;
                thr = level ? thr + (prio_cut(level + 1) - prio_cut(level)) * q : 0xFFFFFFFFu;
                set_priority(level);
            }
        };
        if constexpr (ADAPT) {
            // Two indices in flight, each in a register of its own.
            if (k + K <= fend) tq0 = load_tidx(k);
            if (k + 2 * K <= fend) tq1 = load_tidx(k + K);
            while (ok && k < fast_end) {
                lower_priority();
                ok = super_step<kFast>(k, pre, fend, tq0);
                k += K;
                if (!ok || k >= fast_end) break;
                ok = super_step<kFast>(k, pre, fend, tq1);
                k += K;
            }
        } else {
            for (; ok && k < fast_end; k += K) {
                lower_priority();
                ok = super_step<kFast>(k, pre, fend, tq0);
            }
        }
        for (; ok && k < kmax; k += K) ok = super_step<kPred>(k, pre, 0u, tq0);
        if (!ok && lane == 0) atomicOr(p.err, kDevErrUnderflow);
    }
};

}  // namespace dev
}  // namespace recoil
