// Decoder: g <- peeling_decompress(index, count_sketch) of Algorithm 1 (section 2.2).
//
// One workgroup per sketch partition.  The partition's unknowns are the set bits of the
// merged Index in [bounds[a], bounds[a+1]); its 3*m_sub cells live in LDS for the whole
// peel, so the rounds cost no HBM traffic and no kernel launches.
//
// Peeling is round-synchronous: the unknowns that were alone in a cell when a round began take their
// values from that cell and subtract themselves from their two others; a round that finds none
// ends the peel.  Unknowns left over are reported with value 0 and counted.
//
// The rounds are driven by cells, not by polling unknowns.  Besides its value every cell
// keeps one 32-bit word: (sum of the local ranks of its unresolved unknowns) << 16 | degree.
// When the degree is 1 the upper field *is* the remaining unknown, so a queue of the unknowns
// that have just become the last of a cell is all a round needs.  An unknown leaves a cell by an
// atomic subtraction from that word, whose old degree tells whether another one joins the queue,
// and by a compare-and-swap of the value.  It is queued once, with the cell it is to be read from:
// for the first round that is its first cell of degree 1 (every unknown looks at its three), later
// the one whose wave came first.
// (Float32 cells of an unknown that is alone in several agree up to rounding; cells that were
// rounded to 16 bits on the wire differ by that rounding, and a value with them.)
// Total work is proportional to the unknowns, not to unknowns x rounds.
#include <type_traits>

#include "device_utils.h"
#include "tagc_internal.h"

namespace tagc {

namespace {

// Optional phase timing (build with -DTAGC_PHASE_TIMING): thread 0 of every workgroup
// adds the shader-clock cycles (>> 10) each phase took to status[4 + phase].
#ifdef TAGC_PHASE_TIMING
#define PHASE_MARK(k)                                                        \
    do {                                                                     \
        if (threadIdx.x == 0) {                                              \
            const long long now_ = clock64();                                \
            atomicAdd(&status[4 + (k)], uint32_t((now_ - phase_t0_) >> 10)); \
            phase_t0_ = now_;                                                \
        }                                                                    \
    } while (0)
#define PHASE_INIT() long long phase_t0_ = clock64()
#else
#define PHASE_MARK(k) do { } while (0)
#define PHASE_INIT() do { } while (0)
#endif

constexpr uint32_t kDegBits = 16;  // of a cell's meta word: the degree

// LDS by address: a base in a scalar register and a constant of the instruction, which the compiler does
// not see in a pointer to dynamic LDS (it adds the base, 0, to every address).
template <typename T>
__device__ __forceinline__ T *lds_at(uint32_t address)
{
    return (T *)(__attribute__((address_space(3))) T *)address;
}
__device__ __forceinline__ uint32_t lds_address(void *p)
{
    uint32_t a = uint32_t((uintptr_t)(__attribute__((address_space(3))) char *)p);
    asm("" : "+s"(a));
    return a;
}

// An unknown's three cells: see PartLds::value and meta.
struct Cells {
    uint32_t at[3];
    uint32_t neg;  // bit 4 + j: sign of hash function j is -1
};

// A partition in LDS.  The cells' values and their meta words are two arrays: a wave's accesses are to
// one or the other at random cells, and interleaved they would all meet in half of the banks.
//
// kPacked: an unknown keeps where its cells are and their signs, in 40 bits (sub-tables of 4096
// cells at most); else its c-index, from which they are hashed anew.  Once resolved, its word
// holds its value.  Hashing an unknown again was a third of the vector instructions of the
// rounds (three 32-bit multiplies per hash, at quarter rate).
//
// A queue entry is an unknown and which of its three cells it is alone in.
//
// The packed form's arrays lie where the default partition size has them, whatever the size: the offsets
// of the first ones are constants of the LDS instructions then (16 bits), and a cell's value and meta
// word share an address register.
template <bool kPacked>
struct PartLds {
    static constexpr uint32_t kUnknownBits = kPacked ? 13 : 14, kOne = 1u << kUnknownBits;
    static_assert(kDefaultPartUnknowns <= 1u << 13 && kMaxPartUnknowns <= 1u << 14, "queue entry");
    static_assert(kDefaultPartCells <= 3u << 12, "packed slots are 12 bits");
    // behind n_queued [3] and handed [4] (see peel_rounds), bar (see peel_barrier)
    static constexpr uint32_t kValue = 32;
    static constexpr uint32_t kClaimed = kValue + 4 * kDefaultPartCells;
    static constexpr uint32_t kRest = kClaimed + 4 * ((kDefaultPartUnknowns / 32 + 1 + 3) & ~3u);
    static constexpr uint32_t kMeta = kRest + kDefaultPartUnknowns;
    static constexpr uint32_t kWord = kMeta + 4 * kDefaultPartCells;
    static constexpr uint32_t kQueue = kWord + 4 * kDefaultPartUnknowns;
    static constexpr uint32_t kPackedBytes = kQueue + 2 * kDefaultPartUnknowns;
    static constexpr uint32_t kStaged = kRest - 4;  // (behind the claims: see sum_peel_kernel)
    static_assert(kStaged >= kClaimed + 4 * (kDefaultPartUnknowns / 32 + 1), "a word to spare");
    static_assert(kMeta <= 0xFFFF && kMeta % 16 == 0, "offset of an LDS instruction, 16-byte stores");

    uint32_t base;     // of all of it
    uint32_t meta0;    // [T_cap] meta words
    uint32_t word0;    // [P_cap] packed slots or c-index, then the value
    uint32_t claim0;   // [P_cap/32 + 1] unknowns that are, or were, in the queue
    uint32_t queue0;   // unknown | sub-table of the cell << kUnknownBits, each unknown once
    uint32_t rest0;    // [P_cap] bytes, packed: slot_2 >> 8, and the signs in bits 4 .. 6
    uint32_t cell[3];  // address of sub-table j, less kValue
    uint32_t m_sub, fsw[3];  // folded seed words

    __device__ __forceinline__ PartLds(void *lds, uint32_t T_cap, uint32_t P_cap, uint32_t m)
    {
        base = lds_address(lds);
        if (kPacked) {
            meta0 = base + kMeta;
            word0 = base + kWord;
            claim0 = base + kClaimed;
            queue0 = base + kQueue;
            rest0 = base + kRest;
        } else {
            meta0 = base + kValue + 4 * T_cap;
            word0 = meta0 + 4 * T_cap;
            claim0 = word0 + 4 * P_cap;
            queue0 = claim0 + 4 * (P_cap / 32 + 1);
            rest0 = 0;
        }
        m_sub = m;
        for (uint32_t j = 0; j < 3; ++j) cell[j] = base + 4 * j * m;
    }
    __device__ __forceinline__ uint32_t *value(uint32_t at) const { return lds_at<uint32_t>(at + kValue); }
    __device__ __forceinline__ uint32_t *meta(uint32_t at) const
    {
        return lds_at<uint32_t>(kPacked ? at + kMeta : at + (meta0 - base));
    }
    __device__ __forceinline__ uint32_t *word(uint32_t u) const { return lds_at<uint32_t>(word0 + 4 * u); }
    __device__ __forceinline__ uint8_t *rest(uint32_t u) const
    {
        return lds_at<uint8_t>(kPacked ? base + u + kRest : rest0 + u);
    }
    // the claims of the 32 unknowns that w / 32 names
    __device__ __forceinline__ uint32_t *claims(uint32_t w) const
    {
        return lds_at<uint32_t>(kPacked ? base + 4 * (w >> 5) + kClaimed : claim0 + 4 * (w >> 5));
    }
    __device__ __forceinline__ uint16_t *queue(uint32_t e) const { return lds_at<uint16_t>(queue0 + 2 * e); }
    __device__ __forceinline__ uint32_t *n_queued(uint32_t i) const { return lds_at<uint32_t>(base + 4 * i); }
    __device__ __forceinline__ uint32_t *bar() const { return lds_at<uint32_t>(base + 12); }
    __device__ __forceinline__ uint32_t *staged() const { return lds_at<uint32_t>(base + kStaged); }
    __device__ __forceinline__ uint4 *handed() const { return lds_at<uint4>(base + 16); }
    // nobody in the first `cells` cells, nothing queued (by NT threads)
    template <uint32_t NT>
    __device__ __forceinline__ void clear(uint32_t tid, uint32_t cells) const
    {
        if (kPacked) {
#pragma unroll
            for (uint32_t i = 0; i < kDefaultPartCells / 4; i += NT)
                if (4 * (i + tid) < cells) *lds_at<uint4>(meta0 + 16 * (i + tid)) = make_uint4(0, 0, 0, 0);
        } else {
            for (uint32_t c = tid; c < cells; c += NT) *lds_at<uint32_t>(meta0 + 4 * c) = 0;
        }
        if (tid < 3) *n_queued(tid) = 0;
    }
    __device__ __forceinline__ void seed(uint64_t s, uint32_t salt)
    {
        for (uint32_t j = 0; j < 3; ++j) fsw[j] = fold16(seed_word(s, 3 * salt + j));
    }
    // unknown u has c-index i: keeps what of_unknown needs, and returns the cells
    __device__ __forceinline__ Cells place(uint32_t u, uint32_t i) const
    {
        uint32_t slot[3], neg[3];
        const uint32_t fi = fold16(i);
#pragma unroll
        for (int j = 0; j < 3; ++j) slot[j] = hash_slot_folded(fi, fsw[j], m_sub, &neg[j]);
        Cells r;
#pragma unroll
        for (int j = 0; j < 3; ++j) r.at[j] = cell[j] + 4 * slot[j];
        r.neg = (neg[0] << 4) | (neg[1] << 5) | (neg[2] << 6);
        if (kPacked) {
            *word(u) = slot[0] | (slot[1] << 12) | (slot[2] << 24);
            *rest(u) = uint8_t((slot[2] >> 8) | r.neg);
        } else {
            *word(u) = i;
        }
        return r;
    }
    // an unresolved unknown's cells
    __device__ __forceinline__ Cells of_unknown(uint32_t u) const
    {
        Cells r;
        const uint32_t w = *word(u);
        if (kPacked) {
            const uint32_t b = *rest(u);
            r.at[0] = cell[0] + 4 * (w & 0xFFFu);
            r.at[1] = cell[1] + 4 * ((w >> 12) & 0xFFFu);
            r.at[2] = cell[2] + 4 * (__builtin_amdgcn_alignbit(b, w, 24) & 0xFFFu);
            r.neg = b;
            return r;
        }
        uint32_t neg[3];
        const uint32_t fi = fold16(w);
#pragma unroll
        for (int j = 0; j < 3; ++j) r.at[j] = cell[j] + 4 * hash_slot_folded(fi, fsw[j], m_sub, &neg[j]);
        r.neg = (neg[0] << 4) | (neg[1] << 5) | (neg[2] << 6);
        return r;
    }
};

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0));
}

// First free of n slots taken off *count, by the first active lane for its wave (n uniform).
__device__ __forceinline__ uint32_t take_slots(uint32_t *count, uint32_t n)
{
    const uint32_t leader = __builtin_ctzll(__ballot(true));
    uint32_t at = 0;
    if (lane_id() == leader) at = add_by_lane(count, n);
    return __builtin_amdgcn_readlane(at, leader);
}

// The partition's n unknowns, whose c-indices are in their words, join their cells: thread t has the
// unknowns t, t + NT, ..., kIdx of them at most.  Writes the c-indices out on the way, unless kListed
// (they are there already).
template <uint32_t NT, uint32_t kIdx, bool kListed, bool kPacked>
__device__ __forceinline__ void join_cells(const PartLds<kPacked> &p, uint32_t tid, uint32_t n,
                                           uint32_t *idx_out, uint32_t (&at)[kIdx][3])
{
#pragma unroll
    for (uint32_t q = 0; q < kIdx; ++q) {
        const uint32_t u = tid + q * NT;
#pragma unroll
        for (int j = 0; j < 3; ++j) at[q][j] = p.cell[j];
        if (u < n) {
            const uint32_t i = *p.word(u);
            if (!kListed) idx_out[u] = i;
            const Cells cl = p.place(u, i);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                at[q][j] = cl.at[j];
                atomicAdd(p.meta(cl.at[j]), (u << kDegBits) + 1u);
            }
        }
    }
}

// The first round's queue: the unknowns alone in a cell once all have joined (with the first sub-table
// where it is), which every unknown's own thread finds out from its three cells, so nothing has to
// be claimed and the claims are written whole.  `any`: not if only estimates are wanted.  (Cell by
// cell, with claims in the order of the sub-tables and two barriers for that: three times the
// instructions.  This, the requests in PartAhead and the stores waited for in wait_loads: everything but the
// rounds 23.9 K -> 18.5 K clocks a partition; decoders of 2 ranks of 202 M entries 586 -> 553 us;
// with everything since 563.)
template <uint32_t NT, uint32_t kIdx, bool kPacked>
__device__ __forceinline__ void queue_first(const PartLds<kPacked> &p, uint32_t tid, uint32_t n, bool any,
                                            const uint32_t (&at)[kIdx][3])
{
    constexpr uint32_t kOne = PartLds<kPacked>::kOne;
    const uint32_t lane = lane_id();
    constexpr uint32_t kBatch = kIdx > 12 ? 2 : 4;  // whose cells are requested together
    uint32_t entry[kIdx], total = 0;
    uint64_t alone[kIdx];
#pragma unroll
    for (uint32_t q0 = 0; q0 < kIdx; q0 += kBatch) {
        uint32_t deg[kBatch][3];
#pragma unroll
        for (uint32_t q = q0; q < kIdx && q < q0 + kBatch; ++q)
#pragma unroll
            for (int j = 0; j < 3; ++j) deg[q - q0][j] = *p.meta(at[q][j]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (uint32_t q = q0; q < kIdx && q < q0 + kBatch; ++q) {
            const uint32_t u = tid + q * NT, *d = deg[q - q0];
            const bool one[3] = {uint16_t(d[0]) == 1u, uint16_t(d[1]) == 1u, uint16_t(d[2]) == 1u};
            entry[q] = u | (one[0] ? 0u : (one[1] ? kOne : 2 * kOne));
            alone[q] = __ballot((one[0] | one[1] | one[2]) & (u < n) & any);
            total += uint32_t(__popcll(alone[q]));
            // (lanes 0 and 1 have a word of the wave's 64 claims each)
            const uint32_t w = u - lane + 32 * lane;
            if (lane < 2 && w < n) *p.claims(w) = uint32_t(alone[q] >> (32 * lane));
        }
    }
    if (total == 0) return;
    uint32_t to = take_slots(p.n_queued(1), total);
#pragma unroll
    for (uint32_t q = 0; q < kIdx; ++q) {
        if ((alone[q] >> lane) & 1u) *p.queue(to + lanes_below(alone[q])) = uint16_t(entry[q]);
        to += uint32_t(__popcll(alone[q]));
    }
}

// One queue entry: an unknown that is alone in its cell `own`.  Its value is read there (nobody
// else touches a cell of degree 1) and taken out of its two other cells; an unknown that is
// thereby left alone in one is queued for the next round, from the place on that `room` has for a number
// of them.  Called by any subset of a wave's lanes; returns how many they queued.
//
// A round is a chain of dependent LDS accesses: entry -> slots -> own value, the other cells' values
// and their degrees (counted down on the way) -> the new values, and claims for the next queue ->
// queue.  Every link goes out for all cells together.  The values are swapped right behind
// their reading: cells are shared by unknowns that leave in the same round (in nearly every round of a
// wave), and what a swap found changed is left to the native add: made again, once or twice at some 200 clocks, it held
// up the whole wave (decoders of 2 ranks of 202 M entries with a tenth kept 647 -> 612 us, of 4 ranks of 9 M with two
// fifths 108 -> 104.5).  A wave that is alone with a round (kAlone: 64 entries at most) adds natively at once: a
// partition that gets stuck after 40 rounds, most of them such, 35.7 -> 34.1.  (In all rounds: sixteen waves' adds
// take 49 clocks each, a swap is not felt.)  Measured while failed swaps were still made again: a wave with one entry
// takes 1100 clocks for it, 16 full ones 2100 and a barrier 400, which is latency and the wave's own 130 instructions
// (fewer vector instructions, 87 for 110, changed nothing); a queue for every wave, without a shared count, 826 us where
// 647 were, since every wave then has a few entries of every small round; the arrays as in PartLds, and failed swaps
// made again alone and not both, took a partition's rounds from 38.8 K clocks to 32.0 K (8192 unknowns in 12288 cells, 11
// rounds) and from 51.1 K to 43.3 K (in 10776 cells, 21 rounds).
template <bool kAlone, bool kPacked, typename Room>
__device__ __forceinline__ uint32_t resolve_unknown(const PartLds<kPacked> &p, uint32_t entry, Room &&room)
{
    constexpr int kScope = __HIP_MEMORY_SCOPE_WORKGROUP;
    constexpr uint32_t kSign = 0x80000000u, kOne = PartLds<kPacked>::kOne;
    const uint32_t u = entry & (kOne - 1u);
    const bool j0 = entry < kOne, j2 = entry >= 2 * kOne;  // the sub-table of its own cell is 0; is 2
    const Cells cl = p.of_unknown(u);
    // its cell in the first and in the second of the other sub-tables
    const uint32_t own = j0 ? cl.at[0] : (j2 ? cl.at[2] : cl.at[1]);
    const uint32_t c0 = j0 ? cl.at[1] : cl.at[0], c1 = j2 ? cl.at[1] : cl.at[2];
    const uint32_t dec = (u << kDegBits) + 1u;
    const uint32_t now0 = __hip_atomic_fetch_sub(p.meta(c0), dec, __ATOMIC_RELAXED, kScope) - dec;
    const uint32_t now1 = __hip_atomic_fetch_sub(p.meta(c1), dec, __ATOMIC_RELAXED, kScope) - dec;
    uint32_t x = __hip_atomic_load(p.value(own), __ATOMIC_RELAXED, kScope);
    uint32_t v0 = 0, v1 = 0;
    if (!kAlone) {
        v0 = __hip_atomic_load(p.value(c0), __ATOMIC_RELAXED, kScope);
        v1 = __hip_atomic_load(p.value(c1), __ATOMIC_RELAXED, kScope);
    }
    __builtin_amdgcn_sched_barrier(0);  // (all five on their way before anything waits for one)
    const uint32_t n0 = cl.neg << 27, n1 = cl.neg << 26, n2 = cl.neg << 25;  // the signs in bit 31
    x ^= (j0 ? n0 : (j2 ? n2 : n1)) & kSign;
    const uint32_t t0 = x ^ ((j0 ? n1 : n0) & kSign), t1 = x ^ ((j2 ? n1 : n2) & kSign);
    auto minus = [](uint32_t v, uint32_t t) { return __float_as_uint(__uint_as_float(v) - __uint_as_float(t)); };
    uint32_t r0 = 0, r1 = 0;
    if (kAlone) {
        lds_native_add(p.value(c0), t0 ^ kSign);
        lds_native_add(p.value(c1), t1 ^ kSign);
    } else {
        r0 = atomicCAS(p.value(c0), v0, minus(v0, t0));
        r1 = atomicCAS(p.value(c1), v1, minus(v1, t1));
    }
    *p.word(u) = x;
    // Cells that came down to one unknown: its number is what is left of their sum.  It is claimed
    // in the order of the sub-tables: of two cells that it is left alone in now, it is read from
    // the first (which a wave's lanes settle by this order, and waves by who is first).
    const uint32_t left0 = now0 >> kDegBits, left1 = now1 >> kDegBits;
    const bool one0 = uint16_t(now0) == 1u, one1 = uint16_t(now1) == 1u;
    uint32_t had0 = 0xFFFFFFFFu, mid = 0xFFFFFFFFu, had1 = 0xFFFFFFFFu;
    auto claim = [&](uint32_t w) { return atomicOr(p.claims(w), 1u << (w & 31)); };
    if (one0 & !j0) had0 = claim(left0);
    if ((j0 & one0) | (j2 & one1)) mid = claim(j0 ? left0 : left1);
    if (one1 & !j2) had1 = claim(left1);
    if (j0) had0 = mid;
    if (j2) had1 = mid;
    const bool push0 = !((had0 >> (left0 & 31)) & 1u), push1 = !((had1 >> (left1 & 31)) & 1u);
    const uint64_t b0 = __ballot(push0), b1 = __ballot(push1);
    const uint32_t q0 = __popcll(b0), q1 = __popcll(b1);
    if (q0 + q1) {
        const uint32_t to = room(q0 + q1);
        if (push0) *p.queue(to + lanes_below(b0)) = uint16_t(left0 | (j0 ? kOne : 0u));
        if (push1) *p.queue(to + q0 + lanes_below(b1)) = uint16_t(left1 | (j2 ? kOne : 2 * kOne));
    }
    // Where a swap found another value the native add does it, which nobody waits for: it takes three clocks a
    // lane, but these are few.
    if (r0 != v0) lds_native_add(p.value(c0), t0 ^ kSign);
    if (r1 != v1) lds_native_add(p.value(c1), t1 ^ kSign);
    return q0 + q1;
}

// The rounds of a partition whose first queue has n_queued[1] entries, by NT threads that meet at
// `barrier`: one barrier per round.  The queue's [head, tail) holds the unknowns that the round
// before left alone in a cell.  A cell of degree 1 is touched by its own unknown only, so that
// one may read its value there at any time; every other cell is only ever changed by atomics.
// Removals of a round run concurrently with its readings, which changes
// neither the set of unknowns the round resolves (an unknown left alone in a cell now is queued
// for the next round) nor, beyond rounding order, their values.
// n_queued: per round the number of unknowns it queued for the next one, three slots used in turn:
// round r reads what round r-1 left in slot r%3 and adds to slot (r+1)%3, so a wave that is late
// into round r never sees what faster waves of the same round already write; the slot nobody
// touches in round r is cleared by thread 0 for its next use.  Returns the unknowns resolved.
//
// Rounds of up to 64 entries, of which most peels have a few and one that gets stuck has dozens, are left to
// one wave: it goes on without barriers and without a shared count until the queue is empty or longer.
// (119 partitions of 8166 unknowns in 9393 cells, stuck after 40 rounds: rounds 33.4 K -> 29.0 K clocks, decoder
// 45 -> 39 us.)
template <uint32_t NT, bool kPacked, typename Barrier>
__device__ __forceinline__ uint32_t peel_rounds(const PartLds<kPacked> &p, uint32_t tid,
                                                uint32_t &max_rounds, Barrier &&barrier)
{
    const uint32_t lane = lane_id();
    auto uniform = [](uint32_t x) -> uint32_t { return __builtin_amdgcn_readfirstlane(x); };
    uint32_t head = 0, now = 1, next = 2, spare = 0;
    for (uint32_t r = 0;; ++r) {
        barrier();  // queue, counts and cells of the previous round are complete
        uint32_t n = uniform(*p.n_queued(now));
        if (n - 1 < 64) {
            if (uniform(tid >> 6) == 0) {
                uint32_t h = head, rounds = r;
                do {
                    uint32_t queued = 0;
                    if (lane < n)
                        queued = resolve_unknown<true>(p, *p.queue(h + lane), [&](uint32_t) { return h + n; });
                    h += n;
                    n = uniform(queued);  // (lane 0 had an entry)
                    ++rounds;
                    // (the next entries, and all that is in the cells, may be other lanes' stores)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                } while (n - 1 < 64);
                if (lane == 0) *p.handed() = make_uint4(h, n, rounds, 0);
            }
            barrier();
            const uint4 left = *p.handed();
            head = uniform(left.x);
            n = uniform(left.y);
            r = uniform(left.z);
        }
        if (n == 0) {
            max_rounds = max(max_rounds, r);
            return head;
        }
        if (tid == 0) *p.n_queued(spare) = 0;  // read in the round before, added to again in the next
        const uint32_t tail = head + n;
        for (uint32_t e = head + tid; e < tail; e += NT)
            resolve_unknown<false>(p, *p.queue(e),
                            [&](uint32_t more) { return tail + take_slots(p.n_queued(next), more); });
        head = tail;
        const uint32_t was = now;
        now = next;
        next = spare;
        spare = was;
    }
}

// Output value of unknown u: unknowns never reached stay at 0 or, when the plan asks for it, are
// the median of their three signed readings of the cells as the rounds left them.
template <bool kPacked>
__device__ __forceinline__ float unknown_value(const PartLds<kPacked> &p, uint32_t u, uint32_t mode)
{
    if ((*p.claims(u) >> (u & 31)) & 1u) return __uint_as_float(*p.word(u));
    if (mode == TAGC_DECODE_PEEL) return 0.0f;
    const Cells cl = p.of_unknown(u);
    float r[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const float cv = __uint_as_float(*p.value(cl.at[j]));
        r[j] = ((cl.neg >> (4 + j)) & 1u) ? -cv : cv;
    }
    return fmaxf(fminf(r[0], r[1]), fminf(fmaxf(r[0], r[1]), r[2]));
}

__device__ inline void report_unresolved(uint32_t n, uint32_t mode, uint32_t *status)
{
    if (!n) return;
    atomicAdd(&status[TAGC_ST_UNRESOLVED], n);
    if (mode != TAGC_DECODE_PEEL) atomicAdd(&status[TAGC_ST_ESTIMATED], n);
}

// The merged Index, as the Index aggregation left it.
struct IndexView {
    const uint32_t *bitmap;
    const uint32_t *chunkpre;   // set bits before every chunk
    const uint16_t *grouppre;   // ... and from there before every group of 64 words
    const uint32_t *bounds;     // first c-index of every partition
    uint32_t n_words, n_chunks;
    const uint32_t *list;       // kListed: its set bits, ascending (the caller's idx_out)
};

// Enumerates the set bits of the merged Index in ascending order into idx_out, for the kListed
// forms of the decoder.  One workgroup per 1024-word chunk; chunkpre[] (written by the Index
// aggregation) holds the number of set bits before each chunk, so workgroups are independent.  A
// thread's indices are consecutive in the output but a wave's stores, taken entry by entry, would
// hit 64 different cache lines each; so the chunk's first kEnumStage indices are gathered
// in LDS and leave as contiguous stores.
constexpr uint32_t kEnumStage = 8192;

__global__ void __launch_bounds__(256)
enumerate_kernel(const IndexView index, const uint32_t *__restrict__ header,
                 uint32_t *__restrict__ idx_out)
{
    __shared__ uint32_t scratch[8];
    __shared__ uint32_t stage[kEnumStage];
    const uint32_t U = header[TAGC_HDR_U];
    const uint32_t w0 = blockIdx.x * kChunkWords + threadIdx.x * 4;
    uint32_t w[4] = {0, 0, 0, 0};
    if (w0 + 4 <= index.n_words) {
        const uint4 q = *reinterpret_cast<const uint4 *>(index.bitmap + w0);
        w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
    } else {
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) w[i] = w0 + i < index.n_words ? index.bitmap[w0 + i] : 0u;
    }
    const uint32_t mine = __popc(w[0]) + __popc(w[1]) + __popc(w[2]) + __popc(w[3]);
    uint32_t tot;
    const uint32_t base = index.chunkpre[blockIdx.x];
    uint32_t pl = block_excl_scan<uint32_t, 4>(mine, &tot, scratch);  // position in the chunk
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        for (uint32_t word = w[i]; word; word &= word - 1) {
            const uint32_t v = (w0 + i) * 32 + uint32_t(__builtin_ctz(word));
            if (pl < kEnumStage) stage[pl] = v;
            else if (base + pl < U) idx_out[base + pl] = v;
            ++pl;
        }
    }
    __syncthreads();
    const uint32_t n = min(tot, kEnumStage);
    for (uint32_t i = threadIdx.x; i < n; i += 256)
        if (base + i < U) idx_out[base + i] = stage[i];
}

// The unknowns of a partition are the set bits of the merged Index from bounds[a] on, numbered as
// they come.  A wave turns the Index into unknowns by groups of 64 words, one per lane; since the
// set bits before every group are known, groups are independent of each other.  The kPre groups
// that a wave has of nearly every partition are requested a partition ahead.  (As a kernel of its
// own, whose output the decoder reads back, this takes 5 us on small buckets and 43 to 53 on those of
// 7 to 38 M unknowns; it is left to one where little is set, see launch_decode.)
template <uint32_t NW, uint32_t kPre>
struct PartIndex {
    uint32_t lo, hi;        // the partition's c-indices
    uint32_t g_end;         // behind its last group; 0 if it has no unknowns, and so no groups
    uint32_t word[kPre];    // word `lane` of the wave's groups
    uint32_t before[2];     // lane i: set bits of the whole Index before the i-th of them, to be added up

    static constexpr uint32_t kTail = 8;
    static_assert(kPre <= 64, "a lane per group");
    __device__ __forceinline__ uint32_t load(const IndexView &v, uint32_t g) const
    {
        const uint32_t w = g * kGroupWords + lane_id();
        return g < g_end && w < v.n_words ? v.bitmap[w] : 0u;
    }
    __device__ __forceinline__ static uint32_t bits_before(const IndexView &v, uint32_t g)
    {
        return v.chunkpre[g / 16] + (g < v.n_chunks * 16 ? v.grouppre[g] : 0u);
    }
    __device__ __forceinline__ void request(const IndexView &v, uint32_t from, uint32_t to, uint32_t wave)
    {
        lo = from;
        hi = to;
        // (lo == hi where partitions outnumber the non-zeros, and both are 0 if c-index 0 is one;
        // no group lies behind the Index whatever the bounds hold)
        g_end = lo < hi ? min((hi - 1) / (32 * kGroupWords) + 1, (v.n_words + kGroupWords - 1) / kGroupWords)
                        : 0u;
        const uint32_t g0 = lo / (32 * kGroupWords) + wave;
#pragma unroll
        for (uint32_t i = 0; i < kPre; ++i) word[i] = load(v, g0 + i * NW);
        const uint32_t gl = g0 + lane_id() * NW;
        // (added up where they are needed: nothing here waits for a load)
        const bool ok = lane_id() < kPre && gl < g_end;
        before[0] = ok ? v.chunkpre[gl / 16] : 0u;
        before[1] = ok && gl < v.n_chunks * 16 ? v.grouppre[gl] : 0u;
    }
    // word `lane` of group g, with `pre` set bits before the group: its unknowns' c-indices
    __device__ __forceinline__ void expand(uint32_t *out, uint32_t n, uint32_t rho0, uint32_t g,
                                           uint32_t w, uint32_t pre) const
    {
        const uint32_t inc = wave_incl_scan<uint32_t>(uint32_t(__popc(w)));
        uint32_t u = pre - rho0 + inc - uint32_t(__popc(w));
        const uint32_t c0 = (g * kGroupWords + lane_id()) * 32;
        if (c0 < lo) {  // bits of the partition before
            const uint32_t low = lo - c0 >= 32 ? w : w & ((1u << (lo - c0)) - 1u);
            u += __popc(low);
            w ^= low;
        }
        if (hi - c0 < 32) w &= (1u << (hi - c0)) - 1u;  // (c0 >= hi: below)
        // (nothing lands outside out[0 .. n) whatever the Index holds)
        if (c0 >= hi || u > n || uint32_t(__popc(w)) > n - u) w = 0;
        for (out += u; w; w &= w - 1) *out++ = c0 + uint32_t(__builtin_ctz(w));
    }
    // the partition's n unknowns, of which rho0 lie in partitions before, into out[]
    __device__ __forceinline__ void enumerate(const IndexView &v, uint32_t *out, uint32_t n,
                                              uint32_t rho0, uint32_t wave) const
    {
        const uint32_t g0 = lo / (32 * kGroupWords) + wave, pre = before[0] + before[1];
#pragma unroll
        for (uint32_t i = 0; i < kPre; ++i)
            if (g0 + i * NW < g_end)
                expand(out, n, rho0, g0 + i * NW, word[i], __builtin_amdgcn_readlane(pre, i));
        // The rest (partitions of far fewer unknowns than the plan has room for), 64 of the wave's
        // groups at a time, a lane finding out what lies before each and whether it holds anything:
        // kTail of those that do are on their way together.  (Four at a time, holding anything or
        // not: 10 partitions of 20 M positions 329 us, 189 in this form; 16 at a time 190.)
        for (uint32_t gb = g0 + kPre * NW; gb < g_end; gb += 64 * NW) {
            const uint32_t gl = gb + lane_id() * NW;
            const uint32_t at = gl < g_end ? bits_before(v, gl) : 0u;
            const uint32_t behind = gl < g_end ? bits_before(v, gl + 1) : 0u;
            for (uint64_t some = __ballot(behind != at); some;) {
                uint32_t w[kTail], i[kTail];
#pragma unroll
                for (uint32_t k = 0; k < kTail; ++k) {
                    i[k] = some ? uint32_t(__builtin_ctzll(some)) : 64u;
                    some &= some - 1;
                    w[k] = i[k] < 64 ? load(v, gb + i[k] * NW) : 0u;
                }
#pragma unroll
                for (uint32_t k = 0; k < kTail; ++k)
                    if (i[k] < 64)
                        expand(out, n, rho0, gb + i[k] * NW, w[k], __builtin_amdgcn_readlane(at, i[k]));
            }
        }
    }
};

// A partition's unknowns where they have been listed: requested a partition ahead as well.
template <uint32_t NT, uint32_t kIdx>
struct PartList {
    uint32_t idx[kIdx];

    // n c-indices from `list` on
    __device__ __forceinline__ void request(const uint32_t *list, uint32_t n, uint32_t tid)
    {
#pragma unroll
        for (uint32_t q = 0; q < kIdx; ++q) {
            const uint32_t u = tid + q * NT;
            idx[q] = u < n ? __builtin_nontemporal_load(list + u) : 0u;
        }
    }
    __device__ __forceinline__ void put(uint32_t *out, uint32_t n, uint32_t tid) const
    {
#pragma unroll
        for (uint32_t q = 0; q < kIdx; ++q) {
            const uint32_t u = tid + q * NT;
            if (u < n) out[u] = idx[q];
        }
    }
};

// Rank r's sketch: read from the kernel argument segment (explicit arguments lie there in
// declaration order at their natural alignment, the RankPtrs first), because indexing the argument
// with a run-time r would keep all 32 pointers in registers (a pointer made from an integer has no
// address space the compiler knows: it is declared global here, or every load through it would be
// a flat one, which can only be waited for all at once).
typedef __attribute__((address_space(1))) const float *GlobalCells;
__device__ __forceinline__ GlobalCells rank_sketch(uint32_t r)
{
    typedef __attribute__((address_space(4))) const uint64_t *KernArg;
    KernArg ka = (KernArg)__builtin_amdgcn_kernarg_segment_ptr();
    return (GlobalCells)ka[r];
}

// Four cells of a sketch from any of them on (a partition starts at any multiple of 4 bytes), and put into LDS.
// (One at a time it is four times the instructions, and a wave's loads leave one every 16 clocks: decoders of 2
// ranks of 202 M entries with a tenth kept 671 -> 652 us, sum_peel of 8 ranks of 7 M entries 50.4 -> 48.6.)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void request_four(float *v, GlobalCells src)
{
    const f32x4_any q = __builtin_nontemporal_load((__attribute__((address_space(1))) const f32x4_any *)src);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
}
// cells c .. c + 3 of a partition of `cells`, at `to`
__device__ __forceinline__ void stage_four(uint32_t to, const float *v, uint32_t c, uint32_t cells)
{
    if (c + 4 <= cells) {
        *lds_at<float4>(to) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
            if (c + e < cells) *lds_at<float>(to + 4 * e) = v[e];
    }
}

// A workgroup's partitions a, a + step, ...: partition a has the unknowns [aU/A, (a+1)U/A).  (Divided once
// and counted on: a 64-bit division is some hundred scalar instructions, for every wave.)
struct Partitions {
    uint32_t A, a, step;
    uint32_t rho, rem;            // aU/A, and what is left of it
    uint32_t rho_step, rem_step;  // of step * U
    uint32_t rho_one, rem_one;    // of U

    __device__ __forceinline__ Partitions(uint32_t U, uint32_t n, uint32_t first, uint32_t by)
        : A(n), a(first), step(by)
    {
        rho = uint32_t(uint64_t(a) * U / A);
        rem = uint32_t(uint64_t(a) * U - uint64_t(rho) * A);
        rho_step = uint32_t(uint64_t(step) * U / A);
        rem_step = uint32_t(uint64_t(step) * U - uint64_t(rho_step) * A);
        rho_one = U / A;
        rem_one = U % A;
    }
    __device__ __forceinline__ uint32_t unknowns() const { return rho_one + (rem >= A - rem_one); }
    __device__ __forceinline__ void next()
    {
        const uint32_t carry = rem >= A - rem_step;
        rho += rho_step + carry;
        rem = carry ? rem - (A - rem_step) : rem + rem_step;
        a += step;
    }
};

// Bounds and salt of a partition, requested a partition before they say what else to request.  They were
// written by the kernel before on some other compute die, so they take a microsecond or two: waited for
// where they were needed, they and what waited behind them were 5 K of a partition's 67 K clocks.
struct PartAhead {
    uint32_t v;  // lanes 0 and 1: the bounds, lane 2: the salt
    __device__ __forceinline__ void request(const IndexView &index, const uint32_t *salt, uint32_t a,
                                            uint32_t A)
    {
        v = 0;
        if (a < A) first(index, salt, a);
    }
    // (a is inside the room for partitions, whose salts lie behind the bounds and one more)
    __device__ __forceinline__ void first(const IndexView &index, const uint32_t *salt, uint32_t a)
    {
        const uint32_t lane = lane_id();
        v = index.bounds[a + (lane == 2 ? uint32_t(salt - index.bounds) : uint32_t(lane == 1))];
    }
    __device__ __forceinline__ uint32_t get(uint32_t i) const { return __builtin_amdgcn_readlane(v, i); }
};

// Everything requested so far is there.  Placed where it is so anyway, in front of stores: without it
// the first use behind them would wait for them as well.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)

// The dense output of a partition's range [lo, hi) of c-indices, by a workgroup whose thread t has the
// unknowns t, t + NT, ...: put together in the LDS of the partition, which nobody needs any more, 36864
// floats at a time -- zeros, the unknowns' values among them, out in 16-byte stores that travel while the
// next partition is peeled.  Bound by the LDS (written, written to, read: 43 thousand floats a partition
// take 14 K clocks on top of the peel's 70 K), against 170 us of dense_kernel for 202 M entries, which
// is bound by the stores.
template <uint32_t NT, uint32_t kIdx>
__device__ __forceinline__ void write_dense(const PartLds<true> &p, uint32_t tid, const uint32_t (&idx)[kIdx],
                                            const float (&val)[kIdx], uint32_t lo, uint32_t hi,
                                            float *__restrict__ out)
{
    constexpr uint32_t kTurns = kDensePiece / (4 * NT);
    static_assert(kDensePiece == 4 * kTurns * NT && PartLds<true>::kValue % 16 == 0 &&
                      PartLds<true>::kValue + 4 * kDensePiece <= PartLds<true>::kPackedBytes,
                  "a piece is whole turns and lies inside the partition's LDS");
    const uint32_t area = p.base + PartLds<true>::kValue;
    if (lo >= hi) return;
    DensePieces piece(lo, hi);
    do {
        const uint32_t p0 = piece.at, n = piece.n;
#pragma unroll 3
        for (uint32_t i = 0; i < kTurns; ++i) {
            const uint32_t at = 4 * (tid + i * NT);
            if (at < n) *lds_at<float4>(area + 4 * at) = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < kIdx; ++q)
            if (idx[q] - p0 < n) *lds_at<float>(area + 4 * (idx[q] - p0)) = val[q];
        __syncthreads();
#pragma unroll 3
        for (uint32_t i = 0; i < kTurns; ++i) {
            const uint32_t at = 4 * (tid + i * NT), c = p0 + at;
            if (at >= n) continue;
            const float4 v = *lds_at<float4>(area + 4 * at);
            if (c >= lo && c + 4 <= hi) {
                st_stream(reinterpret_cast<float4 *>(out + c), v);
            } else {  // the neighbours' entries are not this partition's to write
                const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e)
                    if (c + e >= lo && c + e < hi) out[c + e] = x[e];
            }
        }
    } while (piece.next());
}

// The zeros of the dense output, by workgroup `b` of `n` that have no partition: the entries whose Index bit is
// not set, and no others, so that nobody has to wait for whom writes the others; all of them where there is no
// partition (after an overflow, when bits are set all the same).  A wave takes 16 words at a time, the next of
// which are on their way.
constexpr uint32_t kZeroWords = 16;
__device__ __forceinline__ void write_zeros(const IndexView &index, uint32_t b, uint32_t n, bool all,
                                            float *__restrict__ out)
{
    const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t step = n * (kDecodeThreads / 64) * kZeroWords;
    auto request = [&](uint32_t w) { return lane < kZeroWords && w + lane < index.n_words ? index.bitmap[w + lane] : 0u; };
    uint32_t w0 = (b * (kDecodeThreads / 64) + wave) * kZeroWords;
    uint32_t next = w0 < index.n_words ? request(w0) : 0u;
    for (; w0 < index.n_words; w0 += step) {
        const uint32_t word = all ? 0u : next;
        if (w0 + step < index.n_words) next = request(w0 + step);
        float *to = out + 32 * uint64_t(w0) + lane;
#pragma unroll
        for (uint32_t i = 0; i < kZeroWords; i += 2) {
            if (w0 + i >= index.n_words) break;
            const uint32_t lo = __builtin_amdgcn_readlane(word, i), hi = __builtin_amdgcn_readlane(word, i + 1);
            const bool there = lane < 32 || w0 + i + 1 < index.n_words;
            if (there && !(((lane < 32 ? lo : hi) >> (lane & 31)) & 1u)) to[32 * i] = 0.0f;
        }
    }
}

// Peels sketch partitions: unknowns rho .. rho+Pa-1 in order of c-index, cells a*3*m_sub ...
//
// The LDS a partition needs leaves room for one workgroup per CU, and the rounds are bound
// by LDS latency, not by memory.  So the grid is one workgroup per CU, each taking
// partitions b, b+G, ...; while one partition is being peeled the cells and Index words of
// the workgroup's next one are already on their way into registers, and staging it costs
// LDS stores only.
// kCellPre / kIdxPre: cells / unknowns per thread the instantiation can hold.
// kRanks: the cells are summed over the n_in <= kRanks ranks here, in rank order, the ranks' cells of
// the next partition staying in the registers they are loaded to until it is staged.
// kLoop: over any number of ranks, or the summed sketch, added up as they come.  For grids that have a workgroup for
// every partition: there is no next partition whose sum could run beside the rounds, as
// sum_peel_kernel has it (40 partitions of 8 ranks: 27.7 us, 28.9 in that kernel; 51 of 5: 27.5, 30.1; 159 of 8: 31.1,
// 31.3; 239 of 8: 35.6, 34.5; 233 of 12: 39.8, 41.4).  Nor is there one before, whose rounds its cells could travel
// behind: the Index words are requested first and the unknowns enumerated, joined and looked through for the first queue,
// none of which needs a value, while the cells travel (8 ranks of 25 M entries 40.4 -> 38.0, 3 of 36 thousand, one
// partition, 18.6 -> 15.9, 4 of 1 M 20.8 -> 17.9, a summed sketch in 236 partitions 32.0 -> 29.4).
constexpr uint32_t kIndexPre = 6;  // groups of Index words a wave requests ahead
constexpr uint32_t kHeldRanks = 4;  // kRanks of the form for few ranks
constexpr uint32_t kListGroups = 256;  // groups of Index words per partition beyond which its unknowns are listed first
// kListed: the unknowns are in index.list.
// kDense: writes the dense output of the partitions that dense_by_decoder names as well (dense_rest_kernel
// has the others'); with kLoop all of it, its partitions' values where they belong, and the workgroups that have no
// partition the zeros (write_zeros).  Where that is stands behind the ranks' sketches: an argument of its own is two scalar
// registers too many.
constexpr uint32_t kDenseRow = kMaxRanksPerPass - 1;
static_assert(kDenseRow >= kHeldRanks, "the forms that write it have few ranks");
__device__ __forceinline__ float *dense_row() { return (float *)(rank_sketch(kDenseRow)); }
template <uint32_t kCellPre, uint32_t kIdxPre, bool kPacked, uint32_t kRanks, bool kLoop, bool kListed,
          bool kDense>
__global__ void __launch_bounds__(kDecodeThreads)
peel_kernel(const RankPtrs, uint32_t n_in, const IndexView index, const uint32_t *__restrict__ header,
            uint32_t *__restrict__ idx_out, float *__restrict__ val_out,
            uint32_t *status, uint64_t seed, const uint32_t *__restrict__ salt, uint32_t T_cap,
            uint32_t P_cap, uint32_t mode)
{
    extern __shared__ __align__(16) uint64_t lds64[];
    const uint32_t tid = threadIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    PartAhead ahead;
    // (workgroups beyond the room for partitions, which only write zeros, ask for what the last of it holds)
    ahead.first(index, salt, kLoop && kDense ? min(blockIdx.x, uint32_t(salt - index.bounds) - 2u) : blockIdx.x);
    const uint32_t U = header[TAGC_HDR_U], A = header[TAGC_HDR_A];
    const uint32_t m_sub = header[TAGC_HDR_MSUB];
    const uint32_t cells = 3 * m_sub;
    if (blockIdx.x >= A) {
        if (kLoop && kDense) write_zeros(index, blockIdx.x - A, gridDim.x - A, A == 0, dense_row());
        return;
    }
    PartLds<kPacked> part(lds64, T_cap, P_cap, m_sub);

    // the cells and Index words (or unknowns) of partition `p` into registers (zeros beyond their
    // ends)
    float pre_cell[kRanks][kCellPre];
    PartIndex<kDecodeThreads / 64, kIndexPre> pre_index;
    PartList<kDecodeThreads, kIdxPre> pre_list;
    // (the form for larger partitions has no runs of four registers to spare)
    constexpr uint32_t kFour = kPacked ? 4 : 1;
    auto request_cells = [&](float (&v)[kCellPre], uint32_t r, uint64_t tile) {
        const GlobalCells src = rank_sketch(r) + tile;
#pragma unroll
        for (uint32_t q = 0; q < kCellPre; q += kFour) {
            const uint32_t c = kFour * tid + q * kDecodeThreads;
            if (kFour == 1) v[q] = c < cells ? __builtin_nontemporal_load(src + c) : 0.0f;
            else if (c < cells) request_four(v + q, src + c);  // (a sketch has room for three more cells)
            else v[q] = v[q + 1] = v[q + 2] = v[q + 3] = 0.0f;
        }
    };
    // adds the ranks held from the first-th on to the first one
    auto add_cells = [&](uint32_t first, uint32_t n) {
#pragma unroll
        for (uint32_t i = 1; i < kRanks; ++i)
            if (i >= first && i < n)
#pragma unroll
                for (uint32_t q = 0; q < kCellPre; ++q) pre_cell[0][q] += pre_cell[i][q];
    };
    auto request_unknowns = [&](const Partitions &at) {
        if (kListed) pre_list.request(index.list + at.rho, at.unknowns(), tid);
        else pre_index.request(index, ahead.get(0), ahead.get(1), wave);
    };
    auto request_first = [&](uint64_t tile) {
#pragma unroll
        for (uint32_t i = 0; i < kRanks; ++i)
            if (i < n_in) request_cells(pre_cell[i], i, tile);
    };
    // (kLoop) adds up the ranks requested, and requests those from r on
    auto request_more = [&](uint32_t r, uint64_t tile) {
        __builtin_amdgcn_sched_barrier(0);
        add_cells(1, kRanks);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (uint32_t i = 1; i < kRanks; ++i)
            if (r + i - 1 < n_in) request_cells(pre_cell[i], r + i - 1, tile);
            else
#pragma unroll
                for (uint32_t q = 0; q < kCellPre; ++q) pre_cell[i][q] = -0.0f;  // (x + -0 is x)
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr uint32_t kMore = kRanks - 1;  // ranks of a step of it
    Partitions at(U, A, blockIdx.x, gridDim.x);
    uint32_t sa = 0;
    // the partition `at` is at; `ahead` holds what is needed for it, and then that of the one after it
    auto prefetch = [&] {
        sa = ahead.get(2);
        request_unknowns(at);
        ahead.request(index, salt, at.a + at.step, A);
    };
    const uint64_t tile0 = uint64_t(at.a) * cells;
    if (kLoop) {  // (the Index words first: see below)
        prefetch();
        request_first(tile0);
    } else {
        request_first(tile0);  // (these do not need the bounds)
        prefetch();
        wait_loads();
    }

    uint32_t max_rounds = 0;
    while (at.a < A) {
    PHASE_INIT();
    const uint32_t rho0 = at.rho, Pa = at.unknowns();
    // the partition's hash functions: the seed under the salt the encoders used
    part.seed(seed, sa);

    // (addresses that follow from the thread's number are made anew for every partition: kept from one
    // to the next they take the registers that the prefetch needs)
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));

    // ---- stage the partition's cells and unknowns from the registers, clear state
    part.template clear<kDecodeThreads>(tid, cells);
    if (kListed) pre_list.put(part.word(0), Pa, tid);
    else pre_index.enumerate(index, part.word(0), Pa, rho0, wave);
    auto stage_cells = [&] {
        add_cells(1, n_in);
        const uint32_t to = part.base + PartLds<kPacked>::kValue + 4 * kFour * tid;
#pragma unroll
        for (uint32_t q = 0; q < kCellPre; q += kFour) {
            const uint32_t c = kFour * tid + q * kDecodeThreads, at = to + 4 * q * kDecodeThreads;
            if (kFour == 4) stage_four(at, pre_cell[0] + q, c, cells);
            else if (c < cells) *lds_at<float>(at) = pre_cell[0][q];
        }
    };
    if (!kLoop) stage_cells();
    else if (n_in > kRanks) request_more(kRanks, tile0);
    __syncthreads();
    PHASE_MARK(0);

    // The registers are free again: the next partition's data is requested a rank at a time between the steps, and
    // travels during the rounds.  (All of it in front of the rounds kept every wave from its first one for
    // as long as the memory takes for what the whole device requests at that moment: 4 ranks of 9 M entries with two
    // fifths kept 117 -> 108 us, with the dense output, whose stores are on their way first, 652 -> 647.)
    at.next();
    auto request_next = [&](uint32_t r) {
        if (!kLoop && at.a < A && r < n_in) request_cells(pre_cell[r < kRanks ? r : 0], r, uint64_t(at.a) * cells);
    };
    // Ranks requested before the join, and by its end: none before it where a dense output is on its way, and none at all
    // in front of the first queue in the form for larger partitions, which has no registers for that.
    constexpr uint32_t kBefore = kPacked && !(kDense && !kLoop) ? 1 : 0, kJoined = kPacked ? kBefore + 1 : 0;
    if (kBefore && !kLoop && at.a < A) prefetch();
    if (kBefore) request_next(0);
    uint32_t cell[kIdxPre][3];
    join_cells<kDecodeThreads, kIdxPre, kListed>(part, tid, Pa, idx_out + rho0, cell);
    if (kRanks > kBefore && kJoined > kBefore) request_next(kBefore);
    if (kLoop && n_in > kRanks + kMore) request_more(kRanks + kMore, tile0);
    __syncthreads();
    queue_first<kDecodeThreads, kIdxPre>(part, tid, Pa, mode != TAGC_DECODE_ESTIMATE, cell);
    if (!kBefore && !kLoop && at.a < A) prefetch();
#pragma unroll
    for (uint32_t r = kJoined; r < kRanks; ++r) request_next(r);
    // With a workgroup for every partition the ranks' cells travel and are added up beside all that, which needs no
    // values: those are only wanted now.
    if (kLoop) {
        for (uint32_t r = kRanks + 2 * kMore; r < n_in; r += kMore) request_more(r, tile0);
        stage_cells();
    }
    uint32_t idx[kDense ? kIdxPre : 1];
    if constexpr (kDense) {  // (this thread wrote them in join_cells; back long before the rounds are over)
#pragma unroll
        for (uint32_t q = 0; q < kIdxPre; ++q) {
            const uint32_t u = tid + q * kDecodeThreads;
            idx[q] = u < Pa ? idx_out[rho0 + u] : 0xFFFFFFFFu;
        }
    }
    PHASE_MARK(1);

    const uint32_t resolved =
        peel_rounds<kDecodeThreads>(part, tid, max_rounds, [] { __syncthreads(); });
    PHASE_MARK(2);

    // ---- values leave in one contiguous sweep (stored one by one as they were found they
    // would cost a cache-line access each)
    wait_loads();
    if constexpr (kDense) {
        asm volatile("" : "+v"(tid));  // (as above)
        float val[kIdxPre];
#pragma unroll
        for (uint32_t q = 0; q < kIdxPre; ++q) {
            const uint32_t u = tid + q * kDecodeThreads;
            val[q] = u < Pa ? unknown_value(part, u, mode) : 0.0f;
            if (u < Pa) val_out[rho0 + u] = val[q];
            // (a word of the partition that no set bit has filled holds anything, should the Index have changed
            // since it was merged: nothing lands outside the output)
            if (kLoop && idx[q] < 32 * index.n_words) dense_row()[idx[q]] = val[q];
        }
        // all c-indices lie in a partition's range, those before the first unknown in the first one's
        // (read again: kept, the bounds take a vector register to spill)
        const uint32_t a = at.a - at.step;
        const uint32_t lo = !kLoop && a ? index.bounds[a] : 0u;
        const uint32_t hi = kLoop ? 0u : min(index.bounds[a + 1], 32 * index.n_words);
        if (!kLoop && dense_by_decoder(A, gridDim.x, 32 * index.n_words, hi - lo)) {
            __syncthreads();
            write_dense<kDecodeThreads, kIdxPre>(part, tid, idx, val, lo, hi, dense_row());
        }
    } else {
        for (uint32_t u = tid; u < Pa; u += kDecodeThreads)
            val_out[rho0 + u] = unknown_value(part, u, mode);
    }
    if (tid == 0) report_unresolved(Pa - resolved, mode, status);
    PHASE_MARK(3);
    if (kLoop) break;
    __syncthreads();  // before the next partition is staged
    }  // partitions of this workgroup
    if (tid == 0 && max_rounds) atomicMax(&status[TAGC_ST_ROUNDS], max_rounds);
}

// ------------------------------------------------- sketch sum inside the decoder
//
// Reduce(count_sketch) and peeling_decompress of Algorithm 1 in one kernel, without a summed
// sketch in memory.  The rounds of a partition are bound by dependent LDS accesses and leave
// the memory system idle; adding up the ranks' sketches is bound by memory and leaves
// everything else idle; run one after the other they cost the sum.  Here a workgroup's 16
// waves split up: kLoadWaves of them do nothing but add up, in rank order, the cells of the
// workgroup's *next* partition in their registers (48 cells per thread), while the other
// kPeelWaves peel the current one in LDS as peel_kernel does.  The two groups meet once per
// partition, at a hardware barrier: when the peelers are done with the LDS.  The loaders then
// write the summed cells there, say so in an LDS word, and go on; the peelers enumerate, join and queue the
// partition's unknowns, none of which needs a value, and look at that word before the rounds.  (With a
// second barrier there, the peelers of a workgroup's first partition began with the unknowns when its cells
// had been summed.  us, that way / this: 8 ranks of 7 M entries, 325 partitions, 47.7 / 41.4, of 67 M, 433,
// 77.1 / 67.5, 16 of 202 M, 3640, 551 / 552.)  The peelers' own barriers (after the unknowns joined their
// cells, one per round) must not hold up the loaders, which have no part in them and may be waiting for
// memory: they are counted in an LDS word instead (peel_barrier).
constexpr uint32_t kLoadWaves = 4, kPeelWaves = kDecodeThreads / 64 - kLoadWaves;
constexpr uint32_t kLoadThreads = kLoadWaves * 64, kPeelThreads = kPeelWaves * 64;
constexpr uint32_t kLoadCells = (kDefaultPartCells + kLoadThreads - 1) / kLoadThreads;  // per thread
constexpr uint32_t kUnit = 16;  // cells of one rank a loader thread requests at a time
static_assert(kLoadCells == 3 * kUnit, "a rank's cells are three units per loader thread");
constexpr uint32_t kPeelIdx = (kDefaultPartUnknowns + kPeelThreads - 1) / kPeelThreads;

// Barrier among the kPeelWaves peeling waves: every wave adds 1 to an LDS word and goes on
// when the word has reached kPeelWaves x (barriers so far).  All waves of a workgroup are
// resident and every peeling wave reaches every such barrier (they branch on the same LDS
// words), so the wait ends.
__device__ inline void peel_barrier(uint32_t *word, uint32_t &expected)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // this wave's LDS accesses are done
    expected += kPeelWaves;
    if (lane_id() == 0) atomicAdd(word, 1u);
    while (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < expected)
        __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

template <bool kListed>
__global__ void __launch_bounds__(kDecodeThreads)
sum_peel_kernel(const RankPtrs, uint32_t n_in, const IndexView index,
                const uint32_t *__restrict__ header, uint32_t *__restrict__ idx_out,
                float *__restrict__ val_out,
                uint32_t *status, uint64_t seed, const uint32_t *__restrict__ salt,
                uint32_t T_cap, uint32_t P_cap, uint32_t mode)
{
    extern __shared__ __align__(16) uint64_t lds64[];
    const uint32_t tid = threadIdx.x;
    PartAhead ahead;  // (the peelers')
    ahead.first(index, salt, blockIdx.x);
    const uint32_t U = header[TAGC_HDR_U], A = header[TAGC_HDR_A];
    const uint32_t m_sub = header[TAGC_HDR_MSUB];
    const uint32_t cells = 3 * m_sub;
    PartLds<true> part(lds64, T_cap, P_cap, m_sub);
    if (blockIdx.x >= A) return;
    if (tid == 0) *part.bar() = *part.staged() = 0;
    __syncthreads();

    if (tid >= kPeelThreads) {
        // ------------------------------------------------------------ the loaders
        const uint32_t lt = tid - kPeelThreads;
        float acc[kLoadCells];
        float b0[kUnit], b1[kUnit], b2[kUnit];
        // third t (cells [16 t, 16 t + 16) of this thread's 48) of `src`, a rank's partition.
        // A whole tile of the default size is read from the partition's first cell on, also
        // where the partition is smaller: a rank's sketch buffer has that much room behind
        // its cells (tagc_plan_sizes), and only the partition's own cells are staged.
        auto request = [&](float (&b)[kUnit], GlobalCells src, auto third) {
            constexpr uint32_t t = decltype(third)::value;
#pragma unroll
            for (uint32_t i = 0; i < kUnit; i += 4) request_four(b + i, src + 4 * lt + (t * kUnit + i) * kLoadThreads);
        };
        // (the fences keep the compiler from moving the requests of later steps up in front
        // of the adds of earlier ones, which it otherwise does until the registers run out)
        auto add_unit = [&](const float (&b)[kUnit], auto third) {
            constexpr uint32_t t = decltype(third)::value;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (uint32_t i = 0; i < kUnit; ++i) acc[t * kUnit + i] += b[i];
            __builtin_amdgcn_sched_barrier(0);
        };
        constexpr std::integral_constant<uint32_t, 0> T0{};
        constexpr std::integral_constant<uint32_t, 1> T1{};
        constexpr std::integral_constant<uint32_t, 2> T2{};
        // the sum of partition `part` over the ranks, in rank order: the three thirds of a
        // rank are in flight while those of the rank before are added
        auto sum_partition = [&](uint32_t part) {
#pragma unroll
            for (uint32_t q = 0; q < kLoadCells; ++q) acc[q] = 0.0f;
            const uint64_t tile = uint64_t(part) * cells;
            GlobalCells src = rank_sketch(0) + tile;
            request(b0, src, T0);
            request(b1, src, T1);
            request(b2, src, T2);
            for (uint32_t r = 1; r < n_in; ++r) {
                src = rank_sketch(r) + tile;
                add_unit(b0, T0); request(b0, src, T0);
                add_unit(b1, T1); request(b1, src, T1);
                add_unit(b2, T2); request(b2, src, T2);
            }
            add_unit(b0, T0);
            add_unit(b1, T1);
            add_unit(b2, T2);
        };
        sum_partition(blockIdx.x);
        for (uint32_t a = blockIdx.x; a < A; a += gridDim.x) {
            if (a != blockIdx.x) __syncthreads();  // the peelers are done with the LDS
            uint32_t c0 = lt;  // (see peel_kernel's tid)
            asm volatile("" : "+v"(c0));
            const uint32_t to = part.base + PartLds<true>::kValue + 16 * c0;
#pragma unroll
            for (uint32_t q = 0; q < kLoadCells; q += 4)
                stage_four(to + 4 * q * kLoadThreads, acc + q, 4 * c0 + q * kLoadThreads, cells);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // this wave's cells are staged
            if (lane_id() == 0) atomicAdd(part.staged(), 1u);
            if (a + gridDim.x < A) sum_partition(a + gridDim.x);
        }
        return;
    }

    // ---------------------------------------------------------------- the peelers
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    PartIndex<kPeelWaves, kIndexPre> pre_index;
    PartList<kPeelThreads, kPeelIdx> pre_list;
    Partitions at(U, A, blockIdx.x, gridDim.x);
    uint32_t sa = 0;
    auto prefetch = [&] {  // (see peel_kernel)
        sa = ahead.get(2);
        if (kListed) pre_list.request(index.list + at.rho, at.unknowns(), tid);
        else pre_index.request(index, ahead.get(0), ahead.get(1), wave);
        ahead.request(index, salt, at.a + at.step, A);
    };
    prefetch();
    wait_loads();
    uint32_t bar_expected = 0, max_rounds = 0, staged = 0;
    while (at.a < A) {
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const uint32_t rho0 = at.rho, Pa = at.unknowns();
        part.seed(seed, sa);
        if (staged) __syncthreads();  // everybody is done with the previous partition
        part.clear<kPeelThreads>(tid, cells);
        if (kListed) pre_list.put(part.word(0), Pa, tid);
        else pre_index.enumerate(index, part.word(0), Pa, rho0, wave);
        peel_barrier(part.bar(), bar_expected);
        uint32_t cell[kPeelIdx][3];
        join_cells<kPeelThreads, kPeelIdx, kListed>(part, tid, Pa, idx_out + rho0, cell);
        peel_barrier(part.bar(), bar_expected);
        queue_first<kPeelThreads, kPeelIdx>(part, tid, Pa, mode != TAGC_DECODE_ESTIMATE, cell);
        at.next();
        if (at.a < A) prefetch();
        // the loaders have staged the cells: every loader wave of a workgroup says so once for each of its partitions,
        // whatever the peelers do, so the wait ends
        staged += kLoadWaves;
        while (__hip_atomic_load(part.staged(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < staged)
            __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        const uint32_t resolved = peel_rounds<kPeelThreads>(
            part, tid, max_rounds, [&] { peel_barrier(part.bar(), bar_expected); });
        wait_loads();
        for (uint32_t u = tid; u < Pa; u += kPeelThreads) val_out[rho0 + u] = unknown_value(part, u, mode);
        if (tid == 0) report_unresolved(Pa - resolved, mode, status);
    }
    if (tid == 0 && max_rounds) atomicMax(&status[TAGC_ST_ROUNDS], max_rounds);
}

// Dense output: a workgroup writes the 32 NT floats that NT words of the Index cover, zeros
// included.  The Index words, the number of set bits before each
// word, and the words' values (one contiguous run of val_out; its first kDenseStage NT / 1024
// entries, denser words read the rest one by one) are put in LDS; after that a thread
// builds any four consecutive outputs on its own -- the rank of a set bit is the word's
// count plus a popcount -- so the output goes out in plain contiguous 16-byte stores.
constexpr uint32_t kDenseStage = 8192;
// Words of a workgroup of dense_kernel.  Bound by the stores; whole chunks, two workgroups of 1024 threads to a
// compute unit, ended in a turn that was half empty (us, 256 / 512 / 1024 words: 7 M entries 8.9 / 9.1 / 9.6,
// 25 M 20.1 / 20.4 / 22.1, 67 M 50.4 / 50.9 / 51.5, 202 M 151 / 162 / 155).
constexpr uint32_t kDenseWords = 256;

template <uint32_t NT>
__device__ __forceinline__ void write_words(uint32_t piece, const uint32_t *__restrict__ bitmap, uint32_t n_words,
                                            const uint32_t *__restrict__ chunkpre, const uint16_t *__restrict__ grouppre,
                                            uint32_t U, const float *__restrict__ val_out, float *__restrict__ dense_out)
{
    constexpr uint32_t STAGE = kDenseStage * NT / kChunkWords;  // one thread per word
    static_assert(kChunkWords % NT == 0 && NT % kGroupWords == 0, "whole groups of one chunk");
    __shared__ uint32_t scratch[NT / 64];
    __shared__ uint32_t s_word[NT], s_pre[NT];
    __shared__ float vals[STAGE];
    const uint32_t tid = threadIdx.x;
    const uint32_t cw0 = piece * NT;  // first word
    const uint32_t word = cw0 + tid < n_words ? bitmap[cw0 + tid] : 0u;
    const uint32_t base = chunkpre[cw0 / kChunkWords] + (NT < kChunkWords ? grouppre[cw0 / kGroupWords] : 0u);
    uint32_t tot;
    const uint32_t pre = block_excl_scan<uint32_t, NT / 64>(uint32_t(__popc(word)), &tot, scratch);
    s_word[tid] = word;
    s_pre[tid] = pre;
    const uint32_t n_st = min(tot, STAGE);
    for (uint32_t i = tid; i < n_st; i += NT) vals[i] = base + i < U ? val_out[base + i] : 0.f;
    __syncthreads();
    const uint32_t n4 = min(NT, n_words - cw0) * 8;  // float4 groups
    float4 *out = reinterpret_cast<float4 *>(dense_out + uint64_t(cw0) * 32);
    for (uint32_t c = tid; c < n4; c += NT) {
        const uint32_t wd = s_word[c >> 3], sh = (c & 7u) * 4u;
        const uint32_t nib = (wd >> sh) & 0xFu;
        float o[4] = {0.f, 0.f, 0.f, 0.f};
        if (nib) {
            uint32_t r = s_pre[c >> 3] + __popc(wd & ((1u << sh) - 1u));  // rank among the words'
#pragma unroll
            for (uint32_t b = 0; b < 4; ++b) {
                if ((nib >> b) & 1u) {
                    if (r < STAGE) o[b] = vals[r];
                    else if (base + r < U) o[b] = val_out[base + r];
                    ++r;
                }
            }
        }
        st_stream(out + c, make_float4(o[0], o[1], o[2], o[3]));
    }
}

__global__ void __launch_bounds__(kDenseWords)
dense_kernel(const uint32_t *__restrict__ bitmap, uint32_t n_words,
             const uint32_t *__restrict__ chunkpre, const uint16_t *__restrict__ grouppre, const uint32_t *__restrict__ header,
             const float *__restrict__ val_out, float *__restrict__ dense_out)
{
    write_words<kDenseWords>(blockIdx.x, bitmap, n_words, chunkpre, grouppre, header[TAGC_HDR_U], val_out, dense_out);
}

// What a decoder of peel_grid workgroups that writes the dense output has left of it: the chunks that hold
// c-indices of a partition that was not its to write (what else they hold is written again, with the same
// values).  A workgroup has the chunks b, b + grid, ..., marked while all its threads go through the
// partitions' ends.
constexpr uint32_t kRestMarks = 128;  // words of marks: chunks of a workgroup / 32
constexpr uint32_t kRestGrid = (1u << 17) / (32 * kRestMarks);  // fewest workgroups for 2^32 c-indices
static_assert((uint64_t(kRestGrid) * 32 * kRestMarks) * kChunkWords * 32 >= 1ull << 32, "marks for all chunks");
__global__ void __launch_bounds__(kChunkWords)
dense_rest_kernel(const uint32_t *__restrict__ bitmap, uint32_t n_words, const uint32_t *__restrict__ chunkpre,
                  uint32_t n_chunks, const uint32_t *__restrict__ header, const uint32_t *__restrict__ bounds,
                  uint32_t peel_grid, const float *__restrict__ val_out, float *__restrict__ dense_out)
{
    __shared__ uint32_t marks[kRestMarks];
    const uint32_t U = header[TAGC_HDR_U], A = header[TAGC_HDR_A];
    const uint32_t tid = threadIdx.x, b = blockIdx.x, grid = gridDim.x, n_c = 32 * n_words;
    const bool all = !dense_by_decoder(A, peel_grid, n_c, 0);
    if (tid < kRestMarks) marks[tid] = all ? 0xFFFFFFFFu : 0u;
    __syncthreads();
    // (four partitions a thread; the words behind the last bound are the salts)
    for (uint32_t a0 = 4 * tid; !all && a0 < A; a0 += 4 * kChunkWords) {
        const uint4 q = *reinterpret_cast<const uint4 *>(bounds + a0);
        const uint32_t end[5] = {a0 ? q.x : 0u, q.y, q.z, q.w, bounds[a0 + 4]};
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t lo = end[i], hi = min(end[i + 1], n_c);
            if (a0 + i >= A || lo >= hi || dense_by_decoder(A, peel_grid, n_c, hi - lo)) continue;
            // its chunks among b, b + grid, ...
            const uint32_t first = lo / (32 * kChunkWords), last = (hi - 1) / (32 * kChunkWords);
            for (uint32_t k = first > b ? (first - b + grid - 1) / grid : 0u; b + k * grid <= last; ++k)
                atomicOr(&marks[k >> 5], 1u << (k & 31));
        }
    }
    __syncthreads();
    for (uint32_t k = 0; b + k * grid < n_chunks; ++k) {
        if (!((marks[k >> 5] >> (k & 31)) & 1u)) continue;
        write_words<kChunkWords>(b + k * grid, bitmap, n_words, chunkpre, nullptr, U, val_out, dense_out);
        __syncthreads();
    }
}

}  // namespace

// Partitions of the default size at most: sub-tables of 4096 cells, whose slots fit 12 bits.
static bool packed_slots(uint32_t T_cap, uint32_t P_cap)
{
    return T_cap <= kDefaultPartCells && P_cap <= kDefaultPartUnknowns;
}

size_t decode_lds_bytes(uint32_t T_cap, uint32_t P_cap)
{
    // PartLds; in the form that is not packed the queue is as long as there are cells, and 32
    // words are spare
    if (packed_slots(T_cap, P_cap)) return PartLds<true>::kPackedBytes;
    return size_t(T_cap) * 10 + (size_t(P_cap) + (P_cap / 32 + 1)) * 4 + 144;
}

int launch_decode(const tagc_plan_t *p, const tagc_shared_buffers *sh,
                  const tagc_rank_buffers *ranks, uint32_t n_ranks, uint32_t *idx_out,
                  float *val_out, float *dense_out, hipStream_t s)
{
    // ranks != nullptr: no summed sketch, the decoder adds up the ranks' sketches itself
    const bool fused = ranks != nullptr;
    if (fused && (p->T_cap > kDefaultPartCells || p->P_cap > kDefaultPartUnknowns ||
                  n_ranks > kMaxRanksPerPass))
        return TAGC_EUNSUPPORTED;
    const uint32_t n_words = uint32_t(p->n_c / 32);
    const uint32_t n_chunks = uint32_t(p->n_chunks);
    const uint32_t *chunkpre = static_cast<const uint32_t *>(sh->workspace);
    const IndexView index{sh->bitmap, chunkpre, group_prefixes(sh->workspace, n_chunks), sh->bounds,
                          n_words, n_chunks, idx_out};
    const size_t lds = decode_lds_bytes(p->T_cap, p->P_cap);
    // a workgroup takes partitions b, b + grid, ...: any grid size gives the same result
    uint32_t grid = uint32_t(std::min<uint64_t>(p->A_cap, uint64_t(device_cu_count())));
    if (p->cfg.decode_workgroups) grid = std::min(grid, p->cfg.decode_workgroups);
    RankPtrs rp{};
    if (fused) {
        for (uint32_t r = 0; r < n_ranks; ++r) rp.p[r] = ranks[r].sketch;
    } else {
        rp.p[0] = sh->sketch;
        n_ranks = 1;
    }
    // the default partition size gets an instantiation that holds exactly its data
    constexpr uint32_t kC0 = (kDefaultPartCells + kDecodeThreads - 1) / kDecodeThreads;
    constexpr uint32_t kI0 = (kDefaultPartUnknowns + kDecodeThreads - 1) / kDecodeThreads;
    constexpr uint32_t kC1 = (kMaxPartCells + kDecodeThreads - 1) / kDecodeThreads;
    constexpr uint32_t kI1 = (kMaxPartUnknowns + kDecodeThreads - 1) / kDecodeThreads;
    // Partitions that span much of the Index, because little of it can be set: the one workgroup of a partition
    // would go through all of that, most of the device having nothing to do, so a kernel over the whole Index
    // lists the unknowns first.  Decoder alone, us, walking / listing (enumerate and peel), three ranks, by
    // groups a partition: 4 partitions, 64, 128, 192, 256, 400, 600 groups 23.6 / 26.5, 26.1 / 26.2, 27.9 /
    // 26.4, 30.3 / 27.0, 33.6 / 26.2, 38.8 / 26.0; 30, the same 26.1 / 29.3, 27.9 / 28.2, 29.5 / 28.0, 31.6 /
    // 28.3, 35.6 / 28.4, 41.3 / 29.6; 100, 128, 256, 400 29.6 / 30.7, 33.3 / 32.3, 37.3 / 33.8; 164, 256, 320,
    // 400 34.9 / 36.2, 36.3 / 37.2, 39.1 / 37.9; 250, 256, 400 37.9 / 42.0, 43.0 / 46.4; 400, 256 69.3 / 69.7.
    // 8 ranks and one summed sketch the same within 3 %.  So the line is a little high for few partitions and
    // low for those that nearly fill the device; and with the dense output, whose zeros are written beside the
    // walking form only, it is low for 100 partitions (8 ranks, 256, 400 groups 1.34, 0.96 of walking's time)
    // and the same for 4 and 250.
    const bool listed = 16ull * n_chunks > kListGroups * p->A_cap;
    // A workgroup per partition, whatever is summed; else one summed sketch; up to four ranks; any number.
    // (Decoder alone, us, up to four ranks, sixteen waves peeling / sum_peel_kernel, of whose sixteen four sum:
    // one rank of 25, 74, 164 M entries in 300, 900, 2000 partitions 50.5 / 54.9, 98 / 106, 188 / 204; two 51.9
    // / 55.0, 100 / 107, 192 / 208; three 53.4 / 54.8, 102 / 108, 194 / 213; four 55.3 / 55.1, 107 / 112, 200 /
    // 218, of 94 M in 3955 378 / 418.  More ranks' cells do not fit the registers beside the rounds.)
    const uint32_t form = grid == p->A_cap && !listed && packed_slots(p->T_cap, p->P_cap) ? 3u
                          : !fused                ? (packed_slots(p->T_cap, p->P_cap) ? 1u : 0u)
                          : n_ranks <= kHeldRanks ? 2u
                                                  : 4u;
    auto pick = [&](auto list) {
        constexpr bool kList = decltype(list)::value;
        return form == 4   ? sum_peel_kernel<kList>
               : form == 3 ? peel_kernel<kC0, kI0, true, kHeldRanks, true, false, false>
               : form == 2 ? peel_kernel<kC0, kI0, true, kHeldRanks, false, kList, false>
               : form == 1 ? peel_kernel<kC0, kI0, true, 1, false, kList, false>
                           : peel_kernel<kC1, kI1, false, 1, false, kList, false>;
    };
    // A dense output that begins before the last partition is decoded must lie apart from what is still read by
    // then; a launch behind the decoder may put it in the place of a sketch, say.
    auto dense_apart = [&] {
        const uint64_t bytes = 4 * p->n_c;
        bool apart = !overlap(dense_out, bytes, idx_out, 4 * p->U_cap) &&
                     !overlap(dense_out, bytes, sh->bounds, p->sizes.shared_bounds_bytes);
        for (uint32_t r = 0; r < n_ranks; ++r) apart &= !overlap(dense_out, bytes, rp.p[r], 4 * p->m_cap);
        return apart;
    };
    const bool early = dense_out && !listed && !p->cfg.decode_workgroups && dense_apart();
    // The dense output by the decoder itself, whose rounds leave the memory system idle (sum_peel_kernel's
    // do not), where the plan has room for three turns of partitions to hide all but the last turn's behind, and
    // one rank's pairs alone give every compute unit a partition.  That is what the plan can know: which
    // partitions' output it really writes the device decides (dense_by_decoder), and a small launch behind
    // it, 5 us where nothing is left, writes the rest.  Decoder and dense output, us, dense_kernel / by the
    // decoder: 2 ranks of 202 M entries with a tenth kept 710 / 684, in four layers with 5 to 20 % 628 / 593, of
    // 200 M with 2.5 % 296 / 283, of 40 M with a tenth (928 partitions) 165 / 159; one rank of 32 M with a fifth
    // (782) 132 / 133; 200 M nearly all zeros, two partitions, 338 / 341 (6584 by their two workgroups).
    const bool with_dense = early && (form == 1 || form == 2) && p->A_cap >= 3ull * grid &&
                            p->K >= uint64_t(grid) * p->P_cap;
    // Where there are fewer partitions than compute units, workgroups on the others write the dense output's
    // zeros meanwhile, and the decoder its values among them.  Such a workgroup stores 7.7 thousand entries a
    // us, so it may have as many as that makes of what the peel and dense_kernel would take: 100 Ki, 16 for
    // each unknown of a partition, and a 180th of the output (1.4 M entries a us).  Decoder and dense output,
    // us, dense_kernel / this way, by the share of that limit that such a workgroup has, the summed sketch,
    // partitions of 8192: 0.2 32.6 / 28.8 (80 partitions of 3 M entries), 0.5 41.6 / 36.6 (156 of 16 M), 0.7
    // 61.2 / 40.3 (100 of 41 M), 0.8 54.3 / 44.3 (157 of 32 M), 0.9 83.4 / 74.6 (131 of 67 M), 1.0 45.9 / 46.3
    // (200 of 19 M), 1.15 46.1 / 50.0 (200 of 21 M), 1.3 60.4 / 71.3 (187 of 39 M); of 2048 unknowns 0.7 24.8 /
    // 21.4, 1.1 27.9 / 29.8 (200 of 8, 12 M); of 512 0.8 19.9 / 17.2, 1.1 22.2 / 25.6 (200 of 7, 11 M); of 32
    // 0.8 19.4 / 16.2, 1.1 21.3 / 24.2 (200 of 6, 10 M).
    // The sum of many ranks needs the memory itself, and where there is some to write, but not so much that the
    // launch behind it takes long, loses what that would take: 8 ranks, 0.8 M entries 37.7 / 31.1, 3 M 39.1 /
    // 35.2, 6 M 35.1 / 36.0, 8 M 37.3 / 38.7, 12 M 41.6 / 44.8, 16 M 46.4 / 46.4, 19 M 51.5 / 48.7, 24 M 52.9 /
    // 47.6; 16 ranks, 3 M 41.7 / 39.6, 6 M 42.7 / 45.0, 10 M 53.9 / 56.4, 16 M 51.1 / 48.2; 4 ranks, 6 M 34.3 /
    // 34.5, 8 M 38.1 / 38.1, 12 M 38.8 / 37.8.
    // (Plans whose unknowns are listed have no such decoder: it would be one form more.)
    const uint32_t cus = uint32_t(device_cu_count());
    const uint32_t spare = early && form == 3 && p->A_cap < cus ? cus - uint32_t(p->A_cap) : 0u;
    const uint64_t share = 100 * 1024 + 16ull * p->P_cap + p->n_c / 180;
    const bool crowded = n_ranks > kHeldRanks && p->n_c >= 4u << 20 && p->n_c < 16u << 20;
    const bool with_zeros = n_words && n_ranks <= kDenseRow && p->n_c <= spare * share && !crowded;
    constexpr uint32_t kZeroTurn = kZeroWords * (kDecodeThreads / 64);  // words of a workgroup
    if (with_zeros) grid += std::min(spare, (n_words + kZeroTurn - 1) / kZeroTurn);
    const auto kernel = with_zeros ? peel_kernel<kC0, kI0, true, kHeldRanks, true, false, true>
                        : with_dense ? (form == 2 ? peel_kernel<kC0, kI0, true, kHeldRanks, false, false, true>
                                                : peel_kernel<kC0, kI0, true, 1, false, false, true>)
                        : listed   ? pick(std::true_type{})
                                   : pick(std::false_type{});
    static size_t attr_bytes[3][5] = {};
    size_t &attr = attr_bytes[with_dense || with_zeros ? 2 : listed][form];
    if (lds > attr) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)
            return TAGC_EHIP;
        attr = lds;
    }
    if (with_dense || with_zeros) rp.p[kDenseRow] = dense_out;
    if (listed) {
        ProfileScope ps("enumerate", s);
        enumerate_kernel<<<n_chunks, 256, 0, s>>>(index, sh->header, idx_out);
    }
    {
        ProfileScope ps(fused ? "sum_peel" : "peel", s);
        kernel<<<grid, kDecodeThreads, lds, s>>>(rp, n_ranks, index, sh->header, idx_out, val_out,
                                                 sh->status, p->cfg.seed, sh->bounds + p->A_cap + 1,
                                                 p->T_cap, p->P_cap, p->cfg.decode_mode);
    }
    if (with_dense) {
        ProfileScope ps("dense_rest", s);
        const uint32_t n = std::min(n_chunks, std::max(2 * uint32_t(device_cu_count()), kRestGrid));
        dense_rest_kernel<<<n, kChunkWords, 0, s>>>(sh->bitmap, n_words, chunkpre, n_chunks, sh->header, sh->bounds,
                                                    grid, val_out, dense_out);
    } else if (dense_out && n_chunks && !with_zeros) {
        ProfileScope ps("dense", s);
        dense_kernel<<<(n_words + kDenseWords - 1) / kDenseWords, kDenseWords, 0, s>>>(
            sh->bitmap, n_words, chunkpre, index.grouppre, sh->header, val_out, dense_out);
    }
    return hip_ok(hipGetLastError());
}

}  // namespace tagc
