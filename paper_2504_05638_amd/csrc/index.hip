// Index aggregation: what All-Reduce(local_index) yields in Algorithm 1, computed on one
// GPU as the bitwise OR of N ranks' bit maps (section 2.2 names OR as the operation the
// Index needs), followed by everything the later stages derive from the merged Index:
// its number of non-zeros U, the sketch layout (A partitions of 3*m_sub cells) and the
// c-index at which each partition starts.
#include "device_utils.h"
#include "tagc_internal.h"

namespace tagc {

namespace {

// One workgroup per chunk of kChunkWords words of the merged Index; 4 words per thread.
// MODE says how the ranks' wire Indexes combine (section 2.2): the OR the Index needs, or the
// addition that simulates it over a library without OR -- of the 1-bit words themselves
// (carries and all), or of 4-bit counters, four wire words per merged word, a merged bit
// being set where the summed counter is not 0.  Sums wrap as unsigned 32-bit adds do.  With
// more ranks than one launch takes, the running result is carried in `out` (OR, 1-bit add)
// or, for the counters, in `sum4`.
template <int MODE>
__global__ void __launch_bounds__(256)
index_merge_kernel(RankPtrs rp, uint32_t n_in, uint32_t *__restrict__ out, uint32_t n_words,
                   int accumulate, int last, uint32_t *__restrict__ sum4,
                   uint32_t *__restrict__ chunkcnt, uint16_t *__restrict__ grouppre)
{
    static_assert(kChunkWords == 16 * kGroupWords && kGroupWords == 64, "16 groups of a wave's words");
    __shared__ uint32_t smem[16];
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t w0 = blockIdx.x * kChunkWords + threadIdx.x * 4;
    uint32_t pc = 0;
    if (MODE == TAGC_INDEX_ADD4) {
        // a thread merges the words tid, tid + 256, ... of the chunk: the four wire words of
        // one merged word are one 16-byte load per rank, consecutive across the lanes
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t w = blockIdx.x * kChunkWords + k * 256 + threadIdx.x;
            uint32_t set = 0;
            if (w < n_words) {
                const size_t q = 4 * size_t(w);
                uint4 acc = accumulate ? *reinterpret_cast<const uint4 *>(sum4 + q)
                                       : make_uint4(0, 0, 0, 0);
#pragma unroll 8
                for (uint32_t r = 0; r < n_in; ++r) {
                    const uint4 v = ld_stream(reinterpret_cast<const uint4 *>(
                        static_cast<const uint32_t *>(rp.p[r]) + q));
                    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
                }
                if (!last) {
                    *reinterpret_cast<uint4 *>(sum4 + q) = acc;
                } else {
                    const uint32_t m = nibbles_set(acc.x) | (nibbles_set(acc.y) << 8) |
                                       (nibbles_set(acc.z) << 16) | (nibbles_set(acc.w) << 24);
                    out[w] = m;
                    set = __popc(m);
                }
            }
            if (chunkcnt) {  // the wave's words are one group
                set = wave_sum(set);
                if (lane == 0) smem[4 * k + wave] = set;
            }
        }
    } else if (w0 + 4 <= n_words) {
        uint4 acc = accumulate ? *reinterpret_cast<const uint4 *>(out + w0) : make_uint4(0, 0, 0, 0);
        for (uint32_t r = 0; r < n_in; ++r) {
            const uint4 v =
                ld_stream(reinterpret_cast<const uint4 *>(static_cast<const uint32_t *>(rp.p[r]) + w0));
            if (MODE == TAGC_INDEX_OR1) {
                acc.x |= v.x; acc.y |= v.y; acc.z |= v.z; acc.w |= v.w;
            } else {
                acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
            }
        }
        *reinterpret_cast<uint4 *>(out + w0) = acc;
        pc = __popc(acc.x) + __popc(acc.y) + __popc(acc.z) + __popc(acc.w);
    } else {
        for (uint32_t w = w0; w < n_words; ++w) {
            uint32_t acc = accumulate ? out[w] : 0u;
            for (uint32_t r = 0; r < n_in; ++r) {
                const uint32_t v = static_cast<const uint32_t *>(rp.p[r])[w];
                acc = MODE == TAGC_INDEX_OR1 ? (acc | v) : (acc + v);
            }
            out[w] = acc;
            pc += __popc(acc);
        }
    }
    if (!chunkcnt) return;
    // set bits of every group of 64 words: a row of 16 lanes has its four words each
    if (MODE != TAGC_INDEX_ADD4) {
        for (uint32_t d = 1; d < 16; d <<= 1) pc += __shfl_xor(pc, d, 64);
        if ((lane & 15) == 0) smem[threadIdx.x >> 4] = pc;
    }
    __syncthreads();
    if (wave == 0) {
        const uint32_t n = lane < 16 ? smem[lane] : 0u;
        const uint32_t inc = wave_incl_scan<uint32_t>(n);
        if (lane < 16) grouppre[blockIdx.x * 16 + lane] = uint16_t(inc - n);
        if (lane == 15) chunkcnt[blockIdx.x] = inc;
    }
}

struct LayoutParams {
    uint32_t mode, milli, P_cap, T_cap;
    uint64_t M_fixed;  // fixed ratio: target cells, ceil(n_real*1000/milli)
    uint64_t U_cap, A_cap, m_cap;
};
struct Layout {
    uint32_t U, A, m_sub, m, flags;
};

// The sketch layout of a merged Index with U set bits.
//
//   target cells  M = ceil(milli*U/1000)  |  ceil(n_real*1000/milli)
//   partitions    A = max(1, ceil(U/P_cap), ceil(M/(3q))),  q = T_cap/3   (0 if U = 0)
//   sub-table     m_sub = max(1, ceil(M/(3A)))  |  max(1, floor(M/(3A)))
//   total         m = 3*A*m_sub
//
// (U <= U_cap makes everything fit 32 bits: the plan refuses a capacity that does not.)
__device__ inline Layout layout_of(uint32_t U, const LayoutParams &lp)
{
    Layout l{};
    if (U == 0) return l;
    if (U > lp.U_cap) {  // caller broke the plan's bounds
        l.flags = TAGC_FLAG_OVERFLOW;
        return l;
    }
    const bool load = lp.mode == TAGC_SIZE_LOAD_FACTOR;
    const uint32_t M = uint32_t(load ? (uint64_t(lp.milli) * U + 999) / 1000 : lp.M_fixed);
    const uint32_t q = lp.T_cap / 3;
    uint32_t A = max((U - 1) / lp.P_cap + 1, M ? (M - 1) / (3 * q) + 1 : 1u);
    uint32_t m_sub = load ? (M ? (M - 1) / (3 * A) + 1 : 0u) : M / (3 * A);
    m_sub = max(m_sub, 1u);
    const uint64_t m = 3ull * A * m_sub;
    if (A > lp.A_cap || m > lp.m_cap) {
        l.flags = TAGC_FLAG_OVERFLOW;
        return l;
    }
    l.U = U;
    l.A = A;
    l.m_sub = m_sub;
    l.m = uint32_t(m);
    return l;
}

// What a launch needs to know of a rank to find the partitions in its pair list.
struct LayoutRank {
    const uint32_t *idx;
    uint32_t *cnt;
    const uint32_t *wire;  // its Index as it goes on the wire
};
struct LayoutBatch {
    LayoutRank r[kMaxRanksPerPass];
};

// Words 4 w .. 4 w + 3 of the merged Index of the n_in ranks of a launch, as index_merge_kernel has them.
template <int MODE>
__device__ __forceinline__ uint4 merge_four(uint32_t n_in, uint32_t w, uint32_t n_words)
{
    constexpr uint32_t WIRE = MODE == TAGC_INDEX_ADD4 ? 4 : 1;  // 16-byte vectors on the wire
    uint4 acc[WIRE];
#pragma unroll
    for (uint32_t i = 0; i < WIRE; ++i) acc[i] = make_uint4(0, 0, 0, 0);
#pragma unroll 4
    for (uint32_t r = 0; r < n_in; ++r) {
        const uint4 *wire = reinterpret_cast<const uint4 *>(as_global(batch_row<LayoutRank>(r)->wire)) + WIRE * w;
#pragma unroll
        for (uint32_t i = 0; i < WIRE; ++i) {
            if (WIRE > 1 && WIRE * w + i >= n_words) continue;  // (its words' counters are all there is room for)
            const uint4 v = wire[i];
            if (MODE == TAGC_INDEX_OR1) {
                acc[i].x |= v.x; acc[i].y |= v.y; acc[i].z |= v.z; acc[i].w |= v.w;
            } else {
                acc[i].x += v.x; acc[i].y += v.y; acc[i].z += v.z; acc[i].w += v.w;
            }
        }
    }
    if constexpr (MODE == TAGC_INDEX_ADD4) {
        auto word = [](const uint4 &a) {
            return nibbles_set(a.x) | (nibbles_set(a.y) << 8) | (nibbles_set(a.z) << 16) | (nibbles_set(a.w) << 24);
        };
        return make_uint4(word(acc[0]), word(acc[1]), word(acc[2]), word(acc[3]));
    } else {
        return acc[0];
    }
}

// By every 16 lanes of a wave for theirs: the first position in a sorted list whose entry is >= key.  Each step
// cuts the range into 16 parts: 5 or 6 dependent loads for a list of millions where a thread's binary search
// takes over 20 (cut into 64 parts by a whole wave it is 4, of 64 cache lines each: 58 thousand searches of
// 2 M entries were bound by those).
__device__ inline uint32_t lower_bound_by_16(const uint32_t *list, uint32_t n, uint32_t key)
{
    const uint32_t part = lane_id() & 15, shift = lane_id() & 48;
    uint32_t lo = 0, hi = n;
    while (__ballot(lo < hi)) {
        const uint32_t step = (hi - lo + 15) / 16;
        const uint64_t first = lo + uint64_t(part) * step;
        // the last entry of the lane's part
        const uint32_t v = first < hi ? list[min(first + step, uint64_t(hi)) - 1] : 0xFFFFFFFFu;
        // parts wholly below the key; then the part after them, whose last entry is not
        const uint32_t below = uint32_t(__popc(uint32_t(__ballot(v < key) >> shift) & 0xFFFFu));
        const uint64_t at = min(lo + uint64_t(below) * step, uint64_t(hi));
        const uint64_t end = min(at + step, uint64_t(hi));
        lo = uint32_t(at);
        hi = uint32_t(end > at ? end - 1 : at);
    }
    return lo;
}

// Per-partition hash salts (the compression is to be lossless, section 2.2 and Table 1).
// Two non-zeros of a partition that fall into the same three cells can never be peeled
// apart, and with the cells of a non-zero confined to its partition that happens to a few
// pairs per 10^8 non-zeros.  The merged Index reaches every rank before compress(g_shard,
// index) runs (Algorithm 1), so encoder and decoder can both derive from it, for every
// partition, the smallest salt under which all of the partition's (slot_0, slot_1, slot_2)
// are distinct; nothing travels.  Nearly every partition keeps salt 0.
//
// One workgroup per partition at a time, two workgroups per compute unit.  The partition's
// non-zeros are the set bits of the merged Index in [bounds[a], bounds[a+1]).  Each gets a
// number t (any order; a wave takes a run of numbers with one LDS add).  Bound by hashing (three 32-bit
// multiplies per slot, at quarter rate), so nearly all of them are let off with two of their slots: slot_0
// and six bits of slot_1 name a bit of a filter, 64 bits per cell of a sub-table, and whoever finds its bit
// set (one in 64 of 8192) sets one in a second filter, by which all that have the same bits then know
// themselves (one in 30).  Those are listed and compared with all three slots: pushed on the list of their
// slot_0 (an LDS exchange of the list's head), after which each walks what was on that list before it.  A
// partition with more of them than the listing has room for (sub-tables of a few cells) is compared
// that way as a whole.  All of it that way, with a 32-bit tag, a link and a walk for each and all three slots
// hashed, took, us, and takes now: 16 ranks of 202 M entries 149, 125; 2 ranks with a tenth kept 160, 124;
// 8 ranks of 67 M 39, 31, of 25 M 22.4, 20.5; a launch with one partition 0.5 more (two barriers more).
// The same kernel derives everything else the later stages need from the merged Index, each
// step a few dependent loads that would be a launch of their own: every workgroup adds up the
// chunk counts by itself (a few words per thread) and knows the layout; its partitions' bounds
// are found by a wave each (bounds[a] = c-index of the non-zero of rank floor(a*U/A);
// bounds[A] = n_c); and so are their ends in the ranks' sorted pair lists (ranges[a] of a
// rank = number of its pairs whose c-index lies below bounds[a]).  Four launches (header, bounds,
// salt, ranges) were 31 us on an 8-rank bucket of 25 M entries and 48 on one of 67 M, in one launch they
// were 21 and 40 with the same comparison.  A workgroup's first partition waits for memory, in order: chunk
// counts, Index words of the bounds, its own words; then the searches waited 10 to 20 K clocks for four to six
// steps (83 K with 16 ranks of 202 M entries) in which its compute unit hashed nothing.  So some
// workgroups of the launch find the ends in the pair lists, beside the others' salts (us of this kernel, before /
// after: 16 ranks of 202 M entries 125 / 105, one of them with three others' Indexes 52 / 47, 8 ranks of 67 M 27 / 24,
// of 25 M 24.2 / 21.6, of 7 M 20.4 / 18.0, 4 of 1 M 17.0 / 15.0, 3 of 36 thousand 14.3 / 13.0).  (Tried: a step of the searches between the steps of the salts, whose waits are
// longer than those steps, half as much or nothing; the chunk counts kept in LDS for the bounds, nothing; 256
// parts a step and half the steps in small launches, 3 us slower, bound by the lines; words beyond the first
// four requested ahead, 0 to 6 % slower; two searches of a wave at once, 16 ranks of 202 M 141 where one was 135, 8 of
// 7 M 18.9, 18.0; the last, nearly empty turn of the salts taken by the searchers once they are through, 2 of 202 M
// with a tenth 133.5, 4 of 202 M 48.3, 47.2, since they are through last.)
constexpr uint32_t kSaltThreads = 1024;
constexpr uint32_t kLayoutBatch = kSaltThreads / 128;  // partitions whose bounds are found at once
constexpr uint64_t kSearchApart = 2048;  // non-zeros of a partition from which on some workgroups only search
constexpr uint64_t kSplitSearches = 32768;  // (partition, rank) pairs
constexpr uint32_t kSaltLimit = 16;       // salts tried: 0 .. 15
constexpr uint32_t kNoLink = 0xFFFFu;
constexpr uint32_t kFilterBits = 64;      // per cell of a sub-table
constexpr uint32_t kSecondWords = 1024;   // second filter, cleared a word per thread
static_assert(kSecondWords == kSaltThreads, "every thread clears its word");
// Index words up to which the layout merges the ranks' Indexes itself: four of each to a thread, kept in LDS,
// where everything that is looked up in the merged Index then is.  Every workgroup merges them all, so they are
// few and read little.  us of the Index aggregation, merge and layout / layout alone: 33 thousand entries from
// 1, 8, 16 ranks 14.5, 15.7, 17.2 / 11.1, 11.9, 12.4, 66 thousand 16.6, 19.9, 23.4 / 12.3, 13.3, 13.6, 131
// thousand from 1, 4, 8 ranks 16.8, 17.1, 17.5 / 13.1, 13.4, 13.9; in 52 partitions 15.9 / 11.8 (4 ranks).
// 4-bit counters: a thread has four vectors of a rank, and more than eight ranks' go out in too many trips: 8
// thousand entries from 8, 16, 32 ranks 15.3, 15.6, 16.6 / 13.7, 16.5, 21.3, 33 thousand from 8 18.2 / 15.3.
constexpr uint32_t kMergeWords = 4 * kSaltThreads;
constexpr uint32_t kMergeMost = 64;             // partitions of the plan at most
constexpr uint32_t kMergeBytes = 128 * 1024;    // of all ranks' Indexes
constexpr uint32_t kMergeRanks4 = 8;            // ranks of 4-bit counters
constexpr uint32_t kSaltPer = kDefaultPartUnknowns / kSaltThreads;  // non-zeros per thread of a partition of the default size
constexpr uint32_t kSaltPre = 4;          // Index words per thread requested a partition ahead

// The room for the first filter, which is also that for list heads and a 16-bit link per non-zero; and how many
// non-zeros (number, tag, link) can be listed behind the heads.
__host__ __device__ inline uint32_t salt_filter_bytes(uint32_t T_cap, uint32_t P_cap)
{
    const uint32_t q = T_cap / 3, filter = q * (kFilterBits / 8), whole = 4 * q + 2 * P_cap;
    return ((filter > whole ? filter : whole) + 15) & ~15u;
}
__host__ __device__ inline uint32_t salt_listed(uint32_t T_cap, uint32_t P_cap)
{
    return (salt_filter_bytes(T_cap, P_cap) - 4 * (T_cap / 3)) / 8;
}

// (8 waves per SIMD asked for: two workgroups a compute unit; 106 scalar registers leave room for one)
// kMerge: the ranks' Indexes are merged here (MODE says how), and `bitmap`, `chunkcnt` and `grouppre` written.
constexpr int kNoMerge = -1;
template <bool kBounds, bool kSearch, bool kSalts, int MODE>
__global__ void __launch_bounds__(kSaltThreads) __attribute__((amdgpu_waves_per_eu(8)))
layout_kernel(const LayoutBatch, uint32_t n_in, uint32_t all, uint32_t *__restrict__ bitmap,
              uint32_t n_words, uint32_t n_c, uint32_t *__restrict__ chunkcnt, uint16_t *__restrict__ grouppre,
              uint32_t *__restrict__ chunkpre, uint32_t n_chunks, const LayoutParams lp,
              uint32_t *__restrict__ header, uint32_t *__restrict__ status,
              uint32_t *__restrict__ bounds, uint32_t ranges_off, uint32_t pair_cap, uint64_t seed,
              uint32_t n_search, uint32_t search0)
{
    constexpr uint32_t NT = kSaltThreads;
    constexpr bool kMerge = MODE != kNoMerge;
    extern __shared__ uint32_t lds_salt[];
    __shared__ __align__(16) uint32_t s_words[kMerge ? kMergeWords : 1];
    const uint32_t P_cap = lp.P_cap, q_cap = lp.T_cap / 3;
    uint32_t *second = lds_salt;            // [kSecondWords]
    uint32_t *tag = second + kSecondWords;  // [P_cap] c-index; compared as a whole: slot_1 | slot_2 << 16
    // the first filter; behind it in time, list heads and what is compared (see salt_lds_bytes)
    uint32_t *filter = tag + P_cap;         // [kFilterBits / 32 * q_cap]
    uint32_t *head = filter;                // [q_cap]
    const uint32_t n_listed = salt_listed(lp.T_cap, P_cap);
    uint32_t *some_tag = head + q_cap;                                      // [n_listed]
    uint16_t *some = reinterpret_cast<uint16_t *>(some_tag + n_listed);     // [n_listed] their numbers
    uint16_t *some_link = some + n_listed;                                  // [n_listed]
    uint16_t *link = reinterpret_cast<uint16_t *>(head + q_cap);            // [P_cap], as a whole
    __shared__ uint32_t s_n, s_dup, s_some;
    __shared__ uint32_t s_pre[kBounds ? NT : 1];  // set bits before thread t's chunks
    __shared__ uint32_t s_bound[2 * kLayoutBatch];  // first and last bound of the batch's partitions
    __shared__ uint32_t s_pairs[kMaxRanksPerPass];
    __shared__ uint32_t smem[NT / 64];
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // (what every lane holds alike comes from LDS here: said to be uniform, it stays in scalar
    // registers, and the loops below are scalar)
    auto uniform = [](uint32_t x) -> uint32_t { return __builtin_amdgcn_readfirstlane(x); };
    if (kSearch && tid < n_in)
        s_pairs[tid] = min(as_global(batch_row<LayoutRank>(tid)->cnt)[TAGC_CNT_TOTAL], pair_cap);
    // ---- set bits before every thread's chunks, the layout
    const uint32_t per = (n_chunks + NT - 1) / NT;
    Layout lay{};
    if (kBounds) {
        const uint32_t first = tid * per, last = kMerge ? first : min(first + per, n_chunks);
        uint32_t own = 0, total;
        for (uint32_t i = first; i < last; ++i) own += chunkcnt[i];
        uint4 merged = make_uint4(0, 0, 0, 0);
        if (kMerge) {  // (an Index has room for whole vectors; its padding bits are never set, but not so behind its words)
            if (4 * tid < n_words) merged = merge_four<kMerge ? MODE : TAGC_INDEX_OR1>(n_in, tid, n_words);
            if (4 * tid + 1 >= n_words) merged.y = 0;
            if (4 * tid + 2 >= n_words) merged.z = 0;
            if (4 * tid + 3 >= n_words) merged.w = 0;
            reinterpret_cast<uint4 *>(s_words)[tid] = merged;
            own = __popc(merged.x) + __popc(merged.y) + __popc(merged.z) + __popc(merged.w);
        }
        const uint32_t before = block_excl_scan<uint32_t, NT / 64>(own, &total, smem);
        s_pre[tid] = before;
        total = uniform(total);
        lay = layout_of(total, lp);
        if (kMerge) __syncthreads();
        if (kMerge && blockIdx.x == 0) {  // what a merge of its own leaves
            const uint32_t w[4] = {merged.x, merged.y, merged.z, merged.w};
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i)
                if (4 * tid + i < n_words) bitmap[4 * tid + i] = w[i];
            constexpr uint32_t PC = kChunkWords / 4, PG = kGroupWords / 4;  // threads of a chunk, of a group
            if (tid % PC == 0 && tid / PC < n_chunks) {
                chunkcnt[tid / PC] = (tid + PC < NT ? s_pre[tid + PC] : total) - before;
                chunkpre[tid / PC] = before;
            }
            if (tid % PG == 0 && tid / PC < n_chunks) grouppre[tid / PG] = uint16_t(before - s_pre[tid / PC * PC]);
        }
        if (all && blockIdx.x == 0) {
            uint32_t run = before;
            for (uint32_t i = first; i < last; ++i) {
                chunkpre[i] = run;
                run += chunkcnt[i];
            }
            if (tid == 0) {
                chunkpre[n_chunks] = total;
                header[TAGC_HDR_U] = lay.U;
                header[TAGC_HDR_A] = lay.A;
                header[TAGC_HDR_MSUB] = lay.m_sub;
                header[TAGC_HDR_M] = lay.m;
                for (int i = 4; i < TAGC_HDR_WORDS; ++i) header[i] = 0;
                for (int i = 0; i < TAGC_ST_WORDS; ++i) status[i] = 0;
                status[TAGC_ST_FLAGS] = lay.flags;
            }
        }
        __syncthreads();  // s_pre
    } else {
        lay.A = header[TAGC_HDR_A];
        lay.m_sub = header[TAGC_HDR_MSUB];
    }
    const uint32_t U = lay.U, A = lay.A, m_sub = min(lay.m_sub, q_cap);

    // c-index of the set bit of rank rho < U (by a wave, all lanes get it)
    auto bound_of = [&](uint32_t rho) -> uint32_t {
        // the last thread whose chunks start at or before it
        uint32_t t = uint32_t(__popcll(__ballot(s_pre[lane * (NT / 64)] <= rho))) - 1u;
        const uint32_t v = lane < NT / 64 ? s_pre[t * (NT / 64) + lane] : 0xFFFFFFFFu;
        t = t * (NT / 64) + uint32_t(__popcll(__ballot(v <= rho))) - 1u;
        if constexpr (kMerge) {  // its word, then its bit
            uint32_t r = rho - uniform(s_pre[t]), word = 0, i = 0;
            for (; i < 4; ++i) {
                word = uniform(s_words[4 * t + i]);
                const uint32_t c = __popc(word);
                if (r < c) break;
                r -= c;
            }
            const uint64_t hit = __ballot(lane < 32 && ((word >> (lane & 31)) & 1u) &&
                                          uint32_t(__popc(word & ((1u << (lane & 31)) - 1u))) == r);
            return hit ? (4 * t + i) * 32 + uint32_t(__builtin_ctzll(hit)) : n_c;
        }
        // its chunk
        uint32_t run = uniform(s_pre[t]), chunk = t * per, local = 0;
        for (uint32_t j = 0; j < per; j += 64) {
            const uint32_t c = t * per + j + lane;
            const uint32_t n = j + lane < per && c < n_chunks ? chunkcnt[c] : 0u;
            const uint32_t inc = wave_incl_scan<uint32_t>(n);
            const uint32_t tot = __builtin_amdgcn_readlane(inc, 63);
            if (rho - run < tot) {
                const uint32_t k = uint32_t(__popcll(__ballot(run + inc <= rho)));
                chunk = t * per + j + k;
                local = rho - run - (k ? __builtin_amdgcn_readlane(inc, k - 1) : 0u);
                break;
            }
            run += tot;
        }
        // its bit, the wave looking at 16 words per lane
        const uint32_t wbase = chunk * kChunkWords + lane * 16;
        uint32_t w[16], tot = 0;
        if (wbase + 16 <= n_words) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4 x = *reinterpret_cast<const uint4 *>(bitmap + wbase + 4 * i);
                w[4 * i] = x.x; w[4 * i + 1] = x.y; w[4 * i + 2] = x.z; w[4 * i + 3] = x.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) w[i] = (wbase + i < n_words) ? bitmap[wbase + i] : 0u;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) tot += __popc(w[i]);
        const uint32_t incl = wave_incl_scan<uint32_t>(tot);
        const uint32_t excl = incl - tot;
        uint32_t found = n_c;
        const bool mine = excl <= local && local < incl;
        if (mine) {
            uint32_t r = local - excl;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t c = __popc(w[i]);
                if (found == n_c) {
                    if (r < c) {
                        uint32_t x = w[i];
                        for (uint32_t s = 0; s < r; ++s) x &= x - 1;
                        found = (wbase + i) * 32 + __builtin_ctz(x);
                    } else {
                        r -= c;
                    }
                }
            }
        }
        const uint64_t who = __ballot(mine);
        return who ? __builtin_amdgcn_readlane(found, __builtin_ctzll(who)) : n_c;
    };
    if (kBounds && blockIdx.x == 0) {  // the end of the last partition (of none: the only bound)
        if (tid == 0) bounds[A] = n_c;
        // (rank r's words from ranges_off on: positions in its pair list)
        if (kSearch && tid < n_in) as_global(batch_row<LayoutRank>(tid)->cnt)[ranges_off + A] = s_pairs[tid];
    }
    // word `w` of partition [lo, hi); and the same with the bits outside the partition cleared, which is a step
    // of its own because it waits for the word
    auto load_word = [&](uint32_t w, uint32_t lo, uint32_t hi) -> uint32_t {
        const uint32_t end = lo < hi ? min(((hi - 1) >> 5) + 1, n_words) : 0u;
        return w < end ? (kMerge ? s_words[w] : bitmap[w]) : 0u;
    };
    auto clip_word = [&](uint32_t word, uint32_t w, uint32_t lo, uint32_t hi) -> uint32_t {
        if (w == (lo >> 5)) word &= 0xFFFFFFFFu << (lo & 31);
        if (w == ((hi - 1) >> 5) && (hi & 31)) word &= (1u << (hi & 31)) - 1u;
        return word;
    };
    // The workgroup's partitions are me, me + G, me + 2 G, ...
    // (n_search workgroups from search0 on search, the others are for the salts; 0: all are for both.  search0
    // is where the others end; written with that in mind, this kernel came out 0.5 to 3 us slower.)
    const bool searcher = kSearch && blockIdx.x - search0 < n_search;
    const uint32_t me = searcher ? blockIdx.x - search0 : blockIdx.x - (blockIdx.x >= search0 ? n_search : 0u);
    const uint32_t G = searcher ? n_search : gridDim.x - n_search;
    const uint32_t n_mine = me < A ? (A - 1 - me) / G + 1 : 0u;
    for (uint32_t b0 = 0; b0 < n_mine; b0 += kLayoutBatch) {
    const uint32_t nb = min(kLayoutBatch, n_mine - b0);
    __syncthreads();  // s_bound is free
    if (!kBounds) {
        if (tid < 2 * nb) s_bound[tid] = bounds[me + (b0 + (tid >> 1)) * G + (tid & 1)];
    } else if ((wave >> 1) < nb) {
        const uint32_t a = me + (b0 + (wave >> 1)) * G + (wave & 1);
        // (floor(a U / A): 32-bit divisions where they are enough, a 64-bit one is several times the instructions)
        const uint32_t rho = A < 65536 ? a * (U / A) + a * (U % A) / A : uint32_t(uint64_t(a) * U / A);
        const uint32_t x = a == A ? n_c : bound_of(rho);
        if (lane == 0) {
            s_bound[wave] = x;
            if (!(wave & 1) && !(kSalts && searcher)) bounds[a] = x;
        }
    }
    __syncthreads();
    if (searcher || (kSearch && n_search == 0)) {
        // a wave has the tasks wave, wave + NT / 64, ..., each a rank's list and four partitions
        for (uint32_t task = wave; task < n_in * ((nb + 3) / 4); task += NT / 64) {
            const uint32_t r = task % n_in, i = task / n_in * 4 + lane / 16;
            const auto *row = batch_row<LayoutRank>(r);
            const uint32_t at = lower_bound_by_16(as_global(row->idx), i < nb ? s_pairs[r] : 0u, s_bound[2 * min(i, nb - 1)]);
            if ((lane & 15) == 0 && i < nb) as_global(row->cnt)[ranges_off + me + (b0 + i) * G] = at;
        }
    }
    if (searcher) continue;
    // Requests run ahead of the work: the first Index words of a partition while the one before it is checked.
    // (Those of the first ahead of the searches too, where a workgroup does both: no difference.)
    uint32_t lo = uniform(s_bound[0]), hi = uniform(s_bound[1]), pre[kSaltPre];
#pragma unroll
    for (uint32_t k = 0; k < kSaltPre; ++k)
        pre[k] = kSalts ? load_word((lo >> 5) + k * NT + tid, lo, hi) : 0u;
    for (uint32_t i = 0; kSalts && i < nb; ++i) {
        const uint32_t w_lo = lo >> 5, w_hi = lo < hi ? (hi - 1) >> 5 : 0;
        const uint32_t cur_lo = lo, cur_hi = hi;
        uint32_t cur[kSaltPre];
#pragma unroll
        for (uint32_t k = 0; k < kSaltPre; ++k) cur[k] = pre[k];
        if (i + 1 < nb) {
            lo = uniform(s_bound[2 * i + 2]);
            hi = uniform(s_bound[2 * i + 3]);
#pragma unroll
            for (uint32_t k = 0; k < kSaltPre; ++k)
                pre[k] = load_word((lo >> 5) + k * NT + tid, lo, hi);
        }
        uint32_t salt = 0;
        if (cur_lo < cur_hi) {
            // the non-zeros' c-indices into tag[]
            auto enumerate = [&] {
                uint32_t k = 0;
                for (uint32_t base = w_lo + (tid - lane); base <= w_hi; base += kSaltThreads, ++k) {
                    // (wave-uniform loop: the numbering below is a wave-wide scan)
                    uint32_t word = k < kSaltPre ? cur[k < kSaltPre ? k : 0]
                                                 : load_word(base + lane, cur_lo, cur_hi);
                    word = clip_word(word, base + lane, cur_lo, cur_hi);
                    const uint32_t pc = __popc(word);
                    const uint32_t inc = wave_incl_scan<uint32_t>(pc);
                    const uint32_t tot = __builtin_amdgcn_readlane(inc, 63);
                    if (tot == 0) continue;
                    uint32_t start = 0;
                    if (lane == 0) start = atomicAdd(&s_n, tot);
                    start = __builtin_amdgcn_readfirstlane(start);
                    uint32_t t = start + inc - pc;
                    for (; word; word &= word - 1, ++t)  // (a partition holds <= P_cap)
                        if (t < P_cap) tag[t] = (base + lane) * 32 + uint32_t(__builtin_ctz(word));
                }
            };
            // pushes entry t of a list under its slots, then looks for another one with the same
            auto push = [&](uint32_t i, uint32_t t, uint32_t *tags, uint16_t *links, const uint32_t (&fsw)[3]) {
                uint32_t neg;
                const uint32_t fi = fold16(i), c0 = hash_slot_folded(fi, fsw[0], m_sub, &neg);
                tags[t] = hash_slot_folded(fi, fsw[1], m_sub, &neg) |
                          (hash_slot_folded(fi, fsw[2], m_sub, &neg) << 16);
                links[t] = uint16_t(atomicExch(&head[c0], t));
            };
            auto twice = [&](uint32_t t, const uint32_t *tags, const uint16_t *links) {
                const uint32_t mine = tags[t];
                bool dup = false;
                for (uint32_t p = links[t]; p != kNoLink; p = links[p]) dup |= tags[p] == mine;
                return dup;
            };
            // (not kept from one partition to the next in registers that are needed)
            uint32_t tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            bool listed = false;  // tag[] holds the c-indices
            for (salt = 0; salt < kSaltLimit; ++salt) {
                uint32_t fsw[3];
                for (uint32_t j = 0; j < 3; ++j) fsw[j] = fold16(seed_word(seed, 3 * salt + j));
                for (uint32_t c = tid; c < kFilterBits / 32 * m_sub; c += kSaltThreads) filter[c] = 0;
                second[tid] = 0;
                if (tid == 0) {
                    s_dup = s_some = 0;
                    if (!listed) s_n = 0;
                }
                __syncthreads();
                if (!listed) {
                    enumerate();
                    __syncthreads();
                }
                listed = true;
                const uint32_t n = min(s_n, P_cap);
                // every lane busy: the non-zeros are hashed in number order (a lane's own Index word
                // holds anything from none to a dozen of them)
                auto filter_bit = [&](uint32_t t) -> uint32_t {
                    uint32_t neg;
                    const uint32_t fi = fold16(tag[t]), c0 = hash_slot_folded(fi, fsw[0], m_sub, &neg);
                    return c0 * kFilterBits + hash_slot_folded(fi, fsw[1], m_sub, &neg) % kFilterBits;
                };
                auto mark = [&](uint32_t b) {
                    const uint32_t one = 1u << (b & 31);
                    if (atomicOr(&filter[b >> 5], one) & one) atomicOr(&second[(b >> 5) % kSecondWords], one);
                };
                auto list = [&](uint32_t t, uint32_t b) {
                    if (!((second[(b >> 5) % kSecondWords] >> (b & 31)) & 1u)) return;
                    const uint32_t at = add_by_lane(&s_some, 1u);
                    if (at < n_listed) some[at] = uint16_t(t);
                };
                uint32_t bit[kSaltPer];  // (larger partitions: found out twice)
#pragma unroll
                for (uint32_t q = 0; q < kSaltPer; ++q) {
                    const uint32_t t = tid + q * kSaltThreads;
                    if (t < n) mark(bit[q] = filter_bit(t));
                }
                for (uint32_t t = tid + kSaltPer * kSaltThreads; t < n; t += kSaltThreads) mark(filter_bit(t));
                __syncthreads();
                for (uint32_t c = tid; c < m_sub; c += kSaltThreads) head[c] = kNoLink;
#pragma unroll
                for (uint32_t q = 0; q < kSaltPer; ++q) {
                    const uint32_t t = tid + q * kSaltThreads;
                    if (t < n) list(t, bit[q]);
                }
                for (uint32_t t = tid + kSaltPer * kSaltThreads; t < n; t += kSaltThreads) list(t, filter_bit(t));
                __syncthreads();
                const uint32_t n_some = s_some;
                bool dup = false;
                if (n_some <= n_listed) {
                    for (uint32_t t = tid; t < n_some; t += kSaltThreads)
                        push(tag[some[t]], t, some_tag, some_link, fsw);
                    __syncthreads();
                    for (uint32_t t = tid; t < n_some; t += kSaltThreads) dup |= twice(t, some_tag, some_link);
                } else {
                    for (uint32_t t = tid; t < n; t += kSaltThreads) push(tag[t], t, tag, link, fsw);
                    listed = false;
                    __syncthreads();
                    for (uint32_t t = tid; t < n; t += kSaltThreads) dup |= twice(t, tag, link);
                }
                if (dup) s_dup = 1;
                __syncthreads();
                const bool again = s_dup != 0;
                __syncthreads();  // s_dup is cleared by the next try
                if (!again) break;
            }
            salt = min(salt, kSaltLimit - 1);
        }
        // (the salts lie behind the bounds)
        if (tid == 0) bounds[lp.A_cap + 1 + me + (b0 + i) * G] = salt;
    }
    }
}

// The ends of the partitions in the ranks' pair lists as a launch of its own: a thread per (rank,
// partition), whose binary search is 20 dependent loads, but all of them run at once.
__global__ void __launch_bounds__(256)
ranges_kernel(const LayoutBatch, const uint32_t *__restrict__ header,
              const uint32_t *__restrict__ bounds, uint32_t ranges_off, uint32_t pair_cap)
{
    const uint32_t a = blockIdx.x * 256 + threadIdx.x;
    if (a > header[TAGC_HDR_A]) return;  // (bounds[A] = n_c: all of the list)
    const auto *row = batch_row<LayoutRank>(blockIdx.y);
    const uint32_t *list = as_global(row->idx);
    uint32_t *cnt = as_global(row->cnt);
    const uint32_t key = bounds[a];
    uint32_t lo = 0, hi = min(cnt[TAGC_CNT_TOTAL], pair_cap);
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (list[mid] < key) lo = mid + 1; else hi = mid;
    }
    cnt[ranges_off + a] = lo;
}

}  // namespace

size_t salt_lds_bytes(uint32_t T_cap, uint32_t P_cap)
{
    return (kSecondWords + size_t(P_cap)) * 4 + salt_filter_bytes(T_cap, P_cap);
}

int launch_index_or(const tagc_plan_t *p, const tagc_rank_buffers *ranks, uint32_t n_ranks,
                    const tagc_shared_buffers *sh, hipStream_t s)
{
    const uint32_t n_words = uint32_t(p->n_c / 32);
    const uint32_t n_chunks = uint32_t(p->n_chunks);
    // (see index_words) prefix sums of the chunks' set bits, the chunks' set bits, the groups'
    // prefix sums inside their chunks, and the 4-bit running sum
    uint32_t *chunkpre = static_cast<uint32_t *>(sh->workspace);
    uint32_t *chunk = chunkpre + n_chunks + 1;
    uint16_t *grouppre = group_prefixes(chunkpre, n_chunks);
    // Small Indexes are merged by the layout, whose workgroups are few then.  Each reads all of the ranks' Indexes and
    // one writes the merged one meanwhile, so not where that takes a rank's own place (a merge of its own reads
    // and writes word by word).
    const bool add4 = p->cfg.index_mode == TAGC_INDEX_ADD4;
    const uint64_t wire_bytes = uint64_t(n_words) * (add4 ? 16 : 4);
    bool merges = n_chunks && n_words <= kMergeWords && p->A_cap <= kMergeMost &&
                  n_ranks <= (add4 ? kMergeRanks4 : kMaxRanksPerPass) &&
                  n_ranks * wire_bytes <= kMergeBytes;
    for (uint32_t r = 0; merges && r < n_ranks; ++r)
        merges = !overlap(sh->bitmap, 4ull * n_words, ranks[r].bitmap, wire_bytes);
    if (n_chunks && !merges) {
        ProfileScope ps("index_or", s);
        for (uint32_t r0 = 0; r0 < n_ranks; r0 += kMaxRanksPerPass) {
            RankPtrs rp{};
            const uint32_t n_in = std::min(kMaxRanksPerPass, n_ranks - r0);
            for (uint32_t r = 0; r < n_in; ++r) rp.p[r] = ranks[r0 + r].bitmap;
            const bool last = r0 + n_in == n_ranks;
            uint32_t *sum4 = chunkpre + index_words(n_chunks);
            auto kernel = p->cfg.index_mode == TAGC_INDEX_ADD4
                              ? index_merge_kernel<TAGC_INDEX_ADD4>
                              : (p->cfg.index_mode == TAGC_INDEX_ADD1
                                     ? index_merge_kernel<TAGC_INDEX_ADD1>
                                     : index_merge_kernel<TAGC_INDEX_OR1>);
            kernel<<<n_chunks, 256, 0, s>>>(rp, n_in, sh->bitmap, n_words, r0 != 0, last, sum4,
                                            last ? chunk : nullptr, grouppre);
        }
    }
    const LayoutParams lp{p->cfg.sizing,
                          p->cfg.sizing_milli,
                          p->P_cap,
                          p->T_cap,
                          (p->n_real * 1000 + p->cfg.sizing_milli - 1) / p->cfg.sizing_milli,
                          p->U_cap,
                          p->A_cap,
                          p->m_cap};
    const size_t lds = salt_lds_bytes(p->T_cap, p->P_cap);
    const size_t lds_all = lds + 6 * 1024 + (merges ? 4 * kMergeWords : 0);  // with the kernel's own
    const uint32_t per_cu = uint32_t(std::max<size_t>(1, std::min<size_t>(2, kLdsBytes / lds_all)));
    const uint32_t most = uint32_t(device_cu_count()) * per_cu;  // workgroups that fit the device at once
    // Many searches in a plan that says, by a limit on the decoder's workgroups, that other buckets
    // are in flight: three launches.  In the one launch the workgroups that wait for the searches'
    // loads hold a compute unit's local memory, and no other bucket's salts run meanwhile; and 16
    // lanes to a search read more than a thread's binary search does.  16 ranks of 202 M entries,
    // 58 thousand searches: 12 buckets in flight 190 us each in one launch (with the merge), 153 in
    // three.  Alone one launch is the better, 105 and 113 us (without the merge), and it leaves the
    // pair lists in the cache for the encoder (570 us, 582 after three launches).
    const bool split = p->cfg.decode_workgroups && p->A_cap * n_ranks > kSplitSearches;
    const uint32_t batches = uint32_t(std::min<uint64_t>((p->A_cap + kLayoutBatch - 1) / kLayoutBatch,
                                                         uint64_t(device_cu_count()) * 2));
    // Searching workgroups of the one launch, and those that look for salts, each taking partitions b, b + grid,
    // ...  The searches of a partition grow with the ranks, its salt does not: 64 are done before the salts
    // with up to eight ranks, 96 with more (us of layout, 32 / 64 / 96 / 128 of them: 16 ranks of 202 M entries
    // 238 / 138 / 106 / 115, where all workgroups did both in 125; 12 ranks 155 / 93 / 86 / 93; 8 ranks 87 / 65 / 65 /
    // 71; 4 ranks 48 / 48 / 52 / 51; 16 ranks of 9 M with two fifths
    // 98 / 64 / 51 / 54).  None, all of them do both, where all workgroups have a partition each and the salts'
    // alone would not (8 ranks of 49 M entries, 464 partitions, 24.9).  A call may have as few under a plan for more,
    // when ranks share what they keep: two turns (480 partitions, 29.8; 28.7 if all did both, but for the
    // kernel to ask how many there are cost all other calls 0.5 to 1).  Nor where there are more partitions than
    // workgroups, and small ones: the salts are the lesser part then (50 M entries, all do both / 64, or 96, apart: 4
    // ranks with partitions of 40 non-zeros 291 / 405, 320 49 / 63, 640 32 / 39, 1280 25.6 / 25.5, 2560 23.3 / 21.6,
    // 6400 25.9 / 23.8; 8 ranks with 640 56 / 66, 1280 38.8 / 40.5, 2560 30.0 / 27.7; 16 ranks 103 / 125, 69 / 73, 48 / 47).
    // Nor where there are few ranks and many partitions of the default size, whose searches are little beside the
    // salts that 64 workgroups less look for (both / apart: 1 rank, 2000, 3000, 4900 partitions 60 / 60, 81 / 85,
    // 124 / 127; 2 ranks, 2000, 3000, 4640, 8800 60 / 61, 82 / 86, 119 / 124, 198 / 212; 4 ranks, 1900, 2300, 2400, 3200,
    // 4200, 7200 68.5 / 64, 65 / 68, 58.5 / 55.5, 85 / 87, 102 / 107, 169 / 174; 5 ranks, 3200, 5000 87 / 87, 121 / 121;
    // 6 ranks, 2900 82 / 75).
    const uint32_t want = std::min(n_ranks > 8 ? 96u : 64u, batches);
    const bool apart = p->A_cap + want <= most ||
                       (p->A_cap > most && p->U_cap >= kSearchApart * p->A_cap &&
                        (n_ranks > 4 || p->A_cap <= 5 * uint64_t(most)));
    const uint32_t searching = apart ? std::min(want, most / 2) : 0u;
    const uint32_t salting = uint32_t(std::min<uint64_t>(p->A_cap, most - searching));
    const auto layout = !merges ? layout_kernel<true, true, true, kNoMerge>
                        : p->cfg.index_mode == TAGC_INDEX_ADD4 ? layout_kernel<true, true, true, TAGC_INDEX_ADD4>
                        : p->cfg.index_mode == TAGC_INDEX_ADD1 ? layout_kernel<true, true, true, TAGC_INDEX_ADD1>
                                                               : layout_kernel<true, true, true, TAGC_INDEX_OR1>;
    const auto salts = layout_kernel<false, false, true, kNoMerge>;
    static size_t attr_bytes[5] = {};
    size_t &attr = attr_bytes[merges ? 2 + p->cfg.index_mode : split ? 1 : 0];
    if (lds > attr) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(split ? salts : layout),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(lds)) != hipSuccess)
            return TAGC_EHIP;
        attr = lds;
    }
    auto launch = [&](auto kernel, uint32_t n_wgs, size_t lds_bytes, const LayoutBatch &lb,
                      uint32_t n_in, bool all, uint32_t n_search) {
        // (searching workgroups are the last: on a device nearly full of those with a partition each they then
        // share few compute units, 8 ranks of 25 M entries, us a pass, first / last: 239 / 237, with 4-bit
        // counters 281 / 277)
        const uint32_t search0 = n_wgs;
        kernel<<<n_wgs + n_search, kSaltThreads, lds_bytes, s>>>(
            lb, n_in, all, sh->bitmap, n_words, uint32_t(p->n_c), chunk, grouppre, chunkpre, n_chunks, lp,
            sh->header, sh->status, sh->bounds, p->cnt_ranges, uint32_t(p->K), p->cfg.seed, n_search, search0);
    };
    for (uint32_t r0 = 0; r0 < n_ranks; r0 += kMaxRanksPerPass) {
        // (ranks beyond the first launch's only need their pair lists searched)
        LayoutBatch lb{};
        const uint32_t n_in = std::min(kMaxRanksPerPass, n_ranks - r0);
        for (uint32_t r = 0; r < n_in; ++r)
            lb.r[r] = LayoutRank{ranks[r0 + r].idx, ranks[r0 + r].cnt, ranks[r0 + r].bitmap};
        if (r0 == 0 || !split) {
            ProfileScope ps("layout", s);
            if (split) launch(layout_kernel<true, false, false, kNoMerge>, batches, 0, lb, n_in, true, 0);
            else if (r0 == 0) launch(layout, salting, lds, lb, n_in, true, searching);
            else launch(layout_kernel<true, true, false, kNoMerge>, 0, 0, lb, n_in, false, batches);
        }
        if (split) {
            ProfileScope ps("ranges", s);
            ranges_kernel<<<dim3(uint32_t((p->A_cap + 1 + 255) / 256), n_in), 256, 0, s>>>(
                lb, sh->header, sh->bounds, p->cnt_ranges, uint32_t(p->K));
        }
    }
    if (split) {
        ProfileScope ps("salt", s);
        launch(salts, uint32_t(std::min<uint64_t>(p->A_cap, most)), lds, LayoutBatch{}, 0, true, 0);
    }
    return hip_ok(hipGetLastError());
}

}  // namespace tagc
