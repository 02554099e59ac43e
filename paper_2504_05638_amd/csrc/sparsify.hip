// Stage 1 of the hot path: dynamic magnitude sparsifier + local Index.
//
// For every compressed segment of one rank's gradient bucket: find the threshold key T
// such that exactly k_l entries survive (section 3.2: the zeroing value is chosen
// dynamically so that at least theta of the values become zero), then emit the
// survivors as (c-index, float32 value) pairs in ascending c-index together with the
// 1-bit-per-parameter Index (Algorithm 1: sparsify, create_index).
//
// Keys: |g| as an unsigned integer (float32 bit pattern with the sign cleared; bf16 is
// widened first).  Ties at the threshold go to the lower position; exact zeros never
// survive.
//
// Two routes per segment, both exact:
//
//  candidate route (one read of the gradient)
//    prepare      only on the first call after the plan's table was uploaded: a strided
//                 sample gives every segment a conservative pre-threshold bin; afterwards
//                 each call leaves the pre-threshold for the next one in the table
//    scan_spill   streams the segment once: entries with key bin >= the pre-threshold
//                 ("candidates", ~1.3 x k of them) are histogrammed and spilled, in position
//                 order, into fixed slots per 4 KiB chunk -- no cross-wave dependency.  The
//                 workgroup that finishes a segment last selects its exact threshold from
//                 the candidate histogram; if the candidates do not contain k entries (the
//                 pre-threshold misled) the segment is re-routed
//    refine       fp32 only: low 16 key bits inside the threshold bin
//    count        survivors of every super-chunk of candidates (32 chunks)
//    place        ordered pass over the candidates only: pairs + every Index word
//
//  dense route (segments that are short, unaligned, keep more than ~23 %, have no
//  pre-threshold yet, or were re-routed; three reads)
//    hist1        exact histogram of the top 15 key bits of every entry, in LDS windows; the
//                 workgroup that completes a segment's histogram selects its threshold.  A
//                 segment that one workgroup's registers hold is selected by one, fp32 included
//    refine       fp32 only, as above, from the gradient
//    count        survivors of every tile of the gradient
//    place        ordered pass over the gradient: pairs + Index words
//
// count and place are one launch each for both routes.  Ordered output across workgroups
// needs no waiting: place starts when every count is there, and every item adds up the counts
// of the earlier items of its segment by itself.
//
// With a gradient accumulator (error feedback: Algorithm 1, lines 1-2) what is sparsified is
// grad + acc: scan_spill, and accumulate for the segments it does not read, write the sums
// back to acc, from which the dense route then reads; which of them were sent is recorded
// by the rank's own Index and applied when acc is read next (see SentMap).  With 4-bit
// counters on the wire (section 2.2) widen4 turns the Index into them at the end.
//
// Counters that must start at zero (arrivals, the candidate histograms) live in the plan's
// table, which only the library writes: whoever reads them last puts them back to zero, so
// no call spends a launch on clearing (see TableState).
#include <mutex>
#include <type_traits>

#include "device_utils.h"
#include "tagc_internal.h"

namespace tagc {

namespace {

constexpr int kF32 = TAGC_F32, kBF16 = TAGC_BF16;

// What a launch needs to know of one rank.  A launch takes a batch of ranks, blockIdx.y being the
// rank's row: ranks are independent of each other up to the Index merge, and a launch of one
// rank's work spends a good part of its time starting, draining and turning round (a rank's
// scan of 405 MB streams for 57 us and takes 80).
struct SparsifyRank {
    const char *grad;
    char *acc;             // error feedback: the accumulator, or NULL
    const uint32_t *sent;  // error feedback: the Index the rank's previous call left
    char *ws;              // the rank's workspace
    uint32_t *idx;
    float *val;
    uint32_t *bitmap;      // 1-bit Index (in the workspace if the wire takes 4-bit counters)
    uint32_t *wire;        // the rank's Index as it goes on the wire
    uint32_t *cnt;
    uint32_t slot;         // the rank's slot of the table's device state
    uint32_t from;         // the slot whose carried pre-thresholds it starts from
};
struct SparsifyBatch {
    SparsifyRank r[kMaxRanksPerPass];
};
static_assert(sizeof(SparsifyBatch) <= 3072, "kernel arguments are limited to 4 KiB");

// Where things are in a rank's workspace, and how many candidate slots it has; and what the table's
// first words say as well (segments, tiles, super-chunks).  Everything in these kernels waits for that:
// read from the table it is a trip to memory in front of each of them.
struct WsLayout {
    uint64_t hist1d, hist2, group_cnt, sel, tile_cnt, sc_cnt, chunk_info, cand, n_slots;
    uint32_t L, total_tiles, total_sc;
};

// The row of the rank a workgroup works for, its pointers known to be global memory.
struct RankView {
    const char *grad;
    char *acc;
    const uint32_t *sent;
    char *ws;
    uint32_t *idx;
    float *val;
    uint32_t *bitmap;
    uint32_t *wire;
    uint32_t *cnt;
    uint32_t slot, from;
    // what is sparsified: the gradient, or the sums in the accumulator
    __device__ inline const char *src() const { return acc ? acc : grad; }
    template <typename T>
    __device__ inline T *at(uint64_t offset) const { return reinterpret_cast<T *>(ws + offset); }
};
__device__ inline RankView rank_view()
{
    const auto *r = batch_row<SparsifyRank>(blockIdx.y);
    return RankView{as_global(r->grad), as_global(r->acc),    as_global(r->sent), as_global(r->ws),
                    as_global(r->idx),  as_global(r->val),    as_global(r->bitmap),
                    as_global(r->wire), as_global(r->cnt),    r->slot,            r->from};
}

__global__ void __launch_bounds__(256) fill_zero_kernel(uint4 *p, uint64_t n16, uint32_t *cnt,
                                                        uint32_t n_cnt)
{
    const uint4 z = make_uint4(0, 0, 0, 0);
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < n16; i += gridDim.x * 256ull)
        p[i] = z;
    if (blockIdx.x == 0)
        for (uint32_t i = threadIdx.x; i < n_cnt; i += 256) cnt[i] = 0;
}

__device__ inline uint32_t load_elem_bits(const char *base, uint64_t i, int dtype)
{
    if (dtype == kBF16) return uint32_t(reinterpret_cast<const uint16_t *>(base)[i]) << 16;
    return reinterpret_cast<const uint32_t *>(base)[i];
}

// float32 bit pattern of element e of a 16-byte vector
template <int DTYPE>
__device__ inline uint32_t vec_elem_bits(const uint32_t (&w)[4], uint32_t e)
{
    return DTYPE == kBF16 ? ((w[e >> 1] >> (16 * (e & 1))) << 16) : w[e];
}

// g + acc in the gradient's own type (Algorithm 1, line 1; section 3.2, local gradient
// accumulation): one float32 add per entry; a bf16 result is rounded to nearest-even (a NaN
// keeps a mantissa bit).  `g`, `a`: one 32-bit word of each buffer (two bf16 entries).
template <int DTYPE>
__device__ inline uint32_t sum_word(uint32_t g, uint32_t a)
{
    if (DTYPE == kF32) return __float_as_uint(__uint_as_float(g) + __uint_as_float(a));
    const float lo = __uint_as_float(g << 16) + __uint_as_float(a << 16);
    const float hi = __uint_as_float(g & 0xFFFF0000u) + __uint_as_float(a & 0xFFFF0000u);
    return round_to_bf16(lo) | (round_to_bf16(hi) << 16);
}
// the same for one entry given as float32 bit patterns; returns the entry's bit pattern in
// its own type (low 16 bits for bf16)
template <int DTYPE>
__device__ inline uint32_t sum_elem(uint32_t g_f32bits, uint32_t a_f32bits)
{
    const float x = __uint_as_float(g_f32bits) + __uint_as_float(a_f32bits);
    return DTYPE == kF32 ? __float_as_uint(x) : round_to_bf16(x);
}
__device__ inline void store_elem(char *base, uint64_t i, uint32_t bits, int dtype)
{
    if (dtype == kBF16) reinterpret_cast<uint16_t *>(base)[i] = uint16_t(bits);
    else reinterpret_cast<uint32_t *>(base)[i] = bits;
}

// Error feedback keeps the record of what a rank sent in the rank's Index, not in the
// accumulator: clearing ~1 % of the accumulator's entries one by one after the streaming
// pass touched almost half of its cache lines a second time (measured: 140 us per rank on
// 7B-shaped buckets).  Instead an entry of acc whose bit is set in the Index the rank's
// previous call left (`sent`: 1 bit per parameter, or the 4-bit counters) reads as 0, and
// the next call's streaming pass, which rewrites all of acc anyway, applies that.
struct SentMap {
    const uint32_t *map;  // the rank's Index buffer as the previous call left it
    uint32_t wire4;       // 4-bit counters instead of bits
};

// bit e <=> parameter ci + e was sent, for the VEC parameters of one 16-byte vector
// (ci a multiple of VEC, VEC = 4 or 8)
template <uint32_t VEC>
__device__ inline uint32_t sent_bits(const SentMap sm, uint32_t ci)
{
    if (sm.wire4) {
        const uint32_t w = sm.map[ci >> 3];
        return VEC == 8 ? nibbles_set(w) : nibbles_set((w >> (4 * (ci & 4u))) & 0xFFFFu);
    }
    const uint32_t b = reinterpret_cast<const uint8_t *>(sm.map)[ci >> 3];
    return VEC == 8 ? b : (b >> (ci & 4u)) & 0xFu;
}

__device__ inline bool sent_bit(const SentMap sm, uint32_t ci)
{
    if (sm.wire4) return ((sm.map[ci >> 3] >> (4 * (ci & 7u))) & 0xFu) != 0;
    return ((sm.map[ci >> 5] >> (ci & 31u)) & 1u) != 0;
}

// float32 bit pattern of entry i of a segment's accumulator, 0 if it was sent
__device__ inline uint32_t unsent_elem(const char *ab, uint64_t i, uint32_t c_off,
                                       const SentMap sm, int dtype)
{
    return sent_bit(sm, c_off + uint32_t(i)) ? 0u : load_elem_bits(ab, i, dtype);
}

// word j of an accumulator vector with the entries named by `bits` (see sent_bits) cleared
template <int DTYPE>
__device__ inline uint32_t unsent_word(uint32_t a, uint32_t bits, uint32_t j)
{
    if (DTYPE == kF32) return (bits >> j) & 1u ? 0u : a;
    const uint32_t two = (bits >> (2 * j)) & 3u;
    return a & ~((two & 1u ? 0xFFFFu : 0u) | (two & 2u ? 0xFFFF0000u : 0u));
}

// Error feedback for the segments scan_spill never streams (short, unaligned, keeping
// nothing or too much): acc <- grad + acc, entry by entry.  The dense route then reads its
// input from acc.  Workgroups stride over each such segment.
template <int DTYPE>
__global__ void __launch_bounds__(256)
accumulate_kernel(const SparsifyBatch, const uint32_t *__restrict__ table, uint32_t wire4)
{
    const RankView rv = rank_view();
    const char *grad = rv.grad;
    char *acc = rv.acc;
    const SentMap sent{rv.sent, wire4};
    constexpr uint32_t EB = DTYPE == kBF16 ? 2 : 4;
    constexpr uint32_t VEC = 16 / EB;
    const uint32_t L = table[0];
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    for (uint32_t l = 0; l < L; ++l) {
        const SegDev sd = segs[l];
        if (sd.n == 0 || (sd.flags & kSegFast)) continue;
        const char *gb = grad + sd.offset * EB;
        char *ab = acc + sd.offset * EB;
        const uint64_t stride = uint64_t(gridDim.x) * 256;
        if (sd.flags & kSegAligned) {
            const uint64_t nvec = sd.n / VEC;
            for (uint64_t v = uint64_t(blockIdx.x) * 256 + threadIdx.x; v < nvec; v += stride) {
                const uint4 g = ld_stream(reinterpret_cast<const uint4 *>(gb) + v);
                const uint4 a = ld_stream(reinterpret_cast<const uint4 *>(ab) + v);
                const uint32_t sb = sent_bits<VEC>(sent, sd.c_off + uint32_t(v) * VEC);
                reinterpret_cast<uint4 *>(ab)[v] =
                    make_uint4(sum_word<DTYPE>(g.x, unsent_word<DTYPE>(a.x, sb, 0)),
                               sum_word<DTYPE>(g.y, unsent_word<DTYPE>(a.y, sb, 1)),
                               sum_word<DTYPE>(g.z, unsent_word<DTYPE>(a.z, sb, 2)),
                               sum_word<DTYPE>(g.w, unsent_word<DTYPE>(a.w, sb, 3)));
            }
            if (blockIdx.x == 0) {
                const uint64_t i = nvec * VEC + threadIdx.x;
                if (i < sd.n)
                    store_elem(ab, i, sum_elem<DTYPE>(load_elem_bits(gb, i, DTYPE),
                                                      unsent_elem(ab, i, sd.c_off, sent, DTYPE)),
                               DTYPE);
            }
        } else {
            for (uint64_t i = uint64_t(blockIdx.x) * 256 + threadIdx.x; i < sd.n; i += stride)
                store_elem(ab, i, sum_elem<DTYPE>(load_elem_bits(gb, i, DTYPE),
                                                  unsent_elem(ab, i, sd.c_off, sent, DTYPE)),
                           DTYPE);
        }
    }
}

// ----------------------------------------------------------------- select

// For each of two counts `want` (0 = not asked): the largest bin b with
// sum_{x >= b} get(x) >= want and the entries in higher bins; bin = kNoBin if all
// bins together hold fewer.  By a workgroup of NT threads, thread t owning the BPT consecutive
// bins from t * BPT, whose sum it passes as `own`; the thread whose bins hold the answer leaves
// its number, and one wave reads those bins side by side.
constexpr uint32_t kNoBin = 0xFFFFFFFFu;
struct BinFound {
    uint32_t bin, above;
};
template <uint32_t NT, uint32_t BPT, typename Get>
__device__ inline void select_top(Get &&get, uint32_t own, const uint32_t (&want)[2],
                                  BinFound (&found)[2], uint32_t *total_out,
                                  uint32_t *smem /* >= 32 words */)
{
    static_assert(NT >= 128, "a wave per count");
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t total;
    const uint32_t prefix = block_excl_scan<uint32_t, NT / 64>(own, &total, smem);
    const uint32_t suffix = total - prefix;  // bins of this thread and all higher ones
    if (t < 2) smem[16 + 4 * t] = smem[17 + 4 * t] = kNoBin;
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i)
        if (want[i] && suffix >= want[i] && suffix - own < want[i]) {
            smem[16 + 4 * i] = t;
            smem[18 + 4 * i] = suffix - own;
        }
    __syncthreads();
    uint32_t owner = kNoBin, acc = 0;
    if (wave < 2) {
        owner = smem[16 + 4 * wave];
        acc = smem[18 + 4 * wave];
    }
    __syncthreads();  // (the words are written again below)
    if (owner != kNoBin) {  // wave-uniform
        const uint32_t need = wave ? want[1] : want[0];
        constexpr int NB = (BPT + 63) / 64;  // looked at 64 at a time, from the top down
#pragma unroll
        for (int k = NB - 1; k >= 0; --k) {
            const uint32_t b = uint32_t(k) * 64 + lane;
            const uint32_t c = b < BPT ? get(owner * BPT + b) : 0u;
            const uint32_t inc = wave_incl_scan<uint32_t>(c);
            const uint32_t tot = __builtin_amdgcn_readlane(inc, 63);
            const uint32_t above = acc + tot - inc;
            if (above < need && above + c >= need) {
                smem[16 + 4 * wave] = owner * BPT + b;
                smem[17 + 4 * wave] = above;
            }
            acc += tot;
        }
    } else if (wave < 2 && lane == 0) {
        smem[16 + 4 * wave] = kNoBin;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i)
        found[i] = BinFound{smem[16 + 4 * i], smem[17 + 4 * i]};
    *total_out = total;
    __syncthreads();
}

// sum of the BPT bins a thread owns of an array in memory
template <uint32_t BPT>
__device__ inline uint32_t own_bins(const uint32_t *hist)
{
    const uint4 *hv = reinterpret_cast<const uint4 *>(hist + threadIdx.x * BPT);
    uint32_t s = 0;
#pragma unroll 8
    for (uint32_t i = 0; i < BPT / 4; ++i) {
        const uint4 v = hv[i];
        s += v.x + v.y + v.z + v.w;
    }
    return s;
}

// ---------------------------------------------------------------- prepare

// First call after the table's upload.  One workgroup per compressed segment:
// segments on the candidate route that have no pre-threshold yet get one from a strided sample
// of 16-byte vectors: the sample bin above which  k*S/n + 5*sqrt(k*S/n) + 16  sampled entries
// lie.  The margin makes it very unlikely that fewer than k entries of the whole segment pass
// the pre-threshold; if that still happens the selection notices and re-routes the segment.
// A sample that holds too few non-zeros to say anything leaves the segment without one: it
// takes the dense route this time, whose histogram then provides it.
template <int DTYPE>
__global__ void __launch_bounds__(kHistThreads)
prepare_kernel(const SparsifyBatch, uint32_t *table, uint32_t wire4)
{
    extern __shared__ uint32_t h[];
    __shared__ uint32_t smem[32];
    constexpr uint32_t EB = DTYPE == kBF16 ? 2 : 4;
    constexpr uint32_t VEC = 16 / EB;
    const uint32_t L = table[0];
    const uint32_t tid = threadIdx.x;
    const RankView rv = rank_view();
    const char *grad = rv.grad, *acc = rv.acc;
    const SentMap sent{rv.sent, wire4};
    const uint32_t l = blockIdx.x;
    const SegDev sd = reinterpret_cast<const SegDev *>(table + 8)[l];
    const TableState ts = table_state(table, L, rv.slot);
    if (sd.k == 0 || sd.n == 0 || !(sd.flags & kSegFast) || ts.hint[l]) return;
    for (uint32_t i = tid; i < kBins1; i += kHistThreads) h[i] = 0;
    __syncthreads();
    const uint32_t nvec = sd.n / VEC;
    const uint32_t S = min(nvec, kSampleVectors);
    const uint32_t stride = nvec / S;
    const uint4 *vp = reinterpret_cast<const uint4 *>(grad + sd.offset * EB);
    const uint4 *ap = acc ? reinterpret_cast<const uint4 *>(acc + sd.offset * EB) : nullptr;
    for (uint32_t i = tid; i < S; i += kHistThreads) {
        uint4 q = vp[uint64_t(i) * stride + (stride >> 1)];
        if (ap) {  // error feedback: what is sparsified is grad + acc
            const uint32_t v = i * stride + (stride >> 1);
            const uint4 a = ap[v];
            const uint32_t sb = sent_bits<VEC>(sent, sd.c_off + v * VEC);
            q = make_uint4(sum_word<DTYPE>(q.x, unsent_word<DTYPE>(a.x, sb, 0)),
                           sum_word<DTYPE>(q.y, unsent_word<DTYPE>(a.y, sb, 1)),
                           sum_word<DTYPE>(q.z, unsent_word<DTYPE>(a.z, sb, 2)),
                           sum_word<DTYPE>(q.w, unsent_word<DTYPE>(a.w, sb, 3)));
        }
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (uint32_t e = 0; e < VEC; ++e) {
            const uint32_t key = vec_elem_bits<DTYPE>(w, e) & 0x7FFFFFFFu;
            if (key) atomicAdd(&h[key >> 16], 1u);
        }
    }
    __syncthreads();
    const float ks = float(double(sd.k) * double(S * VEC) / double(sd.n));
    const uint32_t need = uint32_t(ks + 5.0f * sqrtf(ks) + 16.0f) + 1u;
    uint32_t total;
    BinFound f[2];
    constexpr uint32_t BPT = kBins1 / kHistThreads;
    select_top<kHistThreads, BPT>([&](uint32_t b) { return h[b]; }, own_bins<BPT>(h), {need, 0u}, f,
                                  &total, smem);
    // bin 0 (|g| < 2^-133) is never a candidate
    if (tid == 0 && f[0].bin != kNoBin) ts.hint[l] = max(f[0].bin, 1u);
}

// ------------------------------------------------------------- scan_spill

// Streams every candidate-route segment once.  A wave owns one chunk (64 lanes x 4 rows
// of 16-byte vectors, contiguous) at a time; candidates (key bin >= binlo) are counted in
// the workgroup's LDS histogram and written in position order to the chunk's slot array.
// bf16 slot: (bf16 bits << 16) | position in chunk.  fp32 slot: value bits in cand[slot],
// position in cand[n_slots_total + slot].
//
// Work assignment: the chunks of all segments form one list (a segment's chunks start at
// its first super-chunk); each workgroup takes one contiguous span of it, its waves
// interleaved inside the span.  A workgroup therefore meets a segment boundary -- where
// the LDS histogram has to be flushed behind barriers -- only if its span straddles one,
// instead of the whole grid draining at every boundary.
//
// Memory operations of a wave complete, as far as the wave can tell, in the order they
// were issued, and a store is acknowledged later than a load returns: a wave that stores
// a chunk's slots and then loads the next chunk waits for the acknowledgement as well,
// about a microsecond per chunk.  So the steady state of this kernel issues loads only.
// The next chunk is requested while the current one is processed, and the slots of a
// dozen chunks pile up in the wave's LDS staging area and leave together (when the area
// is full, and at the end), at which point nothing is waiting behind the stores.
//
// Two 512-thread workgroups per CU.  With the next chunk always in flight that keeps about
// 32 MB of requests outstanding, enough to saturate HBM; more only lengthens the queue the
// last workgroups to start wait in, and they keep that lag to the end of the kernel.  The
// LDS pays for the chunk buffer (candidates are fetched from it by position instead of
// being selected out of sixteen registers) and the staging area.  The histogram covers the
// kWinBins bins from the segment's pre-threshold upwards (12 octaves of magnitude); what lies
// above them is only counted (it survives whenever the threshold is inside the window, and
// otherwise the segment is re-routed).  Slot order inside a chunk comes from a wave-local
// scan of the per-lane counts, so a wave never waits on another.
//
// A workgroup that is done with its part of a segment adds its histogram to the segment's
// in the plan's table and counts itself as arrived; the one that arrives last selects the
// segment's threshold on the spot (select_window) and puts the table words back to zero.
// The kernel's workgroups also clear, as they start, the dense route's histograms in the
// rank workspace, which nothing touches before the kernels after this one.
constexpr uint32_t kSpillThreads = 512;
#ifndef TAGC_SPILL_WGS
#define TAGC_SPILL_WGS 2
#endif
constexpr uint32_t kSpillWgsPerCU = TAGC_SPILL_WGS;  // workgroups launched per compute unit
constexpr uint32_t kSpillSpan = 128;   // chunks a workgroup's span has at least in launches of several rounds
// Slots and chunks a wave stages before they leave.  Stores among the loads cost the scan more than
// their bytes (16 ranks of 202 M bf16 entries: 235 MB of 6.7 GB, a tenth of the time; without its
// stores it would run at 6.2 TB/s), so they leave in runs as long as the LDS of two workgroups per
// compute unit has room for.  bf16, 512 slots and 16 chunks / 1024 and 32, us: one rank 82 / 77,
// 8 ranks of 67 M 201 / 198, with an accumulator 276 / 270, a tenth kept 225 / 220; fp32, which
// needs two words a slot, 58 / 65 (one workgroup per compute unit).  Not so beside other buckets: two workgroups
// with the short stage leave 49 KiB, enough for one of another bucket's encoder (48 KiB and 31 registers), with
// the long one 10.  Buckets of 202 M entries, 12 in flight, ms a step, short / long: 32 from 16 ranks at load factor
// 1.5 87.4 / 88.3, at 1.15 88.3 / 90.2; 12 from 2 ranks with 3 and 5 % kept 7.6 / 7.7 and 9.7 / 9.7, with a tenth,
// where a chunk has hundreds of slots and a run of 512 is a chunk or two, 16.1 / 15.9, with a fifth 26.2 / 25.8.
template <int DTYPE, bool LONG>
constexpr uint32_t kSpillStage = DTYPE == kBF16 && LONG ? 1024 : 512;
template <int DTYPE, bool LONG>
constexpr uint32_t kSpillList = DTYPE == kBF16 && LONG ? 32 : 16;
constexpr uint32_t kWatchCalls = 8;    // calls that extrapolate a falling pre-threshold after a miss
constexpr uint32_t kSpillRaise = 6;    // bins (1/128 octave each) a wave's pre-threshold goes up per try

// Threshold of one candidate-route segment from its candidate histogram `win` (table), by
// the kSpillThreads threads of the scan's last workgroup on the segment.  Leaves SelDev,
// the segment's count, the pre-threshold for the next call, and the table words at zero.
// pre-threshold for the next call from `bin2`, the bin above which 1.3 k entries lie now:
// that bin itself, or, in the calls after a miss (the scale fell by more than the margin
// since the hint was tuned), lower by the factor it fell by since the call before (at most
// half an octave) and 1.5 % more.  Bins are float32 bit patterns >> 16: the magnitudes are
// extrapolated, not the bin numbers, whose width in relative terms varies twofold across an
// octave.
__device__ inline uint32_t next_hint(uint32_t bin2, uint32_t prev, uint32_t watch)
{
    if (!watch || prev <= bin2) return max(bin2, 1u);
    const float now = __uint_as_float(bin2 << 16), before = __uint_as_float(prev << 16);
    const float fall = fmaxf(now / before, 0.7071f);
    return max(__float_as_uint(now * fall * 0.985f) >> 16, 1u);
}

template <int DTYPE>
__device__ inline void select_window(uint32_t l, const SegDev &sd, uint32_t blo,
                                     const TableState ts, const TableState from, SelDev *sel, uint32_t *smem /* >= 32 */)
{
    constexpr uint32_t BPT = kWinBins / kSpillThreads;  // consecutive bins per thread
    static_assert(BPT * kSpillThreads == kWinBins, "every thread owns BPT bins of the window");
    const uint32_t tid = threadIdx.x;
    uint32_t *win = ts.win + size_t(l) * kWinWords;
    uint32_t c[BPT];
#pragma unroll
    for (uint32_t b = 0; b < BPT; ++b) {
        c[b] = win[tid * BPT + b];
        win[tid * BPT + b] = 0;
    }
    const uint32_t above_w = win[kWinBins], nf = win[kWinBins + 1];
    const uint32_t raised = ts.raised[l], overflow = ts.reroute[l];
    const uint32_t prev = from.prev[l], wt = from.watch[l];  // (requested with the rest)
    __syncthreads();  // everybody has read what thread 0 clears next
    if (tid == 0) {
        win[kWinBins] = win[kWinBins + 1] = 0;
        ts.raised[l] = ts.reroute[l] = ts.arrive[l] = 0;
    }
    // the histogram is complete from the highest pre-threshold any wave used upwards
    const uint32_t floor_bin = max(blo, raised), floor_w = floor_bin - blo;
    uint32_t s = 0;
#pragma unroll
    for (uint32_t b = 0; b < BPT; ++b) {
        if (tid * BPT + b < floor_w) c[b] = 0;
        s += c[b];
    }
    uint32_t total;
    const uint32_t prefix = block_excl_scan<uint32_t, kSpillThreads / 64>(s, &total, smem);
    const uint32_t suffix = total - prefix + above_w;  // this thread's bins and everything higher
    // largest bin with at least `need` entries at or above it; twice: the threshold (k), and
    // the pre-threshold for the next call (1.3 k, what the slots per chunk are sized for)
    const uint32_t want = uint32_t(1.3f * float(sd.k)) + 1u;
    if (tid == 0) smem[16] = smem[19] = 0xFFFFFFFFu;
    __syncthreads();
    auto locate = [&](uint32_t need, uint32_t *bin_out, uint32_t *above_out) {
        if (!(s && suffix >= need && suffix - s < need)) return;
        uint32_t acc = suffix - s;  // entries in the bins above the one looked at
#pragma unroll
        for (int b = int(BPT) - 1; b >= 0; --b) {
            if (acc + c[b] >= need) {
                *bin_out = tid * BPT + uint32_t(b);
                if (above_out) *above_out = acc;
                return;
            }
            acc += c[b];
        }
    };
    locate(sd.k, &smem[16], &smem[17]);
    locate(want, &smem[19], nullptr);
    __syncthreads();
    if (tid != 0) return;
    const uint32_t bin_w = smem[16], above = smem[17], bin2_w = smem[19];
    const bool found = bin_w != 0xFFFFFFFFu && !overflow && blo != 0;
    SelDev r{};
    if (!found) {
        // The candidates hold fewer than k entries (the scale fell since the pre-threshold
        // was tuned), the threshold lies above the window, slots overflowed, or there was no
        // pre-threshold: dense route, whose histogram also provides the next pre-threshold.
        r.route = 1;
        ts.watch[l] = blo != 0 && !overflow && above_w < sd.k ? kWatchCalls : wt;
        ts.prev[l] = prev;
        ts.hint[l] = 0;
        sel[l] = r;
        return;
    }
    // The window may not reach down to 1.3 k entries; then one bin below what this call
    // could see.
    const uint32_t bin2 = bin2_w != 0xFFFFFFFFu ? max(blo + bin2_w, 1u) : max(floor_bin, 2u) - 1u;
    ts.hint[l] = next_hint(bin2, prev, wt);
    ts.prev[l] = bin2;
    ts.watch[l] = wt ? wt - 1 : 0u;
    if (nf) atomicAdd(&ts.glob[1], nf);
    const uint32_t T_bin = blo + bin_w;
    if (DTYPE == kBF16) {
        r.T = T_bin << 16;
        r.G = above;
        r.quota = sd.k - above;
        r.cnt = sd.k;
    } else {
        r.bin1 = T_bin;
        r.G1 = above;
        r.need2 = 1;
    }
    sel[l] = r;
}

// ACC: with a gradient accumulator (all ranks of a launch have one, or none).  LONG: the longer stage.
template <int DTYPE, bool ACC, bool LONG>
__global__ void __launch_bounds__(kSpillThreads)
scan_spill_kernel(const SparsifyBatch, uint32_t *table, const WsLayout wl, uint32_t CAP,
                  uint64_t zero_n16, uint32_t wire4)
{
    const RankView rv = rank_view();
    const char *__restrict__ grad = rv.grad;
    char *acc = ACC ? rv.acc : nullptr;
    const SentMap sent{rv.sent, wire4};
    SelDev *sel = rv.at<SelDev>(wl.sel);
    uint32_t *__restrict__ cand = rv.at<uint32_t>(wl.cand);
    uint2 *__restrict__ chunk_info = rv.at<uint2>(wl.chunk_info);
    const uint64_t n_slots_total = wl.n_slots;
    uint4 *zero_base = rv.at<uint4>(0);
    constexpr uint32_t EB = DTYPE == kBF16 ? 2 : 4;
    constexpr uint32_t VEC = 16 / EB;
    constexpr uint32_t ROWS = kCandRows;
    constexpr uint32_t ROW_ELEMS = 64 * VEC;
    constexpr uint32_t CHUNK = ROW_ELEMS * ROWS;
    constexpr uint32_t NW = kSpillThreads / 64;
    constexpr uint32_t STAGE = kSpillStage<DTYPE, LONG>, LIST = kSpillList<DTYPE, LONG>;
    constexpr uint32_t STAGE_WORDS = STAGE * (DTYPE == kBF16 ? 1 : 2);
    static_assert(ROWS == 4 && ROWS * VEC <= 32, "packed masks and row counts below");
    __shared__ uint32_t h[kWinWords];
    __shared__ uint32_t s_sel[32];
    __shared__ uint32_t s_last;
    __shared__ uint32_t s_region;  // slots of the workgroup's part of `cand` handed out so far
    __shared__ uint32_t stage[NW][STAGE_WORDS];
    __shared__ uint32_t list[NW][3][LIST];  // chunk number, staging offset, count
    __shared__ uint4 data[NW][ROWS * 64];         // each wave's current chunk
    const uint32_t L = wl.L;
    const uint32_t total_chunks = wl.total_sc * kCandChunksPerSuper;
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    const TableState ts = table_state(table, L, rv.slot), from = table_state(table, L, rv.from);
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    // wave-uniform by construction; saying so keeps chunk addresses in scalar registers
    const uint32_t wib = __builtin_amdgcn_readfirstlane(tid >> 6);
    {   // the dense route's histograms start at zero (nobody reads them before this kernel ends)
        const uint4 z = make_uint4(0, 0, 0, 0);
        for (uint64_t i = uint64_t(blockIdx.x) * kSpillThreads + tid; i < zero_n16;
             i += uint64_t(gridDim.x) * kSpillThreads)
            zero_base[i] = z;
    }
    uint32_t span = (total_chunks + gridDim.x - 1) / gridDim.x;
    span = (span + NW - 1) / NW * NW;
    const uint64_t g0 = uint64_t(blockIdx.x) * span;
    if (g0 >= total_chunks) return;
    const uint64_t g1 = min(g0 + span, uint64_t(total_chunks));
    for (uint32_t i = tid; i < kWinWords; i += kSpillThreads) h[i] = 0;
    if (tid == 0) s_region = 0;
    // last segment whose first chunk is not beyond the span's start.  Up to 64 segments: lane
    // i holds segment i's row and pre-threshold, all requested at once (a search, the row, the
    // pre-threshold would be several dependent loads, which is time the workgroup's first
    // chunk waits for)
    uint4 row_a = make_uint4(0, 0, 0, 0), row_b = row_a;
    uint32_t row_hint = 0;
    if (L <= 64 && lane < L) {
        const uint4 *row = reinterpret_cast<const uint4 *>(segs + lane);
        row_a = row[0];
        row_b = row[1];
        row_hint = from.hint[lane];
    }
    auto segment = [&](uint32_t l) {
        if (L > 64) return segs[l];
        auto get = [&](uint32_t v) { return uint32_t(__builtin_amdgcn_readlane(v, l)); };
        return SegDev{uint64_t(get(row_a.y)) << 32 | get(row_a.x), get(row_a.z), get(row_a.w),
                      get(row_b.x), get(row_b.y), get(row_b.z), get(row_b.w)};
    };
    uint32_t l0 = 0;
    if (L <= 64) {
        const uint64_t first = lane < L ? uint64_t(row_b.w) * kCandChunksPerSuper : ~0ull;
        l0 = uint32_t(__popcll(__ballot(first <= g0))) - 1u;  // segment 0 starts at chunk 0
    } else {
        for (uint32_t hi = L; hi - l0 > 1;) {
            const uint32_t mid = (l0 + hi) >> 1;
            if (uint64_t(segs[mid].sc_start) * kCandChunksPerSuper <= g0) l0 = mid;
            else hi = mid;
        }
    }
    __syncthreads();  // h[] is clear
    uint32_t *st = stage[wib];
    uint32_t *lst_chunk = list[wib][0], *lst_off = list[wib][1], *lst_cnt = list[wib][2];
    uint4 *dw = data[wib];
    const bool staged = CAP <= STAGE;
    uint32_t n_list = 0, fill = 0;  // wave-uniform

    // The staged chunks' slots and counts go out; only this wave touched what it reads.
    // The slots are packed: the chunks of the workgroup's span own the part
    // [g0 * CAP, g1 * CAP) of `cand`, and every flush takes the next free stretch of it, a
    // whole number of 128-byte lines (a line written only in part costs the memory system a
    // read-modify-write; a stretch never needs more than its chunks' CAP slots each, so the
    // part cannot run out).  Where a chunk's slots went is recorded beside its count.  With
    // one fixed array of CAP slots per chunk, of which a quarter is used on average, every
    // pass over the slots moved twice the bytes.
    auto flush = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t n_out = (fill + 31u) & ~31u;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_region, n_out);
        at = __builtin_amdgcn_readfirstlane(at);
        const uint32_t first = uint32_t(g0) * CAP + at;  // (the plan keeps slot numbers in 32 bits)
        uint32_t *slots = cand + first;
        // the padding words are stale staging content, which no reader looks at
        for (uint32_t i = lane; i < n_out; i += 64) {
            slots[i] = st[i];
            if (DTYPE != kBF16) slots[n_slots_total + i] = st[STAGE + i];
        }
        if (lane < n_list)
            chunk_info[lst_chunk[lane]] = make_uint2(lst_cnt[lane], first + lst_off[lane]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        n_list = 0;
        fill = 0;
    };

    for (uint32_t l = l0; l < L; ++l) {
        const SegDev sd = segment(l);
        const uint64_t s0 = uint64_t(sd.sc_start) * kCandChunksPerSuper;
        if (s0 >= g1) break;
        if (sd.k == 0 || sd.n == 0 || !(sd.flags & kSegFast)) continue;
        const uint32_t n_chunks = (sd.n + CHUNK - 1) / CHUNK;
        const uint32_t lo = g0 > s0 ? uint32_t(g0 - s0) : 0u;
        const uint32_t hi = uint32_t(min(uint64_t(n_chunks), g1 - s0));
        if (lo >= hi) continue;
        // No pre-threshold (the sample could not tell, or the last call withdrew it): the
        // segment takes the dense route this time.
        // With an accumulator (error feedback) the segment is streamed all the same: this
        // pass is also the one that turns acc into grad + acc, which the dense route then
        // reads instead of the gradient.  Its candidates are then never used.
        const uint32_t hint = L <= 64 ? uint32_t(__builtin_amdgcn_readlane(row_hint, l)) : from.hint[l];
        const uint32_t blo = hint ? hint : 0x7F7Fu;  // 1 <= blo <= 0x7FFF
        if (hint || ACC) {
            const char *base = grad + sd.offset * EB;
            char *abase = ACC ? acc + sd.offset * EB : nullptr;
            // The wave's own pre-threshold: starts at the segment's and goes up when a chunk
            // holds more candidates than it has slots (see below).
            uint32_t blo_w = blo, swar_add = (0x8000u - blo) * 0x10001u;
            bool overflow = false;
            // the lane's four vectors of chunk `ch`; entries past the segment's end read as 0
            auto load_chunk = [&](const char *base, uint32_t ch, uint32_t (&w)[ROWS][4]) {
                const uint32_t rel0 = ch * CHUNK;
                if (rel0 + CHUNK <= sd.n) {
                    const uint4 *q = reinterpret_cast<const uint4 *>(base + uint64_t(rel0) * EB) + lane;
#pragma unroll
                    for (uint32_t r = 0; r < ROWS; ++r) {
                        const uint4 v = ld_stream(q + 64 * r);  // read once, never again
                        w[r][0] = v.x; w[r][1] = v.y; w[r][2] = v.z; w[r][3] = v.w;
                    }
                } else {
#pragma unroll
                    for (uint32_t r = 0; r < ROWS; ++r) {
                        const uint32_t rel = rel0 + r * ROW_ELEMS + lane * VEC;
                        w[r][0] = w[r][1] = w[r][2] = w[r][3] = 0;
                        if (rel + VEC <= sd.n) {
                            const uint4 v = *reinterpret_cast<const uint4 *>(base + uint64_t(rel) * EB);
                            w[r][0] = v.x; w[r][1] = v.y; w[r][2] = v.z; w[r][3] = v.w;
                        } else if (rel < sd.n) {
#pragma unroll
                            for (uint32_t e = 0; e < VEC; ++e) {
                                if (rel + e >= sd.n) continue;
                                const uint32_t b = load_elem_bits(base, uint64_t(rel) + e, DTYPE);
                                if (DTYPE == kBF16) w[r][e >> 1] |= (b >> 16) << (16 * (e & 1));
                                else w[r][e] = b;
                            }
                        }
                    }
                }
            };
            // The sums of chunk `ch` back to the accumulator (entries inside the segment only),
            // from the chunk's LDS copy: the stores are issued after the next chunk's loads,
            // whose registers the sums no longer occupy, so that waiting for those loads does
            // not mean waiting for the stores' acknowledgements as well.
            auto store_chunk = [&](uint32_t ch) {
                const uint32_t rel0 = ch * CHUNK;
                if (rel0 + CHUNK <= sd.n) {
                    uint4 *q = reinterpret_cast<uint4 *>(abase + uint64_t(rel0) * EB) + lane;
#pragma unroll
                    for (uint32_t r = 0; r < ROWS; ++r) st_stream(q + 64 * r, dw[r * 64 + lane]);
                } else {
#pragma unroll
                    for (uint32_t r = 0; r < ROWS; ++r) {
                        const uint32_t rel = rel0 + r * ROW_ELEMS + lane * VEC;
                        const uint4 v = dw[r * 64 + lane];
                        const uint32_t x[4] = {v.x, v.y, v.z, v.w};
                        if (rel + VEC <= sd.n) {
                            *reinterpret_cast<uint4 *>(abase + uint64_t(rel) * EB) = v;
                        } else if (rel < sd.n) {
#pragma unroll
                            for (uint32_t e = 0; e < VEC; ++e) {
                                if (rel + e >= sd.n) continue;
                                const uint32_t b = DTYPE == kBF16
                                                       ? (x[e >> 1] >> (16 * (e & 1))) & 0xFFFFu
                                                       : x[e];
                                store_elem(abase, uint64_t(rel) + e, b, DTYPE);
                            }
                        }
                    }
                }
            };
            // which of the lane's accumulator entries of chunk `ch` the previous call sent
            // (one byte or half a byte of the 1-bit Index per vector, one word or half a
            // word of the 4-bit one); vectors past the segment's end have none
            auto load_sent = [&](uint32_t ch, uint32_t (&sb)[ROWS]) {
#pragma unroll
                for (uint32_t r = 0; r < ROWS; ++r) {
                    const uint32_t rel = ch * CHUNK + r * ROW_ELEMS + lane * VEC;
                    sb[r] = rel < sd.n ? sent_bits<VEC>(sent, sd.c_off + rel) : 0u;
                }
            };
            uint32_t w[ROWS][4], aw[ROWS][4], sb[ROWS];
            if (lo + wib < hi) {
                load_chunk(base, lo + wib, w);
                if (ACC) {
                    load_chunk(abase, lo + wib, aw);
                    load_sent(lo + wib, sb);
                }
            }
            for (uint32_t ch = lo + wib; ch < hi; ch += NW) {
                if (ACC) {  // error feedback: sparsify grad + acc, and keep the sums
#pragma unroll
                    for (uint32_t r = 0; r < ROWS; ++r)
#pragma unroll
                        for (uint32_t j = 0; j < 4; ++j)
                            w[r][j] = sum_word<DTYPE>(w[r][j], unsent_word<DTYPE>(aw[r][j], sb[r], j));
                }
                // Keep the chunk in LDS (a lane only ever reads back what it wrote itself).
                // Branch-free classification: bit r*VEC + e of `mask` <=> entry e of the
                // lane's vector in row r is a candidate.
                uint32_t mask = 0, c[ROWS];
#pragma unroll
                for (uint32_t r = 0; r < ROWS; ++r) {
                    dw[r * 64 + lane] = make_uint4(w[r][0], w[r][1], w[r][2], w[r][3]);
                    uint32_t f = 0;
                    if (DTYPE == kBF16) {
                        // both halves of a word at once: adding 0x8000 - binlo to a 15-bit
                        // key sets bit 15 exactly when key >= binlo, without carrying over
#pragma unroll
                        for (uint32_t j = 0; j < 4; ++j) {
                            const uint32_t t = ((w[r][j] & 0x7FFF7FFFu) + swar_add) & 0x80008000u;
                            f |= (t >> 15) << (2 * j);  // low half -> bit 2j, high -> bit 2j+16
                        }
                        c[r] = __popc(f);
                        f = (f & 0xFFFFu) | ((f >> 16) << 1);
                    } else {
#pragma unroll
                        for (uint32_t e = 0; e < VEC; ++e)
                            f |= uint32_t(((w[r][e] & 0x7FFFFFFFu) >> 16) >= blo_w) << e;
                        c[r] = __popc(f);
                    }
                    mask |= f << (r * VEC);
                }
                if (ch + NW < hi) {  // in flight during the rest
                    load_chunk(base, ch + NW, w);
                    if (ACC) {
                        load_chunk(abase, ch + NW, aw);
                        load_sent(ch + NW, sb);
                    }
                }
                if (ACC) store_chunk(ch);
                // slot of each lane's first candidate per row: one scan over the four
                // row counts packed in 16-bit fields (a row holds at most 512 candidates)
                uint32_t p01, p23, total;
                auto place = [&]() {
                    const uint32_t ia = wave_incl_scan<uint32_t>(c[0] | (c[1] << 16));
                    const uint32_t ib = wave_incl_scan<uint32_t>(c[2] | (c[3] << 16));
                    const uint32_t ta = __builtin_amdgcn_readlane(ia, 63);
                    const uint32_t tb = __builtin_amdgcn_readlane(ib, 63);
                    const uint32_t t0 = ta & 0xFFFFu, t1 = ta >> 16, t2 = tb & 0xFFFFu,
                                   t3 = tb >> 16;
                    // exclusive positions, again two per register: rows 0,1 and rows 2,3
                    p01 = ia - (c[0] | (c[1] << 16)) + (t0 << 16);
                    p23 = ib - (c[2] | (c[3] << 16)) + (t0 + t1) * 0x10001u + (t2 << 16);
                    total = t0 + t1 + t2 + t3;
                };
                place();
                // More candidates than the chunk has slots: the pre-threshold this call was
                // given is too low (the gradient's scale went up since it was tuned; with
                // error feedback it does every step).  Rather than giving the segment up to
                // the two-read route, the wave raises its own pre-threshold -- for this chunk,
                // classified again from its LDS copy, and for the chunks it takes after it --
                // until the chunk fits.  Nothing has been counted or stored for the chunk yet.
                // The highest pre-threshold any wave used is recorded: the histogram is only
                // complete from there upwards, which is where the selection then looks.
                while (total > CAP && blo_w < 0x7F7Fu) {
                    blo_w = min(blo_w + kSpillRaise, 0x7F7Fu);
                    swar_add = (0x8000u - blo_w) * 0x10001u;
                    mask = 0;
#pragma unroll
                    for (uint32_t r = 0; r < ROWS; ++r) {
                        const uint4 v = dw[r * 64 + lane];
                        const uint32_t x[4] = {v.x, v.y, v.z, v.w};
                        uint32_t f = 0;
                        if (DTYPE == kBF16) {
#pragma unroll
                            for (uint32_t j = 0; j < 4; ++j) {
                                const uint32_t t = ((x[j] & 0x7FFF7FFFu) + swar_add) & 0x80008000u;
                                f |= (t >> 15) << (2 * j);
                            }
                            c[r] = __popc(f);
                            f = (f & 0xFFFFu) | ((f >> 16) << 1);
                        } else {
#pragma unroll
                            for (uint32_t e = 0; e < VEC; ++e)
                                f |= uint32_t(((x[e] & 0x7FFFFFFFu) >> 16) >= blo_w) << e;
                            c[r] = __popc(f);
                        }
                        mask |= f << (r * VEC);
                    }
                    place();
                }
                const uint32_t chunk_id = uint32_t(s0) + ch;
                // (a chunk's slots start on a 16-byte boundary: they are read in such groups)
                const uint32_t need = min((total + 3u) & ~3u, CAP);
                if (staged && (n_list == LIST || fill + need > STAGE)) flush();
                uint32_t *slots = cand + uint64_t(chunk_id) * CAP;
                uint32_t *slots_pos = slots + n_slots_total;  // fp32 only
                uint32_t *stc = st + fill;
                // Candidates are rare: every lane walks its own few set bits, so the wave
                // issues as many histogram / store instructions as its busiest lane needs.
                for (uint32_t mm = mask; mm;) {
                    const uint32_t e = __builtin_ctz(mm);
                    mm &= mm - 1;
                    const uint32_t r = e / VEC;
                    const uint32_t row_bits = ((1u << VEC) - 1u) << (r * VEC);
                    const uint32_t before = __popc(mask & row_bits & ((1u << e) - 1u));
                    const uint32_t ps = (((r & 2u) ? p23 : p01) >> (16 * (r & 1u)) & 0xFFFFu) + before;
                    const uint32_t rel = r * ROW_ELEMS + lane * VEC + (e % VEC);
                    uint32_t bits;
                    if (DTYPE == kBF16)
                        bits = uint32_t(reinterpret_cast<const uint16_t *>(dw)[rel]) << 16;
                    else
                        bits = reinterpret_cast<const uint32_t *>(dw)[rel];
                    const uint32_t bin = (bits & 0x7FFFFFFFu) >> 16;
                    atomicAdd(&h[min(bin - blo, kWinBins)], 1u);      // in the window, or above it
                    if (bin >= 0x7F80u) atomicAdd(&h[kWinBins + 1], 1u);  // all-ones exponent
                    if (ps < CAP) {
                        if (DTYPE == kBF16) {
                            if (staged) stc[ps] = bits | rel;
                            else slots[ps] = bits | rel;
                        } else {
                            if (staged) {
                                stc[ps] = bits;
                                stc[STAGE + ps] = rel;
                            } else {
                                slots[ps] = bits;
                                slots_pos[ps] = rel;
                            }
                        }
                    }
                }
                if (staged) {
                    if (lane == 0) {
                        lst_chunk[n_list] = chunk_id;
                        lst_off[n_list] = fill;
                        lst_cnt[n_list] = total;
                    }
                    ++n_list;
                    fill += need;
                } else if (lane == 0) {
                    chunk_info[chunk_id] = make_uint2(total, chunk_id * CAP);
                }
                overflow |= total > CAP;
            }
            if (staged && n_list) flush();
            if (blo_w > blo && lane == 0) atomicMax(&ts.raised[l], blo_w);
            if (overflow && lane == 0)  // a chunk denser than its slots: take the dense route
                atomicOr(&ts.reroute[l], 1u);
        }
        __syncthreads();
        uint32_t *win = ts.win + size_t(l) * kWinWords;
        for (uint32_t i = tid; i < kWinWords; i += kSpillThreads) {
            const uint32_t c = h[i];
            if (c) {
                atomicAdd(&win[i], c);
                h[i] = 0;
            }
        }
        // The table updates are device-scope atomics, performed where every CU sees them; a
        // thread only has to wait until its own have been acknowledged before the workgroup
        // counts as arrived.  The workgroup that arrives last drops what it may hold of the
        // table in its caches and selects.
        wait_own_memory_ops();
        __syncthreads();
        if (tid == 0) {
            const uint64_t c_last = s0 + n_chunks - 1;  // segment's chunks: one workgroup per span
            const uint32_t expected = uint32_t(c_last / span) - uint32_t(s0 / span) + 1u;
            s_last = atomicAdd(&ts.arrive[l], 1u) == expected - 1u;
        }
        __syncthreads();
        if (s_last) {  // uniform
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            select_window<DTYPE>(l, sd, hint, ts, from, sel, s_sel);
        }
        __syncthreads();
    }
}

// Whether segment l is on the dense route: by plan (not eligible for the candidate route), or
// because the scan's selection sent it there (no pre-threshold, too few candidates, a chunk
// denser than its slots).  sel[l] of a candidate-route segment has been written by the scan.
__device__ inline bool on_dense_route(const SegDev &sd, const SelDev *sel, uint32_t l)
{
    // (looked up whatever the row says, so that row and route are on their way together; a segment
    // that keeps nothing has no selection, and what lies in its place does not count)
    const uint32_t route = sel[l].route;
    return bool(uint32_t(sd.k != 0) & uint32_t(sd.n != 0) &
                (uint32_t(!(sd.flags & kSegFast)) | uint32_t(route != 0)));
}

// true iff some segment is on the dense route: lane i looks at segments i, i + 64, ...
__device__ inline bool any_dense_route(const SegDev *segs, const SelDev *sel, uint32_t L)
{
    bool any = false;
    for (uint32_t l = threadIdx.x & 63; l < L; l += 64) any |= on_dense_route(segs[l], sel, l);
    return __ballot(any) != 0;
}

// ------------------------------------------------------------------ hist1

// The dense route reads any 16-byte vector of a segment, aligned or not (memory instructions
// take any alignment; a wave's kilobyte then touches one cache line more).
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
__device__ inline uint4 ld_stream_any(const char *p)
{
    const u32x4_any v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// entries rel .. rel + VEC - 1 of a segment of n entries, those past its end as 0
template <int DTYPE>
__device__ inline uint4 load_vec(const char *base, uint32_t rel, uint32_t n)
{
    constexpr uint32_t EB = DTYPE == kBF16 ? 2 : 4;
    constexpr uint32_t VEC = 16 / EB;
    if (rel + VEC <= n) return ld_stream_any(base + uint64_t(rel) * EB);
    uint32_t w[4] = {0, 0, 0, 0};
    if (rel < n) {
#pragma unroll
        for (uint32_t e = 0; e < VEC; ++e) {
            if (rel + e >= n) continue;
            const uint32_t b = load_elem_bits(base, uint64_t(rel) + e, DTYPE);
            if (DTYPE == kBF16) w[e >> 1] |= (b >> 16) << (16 * (e & 1));
            else w[e] = b;
        }
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// fn(level-1 bin of the key, key) for the VEC entries of a vector, exact zeros left out
template <int DTYPE, typename Fn>
__device__ inline void for_keys(uint4 v, Fn &&fn)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    constexpr uint32_t VEC = DTYPE == kBF16 ? 8 : 4;
#pragma unroll
    for (uint32_t e = 0; e < VEC; ++e) {
        const uint32_t key = vec_elem_bits<DTYPE>(w, e) & 0x7FFFFFFFu;
        if (key) fn(key >> 16, key);
    }
}

// What a dense-route segment's level-1 histogram says: writes the selection (fp32: its upper
// half) and, for a segment that was re-routed, the pre-threshold for the next call, the bin
// above which about 1.3 k entries lie (what the slots per chunk are sized for).  One thread `leaves` what it finds in
// the table.
template <int DTYPE>
__device__ inline SelDev dense_selection(uint32_t l, const SegDev &sd, const BinFound &k_th,
                                         const BinFound &want, uint32_t total, uint32_t nonfinite,
                                         const TableState ts, bool leaves = true)
{
    if (leaves && (sd.flags & kSegFast)) {
        // fewer non-zeros than 1.3 k in the whole segment: everything is a candidate
        const uint32_t b2 = want.bin != kNoBin ? max(want.bin, 1u) : 1u;
        // after a miss (the scale fell below what the carried pre-threshold admits) the next
        // calls extrapolate the fall instead of trusting the last value
        ts.hint[l] = next_hint(b2, ts.prev[l], ts.watch[l]);
        ts.prev[l] = b2;
    }
    if (leaves && nonfinite) atomicAdd(&ts.glob[1], nonfinite);
    if (leaves) atomicAdd(&ts.glob[2], 1u);
    SelDev r{};
    r.route = 1;
    if (k_th.bin == kNoBin) {  // fewer non-zeros than k: keep every non-zero
        r.T = 0;
        r.quota = 0;
        r.G = total;
        r.cnt = total;
    } else if (DTYPE == kBF16) {
        r.T = k_th.bin << 16;
        r.G = k_th.above;
        r.quota = sd.k - k_th.above;
        r.cnt = sd.k;
    } else {
        r.bin1 = k_th.bin;
        r.G1 = k_th.above;
        r.need2 = 1;
    }
    return r;
}
__device__ inline uint32_t carried_count(const SegDev &sd)
{
    return (sd.flags & kSegFast) ? uint32_t(1.3f * float(sd.k)) + 1u : 0u;
}

// A segment that one workgroup can hold in its registers: all of it is read once, histogrammed
// in LDS (two 16-bit counts per word: a segment has fewer than 65536 entries), and, in fp32,
// the low 16 key bits of the threshold bin found by two rounds of 256 bins over the same
// registers.  Nothing of it goes through global memory and nobody waits for anybody: with a
// histogram in memory such a segment cost the device a pass of clearing, 256 workgroups'
// flushes and an arrival count (five segments of 400 to 11,000 fp32 entries, three ranks: 75 us
// over two launches; 15 in one in this form, a third of it the time a launch takes).
template <int DTYPE>
__device__ __forceinline__ void load_small(uint4 (&v)[kSmallVecs], const SegDev &sd, const char *base)
{
    constexpr uint32_t VEC = DTYPE == kBF16 ? 8 : 4;
#pragma unroll
    for (uint32_t i = 0; i < kSmallVecs; ++i)
        v[i] = load_vec<DTYPE>(base, (i * kSmallThreads + threadIdx.x) * VEC, sd.n);
}
// `counted` gets the segment's non-zeros as soon as they are known.
template <int DTYPE, typename Counted>
__device__ __forceinline__ SelDev select_small(uint32_t l, const SegDev &sd, const uint4 (&v)[kSmallVecs],
                                               const TableState ts, uint32_t *h16, uint32_t *smem, bool leaves,
                                               Counted &&counted)
{
    constexpr uint32_t NT = kSmallThreads;
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < kBins1 / 8; i += NT)
        reinterpret_cast<uint4 *>(h16)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kSmallVecs; ++i)
        for_keys<DTYPE>(v[i], [&](uint32_t bin, uint32_t) {
            atomicAdd(&h16[bin >> 1], 1u << (16 * (bin & 1u)));
        });
    __syncthreads();
    // a thread's bins are BPT / 2 consecutive words, read from a different one on in every
    // lane (or all lanes would meet in the same LDS banks)
    constexpr uint32_t BPT = kBins1 / NT, WPT = BPT / 2;
    uint32_t two = 0;
#pragma unroll
    for (uint32_t i = 0; i < WPT; ++i) two += h16[tid * WPT + ((i + tid) % WPT)];
    const uint32_t own = (two & 0xFFFFu) + (two >> 16);  // (a segment's total fits 16 bits)
    if (tid == 0) smem[32] = 0;
    __syncthreads();
    if (tid * BPT >= 0x7F80u && own) atomicAdd(&smem[32], own);  // all-ones exponents
    uint32_t total;
    BinFound f[2];
    auto get = [&](uint32_t b) { return (h16[b >> 1] >> (16 * (b & 1u))) & 0xFFFFu; };
    select_top<NT, BPT>(get, own, {sd.k, carried_count(sd)}, f, &total, smem);
    counted(total);
    SelDev r = dense_selection<DTYPE>(l, sd, f[0], f[1], total, smem[32], ts, leaves && tid == 0);
    if (DTYPE == kBF16 || f[0].bin == kNoBin) return r;  // uniform
    uint32_t above = f[0].above, prefix = f[0].bin;  // key >> shift of the bin looked into
    const uint32_t in_bin = get(prefix);
    __syncthreads();  // everybody has read h16
    if (in_bin <= 64) {
        // fp32, and no more entries in the threshold's bin than a wave has lanes, as nearly always: every wave
        // compares them all with each other (the two rounds below are sixteen barriers: small_kernel of 11
        // thousand entries 16.1 us, 13.5 this way)
        const uint32_t lane = tid & 63, want = sd.k - above;
        if (tid == 0) smem[33] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < kSmallVecs; ++i)
            for_keys<DTYPE>(v[i], [&](uint32_t bin, uint32_t key) {
                if (bin == prefix) h16[add_by_lane(&smem[33], 1u)] = key;
            });
        __syncthreads();
        const uint32_t mine = lane < in_bin ? h16[lane] : 0u;
        uint32_t gt = 0, ge = 0;
        for (uint32_t i = 0; i < in_bin; ++i) {
            const uint32_t x = __builtin_amdgcn_readlane(mine, i);
            gt += x > mine;
            ge += x >= mine;
        }
        const uint32_t who = uint32_t(__builtin_ctzll(__ballot(lane < in_bin && gt < want && ge >= want)));
        prefix = __builtin_amdgcn_readlane(mine, who);
        above += __builtin_amdgcn_readlane(gt, who);
    } else {
        // eight key bits a round
#pragma unroll
        for (uint32_t round = 0; round < 2; ++round) {
            const uint32_t shift = 16 - 8 * round;
            if (tid < 256) h16[tid] = 0;
            __syncthreads();
#pragma unroll
            for (uint32_t i = 0; i < kSmallVecs; ++i)
                for_keys<DTYPE>(v[i], [&](uint32_t, uint32_t key) {
                    if ((key >> shift) == prefix) atomicAdd(&h16[(key >> (shift - 8)) & 0xFFu], 1u);
                });
            __syncthreads();
            uint32_t tot2;
            BinFound g[2];
            select_top<NT, 1>([&](uint32_t b) { return h16[b]; }, tid < 256 ? h16[tid] : 0u,
                              {sd.k - above, 0u}, g, &tot2, smem);
            above += g[0].above;
            prefix = (prefix << 8) | g[0].bin;
        }
    }
    r.T = prefix;
    r.G = above;
    r.quota = sd.k - above;
    r.cnt = sd.k;
    r.need2 = 0;
    return r;
}

// Dense route: thresholds of the segments the scan does not select for, by plan or because its
// selection re-routed them.  The last `n_span` workgroups of a rank share the entries of its
// longer segments out in contiguous spans of tiles, each adding what it counted in LDS to the
// segment's histogram in the workspace; whoever completes that histogram selects right away.
// The first workgroups (SMALL: the plan has such segments) take a short segment each.
//
// The LDS histogram is a window of 4096 bins, 32 octaves of magnitude, that every workgroup puts
// where its own first vectors lie; what falls outside goes to the histogram in memory directly.
// With all 32768 bins in LDS (128 KiB) a compute unit held one workgroup, which cleared and
// searched that much for every segment: 95 us for four ranks of 9 M bf16 entries in five
// segments, against 47 in this form (of which reading them takes 12: the rest is LDS adds, one
// per entry).
//
// A plan without such segments launches the kernel only as the safety net of re-routed ones,
// where it leaves at once: small workgroups find room on a busy device, a launch of
// 1024-thread ones cost 7 us with other buckets in flight.
template <int DTYPE, bool SMALL>
__global__ void __launch_bounds__(SMALL ? kSmallThreads : kDenseThreads)
hist1_kernel(const SparsifyBatch, uint32_t *table, const WsLayout wl, uint32_t n_span)
{
    constexpr uint32_t EB = DTYPE == kBF16 ? 2 : 4;
    constexpr uint32_t VEC = 16 / EB;
    constexpr uint32_t NT = SMALL ? kSmallThreads : kDenseThreads;
    constexpr uint32_t BPT = kBins1 / NT;
    constexpr uint32_t TILE = NT * VEC * kDenseRows;
    static_assert(0x7F80u % BPT == 0, "a thread's bins are all finite or none is");
    __shared__ uint32_t h[SMALL ? kBins1 / 2 : kHistWindow];
    __shared__ uint32_t smem[40];
    __shared__ uint32_t s_last, s_top;
    const RankView rv = rank_view();
    const char *grad = rv.src();
    SelDev *sel = rv.at<SelDev>(wl.sel);
    const uint32_t L = wl.L;
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    const TableState ts = table_state(table, L, rv.slot);
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t n_small = gridDim.x - n_span;
    if (blockIdx.x == 0) {  // the tile groups' counts are added to by the next kernel
        uint64_t *gc = rv.at<uint64_t>(wl.group_cnt);
        for (uint32_t i = tid; i <= wl.total_tiles / kTileGroup; i += NT) gc[i] = 0;
    }
    if (SMALL && blockIdx.x < n_small) {
        const uint32_t l = blockIdx.x;
        const SegDev sd = segs[l];
        if (sd.k != 0 && (sd.flags & kSegSmall)) {
            uint4 v[kSmallVecs];
            load_small<DTYPE>(v, sd, grad + sd.offset * EB);
            const SelDev r = select_small<DTYPE>(l, sd, v, ts, h, smem, true, [](uint32_t) {});
            if (tid == 0) sel[l] = r;
        }
        return;
    }
    // tiles of the segment of row l that go through here
    auto tiles_of = [&](uint32_t l) -> uint32_t {
        if (l >= L) return 0u;
        const SegDev sd = segs[l];
        if ((sd.flags & kSegSmall) || !on_dense_route(sd, sel, l)) return 0u;
        return (sd.n + TILE - 1) / TILE;
    };
    uint32_t all = 0;  // (every wave adds them up for itself; all entries are < 2^32, a tile holds 4096 or more)
    for (uint32_t l = lane; l < (L + 63) / 64 * 64; l += 64) all += tiles_of(l);
    all = wave_sum(all);
    if (all == 0) return;
    const uint32_t span = (all + n_span - 1) / n_span;
    const uint32_t g0 = (blockIdx.x - n_small) * span, g1 = min(g0 + span, all);
    if (g0 >= all) return;
    bool clear = false;
    uint32_t first = 0;  // tiles of the segments before
    for (uint32_t l0 = 0; l0 < L && first < g1; l0 += 64) {
        const uint32_t mine = tiles_of(l0 + lane), inc = wave_incl_scan<uint32_t>(mine);
        // segments of this block of 64 rows whose tiles meet the workgroup's
        uint64_t meet = __ballot(mine && first + inc > g0 && first + inc - mine < g1);
        for (; meet; meet &= meet - 1) {
            const uint32_t j = uint32_t(__builtin_ctzll(meet)), l = l0 + j;
            const uint32_t nt = __builtin_amdgcn_readlane(mine, j);
            const uint32_t s0 = first + __builtin_amdgcn_readlane(inc, j) - nt;
            const SegDev sd = segs[l];
            const char *base = grad + sd.offset * EB;
            uint32_t *gh = rv.at<uint32_t>(wl.hist1d) + uint64_t(l) * kBins1;
            const uint32_t t0 = max(g0, s0) - s0, t1 = min(g1, s0 + nt) - s0;
            auto load_tile = [&](uint32_t t, uint4 (&v)[kDenseRows]) {
#pragma unroll
                for (uint32_t r = 0; r < kDenseRows; ++r)
                    v[r] = load_vec<DTYPE>(base, t * TILE + (r * NT + tid) * VEC, sd.n);
            };
            uint4 v[kDenseRows];
            load_tile(t0, v);
            if (!clear)
                for (uint32_t i = tid; i < kHistWindow; i += NT) h[i] = 0;
            clear = true;
            // The window: from 8 octaves above the smallest of the waves' largest finite keys
            // (an odd outlier moves one wave's) 32 octaves down.
            if (tid == 0) s_top = 0x7F7Fu;
            uint32_t top = 0;
#pragma unroll
            for (uint32_t r = 0; r < kDenseRows; ++r)
                for_keys<DTYPE>(v[r], [&](uint32_t bin, uint32_t) {
                    if (bin < 0x7F80u) top = max(top, bin);
                });
#pragma unroll
            for (uint32_t d = 32; d >= 1; d >>= 1) top = max(top, uint32_t(__shfl_xor(top, d, 64)));
            __syncthreads();
            if (lane == 0 && top) atomicMin(&s_top, top);
            __syncthreads();
            const uint32_t end = min(s_top + 1024u, kBins1);
            const uint32_t wbase = end > kHistWindow ? end - kHistWindow : 0u;
            for (uint32_t t = t0; t < t1; ++t) {
                uint4 cur[kDenseRows];
#pragma unroll
                for (uint32_t r = 0; r < kDenseRows; ++r) cur[r] = v[r];
                if (t + 1 < t1) load_tile(t + 1, v);  // on its way while this one is counted
#pragma unroll
                for (uint32_t r = 0; r < kDenseRows; ++r)
                    for_keys<DTYPE>(cur[r], [&](uint32_t bin, uint32_t) {
                        const uint32_t w = bin - wbase;
                        if (w < kHistWindow) atomicAdd(&h[w], 1u);
                        else atomicAdd(&gh[bin], 1u);
                    });
            }
            __syncthreads();
            for (uint32_t i = tid; i < kHistWindow; i += NT) {
                const uint32_t c = h[i];
                if (c) {
                    atomicAdd(&gh[wbase + i], c);
                    h[i] = 0;
                }
            }
            // The histogram updates are device-scope atomics, performed where every CU sees
            // them; a thread only has to wait until its own have been acknowledged before the
            // workgroup is counted as arrived.  The workgroup that arrives last drops what it
            // may hold of the histogram in its caches and selects.
            wait_own_memory_ops();
            __syncthreads();
            if (tid == 0) {
                const uint32_t expected = (s0 + nt - 1) / span - s0 / span + 1u;
                s_last = atomicAdd(&ts.arrive_d[l], 1u) == expected - 1u;
            }
            __syncthreads();
            if (!s_last) continue;  // uniform
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            const uint32_t own = own_bins<BPT>(gh);
            if (tid == 0) {
                ts.arrive_d[l] = 0;  // for the next call
                smem[32] = 0;
            }
            __syncthreads();
            if (tid * BPT >= 0x7F80u && own) atomicAdd(&smem[32], own);  // all-ones exponents
            uint32_t total;
            BinFound f[2];
            select_top<NT, BPT>([&](uint32_t b) { return gh[b]; }, own, {sd.k, carried_count(sd)},
                                f, &total, smem);
            if (tid == 0) sel[l] = dense_selection<DTYPE>(l, sd, f[0], f[1], total, smem[32], ts);
        }
        first += __builtin_amdgcn_readlane(inc, 63);
    }
}

// ------------------------------------------------------------------ small

// Few short segments (tagc_plan says which) take one launch from the gradient to pairs, Index and counts: a
// workgroup that has found its segment's threshold has all its entries at hand.  What it cannot know is how many
// pairs the segments before it emit: as many as they are to keep, unless one has fewer non-zeros than that.  So
// every workgroup tells, with its histogram's total, before it has its threshold; and whoever finds a segment's
// word missing behind its own all the same, because that workgroup has had no compute unit yet, counts the
// segment itself.  Nobody waits for anybody: workgroups that did could wait for good, for some that they keep
// out, where launches of several streams fill the device.  (Every workgroup counting all before its own, a wave a
// segment: 64 of 32 thousand entries nearly all zeros, eight ranks, 416 us; this 69, the three launches 66.)
// us: hist1, count and place of five segments of 72 to 11 thousand fp32 entries, three ranks, 23.5; this 13.1.

// The segment's pairs, from the position of the rank's list on that one wave's `look` leaves in `base`; and its
// Index words.
template <int DTYPE, typename Look>
__device__ __forceinline__ void emit_small(const SegDev &sd, uint4 (&v)[kSmallVecs], const SelDev &se,
                                           const uint32_t *base, uint32_t *idx, float *val, uint32_t *bitmap,
                                           uint32_t *s_rows /* [kSmallVecs * NT / 64] */, Look &&look)
{
    constexpr uint32_t VEC = DTYPE == kBF16 ? 8 : 4, NT = kSmallThreads, NWV = NT / 64, LPW = 32 / VEC;
    static_assert(kSmallVecs * NWV == 128, "two counts a lane");
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // which entries of a vector are above the threshold, and << 16 which are at it; how many (a segment has fewer
    // than 65536)
    uint32_t marks[kSmallVecs], inc[kSmallVecs];
    auto own = [&](uint32_t i) { return uint32_t(__popc(marks[i] & 0xFFFFu)) | (uint32_t(__popc(marks[i] >> 16)) << 16); };
#pragma unroll
    for (uint32_t i = 0; i < kSmallVecs; ++i) {
        const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
        uint32_t gt = 0, eq = 0;
#pragma unroll
        for (uint32_t e = 0; e < VEC; ++e) {
            const uint32_t key = vec_elem_bits<DTYPE>(w, e) & 0x7FFFFFFFu;
            gt |= uint32_t(key > se.T) << e;
            eq |= uint32_t(key == se.T) << e;
        }
        marks[i] = gt | (se.quota ? eq << 16 : 0u);
        inc[i] = wave_incl_scan<uint32_t>(own(i));
        if (lane == 63) s_rows[i * NWV + wave] = inc[i];
    }
    __syncthreads();
    if (wave == 0) {  // what lies before each wave's vectors of a row
        const uint32_t a = s_rows[2 * lane], b = s_rows[2 * lane + 1];
        const uint32_t before = wave_incl_scan<uint32_t>(a + b) - a - b;
        s_rows[2 * lane] = before;
        s_rows[2 * lane + 1] = before + a;
    }
    if (wave == 1) look();
    __syncthreads();
    const uint32_t from = *base;
#pragma unroll
    for (uint32_t i = 0; i < kSmallVecs; ++i) {
        if (i * NT * VEC >= sd.n) break;  // uniform
        const uint32_t at = s_rows[i * NWV + wave] + inc[i] - own(i), rel = (i * NT + tid) * VEC;
        uint32_t gb = at & 0xFFFFu, eb = at >> 16;
        const uint32_t gt = marks[i] & 0xFFFFu, eq = marks[i] >> 16;
        // (unpacked anew: the entries, kept since the marks were made, take registers that are not there)
        asm volatile("" : "+v"(v[i].x), "+v"(v[i].y), "+v"(v[i].z), "+v"(v[i].w));
        const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
        uint32_t kept = gt;
        for (uint32_t m = gt | eq; m; m &= m - 1) {
            const uint32_t e = uint32_t(__builtin_ctz(m));
            const bool above = (gt >> e) & 1u;
            if (above || eb < se.quota) {
                const uint32_t pos = from + gb + min(eb, se.quota);
                // (a register cannot be named by a number that is not known)
                uint32_t bits = 0;
#pragma unroll
                for (uint32_t x = 0; x < VEC; ++x) bits = e == x ? vec_elem_bits<DTYPE>(w, x) : bits;
                idx[pos] = sd.c_off + rel + e;
                val[pos] = __uint_as_float(bits);
                kept |= 1u << e;
            }
            gb += above;
            eb += !above;
        }
        uint32_t x = kept << (VEC * (tid & (LPW - 1)));
#pragma unroll
        for (uint32_t d = 1; d < LPW; d <<= 1) x |= __shfl_xor(x, d, 64);
        const uint32_t rel0 = rel - (tid & (LPW - 1)) * VEC;  // first entry of the word
        if ((tid & (LPW - 1)) == 0 && rel0 < sd.n) bitmap[(sd.c_off + rel0) >> 5] = x;
    }
}

// By a wave: the pairs a segment emits, its non-zeros or what it is to keep, if its `word` does not say so meanwhile.
// (Rarely needed: short, and not wide.)
template <int DTYPE>
__device__ inline uint32_t emitted_small(const SegDev &sd, const char *base, const uint32_t *word)
{
    constexpr uint32_t VEC = DTYPE == kBF16 ? 8 : 4;
    uint32_t n = 0;
    for (uint32_t at = 0; at < sd.n && n < sd.k; at += 64 * VEC) {
        const uint32_t told =
            __builtin_amdgcn_readfirstlane(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        uint32_t own = 0;
        for_keys<DTYPE>(load_vec<DTYPE>(base, at + lane_id() * VEC, sd.n), [&](uint32_t, uint32_t) { ++own; });
        if (int32_t(told) > 0) return told - 1;
        n += __builtin_amdgcn_readlane(wave_incl_scan<uint32_t>(own), 63);
    }
    return min(n, sd.k);
}

constexpr uint32_t kSmallTries = 4;  // looks at the others' words, after the first, before one is done without

template <int DTYPE>
__global__ void __launch_bounds__(kSmallThreads)
small_kernel(const SparsifyBatch, uint32_t *table, const WsLayout wl)
{
    constexpr uint32_t EB = DTYPE == kBF16 ? 2 : 4;
    __shared__ uint32_t h[kBins1 / 2];
    __shared__ uint32_t smem[40];
    __shared__ uint32_t s_base;  // pairs of the segments before
    static_assert(kSmallSegments <= 64, "a lane a segment");
    const RankView rv = rank_view();
    const char *grad = rv.src();
    const uint32_t L = wl.L, l = blockIdx.x, tid = threadIdx.x, lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    const TableState ts = table_state(table, L, rv.slot);
    const SegDev sd = segs[l];
    uint4 v[kSmallVecs];
    load_small<DTYPE>(v, sd, grad + sd.offset * EB);
    uint32_t dense = 0;  // segments that keep something (lane i has looked at segment i: they are 64 at most)
    if (l == L - 1) {
        const SegDev row = segs[min(lane, L - 1)];
        dense = uint32_t(__popcll(__ballot(lane < L && row.k && row.n)));
    }
    const bool keeps = sd.k != 0 && sd.n != 0;
    SelDev r{};  // (no entry is above the largest key)
    r.T = 0xFFFFFFFFu;
    // how many pairs the segment emits, for those behind it (the word is zero between the launches)
    auto tell = [&](uint32_t nonzeros) {
        if (tid == 64 && l != L - 1) atomicAdd(&ts.arrive_d[l], min(nonzeros, sd.k) + 1u);
    };
    if (keeps) r = select_small<DTYPE>(l, sd, v, ts, h, smem, false, tell);
    else tell(0);
    __syncthreads();  // h
    // The entries that are not finite are counted by the last one to say that it has found its segment's, which
    // only has to look if somebody had some; the others' counts are the plan's.
    constexpr uint32_t kSome = 1u << 16;
    static_assert(kSmallSegments < kSome, "arrivals");
    uint32_t came = 0, nonfinite = 0;
    uint32_t word = 1, most = 0;
    if (wave == 1 && lane < l) {
        word = __hip_atomic_load(&ts.arrive_d[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        most = segs[lane].k;
    }
    auto look = [&] {
        for (uint32_t tries = 0;; ++tries) {
            const uint64_t untold = __ballot(int32_t(word) <= 0);
            if (!untold) break;
            if (tries < kSmallTries) {
                if (int32_t(word) <= 0)
                    word = __hip_atomic_load(&ts.arrive_d[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                continue;
            }
            const uint32_t i = uint32_t(__builtin_ctzll(untold));
            const SegDev before = segs[i];
            const uint32_t n = emitted_small<DTYPE>(before, grad + before.offset * EB, ts.arrive_d + i);
            if (lane == i) word = n + 1;
        }
        // (nothing lands outside the list, whatever the words hold)
        const uint32_t pairs = __builtin_amdgcn_readlane(wave_incl_scan<uint32_t>(min(word - 1u, most)), 63);
        if (lane == 0) {
            s_base = pairs;
            nonfinite = keeps ? smem[32] : 0u;
            if (nonfinite) atomicAdd(&ts.glob[1], nonfinite);
            wait_own_memory_ops();  // (what the last one looks at, and the word that it clears)
            came = atomicAdd(&ts.arrive[0], nonfinite ? 1u + kSome : 1u);
        }
    };
    emit_small<DTYPE>(sd, v, r, &s_base, rv.idx, rv.val, rv.bitmap, h, look);
    if (tid == 0) {
        rv.cnt[TAGC_CNT_SEG0 + l] = r.cnt;
        if (l == L - 1) {
            rv.cnt[TAGC_CNT_TOTAL] = s_base + r.cnt;
            rv.cnt[TAGC_CNT_FLAGS] = 0;
            rv.cnt[TAGC_CNT_DENSE] = dense;
            rv.cnt[TAGC_CNT_RESERVED] = 0;
        }
    }
    if (wave == 1 && (__builtin_amdgcn_readfirstlane(came) & (kSome - 1)) == L - 1) {  // everybody has told and looked
        if (lane < L) ts.arrive_d[lane] = 0;
        if (lane == 0) {
            uint32_t all = 0;
            if (came >= kSome || nonfinite) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                all = ts.glob[1];
                ts.glob[1] = 0;
            }
            rv.cnt[TAGC_CNT_NONFINITE] = all;
            ts.arrive[0] = 0;
        }
    }
}

// last l with start(l) <= t, start() read through `field` (tile_start or sc_start)
template <typename F>
__device__ inline uint32_t segment_of(uint32_t L, uint32_t t, F start)
{
    uint32_t lo = 0, hi = L;
    while (hi - lo > 1) {
        uint32_t mid = (lo + hi) >> 1;
        if (start(mid) <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// fp32: the low 16 key bits of the thresholds, for the segments whose level-1 bin is known.  The
// keys of that bin are counted twice, by all 16 bits (memory) and by the upper 8 of them (LDS, then
// the segment's candidate histogram in the table, which is idle from its selection on: key by
// key, its few cache lines would be the bottleneck); the workgroup
// that is done with a segment last looks at 256 counts of each.  Candidate route: the keys come
// from the spilled slots; the super-chunks of all segments form one list, a workgroup takes one
// contiguous span of it and a wave a super-chunk at a time, whose chunks' slots are requested
// kRefineBatch at a time (one chunk after the other, each a chain of two loads, this took 16 us on
// 8 ranks of 7 M entries, and the two launches that followed 5 and 10; all of it now 14).  That list
// is the first n_cand workgroups' work.
// Dense route: from the gradient, by the first n_dense workgroups, kRefineRows vectors per thread at
// a time.  Four workgroups per compute unit at most: each ends in up to 256 atomics on the same few
// lines and an arrival.  (With as many workgroups as the candidate list asked for, and a vector at a
// time, 2 ranks of 1 M entries took 82 us, 11 now; 4 ranks of 9 M 105, 44 now, with eight per
// compute unit 61; one rank of 60 M 104, 63 now.)
constexpr uint32_t kRefineBatch = 16;
constexpr uint32_t kRefineRows = 4;

// By a wave, of 256 counts: the largest b with sum_{x >= b} bins[x] >= want and the entries in
// higher ones; kNoBin if all together hold fewer.
__device__ inline uint32_t top_of_256(const uint32_t *bins, uint32_t want, uint32_t *above)
{
    const uint32_t lane = lane_id();
    const uint4 v = reinterpret_cast<const uint4 *>(bins)[lane];
    const uint32_t c[4] = {v.x, v.y, v.z, v.w};
    const uint32_t own = c[0] + c[1] + c[2] + c[3];
    const uint32_t inc = wave_incl_scan<uint32_t>(own);
    const uint32_t total = __builtin_amdgcn_readlane(inc, 63);
    uint32_t acc = total - inc, bin = kNoBin, at = total;  // acc: in the lanes above
#pragma unroll
    for (int i = 3; i >= 0; --i) {
        if (acc < want && acc + c[i] >= want) {
            bin = 4 * lane + uint32_t(i);
            at = acc;
        }
        acc += c[i];
    }
    const uint64_t who = __ballot(bin != kNoBin);
    const uint32_t l = who ? uint32_t(__builtin_ctzll(who)) : 0u;
    *above = __builtin_amdgcn_readlane(at, l);
    return __builtin_amdgcn_readlane(bin, l);
}

__global__ void __launch_bounds__(256)
refine_kernel(const SparsifyBatch, uint32_t *table, const WsLayout wl, uint32_t CAP, uint32_t n_cand,
              uint32_t n_dense)
{
    constexpr uint32_t CHUNK = 64 * 4 * kCandRows, NCH = kCandChunksPerSuper, NWV = 4;
    __shared__ uint32_t s_last, s_coarse[256];
    const RankView rv = rank_view();
    SelDev *sel = rv.at<SelDev>(wl.sel);
    const uint32_t *cand = rv.at<uint32_t>(wl.cand);
    const uint2 *chunk_info = rv.at<uint2>(wl.chunk_info);
    const uint32_t n_slots_total = uint32_t(wl.n_slots);
    const uint32_t L = wl.L, total_sc = wl.total_sc;
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    const TableState ts = table_state(table, L, rv.slot);
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    s_coarse[tid] = 0;
    __syncthreads();

    auto add_key = [&](uint32_t l, uint32_t bin1, uint32_t key) {
        const bool hit = key && (key >> 16) == bin1;
        const uint64_t hits = __ballot(hit);
        if (!hits) return;
        const uint32_t leader = uint32_t(__builtin_ctzll(hits));
        uint32_t n = 1;
        bool adds = hit;
        // many keys and all the same (quantised values): one add for the wave
        if (__popcll(hits) > 8 && !__ballot(hit && key != __builtin_amdgcn_readlane(key, leader))) {
            n = uint32_t(__popcll(hits));
            adds = lane == leader;
        }
        if (adds) {
            atomicAdd(&rv.at<uint32_t>(wl.hist2)[uint64_t(l) * kBins2 + (key & 0xFFFFu)], n);
            atomicAdd(&s_coarse[(key >> 8) & 0xFFu], n);
        }
    };
    // the workgroup is done with its part of segment l; the last of `expected` selects
    auto finish = [&](uint32_t l, uint32_t k, SelDev r, uint32_t expected) {
        __syncthreads();  // s_coarse is complete
        const uint32_t c = s_coarse[tid];
        s_coarse[tid] = 0;
        if (c) atomicAdd(&ts.win[size_t(l) * kWinWords + tid], c);
        wait_own_memory_ops();
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(&ts.arrive[l], 1u) == expected - 1u;
        __syncthreads();
        if (s_last && wave == 0) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            uint32_t *coarse = ts.win + size_t(l) * kWinWords;
            const uint32_t want = k - r.G1;
            uint32_t hi_above, lo_above = 0, bin = 0;
            const uint32_t hi = top_of_256(coarse, want, &hi_above);
            reinterpret_cast<uint4 *>(coarse)[lane] = make_uint4(0, 0, 0, 0);
            if (hi != kNoBin)
                bin = hi << 8 | top_of_256(rv.at<uint32_t>(wl.hist2) + uint64_t(l) * kBins2 + hi * 256,
                                           want - hi_above, &lo_above);
            else if (lane == 0)  // cannot happen when both histograms saw the same data
                atomicOr(&ts.glob[0], TAGC_FLAG_OVERFLOW);
            if (lane == 0) {
                r.T = (r.bin1 << 16) | bin;
                r.G = r.G1 + hi_above + lo_above;
                r.quota = k - r.G;
                r.cnt = k;
                r.need2 = 0;
                sel[l] = r;
                ts.arrive[l] = 0;
            }
        }
        __syncthreads();  // s_last
    };

    // ---- candidate route: super-chunks [s0, s1) of the list
    const uint32_t span = (total_sc + n_cand - 1) / n_cand;
    const uint32_t s0 = blockIdx.x < n_cand ? min(blockIdx.x * span, total_sc) : total_sc,
                   s1 = min(s0 + span, total_sc);
    // (requested before anything is known of the segments: every link of the chain counts)
    auto info_of = [&](uint32_t sc) {
        return lane < NCH && sc < s1 ? chunk_info[sc * NCH + lane] : make_uint2(0, 0);
    };
    const uint2 info0 = info_of(s0 + wave);
    uint32_t l0 = L;  // the last segment that starts at s0 or before
    if (s0 < s1) {
        if (L <= 64)
            l0 = uint32_t(__popcll(__ballot(lane < L && segs[lane < L ? lane : 0].sc_start <= s0))) - 1u;
        else
            l0 = segment_of(L, s0, [&](uint32_t i) { return segs[i].sc_start; });
    }
    for (uint32_t l = l0; l < L; ++l) {
        const SegDev sd = segs[l];
        const SelDev se = sel[l];
        if (sd.sc_start >= s1) break;
        if (sd.k == 0 || sd.n == 0 || !(sd.flags & kSegFast) || se.route || !se.need2) continue;
        const uint32_t bin1 = se.bin1;
        const uint32_t n_sc = (sd.n + CHUNK * NCH - 1) / (CHUNK * NCH);
        const uint32_t lo = max(s0, sd.sc_start), hi = min(s1, sd.sc_start + n_sc);
        if (lo >= hi) continue;
        for (uint32_t sc = lo + wave; sc < hi; sc += NWV) {
            uint32_t cnt_l = 0, first_l = 0;  // of chunk `lane`
            if (lane < NCH && ((sc - sd.sc_start) * NCH + lane) * CHUNK < sd.n) {
                const uint2 info = sc == s0 + wave ? info0 : info_of(sc);
                cnt_l = min(info.x, CAP);
                first_l = min(info.y, n_slots_total - CAP);
            }
#pragma unroll
            for (uint32_t b0 = 0; b0 < NCH; b0 += kRefineBatch) {
                uint32_t v[kRefineBatch];
#pragma unroll
                for (uint32_t j = 0; j < kRefineBatch; ++j) {
                    const uint32_t c = __builtin_amdgcn_readlane(cnt_l, b0 + j);
                    const uint32_t first = __builtin_amdgcn_readlane(first_l, b0 + j);
                    v[j] = lane < c ? cand[first + lane] : 0u;
                }
#pragma unroll
                for (uint32_t j = 0; j < kRefineBatch; ++j) add_key(l, bin1, v[j] & 0x7FFFFFFFu);
            }
            for (uint64_t more = __ballot(cnt_l > 64); more; more &= more - 1) {
                const uint32_t ch = uint32_t(__builtin_ctzll(more));
                const uint32_t c = __builtin_amdgcn_readlane(cnt_l, ch);
                const uint32_t first = __builtin_amdgcn_readlane(first_l, ch);
                for (uint32_t i = 64 + lane; i < c; i += 64)
                    add_key(l, bin1, cand[first + i] & 0x7FFFFFFFu);
            }
        }
        finish(l, sd.k, se, (sd.sc_start + n_sc - 1) / span - sd.sc_start / span + 1);
    }

    // ---- dense route
    if (blockIdx.x >= n_dense || !any_dense_route(segs, sel, L)) return;
    for (uint32_t l = 0; l < L; ++l) {
        const SegDev sd = segs[l];
        if (!on_dense_route(sd, sel, l)) continue;
        const SelDev se = sel[l];
        if (!se.need2) continue;
        const uint32_t bin1 = se.bin1;
        const char *base = rv.src() + sd.offset * 4;
        const uint32_t nvec = (sd.n + 3) / 4;
        const uint32_t stride = n_dense * 256;
        for (uint32_t v = blockIdx.x * 256 + tid; v < nvec; v += kRefineRows * stride) {
            uint4 q[kRefineRows];
#pragma unroll
            for (uint32_t r = 0; r < kRefineRows; ++r)
                q[r] = load_vec<kF32>(base, 4 * min(v + r * stride, nvec), sd.n);
#pragma unroll
            for (uint32_t r = 0; r < kRefineRows; ++r) {
                add_key(l, bin1, q[r].x & 0x7FFFFFFFu);
                add_key(l, bin1, q[r].y & 0x7FFFFFFFu);
                add_key(l, bin1, q[r].z & 0x7FFFFFFFu);
                add_key(l, bin1, q[r].w & 0x7FFFFFFFu);
            }
        }
        finish(l, sd.k, se, n_dense);
    }
}

// ---------------------------------------------------------- ordered output

// Ordered output (the candidate route's super-chunks, the dense route's tiles) takes two
// launches and no waiting.  `count` leaves, per item, count(key > T) << 31 | count(key == T);
// `place` starts when all of them are there: every item adds up the counts of the earlier
// items of its segment by itself (a few hundred to a few thousand words from the L2) and puts
// its survivors where they belong.  No workgroup ever depends on another one's progress, so
// neither the order in which the device starts them nor other kernels in flight matter.

// pairs segment i emits, as the selection left it (segments that keep nothing have none)
__device__ inline uint32_t segment_count(const SegDev &sd, const SelDev *sel, uint32_t i)
{
    return sd.k == 0 || sd.n == 0 ? 0u : sel[i].cnt;
}

// The rank's count words, from the selections and what the call's kernels accumulated in
// the table (which goes back to zero); by one workgroup of the last kernel.
__device__ inline void write_rank_counts(uint32_t *table, uint32_t L, uint32_t slot, const SelDev *sel,
                                         uint32_t *cnt, uint32_t *smem /* >= 8 */)
{
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    uint32_t total = 0;
    for (uint32_t l = threadIdx.x; l < L; l += kEmitThreads) {
        const uint32_t c = segment_count(segs[l], sel, l);
        cnt[TAGC_CNT_SEG0 + l] = c;
        total += c;
    }
    total = block_sum<uint32_t, kEmitThreads / 64>(total, smem);
    if (threadIdx.x == 0) {
        const TableState ts = table_state(table, L, slot);
        cnt[TAGC_CNT_TOTAL] = total;
        cnt[TAGC_CNT_FLAGS] = ts.glob[0];
        cnt[TAGC_CNT_NONFINITE] = ts.glob[1];
        cnt[TAGC_CNT_DENSE] = ts.glob[2];
        cnt[TAGC_CNT_RESERVED] = 0;
        ts.glob[0] = ts.glob[1] = ts.glob[2] = 0;
    }
}

// ------------------------------------------------------------------- emit

// Candidate route, count.  How many of a super-chunk's slots are above and at the exact threshold does not
// depend on their order, so LPC lanes read 4 LPC slots of a chunk at once, the first of all the wave's chunks are in
// flight, every lane counts its own, and the wave sums once at the end.  Bound by the reads' latency (8 lanes to a
// chunk, two waves to a super-chunk), or by their bytes where the slots lie in memory and not in the last cache
// (MANY: 16 lanes, one wave; see count_from_memory).  us of the kernel, slots classified in order, a thread's own run
// or 64 a step / this: 2 ranks of 202 M entries with a tenth kept 84 / 55, 16 of 202 M 74 / 64, one rank's part of
// those 11.9 / 7.8, 1 rank of 4 M with a fifth 63 / 20.6.
constexpr uint32_t count_items(bool many)  // super-chunks of a workgroup
{
    return kEmitThreads / (many ? 64 : 128);
}

// Whether count reads the slots of n ranks from memory: chunks that hold hundreds, and more of them all than the
// last cache (256 MiB) keeps from the scan.  us of count, from memory / not: 2 ranks of 200 M entries with 12, 15, 20, 23
// percent kept (250, 312, 416, 478 MB) 63 / 70, 74 / 79, 115 / 128, 143 / 153; of 100 M with 20, 23 (208, 239 MB)
// 58 / 42, 80 / 56, 1 of 4 M with 8, 23 percent 18.5 / 11.5, 40 / 23; fp32, two words a slot, 2 of 100 M with 12, 20
// percent (250, 416 MB) 31.7 / 27.5, 40.4 / 42.5.  (Dozens of slots in 193 MB, 16 of 202 M entries: 75 / 64.)
inline bool count_from_memory(const tagc_plan_t *p, uint32_t n)
{
    // (a chunk's pre-threshold lets 1.3 times the kept entries through)
    const double bytes = 1.3 * double(p->K - p->dense_pairs) * n * (p->cfg.dtype == kF32 ? 8 : 4);
    return p->cand_cap >= kManyCandCap && bytes > 244e6;
}

template <int DTYPE, bool MANY>
__device__ __forceinline__ void count_body(uint32_t bid, const uint32_t *__restrict__ table,
                                           const WsLayout &wl, const SelDev *__restrict__ sel,
                                           const uint32_t *__restrict__ cand,
                                           const uint2 *__restrict__ chunk_info, uint32_t CAP, uint64_t *sc_cnt)
{
    constexpr uint32_t CHUNK = 64 * (DTYPE == kBF16 ? 8 : 4) * kCandRows;
    constexpr uint32_t LPC = MANY ? 16 : 8, WPS = MANY ? 1 : 2;
    constexpr uint32_t NCH = kCandChunksPerSuper / WPS;  // chunks of a wave
    constexpr uint32_t STEPS = NCH * LPC / 64;           // requests that cover them
    constexpr uint32_t ITEMS = count_items(MANY);
    static_assert(ITEMS * WPS * 64 == kEmitThreads, "a workgroup's waves");
    __shared__ uint64_t s_n[kEmitThreads / 64];
    const uint32_t L = wl.L, total_sc = wl.total_sc;
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // segment i's table rows in lane i
    uint32_t t_start = 0xFFFFFFFFu, t_n = 0, t_T = 0, t_quota = 0, t_cnt = 0, t_route = 0;
    if (L <= 64 && lane < L) {
        static_assert(sizeof(SegDev) == 32 && sizeof(SelDev) == 32, "two uint4 per row");
        const uint4 *s4 = reinterpret_cast<const uint4 *>(segs + lane);
        const uint4 *e4 = reinterpret_cast<const uint4 *>(sel + lane);
        const uint4 sa = s4[0], sb = s4[1], ea = e4[0], eb = e4[1];
        t_n = sa.z; t_start = sb.w;     // n, sc_start
        if (sb.x != 0 && sa.z != 0) {   // k, n: a segment that keeps nothing has no selection
            t_T = ea.x; t_quota = ea.y; t_cnt = ea.w; t_route = eb.w;  // T, quota, cnt, route
        }
    }
    const uint32_t base = bid * ITEMS;  // (some of the last workgroup's items may be none)
    const bool item = base + wave / WPS < total_sc;
    const uint32_t sc = item ? base + wave / WPS : base;
    const uint32_t ch0 = (wave % WPS) * NCH + lane / LPC;
    // count and first slot of the lane's chunks (only meaningful for a chunk the scan has seen)
    uint2 info[STEPS];
#pragma unroll
    for (uint32_t j = 0; j < STEPS; ++j) info[j] = chunk_info[sc * kCandChunksPerSuper + ch0 + j * (64 / LPC)];
    uint32_t n_seg, sc_first, T, quota, se_cnt, se_route;
    if (L <= 64) {
        const uint32_t l = uint32_t(__popcll(__ballot(t_start <= sc))) - 1u;  // segment 0 starts at 0
        n_seg = __builtin_amdgcn_readlane(t_n, l);
        sc_first = __builtin_amdgcn_readlane(t_start, l);
        T = __builtin_amdgcn_readlane(t_T, l);
        quota = __builtin_amdgcn_readlane(t_quota, l);
        se_cnt = __builtin_amdgcn_readlane(t_cnt, l);
        se_route = __builtin_amdgcn_readlane(t_route, l);
    } else {
        const uint32_t l = segment_of(L, sc, [&](uint32_t i) { return segs[i].sc_start; });
        const SegDev sd = segs[l];
        SelDev se{};
        if (sd.k != 0 && sd.n != 0) se = sel[l];
        n_seg = sd.n; sc_first = sd.sc_start;
        T = se.T; quota = se.quota; se_cnt = se.cnt; se_route = se.route;
    }
    const uint32_t sc_rel0 = (sc - sc_first) * (CHUNK * kCandChunksPerSuper), own = 4 * (lane % LPC);
    uint32_t c[STEPS];   // slots of this lane's chunk of the step, from the lane's own first on
    uint32_t at[STEPS];  // where that lies
#pragma unroll
    for (uint32_t j = 0; j < STEPS; ++j) {
        // (the bounds keep the reads inside `cand` whatever an unseen chunk's record holds)
        const uint32_t rel0 = sc_rel0 + (ch0 + j * (64 / LPC)) * CHUNK;
        const uint32_t n = !se_route && se_cnt != 0 && rel0 < n_seg ? min(info[j].x, CAP) : 0u;
        c[j] = n > own ? n - own : 0u;
        at[j] = (min(info[j].y, uint32_t(wl.n_slots) - CAP) & ~3u) + own;
    }
    uint32_t n_gt = 0, n_eq = 0;
    bool more = true;
    while (more) {
        uint4 q[STEPS];
#pragma unroll
        for (uint32_t j = 0; j < STEPS; ++j)  // (a chunk's slots start on, and have room up to, 16 bytes)
            q[j] = c[j] ? *reinterpret_cast<const uint4 *>(cand + at[j]) : make_uint4(0, 0, 0, 0);
        uint32_t left = 0;
#pragma unroll
        for (uint32_t j = 0; j < STEPS; ++j) {
            const uint32_t v[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t key = (DTYPE == kBF16 ? v[i] & 0xFFFF0000u : v[i]) & 0x7FFFFFFFu;
                n_gt += i < c[j] && key > T;
                n_eq += i < c[j] && key == T;
            }
            c[j] = c[j] > 4 * LPC ? c[j] - 4 * LPC : 0u;
            at[j] += 4 * LPC;
            left |= c[j];
        }
        more = __ballot(left != 0) != 0;
    }
    n_gt = __builtin_amdgcn_readlane(wave_incl_scan<uint32_t>(n_gt), 63);
    n_eq = __builtin_amdgcn_readlane(wave_incl_scan<uint32_t>(n_eq), 63);
    uint64_t sum = (uint64_t(n_gt) << 31) | uint64_t(quota ? n_eq : 0u);
    if (WPS > 1) {
        if (lane == 0) s_n[wave] = sum;
        __syncthreads();
        sum = s_n[wave & ~1u] + s_n[wave | 1u];
    }
    if (item && lane == 0 && wave % WPS == 0) sc_cnt[sc] = sum;
}

// Candidate route, place.  A wave takes a whole super-chunk, classifies its slots against the exact threshold,
// adds up the earlier super-chunks of the segment and places the survivors in ascending c-index.  Bound by
// latency where chunks hold few slots, and by memory where they hold hundreds.  Everything whose address follows
// from the workgroup number alone is requested at once: the chunk counts, and -- lane i taking segment i -- the
// whole segment and selection tables, from which the item's segment, its threshold and the pair offset of
// the segment come by ballot, readlane and a wave sum (tables of more than 64 segments take a slower path).
//
// The chunks' slots are numbered through by groups of 16 bytes, a lane a group: a step is 256 slots whatever
// the chunks hold, and every lane finds the chunk of its group by four steps of a search in the chunks' last
// group numbers.  BATCH steps are in flight, and the request behind a step goes out before that step's own
// stores: loads are waited for in issue order, and so are the stores between them.  A step's survivors are
// neighbours in the output; they are put side by side in LDS and leave as contiguous stores (entry by entry, each
// store would touch up to 64 cache lines).  The Index words of half a super-chunk are collected in
// LDS (all of it would leave room for fewer workgroups) and written whole, zeros included.  (Tried: a quarter, 12 KiB
// a workgroup instead of 20: 2 ranks of 202 M entries with a tenth kept 1382 -> 1399, no less with other buckets in flight.)
//
// us of the kernel, before / after.  Before, chunks of dozens of slots had four threads each and 23 KiB of LDS a
// workgroup: 8 ranks of 67 M entries 47.8 / 30.4, of 25 M 22.5 / 18.9, of 7 M fp32 22.1 / 18.7, 4 of 1 M fp32
// 9.6 / 9.9.  Chunks of hundreds, and large buckets, had 64 slots of one chunk to a step, 32 or more
// steps a super-chunk, and stored survivors as found: 16 ranks of 202 M 227 / 182, 2 of them with a tenth kept
// 162 / 149, one rank's part of a 202 M bucket 23.4 / 17.8.
constexpr uint32_t kEmitWindow = kCandChunksPerSuper / 2;  // chunks whose Index words are collected at a time
template <int DTYPE>
struct EmitLds {
    static constexpr uint32_t kWords = 64 * (DTYPE == kBF16 ? 8 : 4) * kCandRows * kEmitWindow / 32;
    uint32_t bits[kEmitThreads / 64][kWords];
    // a step's survivors: value bits and position in the super-chunk (16 bits); bf16 packs
    // both in one word, like a candidate slot
    uint32_t st_a[kEmitThreads / 64][256];
    uint16_t st_b[kEmitThreads / 64][DTYPE == kF32 ? 256 : 2];
};

template <int DTYPE, uint32_t BATCH>
__device__ __forceinline__ void emit_body(EmitLds<DTYPE> *lds, uint32_t bid,
                                 const uint32_t *__restrict__ table, const WsLayout &wl,
                                 const SelDev *__restrict__ sel,
            const uint32_t *__restrict__ cand, const uint2 *__restrict__ chunk_info,
            uint32_t CAP, const uint64_t *sc_cnt,
            uint32_t *__restrict__ idx_out, float *__restrict__ val_out,
            uint32_t *__restrict__ bitmap)
{
    constexpr uint32_t VEC = DTYPE == kBF16 ? 8 : 4;
    constexpr uint32_t CHUNK = 64 * VEC * kCandRows;
    constexpr uint32_t NCH = kCandChunksPerSuper;
    constexpr uint32_t SC_ELEMS = CHUNK * NCH;
    constexpr uint32_t WORDS = EmitLds<DTYPE>::kWords;
    constexpr uint32_t NWV = kEmitThreads / 64;
    static_assert(NCH == 32 && kEmitWindow == 16, "a lane per chunk, four steps of the search");
    static_assert(SC_ELEMS <= 65536, "a position in the super-chunk fits 16 bits");
    const uint32_t L = wl.L, total_sc = wl.total_sc;
    const uint64_t n_slots_total = wl.n_slots;
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t sc = bid * NWV + wave;
    if (sc >= total_sc) return;
    // (no other wave touches these)
    uint32_t *bits = lds->bits[wave], *st_a = lds->st_a[wave];
    uint16_t *st_b = lds->st_b[wave];
    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    auto total = [](uint32_t x) -> uint32_t {
        return __builtin_amdgcn_readlane(wave_incl_scan<uint32_t>(x), 63);
    };

    // segment i's table rows in lane i
    uint32_t t_start = 0xFFFFFFFFu, t_n = 0, t_coff = 0, t_T = 0, t_quota = 0, t_cnt = 0,
             t_route = 0;
    if (L <= 64 && lane < L) {
        const uint4 *s4 = reinterpret_cast<const uint4 *>(segs + lane);
        const uint4 *e4 = reinterpret_cast<const uint4 *>(sel + lane);
        const uint4 sa = s4[0], sb = s4[1], ea = e4[0], eb4 = e4[1];
        t_n = sa.z; t_coff = sa.w; t_start = sb.w;                 // n, c_off, sc_start
        if (sb.x != 0 && sa.z != 0) {   // k, n: a segment that keeps nothing has no selection
            t_T = ea.x; t_quota = ea.y; t_cnt = ea.w; t_route = eb4.w;  // T, quota, cnt, route
        }
    }
    for (uint32_t i = lane; i < WORDS; i += 64) bits[i] = 0;

    // count and first slot of chunk `lane` (only meaningful for a chunk the scan has seen),
    // requested together with the tables above
    const uint2 info = lane < NCH ? chunk_info[sc * NCH + lane] : make_uint2(0, 0);
    // ---- segment, threshold, pair offset of the segment
    uint32_t l, c_off, n_seg, sc_first, T, quota, seg_base, se_cnt, se_route;
    if (L <= 64) {
        const uint64_t le = __ballot(t_start <= sc);  // a prefix of the lanes
        l = uint32_t(__popcll(le)) - 1u;              // segment 0 starts at 0
        n_seg = __builtin_amdgcn_readlane(t_n, l);
        c_off = __builtin_amdgcn_readlane(t_coff, l);
        sc_first = __builtin_amdgcn_readlane(t_start, l);
        T = __builtin_amdgcn_readlane(t_T, l);
        quota = __builtin_amdgcn_readlane(t_quota, l);
        se_cnt = __builtin_amdgcn_readlane(t_cnt, l);
        se_route = __builtin_amdgcn_readlane(t_route, l);
        seg_base = lane < l ? t_cnt : 0u;
    } else {
        l = segment_of(L, sc, [&](uint32_t i) { return segs[i].sc_start; });
        const SegDev sd = segs[l];
        SelDev se{};
        if (sd.k != 0 && sd.n != 0) se = sel[l];
        n_seg = sd.n; c_off = sd.c_off; sc_first = sd.sc_start;
        T = se.T; quota = se.quota; se_cnt = se.cnt; se_route = se.route;
        uint32_t sum = 0;
        for (uint32_t i = lane; i < l; i += 64) sum += segment_count(segs[i], sel, i);
        seg_base = sum;
    }
    seg_base = total(seg_base);
    if (se_route) return;  // the dense route writes re-routed segments
    const uint32_t sc_rel0 = (sc - sc_first) * SC_ELEMS;

    // ---- chunk `lane` of the super-chunk: its candidates and where their slots are
    // (the bounds keep the reads inside `cand` whatever the record holds)
    uint32_t cnt_l = 0;
    if (lane < NCH && se_cnt != 0 && sc_rel0 + lane * CHUNK < n_seg) cnt_l = min(info.x, CAP);
    const uint32_t ngr_l = (cnt_l + 3u) >> 2;
    const uint32_t gend_l = wave_incl_scan<uint32_t>(ngr_l);  // (lanes from NCH on: the total)
    // slot and slots left at group g: these + 4 g, - 4 g
    const uint32_t at_l = (min(info.y, uint32_t(n_slots_total) - CAP) & ~3u) - 4 * (gend_l - ngr_l);
    const uint32_t left_l = cnt_l + 4 * (gend_l - ngr_l);
    // steps of the first window and of both
    const uint32_t G0 = __builtin_amdgcn_readlane(gend_l, kEmitWindow - 1);
    const uint32_t G1 = __builtin_amdgcn_readlane(gend_l, 63);
    const uint32_t S0 = (G0 + 63) >> 6, S = S0 + ((G1 - G0 + 63) >> 6);
    uint4 q[BATCH], qp[BATCH];
    uint32_t who[BATCH];  // chunk << 8 | slots of the lane's group
    auto request = [&](uint32_t t, uint32_t j) {
        const bool second = t >= S0;
        const uint32_t g = (second ? G0 + (t - S0) * 64 : t * 64) + lane;
        uint32_t ch = second ? kEmitWindow : 0u;  // first chunk that ends behind g
#pragma unroll
        for (uint32_t d = kEmitWindow / 2; d; d >>= 1)
            ch += uint32_t(__shfl(gend_l, int(ch + d - 1), 64)) <= g ? d : 0u;
        const uint32_t at = uint32_t(__shfl(at_l, int(ch), 64)) + 4 * g;
        const uint32_t left = uint32_t(__shfl(left_l, int(ch), 64)) - 4 * g;
        const uint32_t n = g < (second ? G1 : G0) ? min(left, 4u) : 0u;
        who[j] = ch << 8 | n;
        q[j] = qp[j] = make_uint4(0, 0, 0, 0);
        if (n) {  // (a chunk's slots start on, and have room up to, 16 bytes)
            q[j] = *reinterpret_cast<const uint4 *>(cand + at);
            if (DTYPE == kF32) qp[j] = *reinterpret_cast<const uint4 *>(cand + n_slots_total + at);
        }
    };
#pragma unroll
    for (uint32_t j = 0; j < BATCH; ++j)
        if (j < S) request(j, j);  // (on their way while the prefix below is added up)

    // prefix over the segment's earlier super-chunks, whose counts are all there
    // (eight requests at a time; a tenth kept on 202 M entries, 2 ranks: 163 -> 141 us.
    // fp32 slots are two words each, and beside those in flight there is room for two
    // requests: with eight, 24 registers went to scratch memory.  2 ranks, a tenth of 67 M
    // kept, then a hundredth of 202 M: 103 -> 87 us, 66 -> 56)
    constexpr uint32_t PRE = DTYPE == kBF16 ? 8 : 2;
    uint64_t sum = 0;
    for (uint32_t j = sc_first + lane; j < sc; j += PRE * 64) {
        uint64_t c[PRE];
#pragma unroll
        for (uint32_t i = 0; i < PRE; ++i) c[i] = j + 64 * i < sc ? sc_cnt[j + 64 * i] : 0ull;
#pragma unroll
        for (uint32_t i = 0; i < PRE; ++i) sum += c[i];
    }
    // entries above / at the threshold before the current step
    uint32_t gb = total(uint32_t(sum >> 31));
    uint32_t eb = total(uint32_t(sum & 0x7FFFFFFFu));

    // a window's Index words leave, and read zero again
    auto flush = [&](uint32_t window) {
        wave_fence();
#pragma unroll 8
        for (uint32_t i = lane; i < WORDS; i += 64) {
            const uint32_t w = bits[i], rel0 = sc_rel0 + (window * WORDS + i) * 32;
            bits[i] = 0;
            if (rel0 < n_seg) bitmap[(c_off + rel0) >> 5] = w;
        }
        wave_fence();
    };
    for (uint32_t t0 = 0; t0 < S; t0 += BATCH) {
#pragma unroll
        for (uint32_t j = 0; j < BATCH; ++j) {
            const uint32_t t = t0 + j;
            if (t >= S) break;  // uniform
            if (t == S0) flush(0);
            const uint32_t n = who[j] & 0xFFu, base = (who[j] >> 8) * CHUNK;
            const uint32_t a[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
            const uint32_t b[4] = {qp[j].x, qp[j].y, qp[j].z, qp[j].w};
            constexpr uint32_t KEY = DTYPE == kBF16 ? 0x7FFF0000u : 0x7FFFFFFFu;
            uint32_t own = 0;  // entries above << 16 | at the threshold
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t key = a[i] & KEY;
                own += i < n ? (key > T ? 0x10000u : key == T && quota ? 1u : 0u) : 0u;
            }
            if (t + BATCH < S) request(t + BATCH, j);
            const uint32_t inc = wave_incl_scan<uint32_t>(own);
            const uint32_t all = __builtin_amdgcn_readlane(inc, 63);
            // entries above T all survive, ties while the quota lasts
            const uint32_t pos0 = gb + min(eb, quota);  // the step's first survivor
            uint32_t my_gb = gb + ((inc - own) >> 16), my_eb = eb + ((inc - own) & 0xFFFFu);
            gb += all >> 16;
            eb += all & 0xFFFFu;
            const uint32_t kept = gb + min(eb, quota) - pos0;
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t key = a[i] & KEY;
                const bool is_gt = i < n && key > T, is_eq = i < n && key == T && quota;
                if (is_gt || (is_eq && my_eb < quota)) {
                    const uint32_t p = my_gb + min(my_eb, quota) - pos0;
                    const uint32_t rel = base + ((DTYPE == kBF16 ? a[i] : b[i]) & (CHUNK - 1u));
                    st_a[p] = DTYPE == kBF16 ? (a[i] & 0xFFFF0000u) | rel : a[i];
                    if (DTYPE == kF32) st_b[p] = uint16_t(rel);
                    const uint32_t in_window = rel & (WORDS * 32 - 1u);
                    atomicOr(&bits[in_window >> 5], 1u << (in_window & 31));
                }
                my_gb += is_gt;
                my_eb += is_eq;
            }
            wave_fence();
            for (uint32_t i = lane; i < kept; i += 64) {
                const uint32_t w = st_a[i], r = DTYPE == kBF16 ? w & 0xFFFFu : uint32_t(st_b[i]);
                idx_out[seg_base + pos0 + i] = c_off + sc_rel0 + r;
                val_out[seg_base + pos0 + i] = __uint_as_float(DTYPE == kBF16 ? w & 0xFFFF0000u : w);
            }
            wave_fence();
        }
    }
    if (S == S0) flush(0);
    flush(1);
}

// ---------------------------------------------------------------- compact

// Dense route, count and place, over the gradient itself: one tile of kCompactThreads x ROWS
// 16-byte vectors per workgroup and turn.  Also writes the (all-zero) Index words of the
// segments that keep nothing.  The segments the scan never reads have the first `plan_tiles`
// tiles, one workgroup each; the workgroups behind take those of re-routed segments in turns.
//
// STAGED (a plan whose pairs come mostly from here): a tile's survivors are gathered in LDS and leave as
// contiguous stores; entry by entry each store instruction would touch every cache line a
// wave's part of the output covers (8.7 M entries of which two fifths are kept, 4 ranks: place
// 78 us that way, 54 in this).
template <int DTYPE, bool STAGED>
struct CompactLds {
    static constexpr uint32_t kStage = STAGED ? kCompactThreads * (DTYPE == kBF16 ? 8 : 4) * 4 : 1;
    uint32_t v[kStage];  // bf16: value and position in the tile in one word
    uint16_t p[DTYPE == kF32 ? kStage : 1];
};

template <int DTYPE, uint32_t ROWS, bool PLACE, bool STAGED>
__device__ __forceinline__ void compact_body(CompactLds<DTYPE, STAGED> *lds, uint32_t bid, uint32_t nb, uint32_t plan_tiles,
                                             const char *grad, const uint32_t *__restrict__ table, const WsLayout &wl,
                                             const SelDev *__restrict__ sel, uint64_t *tile_cnt,
                                             uint64_t *group_cnt, uint32_t *__restrict__ idx_out,
                                             float *__restrict__ val_out,
                                             uint32_t *__restrict__ bitmap)
{
    constexpr uint32_t VEC = DTYPE == kBF16 ? 8 : 4;
    constexpr uint32_t ROW_ELEMS = kCompactThreads * VEC;
    constexpr uint32_t TILE = ROW_ELEMS * ROWS;
    constexpr uint32_t LPW = 32 / VEC;  // lanes that share one Index word
    constexpr uint32_t NWV = kCompactThreads / 64;
    static_assert(TILE <= 8192 && ROWS <= 4, "counts of a tile fit 16 bits, of its rows two words");
    static_assert(!STAGED || TILE == CompactLds<DTYPE, STAGED>::kStage, "room for all of a tile");
    uint32_t *st_v = lds->v;
    uint16_t *st_p = lds->p;
    __shared__ uint32_t s_wave[NWV][4];
    __shared__ uint64_t s_sum[NWV];

    const uint32_t L = wl.L, total_tiles = wl.total_tiles;
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // tiles plan_tiles and following are work only if a segment has been re-routed
    const bool net = bid >= plan_tiles;
    if (net) {
        bool any = false;
        for (uint32_t l = lane; l < L; l += 64)
            any |= (segs[l].flags & kSegFast) && on_dense_route(segs[l], sel, l);
        if (__ballot(any) == 0) return;
    }
    const uint32_t step = net ? nb - plan_tiles : total_tiles;

    for (uint32_t t = bid; t < total_tiles; t += step) {
        // ---- the tile's segment, its selection, and the pairs of the segments before it.  Up to 64 segments: lane i
        // looks at segment i, rows and selections requested together, where there are registers for that (row behind row
        // these are three trips to memory in front of the tile's: 4 ranks of 9 M entries, count 23.2 -> 21.6 us,
        // place 52.3 -> 49.9).
        constexpr bool kTogether = !PLACE || ROWS == 2 || (STAGED && DTYPE == kBF16);
        uint32_t l = 0, seg_base = 0;
        SegDev sd;
        SelDev se{};
        bool dense;
        if (kTogether && L <= 64) {
            uint4 ra = make_uint4(0, 0, 0, 0), rb = ra, ea = ra, eb = ra;
            if (lane < L) {
                const uint4 *s4 = reinterpret_cast<const uint4 *>(segs + lane), *e4 = reinterpret_cast<const uint4 *>(sel + lane);
                ra = s4[0]; rb = s4[1]; ea = e4[0]; eb = e4[1];
            }
            const bool keeps = rb.x != 0 && ra.z != 0;  // (a segment that keeps nothing has no selection)
            l = uint32_t(__builtin_ctzll(__ballot(lane < L && t >= rb.y && t - rb.y < (ra.z + TILE - 1) / TILE)));
            auto get = [&](uint32_t v) { return uint32_t(__builtin_amdgcn_readlane(v, l)); };
            sd = SegDev{uint64_t(get(ra.y)) << 32 | get(ra.x), get(ra.z), get(ra.w), get(rb.x), get(rb.y), get(rb.z), get(rb.w)};
            dense = sd.k != 0 && sd.n != 0 && (!(sd.flags & kSegFast) || get(eb.w) != 0);
            if (dense) {
                se.T = get(ea.x);
                se.quota = get(ea.y);
                se.cnt = get(ea.w);
            }
            if (PLACE) seg_base = wave_incl_scan<uint32_t>(keeps && lane < l ? ea.w : 0u);
            seg_base = __builtin_amdgcn_readlane(seg_base, 63);
        } else {
            for (uint32_t l0 = 0; l0 < L; l0 += 64) {
                bool mine = false;
                if (l0 + lane < L) {
                    const SegDev row = segs[l0 + lane];
                    mine = t >= row.tile_start && t - row.tile_start < (row.n + TILE - 1) / TILE;
                }
                const uint64_t bal = __ballot(mine);
                if (bal) {
                    l = l0 + uint32_t(__builtin_ctzll(bal));
                    break;
                }
            }
            sd = segs[l];
            dense = on_dense_route(sd, sel, l);
            if (dense) se = sel[l];
            uint32_t sb = 0;
            for (uint32_t i = lane; PLACE && i < l; i += 64) sb += segment_count(segs[i], sel, i);
            seg_base = wave_sum<uint32_t>(sb);
        }
        // (the candidate route writes the other segments that keep something; a segment that
        // keeps nothing only needs its Index words, which place writes as zeros)
        if (!dense && !(PLACE && sd.k == 0)) continue;  // uniform
        const uint32_t base_rel = (t - sd.tile_start) * TILE;
        const char *base = grad + sd.offset * (DTYPE == kBF16 ? 2 : 4);

        // ---- load (rows of 256 16-byte vectors, lane-contiguous) and classify.  Elements past
        // the end are loaded as 0 and never kept.
        uint32_t w[ROWS][4];
        uint32_t gtm[ROWS], eqm[ROWS];
#pragma unroll
        for (uint32_t r = 0; r < ROWS; ++r) {
            w[r][0] = w[r][1] = w[r][2] = w[r][3] = 0;
            gtm[r] = eqm[r] = 0;
        }
        if (se.cnt != 0) {
#pragma unroll
            for (uint32_t r = 0; r < ROWS; ++r) {
                const uint4 q = load_vec<DTYPE>(base, base_rel + r * ROW_ELEMS + tid * VEC, sd.n);
                w[r][0] = q.x; w[r][1] = q.y; w[r][2] = q.z; w[r][3] = q.w;
            }
#pragma unroll
            for (uint32_t r = 0; r < ROWS; ++r) {
#pragma unroll
                for (uint32_t e = 0; e < VEC; ++e) {
                    const uint32_t key = vec_elem_bits<DTYPE>(w[r], e) & 0x7FFFFFFFu;
                    gtm[r] |= uint32_t(key > se.T) << e;
                    eqm[r] |= uint32_t(key == se.T) << e;
                }
                if (!se.quota) eqm[r] = 0;
            }
        }
        if (!PLACE) {
            // the tile's counts, and added to those of its group of kTileGroup tiles (groups
            // are cut from the bucket's tile numbers, whatever the segments)
            uint32_t both = 0;
#pragma unroll
            for (uint32_t r = 0; r < ROWS; ++r) both += __popc(gtm[r]) | (__popc(eqm[r]) << 16);
            const uint32_t inc = wave_incl_scan<uint32_t>(both);
            if (lane == 63) s_wave[wave][0] = inc;
            __syncthreads();
            if (tid == 0) {
                uint32_t sum = 0;
#pragma unroll
                for (uint32_t i = 0; i < NWV; ++i) sum += s_wave[i][0];
                const uint64_t v = (uint64_t(sum & 0xFFFFu) << 31) | (sum >> 16);
                tile_cnt[t] = v;
                atomicAdd(reinterpret_cast<unsigned long long *>(&group_cnt[t / kTileGroup]), v);
            }
            __syncthreads();
            continue;
        }
        // ---- order inside the tile: the rows' counts, two to a word
        uint32_t own[4] = {0, 0, 0, 0}, inc[4];  // above rows 0/1, 2/3; ties rows 0/1, 2/3
#pragma unroll
        for (uint32_t r = 0; r < ROWS; ++r) {
            own[r >> 1] |= __popc(gtm[r]) << (16 * (r & 1));
            own[2 + (r >> 1)] |= __popc(eqm[r]) << (16 * (r & 1));
        }
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            inc[i] = wave_incl_scan<uint32_t>(own[i]);
            if (lane == 63) s_wave[wave][i] = inc[i];
        }
        // ---- add up the counts of the segment's earlier tiles: whole groups that lie inside
        // the segment by their sums, the tiles before and after them one by one (a few
        // hundred words at most, from the L2)
        {
            uint64_t sum = 0;
            if (dense) {
                const uint32_t t0 = sd.tile_start;
                const uint32_t g0 = (t0 + kTileGroup - 1) / kTileGroup, g1 = t / kTileGroup;
                if (g0 < g1) {
                    for (uint32_t j = t0 + tid; j < g0 * kTileGroup; j += kCompactThreads) sum += tile_cnt[j];
                    for (uint32_t j = g0 + tid; j < g1; j += kCompactThreads) sum += group_cnt[j];
                    for (uint32_t j = g1 * kTileGroup + tid; j < t; j += kCompactThreads) sum += tile_cnt[j];
                } else {
                    for (uint32_t j = t0 + tid; j < t; j += kCompactThreads) sum += tile_cnt[j];
                }
            }
            sum = wave_sum<uint64_t>(sum);
            if (lane == 0) s_sum[wave] = sum;
        }
        __syncthreads();
        uint32_t tot[4] = {0, 0, 0, 0}, ex[4];
        uint64_t before = 0;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) ex[i] = inc[i] - own[i];
#pragma unroll
        for (uint32_t q = 0; q < NWV; ++q) {
            before += s_sum[q];
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t x = s_wave[q][i];
                if (q < wave) ex[i] += x;
                tot[i] += x;
            }
        }
        uint32_t grun = uint32_t(before >> 31), erun = uint32_t(before & 0x7FFFFFFFu);
        const uint32_t tile_pos = grun + min(erun, se.quota);  // first survivor, in the segment

        // ---- pairs and Index words
        uint32_t keepm[ROWS];
#pragma unroll
        for (uint32_t r = 0; r < ROWS; ++r) {
            const uint32_t sh = 16 * (r & 1);
            uint32_t gb = grun + ((ex[r >> 1] >> sh) & 0xFFFFu);
            uint32_t eb = erun + ((ex[2 + (r >> 1)] >> sh) & 0xFFFFu);
            const uint32_t rel_t = r * ROW_ELEMS + tid * VEC;  // position in the tile
            uint32_t km = gtm[r];
            auto keep_entry = [&](uint32_t e, uint32_t bits, uint32_t pos) {
                if (STAGED) {
                    if (DTYPE == kBF16) {
                        st_v[pos - tile_pos] = bits | (rel_t + e);
                    } else {
                        st_v[pos - tile_pos] = bits;
                        st_p[DTYPE == kF32 ? pos - tile_pos : 0] = uint16_t(rel_t + e);
                    }
                } else {
                    idx_out[seg_base + pos] = sd.c_off + base_rel + rel_t + e;
                    val_out[seg_base + pos] = __uint_as_float(bits);
                }
            };
#pragma unroll
            for (uint32_t e = 0; e < VEC; ++e) {
                const uint32_t bits = vec_elem_bits<DTYPE>(w[r], e);
                if ((gtm[r] >> e) & 1u) {
                    keep_entry(e, bits, gb + min(eb, se.quota));
                    ++gb;
                } else if ((eqm[r] >> e) & 1u) {
                    if (eb < se.quota) {
                        km |= 1u << e;
                        keep_entry(e, bits, gb + eb);
                    }
                    ++eb;
                }
            }
            keepm[r] = km;
            grun += (tot[r >> 1] >> sh) & 0xFFFFu;
            erun += (tot[2 + (r >> 1)] >> sh) & 0xFFFFu;
        }
#pragma unroll
        for (uint32_t r = 0; r < ROWS; ++r) {
            const uint32_t rel = base_rel + r * ROW_ELEMS + tid * VEC;
            uint32_t v = keepm[r] << (VEC * (tid & (LPW - 1)));
#pragma unroll
            for (uint32_t d = 1; d < LPW; d <<= 1) v |= __shfl_xor(v, d, 64);
            const uint32_t rel0 = rel - (tid & (LPW - 1)) * VEC;  // first element of the word
            if ((tid & (LPW - 1)) == 0 && rel0 < sd.n) bitmap[(sd.c_off + rel0) >> 5] = v;
        }
        __syncthreads();
        if (STAGED) {
            const uint32_t n_out = grun + min(erun, se.quota) - tile_pos;
            uint32_t *io = idx_out + seg_base + tile_pos;
            float *vo = val_out + seg_base + tile_pos;
            for (uint32_t i = tid; i < n_out; i += kCompactThreads) {
                const uint32_t a = st_v[i];
                const uint32_t rel = DTYPE == kBF16 ? (a & 0xFFFFu) : st_p[DTYPE == kF32 ? i : 0];
                io[i] = sd.c_off + base_rel + rel;
                vo[i] = __uint_as_float(DTYPE == kBF16 ? (a & 0xFFFF0000u) : a);
            }
            __syncthreads();  // LDS is reused by the next iteration
        }
    }
}

// --------------------------------------------------------- count and place

// The last two kernels of PHASE_INDEX.  In each, the first `n_emit` workgroups work on the
// candidate-route segments and the rest on the dense-route ones (pairs and Index words of
// different segments): one launch instead of two, and when a bucket has no dense-route work
// that part costs nothing, not even an empty kernel's turn-around.
static_assert(kEmitThreads == kCompactThreads, "one launch for both parts");

template <int DTYPE, uint32_t COMPACT_ROWS, bool MANY>
__global__ void __launch_bounds__(kEmitThreads)
count_kernel(const SparsifyBatch, uint32_t n_emit, uint32_t plan_tiles,
             const uint32_t *__restrict__ table, const WsLayout wl, uint32_t CAP)
{
    const RankView rv = rank_view();
    const SelDev *sel = rv.at<SelDev>(wl.sel);
    if (blockIdx.x < n_emit) {
        count_body<DTYPE, MANY>(blockIdx.x, table, wl, sel, rv.at<uint32_t>(wl.cand),
                                rv.at<uint2>(wl.chunk_info), CAP, rv.at<uint64_t>(wl.sc_cnt));
    } else
        compact_body<DTYPE, COMPACT_ROWS, false, false>(
            nullptr, blockIdx.x - n_emit, gridDim.x - n_emit, plan_tiles, rv.src(), table, wl, sel,
            rv.at<uint64_t>(wl.tile_cnt), rv.at<uint64_t>(wl.group_cnt), nullptr, nullptr, nullptr);
}

template <int DTYPE, uint32_t COMPACT_ROWS, bool STAGED>
__global__ void __launch_bounds__(kEmitThreads)
    __attribute__((amdgpu_waves_per_eu(COMPACT_ROWS == 2 ? 7 : STAGED && DTYPE == kBF16 ? 4 : 6, 8)))
place_kernel(const SparsifyBatch, uint32_t n_emit, uint32_t plan_tiles, uint32_t *table,
             const WsLayout wl, uint32_t CAP)
{
    union Lds {
        EmitLds<DTYPE> emit;
        CompactLds<DTYPE, STAGED> compact;
    };
    __shared__ Lds lds;
    const RankView rv = rank_view();
    const SelDev *sel = rv.at<SelDev>(wl.sel);
    if (blockIdx.x == gridDim.x - 1) {  // (any one workgroup: the last has the least to do)
        __shared__ uint32_t s_cnt[8];
        write_rank_counts(table, wl.L, rv.slot, sel, rv.cnt, s_cnt);
    }
    if (blockIdx.x < n_emit) {
        const uint32_t *cand = rv.at<uint32_t>(wl.cand);
        const uint2 *chunk_info = rv.at<uint2>(wl.chunk_info);
        const uint64_t *sc_cnt = rv.at<uint64_t>(wl.sc_cnt);
        emit_body<DTYPE, DTYPE == kBF16 ? 4 : 2>(&lds.emit, blockIdx.x, table, wl, sel, cand, chunk_info, CAP,
                                                 sc_cnt, rv.idx, rv.val, rv.bitmap);
    } else
        compact_body<DTYPE, COMPACT_ROWS, true, STAGED>(
            &lds.compact, blockIdx.x - n_emit, gridDim.x - n_emit, plan_tiles, rv.src(), table, wl, sel,
            rv.at<uint64_t>(wl.tile_cnt), rv.at<uint64_t>(wl.group_cnt), rv.idx, rv.val, rv.bitmap);
}

template <typename K>
int resident_blocks_per_cu(K kernel, int threads, size_t lds, int *cache)
{
    if (*cache == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, lds) != hipSuccess ||
            n <= 0)
            return 0;
        *cache = n;
    }
    return *cache;
}

template <typename K>
int allow_lds(K kernel, size_t lds, bool *done)
{
    if (*done) return TAGC_OK;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)
        return TAGC_EHIP;
    *done = true;
    return TAGC_OK;
}

// Error feedback, on request: clears the entries of acc that the rank's Index names, after
// which acc is acc_next of Algorithm 1 as a plain array (for inspection or a checkpoint;
// the next PHASE_INDEX call does not need it and gives the same results either way).  One
// thread per 32 parameters of the c-index space; ~1 % of the entries get a store.
__global__ void __launch_bounds__(256)
feedback_apply_kernel(const uint32_t *__restrict__ table, const SentMap sent, uint32_t n_words,
                      char *acc, int dtype)
{
    const uint32_t w = blockIdx.x * 256 + threadIdx.x;
    if (w >= n_words) return;
    uint32_t bits;
    if (sent.wire4) {
        const uint4 q = *reinterpret_cast<const uint4 *>(sent.map + 4 * size_t(w));
        bits = nibbles_set(q.x) | (nibbles_set(q.y) << 8) | (nibbles_set(q.z) << 16) |
               (nibbles_set(q.w) << 24);
    } else {
        bits = sent.map[w];
    }
    if (!bits) return;
    const uint32_t L = table[0];
    const SegDev *segs = reinterpret_cast<const SegDev *>(table + 8);
    // a word of the Index lies inside one segment (c-offsets are multiples of 32); of several
    // segments starting at the same c-index only the last is not empty
    const uint32_t l = segment_of(L, w * 32, [&](uint32_t i) { return segs[i].c_off; });
    const SegDev sd = segs[l];
    char *ab = acc + sd.offset * (dtype == kBF16 ? 2 : 4);
    const uint32_t rel0 = w * 32 - sd.c_off;
    for (; bits; bits &= bits - 1) {
        const uint32_t rel = rel0 + __builtin_ctz(bits);
        if (rel < sd.n) store_elem(ab, rel, 0u, dtype);
    }
}

// 4-bit wire Index (section 2.2: the stable, four times bigger variant that an All-Reduce
// by addition can merge): one 0/1 counter per parameter, parameter j in bits 4*(j&7).. of
// word j>>3.  One thread per word of the 1-bit Index: 4 bytes in, one 16-byte store out.
__device__ __forceinline__ uint32_t spread8(uint32_t b)  // bit p of a byte -> bit 4p
{
    uint32_t x = (b | (b << 12)) & 0x000F000Fu;  // nibbles 0,1 -> 16-bit fields
    x = (x | (x << 6)) & 0x03030303u;            // 2 bits per byte
    x = (x | (x << 3)) & 0x11111111u;            // 1 bit per nibble
    return x;
}

__global__ void __launch_bounds__(256)
widen4_kernel(const SparsifyBatch, uint32_t n_words)
{
    const RankView rv = rank_view();
    const uint32_t *__restrict__ map = rv.bitmap;
    uint32_t *__restrict__ wire = rv.wire;
    const uint32_t w = blockIdx.x * 256 + threadIdx.x;
    if (w >= n_words) return;
    const uint32_t m = map[w];
    st_stream(reinterpret_cast<uint4 *>(wire + 4 * size_t(w)),
              make_uint4(spread8(m & 0xFFu), spread8((m >> 8) & 0xFFu),
                         spread8((m >> 16) & 0xFFu), spread8(m >> 24)));
}

WsLayout ws_layout(const tagc_plan_t *p)
{
    return WsLayout{p->ws.hist1d,   p->ws.hist2,  p->ws.group_cnt,  p->ws.sel,
                    p->ws.tile_cnt, p->ws.sc_cnt, p->ws.chunk_info, p->ws.cand,
                    uint64_t(p->total_sc) * kCandChunksPerSuper * p->cand_cap,
                    uint32_t(p->table.size()), p->total_tiles, p->total_sc};
}

SparsifyRank sparsify_rank(const tagc_plan_t *p, const void *grad, const tagc_rank_buffers &rk,
                           uint32_t slot, uint32_t from)
{
    char *ws = static_cast<char *>(rk.workspace);
    // with 4-bit counters on the wire the 1-bit Index is built in the workspace and widened
    return SparsifyRank{static_cast<const char *>(grad),
                        static_cast<char *>(rk.acc),
                        rk.bitmap,
                        ws,
                        rk.idx,
                        rk.val,
                        p->cfg.index_mode == TAGC_INDEX_ADD4
                            ? reinterpret_cast<uint32_t *>(ws + p->ws.bitmap1)
                            : rk.bitmap,
                        rk.bitmap,
                        rk.cnt,
                        slot,
                        from};
}

// The first kernels of PHASE_INDEX, up to every segment's threshold (fp32: its upper half), for
// n ranks with workspaces and table slots of their own, all with an accumulator (`acc`) or none
// with one.  `sample`: no pre-threshold is known yet.  `one`: small_kernel does it all, launch_output's part as well.
//
// Error feedback: scan_spill (candidate route) and accumulate_kernel (all other segments) turn
// acc into grad + acc; whoever reads the input after them reads it from acc.  Both read acc
// through the Index this rank's previous call left in rk->bitmap (what was sent reads as 0)
// before place / widen4 overwrite that Index with the new one.
template <int DTYPE>
int launch_select(const tagc_plan_t *p, const SparsifyBatch &sb, uint32_t n, bool acc, bool sample, bool one,
                  uint32_t *table, hipStream_t s)
{
    const WsLayout wl = ws_layout(p);
    const bool wide = p->cfg.index_mode == TAGC_INDEX_ADD4;
    const int cus = device_cu_count();
    const size_t lds_hist = kBins1 * sizeof(uint32_t);
    static bool a_prepare = false;
    if (allow_lds(prepare_kernel<DTYPE>, lds_hist, &a_prepare)) return TAGC_EHIP;
    // `total` workgroups shared out to the ranks
    auto per_rank = [&](uint32_t total) { return std::max(1u, total / n); };
    if (acc && p->any_nonfast) {
        ProfileScope ps("accumulate", s);
        accumulate_kernel<DTYPE><<<dim3(per_rank(cus * 4), n), 256, 0, s>>>(sb, table, wide);
    }
    if (one) {
        ProfileScope ps("small", s);
        small_kernel<DTYPE><<<dim3(uint32_t(p->table.size()), n), kSmallThreads, 0, s>>>(sb, table, wl);
        return TAGC_OK;
    }
    if (sample) {
        ProfileScope ps("prepare", s);
        prepare_kernel<DTYPE><<<dim3(uint32_t(p->table.size()), n), kHistThreads, lds_hist, s>>>(
            sb, table, wide);
    }
    if (p->any_fast || p->span_dense) {
        // (also clears the histograms in memory; short segments need neither)
        ProfileScope ps("scan_spill", s);
        // (the longer stage unless other buckets are in flight and chunks hold dozens of candidates: see
        // kSpillStage)
        constexpr bool kCanLong = DTYPE == kBF16;
        const bool lng = kCanLong && (!p->cfg.decode_workgroups || p->cand_cap >= kManyCandCap);
        auto scan = lng ? (acc ? scan_spill_kernel<DTYPE, true, kCanLong> : scan_spill_kernel<DTYPE, false, kCanLong>)
                        : (acc ? scan_spill_kernel<DTYPE, true, false> : scan_spill_kernel<DTYPE, false, false>);
        // Workgroups that fit the device at once, or, where their spans stay long enough for what
        // a span costs (its window's atomics, its first loads), up to eight rounds of them:
        // compute units do not stream at one rate, and short spans even that out (16 ranks of
        // 202 M entries: 3112 us for the whole path with one round, 3060 with eight).
        const uint32_t resident = per_rank(cus * kSpillWgsPerCU);
        const uint32_t spans = p->total_sc * kCandChunksPerSuper / kSpillSpan;
        const uint32_t rounds = std::min(8u, std::max(1u, spans / resident));
        scan<<<dim3(resident * rounds, n), kSpillThreads, 0, s>>>(
            sb, table, wl, p->cand_cap, p->zero_bytes / 16, wide);
    }
    {
        // Two workgroups of 512 threads per compute unit for work that is certain, as many as
        // there are tiles of a few KiB at most; the net of re-routed segments leaves at once
        // nearly always.
        ProfileScope ps("hist1", s);
        const bool small = p->small_dense;
        const uint32_t threads = small ? kSmallThreads : kDenseThreads;
        const uint32_t most = per_rank(uint32_t(cus) * 2048 / (threads * 2));
        const uint64_t tile = uint64_t(threads) * p->vec_elems * kDenseRows;
        const uint32_t planned = uint32_t(std::min<uint64_t>(most, (p->span_dense + tile - 1) / tile));
        const uint32_t n_span = std::max(p->any_fast ? most : 1u, planned);
        const dim3 grid(n_span + (small ? uint32_t(p->table.size()) : 0u), n);
        auto hist1 = small ? hist1_kernel<DTYPE, true> : hist1_kernel<DTYPE, false>;
        hist1<<<grid, threads, 0, s>>>(sb, table, wl, n_span);
    }
    return TAGC_OK;
}

// The rest of PHASE_INDEX for the same ranks: the thresholds' lower half (fp32), counts, output.
template <int DTYPE>
int launch_output(const tagc_plan_t *p, const SparsifyBatch &sb, uint32_t n, bool one, uint32_t *table,
                  hipStream_t s)
{
    const WsLayout wl = ws_layout(p);
    const int cus = device_cu_count();
    static int occ_place[3] = {};
    auto per_rank = [&](uint32_t total) { return std::max(1u, total / n); };
    if (DTYPE == kF32 && (p->any_fast || p->span_dense)) {
        // candidate list: four super-chunks (a wave each) to a workgroup, no more of them than fit
        // the device; dense route: a workgroup per kRefineRows vectors of its threads where the work
        // is certain, a sixteenth of that for what may be re-routed (idle workgroups, which a
        // bucket of 7 M entries on 8 ranks notices: with a quarter of it 3 us)
        ProfileScope ps("refine", s);
        const uint32_t n_cand = std::min(per_rank(cus * 8), std::max(1u, (p->total_sc + 3) / 4));
        const uint64_t turn = 256 * 4 * kRefineRows;  // entries
        const uint64_t dense = std::max((p->span_dense + turn - 1) / turn,
                                        p->any_fast ? p->n_real / (16 * turn) : uint64_t(0));
        const uint32_t n_dense = uint32_t(
            std::min<uint64_t>(per_rank(cus * 4), std::max<uint64_t>(1, dense)));
        const uint32_t grid = std::max(n_cand, n_dense);
        refine_kernel<<<dim3(grid, n), 256, 0, s>>>(sb, table, wl, p->cand_cap, n_cand, n_dense);
    }
    if (!one) {
        // the plan fixed the compaction tile's height, and with it which kernels these are
        const bool rows4 = p->compact_rows == 4;
        const bool many = count_from_memory(p, n);
        auto count = many ? (rows4 ? count_kernel<DTYPE, 4, true> : count_kernel<DTYPE, 2, true>)
                          : (rows4 ? count_kernel<DTYPE, 4, false> : count_kernel<DTYPE, 2, false>);
        // place stages the dense route's tiles where most pairs can come from them.  Beside large
        // candidate-route segments a short one of the dense route would have every workgroup hold
        // 33 KiB of LDS and 107 registers for it instead of 20 KiB and 75 (us of place, staged / not, 4 ranks
        // of 202 M entries and 5 thousand 49.3 / 44.0; of 25 M and 9 M of which two fifths are kept 58 / 86,
        // of 25 M and 1 M 18.4 / 22.5, of 100 M and 3 M 43.5 / 52; the line could lie a little lower: of
        // 100 M and 1 M 32.2 / 34.7; one rank, or fp32: the same way by less).
        const bool staged = rows4 && 2 * p->dense_pairs > p->K;
        auto place = staged ? place_kernel<DTYPE, 4, true>
                     : rows4 ? place_kernel<DTYPE, 4, false> : place_kernel<DTYPE, 2, false>;
        const int occ = resident_blocks_per_cu(place, kEmitThreads, 0, &occ_place[rows4 + staged]);
        if (occ <= 0) return TAGC_EHIP;
        auto n_emit = [&](uint32_t per_wg) {
            return p->any_fast ? (p->total_sc + per_wg - 1) / per_wg : 0u;
        };
        const uint32_t n_count = n_emit(count_items(many)), n_place = n_emit(kEmitThreads / 64);
        // Dense route: one tile per workgroup where the work is certain.  The tiles of the
        // candidate route's segments are only a safety net for re-routed ones and the
        // workgroups for them nearly always exit at once: a grid that fits the device takes
        // those tiles in turns.
        const uint32_t n_net = std::min<uint32_t>(p->total_tiles - p->plan_tiles,
                                                  per_rank(uint32_t(cus) * uint32_t(occ)));
        auto grid = [&](uint32_t n_cand) { return dim3(n_cand + p->plan_tiles + n_net, n); };
        {
            ProfileScope ps("count", s);
            count<<<grid(n_count), kEmitThreads, 0, s>>>(sb, n_count, p->plan_tiles, table, wl, p->cand_cap);
        }
        {
            ProfileScope ps("place", s);
            place<<<grid(n_place), kEmitThreads, 0, s>>>(sb, n_place, p->plan_tiles, table, wl, p->cand_cap);
        }
    }
    if (p->cfg.index_mode == TAGC_INDEX_ADD4 && p->n_c) {
        ProfileScope ps("widen4", s);
        const uint32_t n_words = uint32_t(p->n_c / 32);
        widen4_kernel<<<dim3((n_words + 255) / 256, n), 256, 0, s>>>(sb, n_words);
    }
    return hip_ok(hipGetLastError());
}

// PHASE_INDEX of n ranks with workspaces and table slots (0 .. n-1) of their own.
template <int DTYPE>
int launch_sparsify_t(const tagc_plan_t *p, const void *const *grads, const tagc_rank_buffers *ranks,
                      uint32_t n, const tagc_shared_buffers *sh, hipStream_t s)
{
    const uint32_t L = uint32_t(p->table.size());
    // the table is the plan's device state as well (pre-thresholds, counters): written here
    uint32_t *table = static_cast<uint32_t *>(const_cast<void *>(sh->table));
    if (L == 0 || (p->total_sc == 0 && p->total_tiles == 0)) {
        // nothing is compressed (or every compressed segment is empty): only the counts
        // have to read zero
        for (uint32_t r = 0; r < n; ++r) {
            ProfileScope ps("fill_zero", s);
            fill_zero_kernel<<<1, 256, 0, s>>>(static_cast<uint4 *>(ranks[r].workspace), 0,
                                               ranks[r].cnt, TAGC_CNT_SEG0 + L);
        }
        return hip_ok(hipGetLastError());
    }
    const bool acc = ranks[0].acc != nullptr;
    // One launch for short segments: a workgroup fills a compute unit, so as long as they are two turns of them
    // (bf16) or four.  PHASE_INDEX, us, three launches / one, gradients nearly all zeros (the same without zeros,
    // 1 % kept), by workgroups: bf16 448 24.4 / 21.8 (24.8 / 22.0), 512 24.4 / 22.3 (25.9 / 22.7), 640 29.9 / 32.2 (30.6
    // / 33.0), 1024 36.8 / 43.4 (39.4 / 44.1); fp32 512 25.5 / 18.0 (38.8 / 19.8), 640 26.0 / 24.7 (40.1 / 28.3), 896
    // 31.9 / 31.7 (50.6 / 37.0), 1024 40.8 / 35.2 (51.0 / 37.6), 2048 57.6 / 66.3 (94.1 / 74.0).
    const uint32_t turns = DTYPE == kBF16 ? 2 : 4;
    const bool one = p->all_small && uint64_t(L) * n <= turns * uint64_t(device_cu_count());
    SparsifyBatch sb{};
    SparsifyBatch part{};  // the ranks whose thresholds are launched next
    uint32_t n_part = 0;
    bool sample = false;
    auto select = [&]() -> int {
        if (!n_part) return TAGC_OK;
        const int rc = launch_select<DTYPE>(p, part, n_part, acc, sample, one, table, s);
        n_part = 0;
        sample = false;
        return rc;
    };
    for (uint32_t r = 0; r < n; ++r) {
        // A rank whose slot of the table's state has not been used since the upload starts
        // from the pre-thresholds of the rank before it (slot 0: from a sample), so it has
        // to wait for those: one launch of the first kernels each, just this once.
        const uint32_t slot = r, bit = 1u << slot;
        const bool fresh = !(p->used.fetch_or(bit, std::memory_order_relaxed) & bit);
        if (fresh)
            if (const int rc = select()) return rc;
        sb.r[r] = part.r[n_part++] =
            sparsify_rank(p, grads[r], ranks[r], slot, fresh && slot ? slot - 1 : slot);
        sample = fresh && slot == 0;
        if (fresh)
            if (const int rc = select()) return rc;
    }
    if (const int rc = select()) return rc;
    return launch_output<DTYPE>(p, sb, n, one, table, s);
}

}  // namespace

int launch_feedback_apply(const tagc_plan_t *p, const tagc_rank_buffers *rk,
                          const tagc_shared_buffers *sh, hipStream_t s)
{
    const uint32_t n_words = uint32_t(p->n_c / 32);
    if (!n_words) return TAGC_OK;
    ProfileScope ps("feedback_apply", s);
    const SentMap sent{rk->bitmap, p->cfg.index_mode == TAGC_INDEX_ADD4 ? 1u : 0u};
    feedback_apply_kernel<<<(n_words + 255) / 256, 256, 0, s>>>(
        static_cast<const uint32_t *>(sh->table), sent, n_words, static_cast<char *>(rk->acc),
        p->cfg.dtype == TAGC_BF16 ? kBF16 : kF32);
    return hip_ok(hipGetLastError());
}

int launch_sparsify(const tagc_plan_t *p, const void *const *grads, const tagc_rank_buffers *ranks,
                    uint32_t n_ranks, const tagc_shared_buffers *sh, hipStream_t s)
{
    for (uint32_t r0 = 0; r0 < n_ranks;) {
        // The longest run of ranks that can go together: buffers of their own (ranks that share a
        // workspace or anything else they write have to take turns), a slot of the table's state
        // each, and all with an accumulator or none with one.
        uint32_t n = 1;
        auto joins = [&](uint32_t r) {
            const tagc_rank_buffers &b = ranks[r];
            if ((b.acc != nullptr) != (ranks[r0].acc != nullptr)) return false;
            for (uint32_t q = r0; q < r; ++q) {
                const tagc_rank_buffers &a = ranks[q];
                if (a.workspace == b.workspace || a.idx == b.idx || a.val == b.val ||
                    a.cnt == b.cnt || a.bitmap == b.bitmap || (a.acc && a.acc == b.acc))
                    return false;
            }
            return true;
        };
        while (r0 + n < n_ranks && n < p->slots && joins(r0 + n)) ++n;
        const int rc = p->cfg.dtype == TAGC_BF16
                           ? launch_sparsify_t<kBF16>(p, grads + r0, ranks + r0, n, sh, s)
                           : launch_sparsify_t<kF32>(p, grads + r0, ranks + r0, n, sh, s);
        if (rc) return rc;
        r0 += n;
    }
    return TAGC_OK;
}

// ------------------------------------------------ workspace without a caller
//
// For callers that cannot hand over (or allocate) a rank workspace: the same kernels work
// on this array instead.  In host code `scratch` is only a stand-in for the symbol, not a
// device address; the address on the current device is looked up once per device and kept.
// Every GPU holds its own copy of the array at its own address until the process ends.
static __device__ __align__(256) unsigned char scratch[TAGC_STATIC_WORKSPACE_BYTES];

int static_workspace(void **out)
{
    static std::mutex mu;
    static void *ptr[64] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return TAGC_EHIP;
    std::lock_guard<std::mutex> lk(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TAGC_EHIP;
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return TAGC_OK;
}

}  // namespace tagc
