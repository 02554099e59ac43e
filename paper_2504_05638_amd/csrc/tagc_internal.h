// Internal declarations shared by the libtagc sources (host plan + HIP kernels).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <vector>

#include "tagc.h"

namespace tagc {

// ---------------------------------------------------------------- constants

constexpr uint32_t kBins1 = 32768;   // top 15 key bits: all of a bf16 key, key>>16 of fp32
constexpr uint32_t kBins2 = 65536;   // low 16 key bits (fp32 only)
constexpr uint32_t kHistThreads = 1024;
constexpr uint32_t kCompactThreads = 256;
constexpr uint32_t kDenseThreads = 256;   // dense route's histogram; ...
constexpr uint32_t kSmallThreads = 1024;  // ... of a plan with segments one workgroup holds
constexpr uint32_t kDenseRows = 4;        // 16-byte vectors per thread and tile of it
constexpr uint32_t kSmallVecs = 8;        // 16-byte vectors per thread such a segment has at most
constexpr uint32_t kSmallSegments = 64;   // segments up to which a plan of such segments takes one launch, ...
constexpr uint32_t kSmallPairs = 80 * 1024;    // ... entries and four times those kept of each (see tagc_plan)
constexpr uint32_t kHistWindow = 4096;
constexpr uint32_t kCandRows = 4;        // 16-byte vectors per lane per candidate chunk
constexpr uint32_t kCandChunksPerSuper = 32;  // chunks that a wave of place takes
constexpr uint32_t kEmitThreads = 256;
constexpr uint32_t kSampleVectors = 4096;     // 16-byte vectors sampled per segment
constexpr uint32_t kFastMinElems = 1u << 17;  // shorter segments take the dense path
constexpr uint32_t kFastMinKeep = 64;
constexpr uint32_t kManyCandCap = 192;  // candidate slots per chunk from which a chunk holds hundreds of them
constexpr double kFastMaxCandFrac = 0.30;  // expected candidates per element beyond which the dense path is planned
constexpr uint32_t kChunkWords = 1024;  // Index words per popcount chunk, ...
constexpr uint32_t kGroupWords = 64;    // ... and per group of it
constexpr uint32_t kTileGroup = 64;     // dense-route tiles whose counts are also kept as one sum
// A partition keeps, in LDS, 8 bytes per cell (value, meta word) and 7 and a bit per unknown (its
// packed slots, then its value; a queue entry; claimed or not): 12288 cells and 8192 unknowns
// take 153 of the 160 KiB.  (Larger ones: 10 per cell and 4 and a bit per unknown.)
constexpr uint32_t kDefaultPartCells = 12288;
constexpr uint32_t kDefaultPartUnknowns = 8192;
constexpr uint32_t kMaxPartCells = 16383;      // 16 registers of cells per decoder thread
constexpr uint32_t kMaxPartUnknowns = 16384;   // local ranks fit 14 bits
constexpr uint32_t kDecodeThreads = 1024;
constexpr uint32_t kLdsBytes = 160 * 1024;
constexpr uint32_t kMaxRanksPerPass = 32;
// A range [lo, hi) of c-indices in the pieces in which the decoder's workgroup puts its dense output
// together: n floats from c-index `at` (a multiple of 4) on.  lo < hi.
constexpr uint32_t kDensePiece = 36 * kDecodeThreads;
struct DensePieces {
    uint32_t at, n, end;
    __host__ __device__ DensePieces(uint32_t lo, uint32_t hi) : at(lo & ~3u), n(0), end(hi) { size(); }
    __host__ __device__ bool next()
    {
        if (end - at <= kDensePiece) return false;  // (a step could go past 2^32)
        at += kDensePiece;
        size();
        return true;
    }
    __host__ __device__ void size()
    {
        const uint32_t left = (end - at + 3u) & ~3u;
        n = left < kDensePiece ? left : kDensePiece;
    }
};
// Whether a decoder of `grid` workgroups writes the dense output of a partition's `len` c-indices itself, A
// partitions sharing n_c c-indices: only if there are three turns of partitions to hide it behind, and
// the partition has no more than kDenseShare times an even share.  Both depend on what the device finds: exact
// zeros are never kept, so that few partitions may be left of a large plan, and a layer of which little is
// kept is a few partitions however long it is; one workgroup stores some 30 GB/s.  (A share of 2 / 4 / 8,
// decoder and dense output, us: 2 ranks of 200 M entries in four layers with 5 to 20 % kept 627 / 593 / 594; 150 M
// with 1 % beside 50 M with 20 % 432 / 431 / 451.)
constexpr uint32_t kDenseShare = 4;
__host__ __device__ inline bool dense_by_decoder(uint32_t A, uint32_t grid, uint32_t n_c, uint32_t len)
{
    return A >= 3ull * grid && len / kDenseShare <= n_c / A;
}
// Candidate histogram of the single-read route: the bins from a segment's pre-threshold
// upwards (12 octaves of magnitude: a gradient may grow 4000-fold between two calls before
// its threshold leaves the window); then one count of everything above them, one of the
// non-finite entries, padding.
constexpr uint32_t kWinBins = 1536;
constexpr uint32_t kWinWords = 1544;

// Device copy of one compressed segment.
struct SegDev {
    uint64_t offset;      // element offset in the gradient buffer
    uint32_t n;           // elements
    uint32_t c_off;       // c-index of element 0 (multiple of 32)
    uint32_t k;           // keep count
    uint32_t tile_start;  // first compaction tile of this segment (dense path)
    uint32_t flags;       // kSegAligned | kSegFast | kSegSmall
    uint32_t sc_start;    // first super-chunk of this segment (candidate path)
};
constexpr uint32_t kSegAligned = 1;  // offset is a multiple of the 16-byte vector
constexpr uint32_t kSegFast = 2;     // eligible for the single-read candidate path
constexpr uint32_t kSegSmall = 4;    // one workgroup's registers hold the whole segment
static_assert(sizeof(SegDev) == 32, "SegDev layout");

// Result of the threshold search for one segment (device memory).  Written for every
// segment with k > 0 and n > 0: by the scan's last workgroup on the segment, by the dense
// route's selection, and (fp32) completed by the second-level selection.
struct SelDev {
    uint32_t T;       // threshold key; keep key > T, and `quota` lowest-position ties
    uint32_t quota;   // ties (key == T) to keep
    uint32_t G;       // count(key > T)
    uint32_t cnt;     // pairs this segment emits = G + min(E, quota)
    uint32_t bin1;    // fp32: level-1 bin that holds T
    uint32_t G1;      // fp32: count of keys in higher level-1 bins
    uint32_t need2;   // fp32: 1 if the low 16 bits still have to be searched
    uint32_t route;   // 0: candidate path, 1: dense path (by plan, or after a miss)
};
static_assert(sizeof(SelDev) == 32, "SelDev layout");

struct RankPtrs {
    const void *p[kMaxRanksPerPass];
};

// ------------------------------------------------------------------- plan

struct Workspace {  // byte offsets inside a rank workspace
    uint64_t hist1d, hist2, group_cnt;  // cleared by every PHASE_INDEX call before they are added to
    uint64_t sel, tile_cnt, sc_cnt, chunk_info, cand, bitmap1, total;
};

// Device state of a plan (per rank slot), kept behind the segment rows of its table: all zero after
// tagc_plan_upload, and every PHASE_INDEX call leaves it as it found it except for the
// pre-thresholds, which are what is carried from call to call.  It lives with the table and
// not in a rank workspace because nobody but the library writes the table: counters that
// have to start at zero can rely on it without a clearing pass per call.
struct TableState {
    uint32_t *hint;      // [L] pre-threshold bin for the next call, 0 = none
    uint32_t *watch;     // [L] calls that still follow the falling trend after a miss
    uint32_t *prev;      // [L] the bin above which 1.3 k entries lay at the last call
    uint32_t *arrive;    // [L] workgroups of the scan that are done with the segment
    uint32_t *arrive_d;  // [L] the same for the dense route's histogram; small_kernel: pairs of the segment + 1
    uint32_t *raised;    // [L] highest pre-threshold a wave of the scan used
    uint32_t *reroute;   // [L] a chunk overflowed its slots
    uint32_t *glob;      // [8] flags, non-finite inputs, dense-route segments of the call
    uint32_t *win;       // [L][kWinWords] candidate histograms
};
// A table holds one such state per rank slot: ranks whose work is in the same launches
// (tagc_compress_ranks) must not share counters, and each then carries its own pre-thresholds.
constexpr uint64_t table_slot_words(uint64_t L)
{
    return L * kWinWords + 8 + (7 * L + 7) / 8 * 8;
}
__host__ __device__ inline TableState table_state(uint32_t *table, uint32_t L, uint32_t slot)
{
    // behind the 32-byte rows, per slot: the histograms (a multiple of 32 bytes each), the rest
    uint32_t *w = table + 8 + 8 * size_t(L) + slot * table_slot_words(L);
    uint32_t *p = w + size_t(L) * kWinWords + 8;
    return TableState{p,         p + L,     p + 2 * L, p + 3 * L, p + 4 * L,
                      p + 5 * L, p + 6 * L, p - 8,     w};
}
static_assert(kWinWords % 8 == 0, "histograms stay 32-byte aligned");

}  // namespace tagc

struct tagc_plan_s {
    tagc_config cfg;
    std::vector<tagc_segment> segments;       // as given
    std::vector<tagc::SegDev> table;          // compressed segments only
    uint32_t elem_bytes, vec_elems;
    uint32_t compact_rows;                    // 16-byte vectors per thread per compaction tile (2 or 4)
    uint32_t tile_elems;                      // elements per compaction tile
    uint32_t total_tiles;
    uint32_t plan_tiles;                      // tiles of the segments scan_spill never reads, the first ones
    uint32_t total_sc;                        // super-chunks of the candidate path
    uint32_t chunk_elems, cand_cap;           // elements / candidate slots per chunk
    uint32_t cnt_ranges;                      // word offset of the partition ranges in a rank's cnt buffer
    bool any_nonfast;                         // some non-empty segment is never streamed by scan_spill
    bool static_dense;                        // some segment with k > 0 never takes the candidate route
    bool any_fast;                            // some segment takes it
    bool small_dense;                         // some dense-route segment is kSegSmall
    bool all_small;                           // a workgroup a segment is the faster sparsifier if there are not too many
    uint64_t span_dense;                      // entries of the dense-route segments that are not
    uint64_t dense_pairs;                     // pairs the dense-route segments emit at most
    uint64_t n_real, n_c, K, U_cap, A_cap, m_cap;
    uint32_t P_cap, T_cap;
    tagc::Workspace ws;
    uint64_t zero_bytes;                      // prefix of the rank workspace cleared per call
    uint32_t slots;                           // rank slots of the table's device state
    // rank slots that a PHASE_INDEX call has used since the table was uploaded (one bit each)
    mutable std::atomic<uint32_t> used{0xFFFFFFFFu};
    uint64_t n_chunks;                        // popcount chunks of the Index
    tagc_sizes sizes;
};

namespace tagc {

// The shared workspace: set bits before every chunk of the merged Index (and in all), set bits of
// every chunk, set bits of a chunk before each of its 16 groups of 64 words (16 bits each); then,
// when the 4-bit Index of more ranks than one pass takes is summed, the running sum.
inline uint16_t *group_prefixes(void *workspace, uint64_t n_chunks)
{
    return static_cast<uint16_t *>(workspace) + 2 * (2 * n_chunks + 1);
}
inline uint64_t index_words(uint64_t n_chunks) { return (2 * n_chunks + 1 + 8 * n_chunks + 3) & ~uint64_t(3); }

// ------------------------------------------------------------------- hash

__host__ __device__ inline uint32_t fold16(uint32_t x) { return x ^ (x >> 16); }

// mix32 behind its first step
__host__ __device__ inline uint32_t mix32_folded(uint32_t x)
{
    x *= 0x6A09E667u;
    x ^= x >> 15;
    x *= 0xBB67AE85u;
    x ^= x >> 16;
    return x;
}

__host__ __device__ inline uint32_t mix32(uint32_t x) { return mix32_folded(fold16(x)); }

__host__ __device__ inline uint32_t seed_word(uint64_t seed, uint32_t j)
{
    return mix32(uint32_t(seed) ^ mix32(uint32_t(seed >> 32) + 0x9E3779B9u * (j + 1)));
}

// slot in [0, m_sub) in the upper bits, sign flag (1 = negative) in bit 31... returned
// separately: slot via multiply-shift range reduction, sign from the low hash bit.
// The first step of mix32 is linear: fold16(i ^ sw) = fold16(i) ^ fold16(sw), so a kernel that takes
// several hash functions of an index folds the index once and the seed words once per partition
// (hash_slot_folded: two instructions less per hash function).
__host__ __device__ inline uint32_t hash_slot_folded(uint32_t fi, uint32_t fsw, uint32_t m_sub,
                                                     uint32_t *neg)
{
    const uint32_t h = mix32_folded(fi ^ fsw);
    *neg = h & 1u;
#if defined(__HIP_DEVICE_COMPILE__)
    return __umulhi(h, m_sub);
#else
    return uint32_t((uint64_t(h) * m_sub) >> 32);
#endif
}

__host__ __device__ inline uint32_t hash_slot(uint32_t i, uint32_t sw, uint32_t m_sub, uint32_t *neg)
{
    return hash_slot_folded(fold16(i), fold16(sw), m_sub, neg);
}

// ---------------------------------------------------------------- profile

void profile_begin(const char *name, hipStream_t s);
void profile_end(hipStream_t s);

struct ProfileScope {
    hipStream_t s;
    ProfileScope(const char *name, hipStream_t st) : s(st) { profile_begin(name, st); }
    ~ProfileScope() { profile_end(s); }
};

int device_cu_count();

// ------------------------------------------------------ stage entry points

int launch_sparsify(const tagc_plan_t *p, const void *const *grads, const tagc_rank_buffers *ranks,
                    uint32_t n_ranks, const tagc_shared_buffers *sh, hipStream_t s);
int launch_feedback_apply(const tagc_plan_t *p, const tagc_rank_buffers *rk,
                          const tagc_shared_buffers *sh, hipStream_t s);
int launch_encode(const tagc_plan_t *p, const tagc_rank_buffers *ranks, uint32_t n_ranks,
                  const tagc_shared_buffers *sh, hipStream_t s);
int launch_index_or(const tagc_plan_t *p, const tagc_rank_buffers *ranks, uint32_t n_ranks,
                    const tagc_shared_buffers *sh, hipStream_t s);
int launch_sketch_sum(const tagc_plan_t *p, const tagc_rank_buffers *ranks, uint32_t n_ranks,
                      const tagc_shared_buffers *sh, hipStream_t s);
int launch_decode(const tagc_plan_t *p, const tagc_shared_buffers *sh,
                  const tagc_rank_buffers *ranks, uint32_t n_ranks, uint32_t *idx_out,
                  float *val_out, float *dense_out, hipStream_t s);

size_t decode_lds_bytes(uint32_t T_cap, uint32_t P_cap);
size_t salt_lds_bytes(uint32_t T_cap, uint32_t P_cap);

// device address, on the current device, of the library's own rank workspace
// (TAGC_STATIC_WORKSPACE_BYTES); looked up on the first call per device, never allocated
int static_workspace(void **out);

// whether two ranges of device memory share a byte
inline bool overlap(const void *a, uint64_t bytes_a, const void *b, uint64_t bytes_b)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + bytes_b && y < x + bytes_a;
}

inline int hip_ok(hipError_t e) { return e == hipSuccess ? TAGC_OK : TAGC_EHIP; }

}  // namespace tagc
