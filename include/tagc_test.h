/*
 * libtagc -- exports for tests and tools only; not part of the hot path's
 * interface (that is tagc.h).
 */
#ifndef TAGC_TEST_H
#define TAGC_TEST_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Hash function j (0..2) of c-index i under partition salt `salt`, for a
 * sub-table of m_sub cells, exactly as the device code computes it (the three
 * hash functions with +-1 signs of the Count Sketch, section 2.2): slot in
 * [0, m_sub), sign +1 or -1.  Host memory only; never touches the device.
 */
void tagc_hash_host(uint32_t i, uint64_t seed, uint32_t j, uint32_t salt, uint32_t m_sub,
                    uint32_t *slot, int32_t *sign);

/*
 * The pieces in which a decoder workgroup writes the dense output of the c-indices
 * [lo, hi), lo < hi: piece i is n[i] floats from c-index at[i] on (floats before lo
 * or from hi on are not stored).  Returns how many there are; goes no further than
 * cap + 1, and writes no more than cap.  Host memory only.
 */
uint32_t tagc_dense_pieces_host(uint32_t lo, uint32_t hi, uint32_t *at, uint32_t *n, uint32_t cap);

#ifdef __cplusplus
}
#endif
#endif /* TAGC_TEST_H */
