// Arguments of a batch of key-switched rotations and the access to its keys, shared by the key-switching kernels.
#pragma once
#include "ckks_internal.h"
#include "ntt_core.h"
#include "philox.h"

constexpr int kRotBatch = 32;  // rotations per batched launch

// the NTT-domain position that sigma_g moves to position j: 2 brev(j') + 1 = (2 brev(j) + 1) g mod 2N
__device__ __forceinline__ uint32_t auto_index(uint32_t j, uint32_t g, uint32_t log_n)
{
    const uint32_t two_n_mask = (2u << log_n) - 1;
    const uint32_t k = 2u * (__brev(j) >> (32 - log_n)) + 1u;
    const uint32_t kg = (uint32_t)(((uint64_t)k * g) & two_n_mask);
    return __brev((kg - 1u) >> 1) >> (32 - log_n);
}

// Batched rotations: rotation r of the batch uses Galois element g[r], key
// key[r], the ModUp digits dig[r] and c0[r] of its input, and writes out[r];
// hoisted rotations of one ciphertext share dig and c0.
struct RotArgs {
    uint32_t count;
    uint32_t g[kRotBatch];
    const uint64_t *key[kRotBatch];
    uint64_t *out[kRotBatch];
    const uint64_t *dig[kRotBatch];  // ModUp digits [nd][ext][N] of the rotated ciphertext
    const uint64_t *c0[kRotBatch];   // its c0 [level+1][N]
    const uint64_t *add1[kRotBatch]; // added to the second component ([level+1][N]; null: nothing)
    // seed-expanded keys (the SEEDED kernels): key[r] is the b half [nd][key_rows][N] and seed[r] the seed of a
    uint64_t seed[kRotBatch][2];
};

// Where rotation r's key words for digit j, key row `krow`, position `pos` come from: b (and, stored, a) from the
// key; a seed-expanded key computes a (q = the row's modulus) from its seed, four digits per Philox block.
template <bool SEEDED>
struct KeyRow {
    const uint64_t *key;
    size_t kstride;      // words between the b and a halves (stored keys)
    uint32_t key_rows, log_n, prime, pos, shift;
    uint64_t q, s0, s1;
    uint64_t blk[4];
    __device__ KeyRow(const RotArgs &ra, uint32_t r, uint32_t key_rows_, uint32_t log_n_, uint32_t prime_,
                      uint32_t pos_, uint64_t q_)
        : key(ra.key[r]), kstride((size_t)key_rows_ << log_n_), key_rows(key_rows_), log_n(log_n_), prime(prime_),
          pos(pos_), shift(seedk::shift_of(q_)), q(q_), s0(ra.seed[r][0]), s1(ra.seed[r][1])
    {
    }
    __device__ uint64_t b(uint32_t j) const
    {
        const size_t row = SEEDED ? (size_t)j * key_rows + prime : (size_t)j * 2 * key_rows + prime;
        return nttc::ld_stream(key + (row << log_n) + pos);
    }
    __device__ uint64_t a(uint32_t j)
    {
        if (!SEEDED) return nttc::ld_stream(key + (((size_t)j * 2 * key_rows + prime) << log_n) + kstride + pos);
        const uint32_t m = j & 3;
        if (m == 0) seedk::block_residues(s0, s1, pos, prime, j >> 2, q, shift, blk);
        return m == 0 ? blk[0] : m == 1 ? blk[1] : m == 2 ? blk[2] : blk[3];
    }
};
