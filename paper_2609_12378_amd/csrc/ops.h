// Launchers of the element-wise, structural, key-switching, encoding and
// projection kernels (definitions in ops.hip, keyswitch.hip, encode.hip,
// project.hip).
#pragma once
#include "ckks_internal.h"

enum { EW_ADD = 0, EW_SUB = 1, EW_MUL = 2 };

ckks_status launch_binary(ckks_ctx *ctx, uint64_t *out, const uint64_t *a, const uint64_t *b, uint32_t rows,
                          const LimbMap &map, int op);
ckks_status launch_mul_plain(ckks_ctx *ctx, uint64_t *out, const uint64_t *ct, const uint64_t *pt, uint32_t polys,
                             uint32_t limbs);
ckks_status launch_tensor(ckks_ctx *ctx, uint64_t *d0, uint64_t *d1, uint64_t *d2, const uint64_t *a,
                          const uint64_t *b, uint32_t limbs);
// `count` independent entries in one launch (at most 65535), each pointer advanced by its own stride in words
ckks_status launch_binary_batch(ckks_ctx *ctx, uint64_t *out, size_t out_stride, const uint64_t *a,
                                size_t a_stride, const uint64_t *b, size_t b_stride, uint32_t count, uint32_t rows,
                                const LimbMap &map, int op);
ckks_status launch_tensor_batch(ckks_ctx *ctx, uint64_t *d0, uint64_t *d1, uint64_t *d2, size_t d_stride,
                                const uint64_t *a, size_t a_stride, const uint64_t *b, size_t b_stride,
                                uint32_t count, uint32_t limbs);
ckks_status launch_expand_i8(ckks_ctx *ctx, uint64_t *out, const int8_t *v, const LimbMap &map);
ckks_status launch_expand_i32(ckks_ctx *ctx, uint64_t *out, const int32_t *v, const LimbMap &map);
ckks_status launch_encrypt(ckks_ctx *ctx, uint64_t *c0, uint64_t *c1, const uint64_t *a, const uint64_t *s,
                           const uint64_t *e, const uint64_t *m, const LimbMap &map);
ckks_status launch_keygen_digit(ckks_ctx *ctx, uint64_t *b_out, uint64_t *a_out, const uint64_t *a,
                                const uint64_t *s, const uint64_t *e, const uint64_t *t, uint32_t dig_lo,
                                uint32_t dig_hi);
// count entries of `words` contiguous words: entry b at src + b src_stride copied to dst_a + b a_stride and, when
// dst_b is not null, to dst_b + b b_stride (strides in words; 16-byte accesses where every pointer and stride
// allows them); count <= 65535
ckks_status launch_copy_rows(ckks_ctx *ctx, uint64_t *dst_a, size_t a_stride, uint64_t *dst_b, size_t b_stride,
                             const uint64_t *src, size_t src_stride, size_t words, uint32_t count);
// top ([polys][N], canonical mod q_l) to centred int64 in place
ckks_status launch_rescale_centre(ckks_ctx *ctx, uint64_t *top, uint32_t polys, uint32_t l);
ckks_status launch_rescale_finish(ckks_ctx *ctx, uint64_t *out, const uint64_t *c, const uint64_t *r,
                                  uint32_t polys, uint32_t l);

// key switching (keyswitch.hip)
// digits: [nd][level+1+K][N] from c ([level+1][N]), followed by stage_rows >= alpha staging rows (as ks_modup_batch)
ckks_status ks_modup(ckks_ctx *ctx, const uint64_t *c, uint32_t level, uint64_t *digits, size_t stage_rows);
// rows after the digits of `count` ciphertexts in a region of ks_scratch_words(ctx, level, batch, count) words: the
// staging rows and the rotations' own scratch, which a ModUp may use before the rotations run
inline size_t ks_stage_rows(const ckks_ctx *ctx, uint32_t level, uint32_t batch, uint32_t count)
{
    return (size_t)count * ctx->alpha + (size_t)batch * (2 * (level + 1 + ctx->n_p) + 2 * (level + 1));
}
// ModUp of `count` ciphertexts at once: c1 of ciphertext r at c1 + r * in_stride (words); digits: [count][nd][ext][N]
// followed by stage_rows staging rows: at least count * alpha; with count * (level+1) the whole-row kernels run
// where the ring has them
ckks_status ks_modup_batch(ckks_ctx *ctx, const uint64_t *c1, size_t in_stride, uint32_t count, uint32_t level,
                           uint64_t *digits, size_t stage_rows);
// out_k = (u_k - Conv(INTT([u_k]_P))) P^-1 (+ add_k), k < polys; u ([polys][level+1+K][N]) is clobbered.
// add0/add1: [level+1][N] or null, add0 read through the automorphism add0_g (1 = none);
// out: [polys][level+1][N]; work: [polys][level+1][N]
ckks_status ks_moddown(ckks_ctx *ctx, uint64_t *u, uint32_t polys, uint32_t level, const uint64_t *add0,
                       uint32_t add0_g, const uint64_t *add1, uint64_t *out, uint64_t *work);
// scratch words for rotations at `level` processed `batch` at a time (see rotate_core)
size_t ks_scratch_words(const ckks_ctx *ctx, uint32_t level, uint32_t batch, uint32_t n_ct = 1);
// rotations per batched launch for `count` requested rotations
uint32_t ks_rot_batch(uint32_t count);
// the a half [dnum][n_q + n_p][N] of the seed-expanded key with seed (s0, s1) (philox.h)
ckks_status launch_expand_key_a(ckks_ctx *ctx, uint64_t s0, uint64_t s1, uint64_t *a);
// `count` (<= 32) rotations: rotation r applies the automorphism g[r] with key keys[r] to the ciphertext whose
// c0 is c0s[r] and whose ModUp digits are digs[r] (hoisted rotations of one ciphertext share both): key inner
// product, ModDown and the sigma_{g_r}(c0) addition, each stage one launch for all r.
// work: count * (2 ext + 2 (level+1)) N words.  seeds (nullable, [count][2]): seed-expanded keys, keys[r] then holds
// the b half [dnum][n_q + n_p][N] and the a half comes from seeds[2r], seeds[2r + 1] (philox.h).  add1 (nullable):
// add1[r] ([level+1][N]) is added to the second component of output r
ckks_status ks_rotate_batch(ckks_ctx *ctx, uint32_t level, uint32_t count, const uint64_t *const *c0s,
                            const uint64_t *const *digs, const uint32_t *g, const uint64_t *const *keys,
                            uint64_t *const *outs, uint64_t *work, const uint64_t *seeds = nullptr,
                            const uint64_t *const *add1 = nullptr);

// lazy ModDown: accs[r mod n_accs] ([2][level+1+K][N]) (+)= the key inner product of
// rotation r over Q_level u P plus P * sigma_{g_r}(c0_r) on the q rows; count <= 32.  ks_moddown of the accumulator
// then gives the sum of the rotations.
ckks_status ks_ip_accumulate(ckks_ctx *ctx, uint32_t level, uint32_t count, const uint64_t *const *c0s,
                             const uint64_t *const *digs, const uint32_t *g, const uint64_t *const *keys,
                             uint64_t *const *accs, uint32_t n_accs, bool accumulate);

// Row passes with the element-wise work that follows the transform (fused_row.hip): N >= 2^12, either arithmetic.
bool fused_rows_ok(const ckks_ctx *ctx);
// rescale of `polys` polynomials c ([polys][l+1][N]) into out ([polys][l][N]) or, out null, of polys / 2 <= 32
// ciphertexts into outs[r] ([2][l][N]); work: polys (1 + l) N words
ckks_status fused_rescale(ckks_ctx *ctx, const uint64_t *c, uint32_t polys, uint32_t l, uint64_t *out,
                          uint64_t *const *outs, uint64_t *work);
// the last step of a rotation batch in the integer arithmetic: u [count][2][level+1+n_p][N], cw [count][2][level+1][N]
// after the column pass
struct RotArgs;
ckks_status fused_moddown_int(ckks_ctx *ctx, uint32_t level, const RotArgs &ra, const uint64_t *u, const uint64_t *cw);
// work: limbs N words, 2 limbs N words
ckks_status fused_decrypt(ckks_ctx *ctx, uint64_t *pt, const uint64_t *c0, const uint64_t *c1, const int8_t *s,
                          uint32_t limbs, uint64_t *work);
ckks_status fused_encrypt(ckks_ctx *ctx, uint64_t *c0, uint64_t *c1, const uint64_t *a, const int8_t *s,
                          const int32_t *e, const uint64_t *m, uint32_t limbs, uint64_t *work);

// ModUp and ModDown conversions in fp64 (modup.hip): N >= 2^12, at most 16 source limbs a conversion whose constants
// are exact in fp64
bool up_conv_ok(const ckks_ctx *ctx, const ConvDev *cd);
// every prime of the level and of P below 2^50 and every conversion of the level such (computed once per context:
// ckks_ctx::f64_level)
bool f64_level_ok(const ckks_ctx *ctx, uint32_t level);
inline bool f64_switch(const ckks_ctx *ctx, uint32_t level)
{
    return !ctx->int_only && level < ctx->f64_level.size() && ctx->f64_level[level];
}
// ModUp of `count` polynomials at c1 + r stride into digits [count][nd][level+1+n_p][N]; needs no other memory
ckks_status up_modup(ckks_ctx *ctx, const uint64_t *c1, size_t stride, uint32_t count, uint32_t level,
                     uint64_t *digits);
// up: [polys][n_p][N] rows modulo P after the row pass of their inverse transform (raw doubles below 2q): finishes it,
// converts to the level's q limbs and runs the first forward pass into cw ([polys][level+1][N] raw doubles)
ckks_status up_moddown(ckks_ctx *ctx, uint64_t *up, uint32_t polys, uint32_t level, uint64_t *cw);

// Whole rows per block (ring_block.hip): fp64 primes, N = 2^12 and 2^13, at 2^14 for launches of many rows.
// the ring has them and the fp64 arithmetic is not switched off
bool blk_ring(const ckks_ctx *ctx);
// they are the faster transform for a launch of `rows` rows, the faster rescale to `rows` rows in all, the faster
// transform of signed coefficients
bool blk_rows(const ckks_ctx *ctx, size_t rows);
bool blk_rescales(const ckks_ctx *ctx, size_t rows);
bool blk_from_i64(const ckks_ctx *ctx);
// they are the faster encryption and decryption of `limbs` limbs
bool blk_crypt(const ckks_ctx *ctx, uint32_t limbs);
// they are the faster ModUp and key switching at `level`
bool blk_switch(const ckks_ctx *ctx, uint32_t level);
// they are the faster ModDown of `polys` polynomials at `level`
bool blk_moddowns(const ckks_ctx *ctx, uint32_t level, uint32_t polys);
// transform of `batch` groups of map.n rows from src (group stride src_stride rows) to dst; dst may be src
ckks_status blk_ntt(ckks_ctx *ctx, uint64_t *dst, uint32_t dst_stride, const uint64_t *src, uint32_t src_stride,
                    uint32_t batch, const LimbMap &map, bool inverse);
ckks_status blk_ntt_from_i64(ckks_ctx *ctx, const int64_t *m, uint64_t *out, uint32_t batch, uint32_t limbs);
ckks_status blk_encrypt(ckks_ctx *ctx, uint64_t *c0, uint64_t *c1, const uint64_t *a, const int8_t *s,
                        const int32_t *e, const uint64_t *m, uint32_t limbs);
ckks_status blk_decrypt(ckks_ctx *ctx, uint64_t *pt, const uint64_t *c0, const uint64_t *c1, const int8_t *s,
                        uint32_t limbs);
// rescale of `polys` polynomials c ([polys][l+1][N]) into out ([polys][l][N]); work: polys N words
ckks_status blk_rescale(ckks_ctx *ctx, const uint64_t *c, uint32_t polys, uint32_t l, uint64_t *out, uint64_t *work);
// ModUp of `count` polynomials at c1 + r stride, or (b set, count 1) of the product of the second components of the
// ciphertexts whose second components start at c1 and at b + (level+1) N; stage: count (level+1) N words
ckks_status blk_modup(ckks_ctx *ctx, const uint64_t *c1, size_t stride, const uint64_t *b, uint32_t count,
                      uint32_t level, uint64_t *digits, uint64_t *stage);
// a rotation batch; with ta, tb2 (ciphertexts) the addends are the first two components of their tensor product.
// work: count 2 (level+1+n_p) N words
struct RotArgs;
ckks_status blk_rotate_batch(ckks_ctx *ctx, uint32_t level, const RotArgs &ra, uint64_t *work,
                             const uint64_t *ta = nullptr, const uint64_t *tb2 = nullptr);
// as ks_moddown
ckks_status blk_moddown(ckks_ctx *ctx, uint64_t *u, uint32_t polys, uint32_t level, const uint64_t *add0,
                        uint32_t add0_g, const uint64_t *add1, uint64_t *out);
// a, b [2][level+1][N]: out = a b relinearised with rlk, every step in the kernels above; out must overlap neither
// input.  work: ks_scratch_words(level, 1) words
ckks_status ks_mul_relin_blk(ckks_ctx *ctx, const uint64_t *a, const uint64_t *b, const uint64_t *rlk, uint32_t level,
                             uint64_t *out, uint64_t *work);

// encoding (encode.hip)
struct SlotSource {
    // explicit slots: re/im [batch][N/2] (im may be null)
    const double *re = nullptr, *im = nullptr;
    // or the projection's weight plaintexts, generated from W (d_in x d_out, row-major):
    // plaintext p of the batch is (output block j0 + (p / pairs) % jc, pair ib0 + p % pairs), where
    // pair = i * bcount + b names input block i and baby step b of giant step g (n1g = n1 * g)
    const double *W = nullptr;
    uint32_t d_out = 0, tokens = 0, feats = 0;
    uint32_t n1g = 0, bcount = 0;
    // several giant steps in one batch: plaintext p belongs to block jr = p / pairs, output j0 + jr % jc of giant step
    // g + jr / jc (n1g + n1 (jr / jc))
    uint32_t jc = 1, n1 = 0;
    uint32_t j0 = 0, ib0 = 0, pairs = 1;
    // optional, for feats <= 256 and N >= 2^12: W re-laid as its cyclic diagonals,
    // Wd[((jb * n_in + i) * D + k) * D + o] = D_k(A_{jb,i})[o], and feat_of_pos[x] = (slot at FFT position x) / tokens
    const double *Wd = nullptr;
    const uint32_t *feat_of_pos = nullptr;
    uint32_t n_in = 0;
};
// m_out: [batch][N] int64 rounded coefficients; work: [batch][N/2] double2
ckks_status enc_coeffs(ckks_ctx *ctx, const SlotSource &src, uint32_t batch, double scale, double2 *work,
                       int64_t *m_out);
// encoding of a projection sub-batch fused with the first NTT pass (N = 2^16, fp64 primes 0..limbs-1):
// FFT pass A into work, then pass B, twist, rounding and the column transforms of every limb in one kernel;
// out: [batch][limbs][N] in the inter-pass form of launch_ntt_col_i64
bool enc_fused_ok(const ckks_ctx *ctx, uint32_t limbs);
// bound below which the fp64 range reduction modulo every prime q_0 .. q_{limbs-1} is the identity
int64_t identity_reduction_bound(const ckks_ctx *ctx, uint32_t limbs);
ckks_status enc_ntt_first_pass(ckks_ctx *ctx, const SlotSource &src, uint32_t batch, double scale, double2 *work,
                               uint32_t limbs, uint64_t *out);
// out[x] = (slot index held at FFT position x) / tokens, x < N/2
ckks_status enc_feat_of_pos(ckks_ctx *ctx, uint32_t tokens, uint32_t *out);
// residues of m ([batch][N]) into out ([batch][limbs][N]), primes 0..limbs-1
ckks_status enc_to_rns(ckks_ctx *ctx, const int64_t *m, uint32_t batch, uint32_t limbs, uint64_t *out);
size_t enc_work_bytes(const ckks_ctx *ctx, uint32_t batch);
size_t proj_workspace_bytes(const ckks_ctx *ctx, uint32_t L, uint32_t tokens, uint32_t d_in, uint32_t d_out,
                            uint32_t n1);
size_t proj_tm_workspace_bytes(const ckks_ctx *ctx, uint32_t L, uint32_t tokens, uint32_t d_in, uint32_t d_out,
                               uint32_t n1);
size_t attn_scores_workspace_bytes(const ckks_ctx *ctx, uint32_t L, uint32_t tokens, uint32_t head_dim);
size_t attn_apply_workspace_bytes(const ckks_ctx *ctx, uint32_t Lp, uint32_t Lv, uint32_t tokens, uint32_t head_dim);

// projection helpers (project.hip): W's cyclic diagonals Wd[((jb * n_in + i) * D + k) * D + o] =
// W[(i D + (k + o) mod D) * d_out + jb D + o]; canonical residues -> the same integers as doubles, in place
ckks_status launch_diag_layout(ckks_ctx *ctx, double *Wd, const double *W, uint32_t D, uint32_t n_in,
                               uint32_t d_out);
ckks_status launch_to_f64(ckks_ctx *ctx, uint64_t *v, size_t words);

// ciphertext-level steps shared by the API calls and the projections (api_ops.hip)
// The gc giant steps g, g + 1, ... of a projection's tile of jc outputs, their partial sums at acc ([gc][jc]
// ciphertexts): that of step 0 to tot ([jc]), the others rotated by step * (g + gg) with gkeys[g + gg] and added to
// tot, or (lazy) their key-switching sums to uacc ([jc][2][level+1+n_p][N]).  rot: gc jc ciphertexts; work:
// ks_scratch_words(ctx, level, ks_rot_batch(gc jc), gc jc) words; jc <= 32
ckks_status giant_steps(ckks_ctx *ctx, const uint64_t *acc, uint64_t *tot, uint64_t *rot, uint64_t *uacc, uint32_t jc,
                        uint32_t g, uint32_t gc, int32_t step, const uint64_t *const *gkeys, uint32_t level, bool lazy,
                        uint64_t *work);
// rotations of one ciphertext sharing a single ModUp; work: ks_scratch_words(level, ks_rot_batch(count))
ckks_status rotate_core(ckks_ctx *ctx, const uint64_t *c, uint32_t level, const int32_t *steps,
                        const uint64_t *const *keys, uint32_t count, uint64_t *const *outs, uint64_t *work,
                        const uint64_t *seeds = nullptr);
// rescale of one ciphertext at level l; work: (2 + 2 l) N words
ckks_status rescale_core(ckks_ctx *ctx, const uint64_t *c, uint32_t l, uint64_t *out, uint64_t *work);
// `count` ciphertexts (at cs + r * stride) each rotated by its own step with its own key; one batched ModUp.
// work: ks_scratch_words(ctx, level, ks_rot_batch(count), count) words
ckks_status rotate_each(ckks_ctx *ctx, const uint64_t *cs, size_t stride, uint32_t count, uint32_t level,
                        const int32_t *steps, const uint64_t *const *keys, uint64_t *const *outs, uint64_t *work);
// rescale of `count` contiguous ciphertexts c ([count][2][l+1][N]) into out ([count][2][l][N]);
// work: 2 count (1 + l) N words
ckks_status rescale_many(ckks_ctx *ctx, const uint64_t *c, uint32_t count, uint32_t l, uint64_t *out,
                         uint64_t *work);
// the same into separate outputs outs[r] ([2][l][N]); count <= 32
ckks_status rescale_each(ckks_ctx *ctx, const uint64_t *c, uint32_t count, uint32_t l, uint64_t *const *outs,
                         uint64_t *work);

// matrix-core multiply-accumulate over residues (project_tm.hip): acc[jj] (+)= sum_kappa Q[kappa][jj] x_kappa for
// jj < jc and the K ciphertexts kappa_base .. kappa_base + K - 1 of a digit layout Xd, per limb l and run x of
// 2^logT positions: Q is [L][D2][K][jc] canonical residues as doubles (D2 runs), acc [jc][2][L][N] canonical.
uint32_t mac_kt_pad(uint32_t kt);
size_t mac_digit_bytes(const ckks_ctx *ctx, uint32_t L, uint32_t kt_pad);
uint32_t mac_max_outputs();
// x2 ([kt][2][L][N] canonical) -> Xd, the digit layout of kt ciphertexts (mac_digit_bytes bytes)
ckks_status launch_xdigits(ckks_ctx *ctx, const uint64_t *x2, int8_t *Xd, uint32_t L, uint32_t kt, uint32_t kt_pad);
ckks_status launch_mac_mfma(ckks_ctx *ctx, uint64_t *acc, const int8_t *Xd, const double *Q, uint32_t jc, uint32_t K,
                            uint32_t kbase, uint32_t kt_pad, uint32_t D2, uint32_t L, uint32_t logT, bool accumulate);
// periodic plaintexts of `count` explicit period vectors U ([count][D]) at scale delta: Q[l][x][pt] (x < 2D) holds
// plaintext pt's NTT values on run x (positions x N/2D ..) modulo q_l, l < L, as doubles
ckks_status launch_enc_vectors(ckks_ctx *ctx, const double *U, uint32_t D, uint32_t count, double delta, uint32_t L,
                               double *Q);

// Lazy sums of rotations (one ModDown per output): ciphertext r (at cs + r * stride) rotated by steps[r] with keys[r]
// is added to accumulator uacc + (r mod n_accs) * 2 ext N; accumulate = false starts the accumulators.  count is a
// multiple of n_accs <= 32.  work: ks_scratch_words(ctx, level, ks_rot_batch(count), count) words
ckks_status rotate_each_lazy(ckks_ctx *ctx, const uint64_t *cs, size_t stride, uint32_t count, uint32_t level,
                             const int32_t *steps, const uint64_t *const *keys, uint64_t *uacc, uint32_t n_accs,
                             bool accumulate, uint64_t *work);

// decode: coef = coefficient form of limbs 0..min(limbs,2)-1 ([limbs][N]); writes N/2 slots
ckks_status dec_slots(ckks_ctx *ctx, const uint64_t *coef, uint32_t limbs, double scale, double2 *work, double *re,
                      double *im);
