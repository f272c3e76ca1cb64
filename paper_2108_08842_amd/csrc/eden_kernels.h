// Host-callable launchers of the EDEN kernels (all asynchronous on the given stream).
#ifndef EDEN_KERNELS_H
#define EDEN_KERNELS_H

#include "eden.h"
#include "eden_device.h"

namespace eden {

// Encode runs the contiguous pass first (it reads x) and the strided passes after it, the last one quantizing and
// packing; decode runs the strided passes first (the first one unpacks) and the contiguous pass last (it sums the
// senders into acc).  Launchers of kernels that leave per-workgroup partial sums return how many partials each
// sender got.

// wave-tile passes (eden_kernels.hip)
// `d` with a `pre` flag next to it is the caller's dimension; pre != 0 (b = 1/2 with the sparsification before the
// rotation) means the transformed vector has dimension ceil(d/2).  Every other `d` is the transformed dimension.
// `tail`: see EncTail (eden_device.h)
uint32_t launch_enc_hi_last(int M, const EncBatch &B, uint32_t n, uint64_t valid_elems, int log2D, int p, uint64_t seed,
                            const float *T, double *partials, uint32_t partial_stride, const CoinTables &ct, const EncTail &tail,
                            hipStream_t st);
// coin budgets (multi-pass sizes): the coins of the senders that have such a budget, with their prefix sums; `part_b`
// (encode) points at the second part of every such sender's payload, which is cleared; null on the receiver's side
void launch_coin_pack(const uint32_t *b_q8, const uint32_t *const *pieces, void *const *part_b, uint32_t n, int log2D,
                      const CoinTables &ct, hipStream_t st);
// `scan` = false: the caller's launch_enc_norm or launch_dec_prepare adds the groups' totals up
void launch_coin_tables(const uint32_t *clients, const uint32_t *b_q8, void *const *part_b, uint32_t n, uint64_t seed, int log2D,
                        const CoinTables &ct, bool scan, hipStream_t st);
// wide strided tiles (8 rows x 512 columns per wave) for the top three index bits of D >= 2^25, one-byte budgets only
uint32_t launch_enc_wide_last(const EncBatch &B, uint32_t n, uint64_t valid_elems, int log2D, const float *T, double *partials,
                              uint32_t partial_stride, const EncScratch *scratch, hipStream_t st);
void launch_dec_wide_first(const DecBatch &B, uint32_t n, uint64_t keep_elems, int log2D, const DecScratch *scratch, float *T,
                           hipStream_t st);
void launch_enc_norm(const EncBatch &B, uint32_t n, const double *partials, uint32_t partial_stride, uint32_t nparts,
                     EncScratch *scratch, const DevTables *tab, int log2D, const CoinTables *coins /* not null: their scan too */, hipStream_t st);
void launch_enc_finish(const EncBatch &B, uint32_t n, uint64_t hdr_d, int log2D, uint64_t seed,
                       const double *partials_n2, uint32_t nparts_n2, const double *partials_ip, uint32_t nparts_ip,
                       uint32_t partial_stride, uint32_t *dev_status, const uint32_t *coin_total, hipStream_t st);
void launch_dec_prepare(const DecBatch &B, uint32_t n, uint64_t hdr_d, int log2D, uint64_t seed, const DevTables *tab,
                        DecScratch *scratch, uint32_t *dev_status, const CoinTables &ct, bool scan, uint32_t *msg_flags,
                        hipStream_t st);
// Does the work of launch_dec_prepare itself.  `narrow`: the slots of b <= 1 senders hold 0 = values, 1 = the integers before the scale
// as fp16, 2 = as fp32
void launch_dec_hi_first(int M, const DecBatch &B, uint32_t n, uint64_t keep_elems, int log2D, int p, uint64_t seed,
                         const DecPrepareArgs &prep, int narrow, float *T, const CoinTables &ct, hipStream_t st);
// pre: 0 = sum the senders into acc; 1 = the same with the pairs scatter of EDEN_B_HALF_PRE; 2 = no sum, every sender's
// decoded vector goes back into its own workspace slot.  The workspace is fp32; for pre 0 and 1 the slots of b <= 1 senders hold
// integers (`narrow` = 2 of launch_dec_hi_first).  mean_n > 0: acc is written with the sum divided by mean_n.
void launch_dec_lo_last(const DecBatch &B, uint32_t n, uint64_t d, int pre, int log2D, uint64_t seed, float *T,
                        const DecScratch *scratch, float *acc, float mean_n, hipStream_t st);
void launch_finalize_mean(const float *acc, uint64_t d, uint32_t n, float *mean, hipStream_t st);
// D <= 4096 (eden_kernels_small.hip): one launch per direction.
// `msg_flags` (may be null): one status word per message of the launch, written by the kernel that checks the headers.
// `pre` as in launch_dec_lo_last (2: into `slots`); `partial`: room for n * (output length of a sender) floats, used when the
// senders do not fit one workgroup; `arrived`: kDecCounters counters that are 0 between launches, `turn`: the one of this
// launch (the next one of the context for every launch); mean_n > 0: acc is written with the sum divided by mean_n instead of added to.
void launch_enc_small(const EncBatch &B, uint32_t n, uint64_t d, int pre, uint64_t hdr_d, int log2D, uint64_t seed,
                      const DevTables *tab, uint32_t *dev_status, hipStream_t st);
void launch_dec_small(const DecBatch &B, uint32_t n, uint64_t d, int pre, uint64_t hdr_d, int log2D, uint64_t seed,
                      const DevTables *tab, float *acc, float mean_n, float *slots, float *partial, uint32_t *arrived, uint32_t turn,
                      uint32_t *dev_status, uint32_t *msg_flags, hipStream_t st);
// b = m/64 (eden_kernels_sparse.hip): the kept coordinates of every x_c (m per block of 64) packed into out + (c << log2_stride),
// and added back from there into acc, sender by sender; mean_n > 0: acc is written with the sum divided by mean_n instead
void launch_sparse_gather(const EncBatch &B, uint32_t n, uint64_t d, uint32_t m, uint64_t seed, float *out, int log2_stride, hipStream_t st);
void launch_sparse_scatter(const DecBatch &B, uint32_t n, uint64_t d, uint32_t m, uint64_t seed, const float *in, int log2_stride,
                           float *acc, float mean_n, hipStream_t st);
// b = 5, 6, 7: one-byte indices (B.codes[c], null for other senders) <-> the packed payload
void launch_pack_bits(const EncBatch &B, uint32_t n, int log2D, hipStream_t st);
void launch_unpack_bits(const DecBatch &B, uint32_t n, int log2D, uint8_t *codes_all, hipStream_t st);
void launch_fill_zero(float *p, uint64_t count, hipStream_t st);
// dst[i] = src_host[i], i < count <= kArgDoubles: the values travel as kernel arguments (no copy is staged)
constexpr int kArgDoubles = 256;
void launch_store_doubles(const double *src_host, uint32_t count, double *dst, hipStream_t st);
void launch_byte_entropy(const uint8_t *bytes, uint64_t count, uint32_t *hist, double *out, hipStream_t st);
void launch_sq_error(const float *a, const float *b, uint64_t d, double *partials, uint32_t max_parts, double *out,
                     hipStream_t st);
void launch_hash_bits(uint64_t key, uint64_t nwords, uint64_t *out, hipStream_t st);
void launch_loss_bitmap(uint64_t key, uint32_t npk, uint32_t drop_q32, uint32_t *bitmap, hipStream_t st);

// workgroup-tile strided passes for D >= 2^21: M bits on top of a contiguous pass over P bits (eden_kernels_wg.hip,
// eden_kernels_wg_dec.hip)
uint32_t launch_enc_hix_last(int M, int P, int blocked, const EncBatch &B, uint32_t n, uint64_t d, int log2D, uint64_t seed, const float *T,
                             double *partials, uint32_t partial_stride, const EncScratch *scratch, const CoinTables &ct,
                             hipStream_t st);
void launch_hix_mid(int M, uint32_t n, float *T, int log2D, uint64_t load_elems, uint64_t store_elems, hipStream_t st);
bool launch_dec_hix_first(int M, int P, const DecBatch &B, uint32_t n, uint64_t d, int log2D, uint64_t seed,
                          const DecScratch *scratch, int narrow, float *T, const CoinTables &ct, const DecPrepareArgs *prep,
                          uint32_t compute_units, hipStream_t st);
// whether launch_dec_hix_first would do so for this batch
bool dec_hix_first_prepares(int M, int P, const DecBatch &B, uint32_t n, int narrow);

// 12- and 14-bit contiguous passes for D <= 2^24 (eden_kernels_lo14.hip)
// `blocked` (P = 14): write the workspace in the blocked layout (eden_device.h: blocked_offset) that launch_enc_hix_last reads
// when told so; not for a first pass that works in place on the workspace
// `compute_units`: of the device; a launch that gives every workgroup one of its own takes more waves per workgroup
uint32_t launch_enc_lo_first(int P, const EncBatch &B, uint32_t n, uint64_t d, int pre, int blocked, int log2D, uint64_t seed, float *T,
                             double *partials, uint32_t partial_stride, const EncTail &tail, uint32_t compute_units, hipStream_t st);
// `resident`: workgroups of the kernel the device holds at once (2 per CU); `partial`: room for `partial_tiles`
// tiles of 2^14 floats, used when tiles are split over several workgroups by sender.
// `mean_n` > 0 (pre == 0 only): acc is not read; acc[i] = (0 + the sum over the senders) / mean_n
// pre == 2: sender c's decoded vector goes to out + (c << log2D); that may be T itself unless `narrow` (fp16 slots)
void launch_dec_lo14_last(const DecBatch &B, uint32_t n, uint64_t d, int pre, int log2D, uint64_t seed, const float *T,
                          const DecScratch *scratch, int narrow, float *acc, float *out, uint32_t resident, float *partial,
                          uint32_t partial_tiles, float mean_n, hipStream_t st);

// 15- and 16-bit contiguous passes for D = 2^25 .. 2^27 (eden_kernels_lo15.hip): the encoder's always writes the blocked layout,
// the decoder's takes every b <= 1 sender's slot as fp16; pre == 2 (one output per sender) does not exist here
uint32_t launch_enc_lo15_first(int P, const EncBatch &B, uint32_t n, uint64_t d, int pre, int log2D, uint64_t seed, float *T,
                               double *partials, uint32_t partial_stride, uint32_t compute_units, hipStream_t st);
void launch_dec_lo15_last(int P, const DecBatch &B, uint32_t n, uint64_t d, int pre, int log2D, uint64_t seed, const float *T,
                          const DecScratch *scratch, float *acc, float mean_n, uint32_t compute_units, hipStream_t st);

}  // namespace eden
#endif
