/*
 * kvtc_test_hooks.h -- internal: exports of the library that let tests run, for the most part without a GPU, the
 * scalar quantiser numerics (csrc/kvtc_numeric.h: the directed fp32 -> fp16 roundings of the shared
 * shift (down) and scale (up), paper Section "Quantization", the group header, and the code decision
 * for one value) and the rules by which a call's route is chosen.  Not part of the coder's API;
 * applications include kvtc.h only.
 */
#ifndef KVTC_TEST_HOOKS_H
#define KVTC_TEST_HOOKS_H

#include <stdint.h>
#include "kvtc.h"

#ifdef __cplusplus
extern "C" {
#endif

uint16_t kvtc_host_f16_round_down(float x);
uint16_t kvtc_host_f16_round_up(float x);
void kvtc_host_group_header(float lo, float hi, int bits, uint16_t* shift16, uint16_t* scale16);
uint32_t kvtc_host_code(float d, uint16_t shift16, uint16_t scale16, int bits);

/* 1: a feature array at this address lies on whole cache lines, so a large one is read or written past the
 * caches; 0: it does not, so none is; -1: the library refuses the array. */
int kvtc_host_whole_lines(uint64_t x_address, kvtc_dtype dtype, int p, const kvtc_layout* layout);

/* Bytes of a call's features from which on its encode reads them past the caches, for a plan that runs as this many tiles of
 * 32 coordinates (2, 4, 6, 8, 10, 12, 16, 20, 24 or 32); UINT64_MAX: never. */
uint64_t kvtc_host_encode_pass_bytes(int tiles, kvtc_dtype dtype);

/* Bytes of a call's output from which on its decode stores past the caches, for plans of this many tiles of 32 coordinates whose
 * bases have this many bytes together, in one tensor's call (single) or a batch; UINT64_MAX: never. */
uint64_t kvtc_host_decode_pass_bytes(int tiles, kvtc_dtype dtype, uint64_t bases, int single);

/* On the GPU, over all fp32 bit patterns: adds to counts_dev[0] how many of them are numbers, and to [1], [2] and [3] how many
 * roundings to fp16, group headers and codes of this many bits come out differently as the kernels work them out and as the
 * kvtc_host_* functions do. */
kvtc_status kvtc_test_numeric(int bits, uint64_t* counts_dev, kvtc_stream stream);

/* On the GPU: *passes_dev = 1 if a launch over these jobs takes a call's features, tokens times features over all jobs that
 * are valid, for `elements` or more, else 0. */
kvtc_status kvtc_test_batch_passes(const kvtc_batch* batch, const kvtc_job* jobs_dev, int n_jobs, const uint64_t* offsets_dev, size_t stream_bytes,
                                   uint64_t elements, uint32_t* passes_dev, kvtc_stream stream);

#ifdef __cplusplus
}
#endif
#endif /* KVTC_TEST_HOOKS_H */
