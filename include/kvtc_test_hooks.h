/*
 * kvtc_test_hooks.h -- internal: exports of the library that let tests run, without a GPU, the
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

#ifdef __cplusplus
}
#endif
#endif /* KVTC_TEST_HOOKS_H */
