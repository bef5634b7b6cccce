// Shared by the encoder's two forms (icq_encode.hip, icq_encode_wave.hip).
#pragma once
#include "icq_internal.h"

// 32-wide slices the codewords' halves have (zero beyond d): the numbers encode_wave_kernel is made for, above 512
// dimensions no spare ones.
static inline int icq_enc_slices(int d_pad) {
    const int n = (d_pad + 31) / 32;
    return n <= 4 || n > 16 ? n : n <= 6 ? 6 : n <= 8 ? 8 : n <= 12 ? 12 : 16;
}
// Whether encode_wave_kernel takes every call on such codebooks; then nothing reads the halves' remainders.
static inline bool icq_enc_wave_only(int d_pad) { return d_pad <= 128; }

// 2^(bits - e) with e the smallest integer for which x < 2^e (clamped): x times this is below 2^bits
__device__ __forceinline__ float icq_enc_scale_below(float x, int bits) {
    const int e = (int)((__float_as_uint(x) >> 23) & 255u) - 126;
    int f = bits - e + 127;
    f = f < 67 ? 67 : f > 187 ? 187 : f;                   // 2^-60 .. 2^60: products of two scales stay finite
    return __uint_as_float((uint32_t)f << 23);
}

// At most 16 slices.  icm: coordinate descent from the codes there, else greedy assignment (sweeps = 1).  res [N][d_pad].
int icq_launch_encode_wave(const icq_index *ix, const float *x, int64_t N, uint8_t *codes, bool icm, int sweeps,
                           float *res, uint32_t *changed, hipStream_t s);
