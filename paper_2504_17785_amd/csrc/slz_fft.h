// Exact negacyclic products through double-precision complex transforms: the pieces shared by the host code, the key
// preparation and the N = 512, 1024, 2048 and 4096 blind rotations.
//
// A key word is cut into SLZ_FFT_PIECES balanced digits of SLZ_FFT_PIECE_BITS bits, w = sum_j K_j 2^(13 j) mod 2^64 with
// |K_j| <= 2^12 (N = 512, whose bases are smaller: three digits of 22 bits).  For every piece the integer polynomial y_j = sum_r d_r K_(r,j) mod X^N + 1 (d_r: gadget digits) is
// computed with floating-point transforms of N / 2 complex points (coefficients c and c + N/2 as real and imaginary part,
// evaluated at the roots of Z^(N/2) = i) and rounded to the nearest integer.  slz_fft_error_bound proves for every input
// that the error before rounding is below 1/2, so the rounded y_j, and with them sum_j y_j 2^(13 j) mod 2^64, are exact.
#pragma once
#include "slz_internal.h"

#define SLZ_FFT_PIECES 5
#define SLZ_FFT_PIECE_BITS 13

// Tables of the N = 2048 kernels (complex entries; device memory, built by slz_fft_init).  M = 1024 points; W(m, b) is the
// twiddle of block b at the forward stage with m blocks: the square root of the constant of that block's Z^n = c.
//   F2 [15][16]      forward strides 32/16 (v, v^2, v^3) and 8/4 (four blocks of three), by the four top position bits
//   F3 [2][6][64]    forward strides 2/1, by (top bit, lane): two blocks of three
//   I2 [8][8]        inverse half-sizes 8..64, by the three lowest position bits, as (cos, tan)
//   I3 [19][64]      inverse half-sizes 128 (1), 256 (2) as (cos, tan); 512: eight (c1, c2) pairs, c1 = psi^-j plain, c2 = psi^-j w as (cos, tan)
#define FFT_F2_OFF 0u
#define FFT_F2_LEN (15u * 16u)
#define FFT_I2_OFF (FFT_F2_OFF + FFT_F2_LEN)
#define FFT_I2_LEN (8u * 8u)
#define FFT_I3_OFF (FFT_I2_OFF + FFT_I2_LEN)
#define FFT_I3_LEN (19u * 64u)
#define FFT_LDS_TAB (FFT_I3_OFF + FFT_I3_LEN)          // everything up to here is staged in LDS
#define FFT_F3_OFF FFT_LDS_TAB
#define FFT_F3_LEN (2u * 6u * 64u)
// eight waves per ciphertext (slz_fft2048_team.hip), offsets from FFT_T_OFF:
//   T2 [3][4]        inverse half-sizes 4 and 8 as one radix-4 layer (v, v^2, v^3), by the two lowest position bits
//   T3 [2][16], T4 [2][64]   half-sizes 16, 32 and 64, 128 as (cos, tan), by the four and six lowest position bits
//   T5 [5][256]      256 as (cos, tan); 512: two (c1, c2) pairs as above
#define FFT_T_OFF (FFT_F3_OFF + FFT_F3_LEN)
#define FFT_T2_OFF 0u
#define FFT_T3_OFF 12u
#define FFT_T4_OFF 44u
#define FFT_T5_OFF 172u
#define FFT_T_LEN (FFT_T5_OFF + 5u * 256u)
#define FFT_TAB_LEN (FFT_T_OFF + FFT_T_LEN)

// complex entries of the transform-domain key of one step: [piece][half g][k][row, component][lane]
#define FFT_KEY_STEP (SLZ_FFT_PIECES * 2u * 8u * 4u * 64u)

// Tables of the N = 1024 kernel, M = 512, all entries (cos, tan); the second of two sibling blocks takes i times the first one's:
//   F2 [4][8]        forward strides 32 (1), 16 (1), 8 (2), by the three top position bits
//   I2 [4][8]        inverse half-sizes 8 (1), 16 (1), 32 (2), by the three lowest position bits
//   I3 [10][64]      inverse half-sizes 64 (1), 128 (1); 256: four (c1, c2) pairs as above
//   F3 [4][64]       forward strides 4 (1), 2 (1), 1 (2), by the six top position bits
#define F10_F2_OFF 0u
#define F10_I2_OFF 32u
#define F10_I3_OFF 64u
#define F10_LDS_TAB (F10_I3_OFF + 640u)
#define F10_F3_OFF F10_LDS_TAB
#define F10_TAB_LEN (F10_F3_OFF + 256u)
// complex entries of the transform-domain key of one step: [piece][k][row, component][lane]
#define F10_KEY_STEP (SLZ_FFT_PIECES * 8u * 4u * 64u)

// Tables of the N = 512 kernel, M = 256, in the same form:
//   F2 [4][8]        forward strides 16 (1), 8 (1), 4 (2), by the three top position bits
//   I2 [4][4]        inverse half-sizes 4 (1), 8 (1), 16 (2), by the two lowest position bits
//   I3 [10][32]      inverse half-sizes 32 (1), 64 (1); 128: four (c1, c2) pairs
//   F3 [2][64]       forward strides 2 (1), 1 (1), by the six top position bits
#define F9_PIECES 3
#define F9_PIECE_BITS 22
#define F9_F2_OFF 0u
#define F9_I2_OFF 32u
#define F9_I3_OFF 48u
#define F9_LDS_TAB (F9_I3_OFF + 320u)
#define F9_F3_OFF F9_LDS_TAB
#define F9_TAB_LEN (F9_F3_OFF + 128u)
// complex entries of the transform-domain key of one step: [piece][k][row, component][lane]
#define F9_KEY_STEP (F9_PIECES * 4u * 8u * 64u)

// Tables of the N = 4096 kernel, M = 2048:
//   F2 [7][8]        forward strides 128, 64, 32 as one radix-8 layer (u .. u^7), by the three top position bits
//   F3 [7][64]       forward strides 16, 8, 4 likewise, by the six top position bits
//   I2 [5][8]        inverse half-sizes 8 and 16 as one radix-4 layer (v, v^2, v^3), 32 (2, as (cos, tan)), by the three lowest position bits
//   I3 [5][64]       inverse half-sizes 64 and 128, 256 (2) likewise
//   I4 [9][256]      inverse half-sizes 512 (1, as (cos, tan)); 1024: four (c1, c2) pairs as above
//   F4 [4][6][64]    forward strides 2/1, by (two top bits, lane): two blocks of three
#define F12_F2_OFF 0u
#define F12_F3_OFF 56u
#define F12_I2_OFF (F12_F3_OFF + 448u)
#define F12_I3_OFF (F12_I2_OFF + 40u)
#define F12_I4_OFF (F12_I3_OFF + 320u)
#define F12_LDS_TAB (F12_I4_OFF + 9u * 256u)
#define F12_F4_OFF F12_LDS_TAB
#define F12_TAB_LEN (F12_F4_OFF + 4u * 6u * 64u)
// complex entries of the transform-domain key of one step: [piece][quarter g][k][row, component][lane]
#define F12_KEY_STEP (SLZ_FFT_PIECES * 4u * 8u * 4u * 64u)

// Worst-case error (absolute, before rounding) of one y_j over all inputs, see slz_fft.hip.
double slz_fft_error_bound(uint32_t N, uint32_t rows, uint32_t beta);
