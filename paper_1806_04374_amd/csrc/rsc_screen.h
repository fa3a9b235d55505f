// Shape of the screened encoder (rsc_encode_screen.hip), shared by the host code that
// arranges its operands and by the kernel.
//
// The screen multiplies 32 patches per wave on v_mfma_f32_32x32x16 with 16-bit operands.
// Stage 1 has 32 rows and 16 contraction slots (8 per half-wave: Re parts of the residual in
// the low half, Im parts in the high one; harmonic 0 has its even profiles low, odd ones
// high).  With up to 8 harmonics (OPS = 1) the rows are (Re, Im) of 16 atoms and one
// instruction takes one harmonic.  With 9..16 harmonics (OPS = 2) the rows are (Re, Im) of 8
// atoms for harmonic j, then the same for harmonic j + 8, whose profiles share the slots
// (their counts add up to at most 8 in the ragged basis that this serves), so stage 1 still
// takes 8 instructions per 16 row pairs and an atom's stage-2 operand is two registers sets
// of 8 slots: harmonics 0..7 from row pair a, 8..15 from row pair a + 8.
#pragma once

namespace rsc {

constexpr int screen_ops(int T) { return T + 1 <= 8 ? 1 : 2; }
constexpr int screen_group_atoms(int T) { return 16 / screen_ops(T); }
constexpr int screen_steps(int T) { return T + 1 <= 8 ? T + 1 : 8; }   // stage-1 instructions per group

// Floats of a dictionary row in the screened encoder's LDS: harmonic 0 (padded to an even count),
// then for each harmonic k >= 1 its profiles as (Re, Im) pairs, so that a pair is one 8-byte read.
// Every lane reads its own atom's row, and the angle table at its own angle: both strides are
// twice an odd number of words, so that the lanes spread over all the 8-byte bank pairs (a
// stride of 56 words takes 8 of the 32, one of 32 words takes 2).
constexpr int screen_row(int B, int s0) { return B + s0 % 2 + ((B + s0 % 2) / 2 % 2 == 0 ? 2 : 0); }
constexpr int screen_angle_stride(int T) { return (T + 1) | 1; }   // (cos, sin) pairs per angle

// LDS per patch that holds the least-squares state while the screen runs, in 16-byte units: the
// factor's strict lower triangle, its inverse diagonal, right-hand sides and coefficients, and
// the selections, two to a word.  The least-squares step uses the same space for arrays that it
// indexes at run time (at most 2 kmax words).
constexpr int screen_state_f4(int kmax) { return (kmax * (kmax - 1) / 2 + 3 * kmax + (kmax + 1) / 2 + 3) / 4; }

}  // namespace rsc
