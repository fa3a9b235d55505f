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

// LDS floats per patch that hold the least-squares state while the screen runs: the factor's
// strict lower triangle, its inverse diagonal, right-hand sides and coefficients, in float4s.
constexpr int screen_state_f4(int kmax) { return (kmax * (kmax - 1) / 2 + 3 * kmax + 3) / 4; }

}  // namespace rsc
