// The wave-wide operations of the convolution kernel's matrix path, on top of
// hip_emu.h: a 64-lane ballot and v_mfma_f32_4x4x1_16b with its A operand
// broadcast from one block (cbsz 4). Every lane of a wave must call them
// together, as the kernel does: each publishes its value, waits for its wave,
// reads the others', waits again.
#pragma once

#include "hip_emu.h"

#define CONV_EMULATED_MFMA 1

constexpr int kEmuMaxWaves = 4;
inline std::barrier<>* emu_matrix_wave(unsigned wave)
{
    static std::barrier<> bars[kEmuMaxWaves]{std::barrier<>(64), std::barrier<>(64), std::barrier<>(64),
                                             std::barrier<>(64)};
    assert(wave < kEmuMaxWaves);
    return &bars[wave];
}
inline float emu_matrix_a[64 * kEmuMaxWaves];
inline int emu_matrix_pred[64 * kEmuMaxWaves];

inline uint64_t __builtin_amdgcn_ballot_w64(bool p)
{
    const unsigned t = threadIdx.x, wave0 = t - t % 64;
    emu_matrix_pred[t] = p;
    emu_matrix_wave(t / 64)->arrive_and_wait();
    uint64_t r = 0;
    for (int k = 0; k < 64; ++k)
        r |= (uint64_t)(emu_matrix_pred[wave0 + k] != 0) << k;
    emu_matrix_wave(t / 64)->arrive_and_wait();
    return r;
}

// D[m] += A[block abid][m] * B[lane] in each lane, fused, round to nearest.
template <class V4>
inline V4 __builtin_amdgcn_mfma_f32_4x4x1f32(float a, float b, V4 c, int cbsz, int abid, int blgp)
{
    assert(cbsz == 4 && abid >= 0 && abid < 16 && blgp == 0);
    const unsigned t = threadIdx.x, wave0 = t - t % 64;
    emu_matrix_a[t] = a;
    emu_matrix_wave(t / 64)->arrive_and_wait();
    for (int m = 0; m < 4; ++m)
        c[m] = std::fmaf(emu_matrix_a[wave0 + 4 * abid + m], b, c[m]);
    emu_matrix_wave(t / 64)->arrive_and_wait();
    return c;
}
