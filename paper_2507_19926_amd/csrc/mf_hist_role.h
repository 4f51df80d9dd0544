// Roles of the four waves of a two-word sliding-histogram work-group
// (mf_hist_kernel.h): plain arithmetic, also compiled for the host by its test.
#pragma once

#include <stdint.h>

#ifndef MF_HOST_DEVICE
#define MF_HOST_DEVICE
#endif

// What a wave publishes about itself: its SIMD (bits 0..1) and whether its
// work-group lies above the CU's lowest LDS (bit 2).
MF_HOST_DEVICE constexpr uint32_t hist_role_word(uint32_t simd, uint32_t lds_base)
{
    return (simd & 3u) | (lds_base != 0 ? 4u : 0u);
}

// Role of wave `wave` from the words of all four, the same four for every wave:
// the SIMD number, exchanged by halves for the upper work-group, and the wave
// number unless the waves are on four SIMDs. The roles of the four waves differ
// whatever the words say. The LDS base counts by wave 0's word alone: read at
// different times, waves of one work-group may see different ones (it may have
// been moved between the reads).
MF_HOST_DEVICE constexpr int hist_role(const uint32_t (&words)[4], int wave)
{
    uint32_t simds = 0, own = 0;
    for (int i = 0; i < 4; ++i) {
        simds |= 1u << (words[i] & 3u);
        if (i == wave) own = words[i] & 3u;
    }
    return simds != 15u ? wave : (int)(own ^ ((words[0] >> 1) & 2u));
}
