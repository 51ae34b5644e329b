// Launchers that live in translation units of their own.
#pragma once
#include "apt_device.h"

// dynamic LDS beyond 64 KB has to be allowed per kernel (per-device set-up)
template <typename K> static inline bool apt_raise_lds_limit(K kern) {
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess;
}

// apt_mfma.inc: hidden-kind items on packed weights (then the KV-kind items, in the same launch).  DT: 1 = fp16, 2 = bf16; DEAL: the
// heads that not every queue has are dealt to all XCDs
template <int DT, bool DEAL> int apt_launch_mfma(const ItemParams& p, int n_wg, hipStream_t st);
template <int DT, bool DEAL> bool apt_setup_mfma();
template <> int apt_launch_mfma<1, false>(const ItemParams& p, int n_wg, hipStream_t st);
template <> int apt_launch_mfma<1, true>(const ItemParams& p, int n_wg, hipStream_t st);
template <> int apt_launch_mfma<2, false>(const ItemParams& p, int n_wg, hipStream_t st);
template <> int apt_launch_mfma<2, true>(const ItemParams& p, int n_wg, hipStream_t st);
template <> bool apt_setup_mfma<1, false>();
template <> bool apt_setup_mfma<1, true>();
template <> bool apt_setup_mfma<2, false>();
template <> bool apt_setup_mfma<2, true>();

// apt_raw16.hip: 16-bit inputs, hidden-kind items on the raw weights (and the KV-kind items, in the same launch)
int apt_launch_raw16(const ItemParams& p, int dtype, int head_dim, hipStream_t st);
bool apt_setup_raw16();

// apt_raw32.hip: fp32 inputs, the same
int apt_launch_raw32(const ItemParams& p, int head_dim, hipStream_t st);

// apt_absorb16.hip: absorbed-weight path, 16-bit inputs
int apt_launch_absorb_scores16(const ItemParams& p, int dtype, int head_dim, hipStream_t st);
bool apt_setup_absorb_scores16();
int apt_launch_absorb_pv16(const ItemParams& p, int dtype, int n_cus, hipStream_t st);
bool apt_setup_absorb_pv16();
int apt_absorb_out16_slices(const ItemParams& p, int n_cus, int most);
int apt_launch_absorb_out16(const ItemParams& p, int dtype, int head_dim, hipStream_t st);
bool apt_setup_absorb_out16();
