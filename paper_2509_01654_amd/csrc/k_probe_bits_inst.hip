// k_probe_bits_inst.hip -- the bit-plane threshold pre-pass and its launcher, a
// translation unit of its own (every row length in one kernel).
#include <cstdlib>
#include <cstring>

#include "k_probe_bits.h"

namespace nw {

// NW_PREPASS=packed keeps the packed selection where this form would apply
// (both give the same keys; for comparisons).
static bool packed_prepass_only()
{
    static const bool only = [] {
        const char *e = std::getenv("NW_PREPASS");
        return e && std::strcmp(e, "packed") == 0;
    }();
    return only;
}

static uint32_t probe_bits_lds(const DevVocab &V)
{
    const uint32_t one = bit_group_bytes(V.lmax, Bits2::kTab, V.alphabet);
    if (one > kProbeTabLds) return 0;
    return kProbeTabLds + (uint32_t)(V.hi - V.lo + 2) / 2u * 256u * (uint32_t)(kThreads / 64);
}

bool probe_bits_applies(const DevVocab &V, int m, uint64_t scratch_bytes)
{
    if (V.bits != 2 || packed_prepass_only() || V.n < kProbeBitsMinWords || V.lmax > kProbeBitsMaxLen || V.nprobe < m) return false;
    const uint32_t lds = probe_bits_lds(V);
    if (lds == 0 || lds > kMaxLdsBytes / 2) return false;
    const uint32_t groups = (uint32_t)(V.pslots / kBitRows) + ((uint32_t)V.nprobe + kBitRows - 1) / kBitRows;
    return probe_bits_lens_bytes(groups) + (uint64_t)groups * bit_group_bytes(V.lmax, Bits2::kTab, V.alphabet) <= scratch_bytes;
}

hipError_t launch_probe_bits(const DevVocab &V, int m, uint64_t *thr, void *scratch, hipStream_t stream)
{
    ProbeBitsArgs Q;
    Q.scratch = static_cast<uint8_t *>(scratch);
    Q.gstride = bit_group_bytes(V.lmax, Bits2::kTab, V.alphabet);
    Q.nA = (uint32_t)(V.pslots / kBitRows);
    Q.nB = ((uint32_t)V.nprobe + kBitRows - 1) / kBitRows;
    Q.npad = (uint32_t)(V.pslots - V.nprobe);
    Q.m = m;
    Q.thr = thr;
    hipLaunchKernelGGL(k_probe_tables, dim3(Q.nA + Q.nB), dim3(kThreads), Q.gstride, stream, V, Q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint32_t lds = probe_bits_lds(V);
    if (lds > 65536) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_probe_bits), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const uint32_t wgs = (uint32_t)((int64_t)V.nb * V.CB / kThreads);
    hipLaunchKernelGGL(k_probe_bits, dim3(wgs), dim3(kThreads), lds, stream, V, Q);
    return hipGetLastError();
}

}  // namespace nw
