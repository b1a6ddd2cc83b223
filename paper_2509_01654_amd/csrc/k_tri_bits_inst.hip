// k_tri_bits_inst.hip -- instantiates one bit-plane triangle or edge kernel:
// variant NW_VARIANT (Bits2 int8, Bits2 int16, Bits3 int8, Bits3 int16, Bits3
// int16 with 16-bit staging, Bits2 edges, Bits3 edges), range NW_RANGE of row
// lengths.  One per translation unit so they build in parallel;
// nw_fill_tri_bits_<variant>_<range> exports it.
#include "k_edges_bits.h"
#include "k_tri_bits.h"
#include "nw_kernels.h"

#define NW_CAT4(a, b, c, d) a##b##c##d
#define NW_CAT(a, b, c, d) NW_CAT4(a, b, c, d)

namespace nw {

using Scheme = std::conditional_t<(NW_VARIANT < 2 || NW_VARIANT == 5), Bits2, Bits3>;
constexpr int kEs = NW_VARIANT == 0 || NW_VARIANT == 2 ? 1 : 2;
constexpr int kSpan = bits_span<Scheme>();
constexpr int kLo = NW_RANGE == 0 ? 0 : NW_RANGE * kSpan + 1, kHi = (NW_RANGE + 1) * kSpan;

void NW_CAT(nw_fill_tri_bits_, NW_VARIANT, _, NW_RANGE)(KernelTables &t)
{
#if NW_VARIANT < 5
    t.tri_bits[NW_VARIANT][NW_RANGE] = reinterpret_cast<const void *>(&k_tri_bits<kLo, kHi, Scheme, kEs, NW_VARIANT == 4>);
    t.tri_bits_threads[NW_VARIANT][NW_RANGE] = tri_bits_threads<kHi, NW_VARIANT == 4>();
#else
    t.edges_bits[NW_VARIANT - 5][NW_RANGE] = reinterpret_cast<const void *>(&k_edges_bits<kLo, kHi, Scheme>);
#endif
}

}  // namespace nw
