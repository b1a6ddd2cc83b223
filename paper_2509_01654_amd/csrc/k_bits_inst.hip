// k_bits_inst.hip -- instantiates the bit-plane top-k kernels for the classes of
// row lengths NW_BITS_LO .. NW_BITS_HI, a few per translation unit so they
// build in parallel.  Exports them through nw_fill_bits_<NW_BITS_LO>.
#include <utility>

#include "k_topk_bits.h"
#include "nw_kernels.h"

#define NW_CAT2(a, b) a##b
#define NW_CAT(a, b) NW_CAT2(a, b)

namespace nw {

template <int C, class S>
static void fill_one(KernelTables &t)
{
    constexpr int s = S::kPlanes - 2;
    t.topk_bits[s][0][C] = reinterpret_cast<const void *>(&k_topk_bits<C, S, false>);
    t.topk_bits[s][1][C] = reinterpret_cast<const void *>(&k_topk_bits<C, S, true>);
}

template <int LO, int... Is>
static void fill(KernelTables &t, std::integer_sequence<int, Is...>)
{
    (fill_one<LO + Is, Bits2>(t), ...);
    (fill_one<LO + Is, Bits3>(t), ...);
}

void NW_CAT(nw_fill_bits_, NW_BITS_LO)(KernelTables &t)
{
    fill<NW_BITS_LO>(t, std::make_integer_sequence<int, NW_BITS_HI - NW_BITS_LO + 1>{});
}

}  // namespace nw
