// k_query_inst.hip -- instantiates the query kernel of the row lengths NW_QUERY_LO ..
// NW_QUERY_HI, one range per translation unit so they build in parallel;
// nw_fill_query_<NW_QUERY_LO> exports it.
#include "k_query.h"
#include "nw_kernels.h"

#define NW_CAT2(a, b) a##b
#define NW_CAT(a, b) NW_CAT2(a, b)

namespace nw {

void NW_CAT(nw_fill_query_, NW_QUERY_LO)(KernelTables &t)
{
    t.query[NW_QUERY_LO / kQuerySpan] = reinterpret_cast<const void *>(&k_query_class<NW_QUERY_LO, NW_QUERY_HI>);
}

}  // namespace nw
