// minor_pairs_b6.hip -- leave-one-column-out walk over pairs, up to 48 columns.
#include "kernels.hpp"
#include "minor_pairs.hpp"

namespace bbfg {

const void* minor_pairs_fn_b6() { return reinterpret_cast<const void*>(&minor_pairs_kernel<6>); }

}  // namespace bbfg
