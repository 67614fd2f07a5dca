// minor_pairs_b3.hip -- leave-one-column-out walk over pairs, up to 24 columns.
#include "kernels.hpp"
#include "minor_pairs.hpp"

namespace bbfg {

const void* minor_pairs_fn_b3() { return reinterpret_cast<const void*>(&minor_pairs_kernel<3>); }

}  // namespace bbfg
