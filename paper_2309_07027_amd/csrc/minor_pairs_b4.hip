// minor_pairs_b4.hip -- leave-one-column-out walk over pairs, up to 32 columns.
#include "kernels.hpp"
#include "minor_pairs.hpp"

namespace bbfg {

const void* minor_pairs_fn_b4() { return reinterpret_cast<const void*>(&minor_pairs_kernel<4>); }

}  // namespace bbfg
