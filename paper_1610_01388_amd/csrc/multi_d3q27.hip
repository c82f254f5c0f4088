// multi_d3q27.hip -- several steps per launch, small domains, D3Q27.
#include "multi_impl.hpp"

namespace lbm {
template hipError_t launch_multi_lattice<2>(int, int, const MultiArgs&, size_t, hipStream_t, int*);
}
