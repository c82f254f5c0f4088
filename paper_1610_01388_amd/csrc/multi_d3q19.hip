// multi_d3q19.hip -- several steps per launch, small domains, D3Q19.
#include "multi_impl.hpp"

namespace lbm {
template hipError_t launch_multi_lattice<1>(int, int, const MultiArgs&, size_t, hipStream_t, int*);
}
