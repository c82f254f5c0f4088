// multi_d2q9.hip -- several steps per launch, small domains, D2Q9.
#include "multi_impl.hpp"

namespace lbm {
template hipError_t launch_multi_lattice<0>(int, int, const MultiArgs&, size_t, hipStream_t, int*);
}
