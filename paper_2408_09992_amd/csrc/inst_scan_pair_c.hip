// Instantiates the catalogue-scan kernels that take two queries per workgroup (see the instance lists in kernels.hpp).
#define PQ_INSTANCE_TU
#include "kernels.hpp"
namespace pqk {
PQ_PAIR_INSTANCES_C(PQ_PAIR_DEFINE)
}
