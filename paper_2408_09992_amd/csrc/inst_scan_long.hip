// Instantiates the candidate-list kernels for short lists (see the instance lists in kernels.hpp).
#define PQ_INSTANCE_TU
#include "kernels.hpp"
namespace pqk {
PQ_LONG_INSTANCES(PQ_LONG_DEFINE)
}
