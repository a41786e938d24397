// Instantiates one group of the batches' filter kernels (see the instance lists in kernels.hpp).
#define PQ_INSTANCE_TU
#include "kernels.hpp"
namespace pqk {
PQ_FILTER_INSTANCES_STAMPED(PQ_FILTER_DEFINE8)
PQ_FILTER_INSTANCES_NEAR_STAMPED(PQ_FILTER_DEFINE10)
}
