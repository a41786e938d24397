// Instantiates one group of the catalogue-scan kernels (see the instance lists in kernels.hpp).
#define PQ_INSTANCE_TU
#include "kernels.hpp"
namespace pqk {
PQ_BYTES_INSTANCES(PQ_BYTES_DEFINE)
}
