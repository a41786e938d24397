// Instantiates the candidate-list (two queries per workgroup) kernels for short lists (see the instance lists in kernels.hpp).
#define PQ_INSTANCE_TU
#include "kernels.hpp"
namespace pqk {
PQ_SUBSETP_INSTANCES(PQ_SUBSETP_DEFINE)
}
