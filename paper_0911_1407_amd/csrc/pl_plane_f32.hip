// FP32 instantiation of the plane passes.
#define PL_T float
#define PL_T_IS_DOUBLE 0
#include "pl_plane_impl.hpp"
