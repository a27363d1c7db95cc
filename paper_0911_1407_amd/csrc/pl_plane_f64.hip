// FP64 instantiation of the plane passes.
#define PL_T double
#define PL_T_IS_DOUBLE 1
#include "pl_plane_impl.hpp"
