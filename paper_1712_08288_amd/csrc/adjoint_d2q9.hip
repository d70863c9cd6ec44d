#include "adjoint.hpp"

template hipError_t lbe::launch_adjoint_nodes<lbe::D2Q9>(const lbe::Engine&,
                                                       const lbe::AdjointLaunch&);
