#include "adjoint.hpp"

template hipError_t lbe::launch_adjoint_nodes<lbe::D3Q19>(const lbe::Engine&,
                                                       const lbe::AdjointLaunch&);
