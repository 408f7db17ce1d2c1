// fp32 forward on split operands (fipa_f32_split.hip), as fipa_f32.hip chooses it.
#pragma once

#include "fipa_internal.h"

namespace fipa {

bool f32_split_applies(const fipa_desc &d, bool masked);  // the shapes that it is built for and is the faster one at
size_t f32_split_workspace(const fipa_desc &d);        // what it asks for (0: no use)
size_t f32_split_workspace_min(const fipa_desc &d);    // without the space for split key ranges
hipError_t f32_split_forward(const fipa_desc &d, const FwdArgs &a, void *ws, size_t ws_bytes, hipStream_t stream);

}  // namespace fipa
