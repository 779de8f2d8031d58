// Blocked Walsh-Hadamard transform of the gate-level path (k_wht.hip), used by api.hip.
#pragma once

#include "internal.h"

namespace grover {

// H^n with the normalisation 2^(-n/2), one pass over the state per group of qubits.
hipError_t launch_hadamard_all_blocked(grover_ctx *c);
// k iterations of H^n (2|0><0| - I) H^n after the oracle, the neighbouring passes of one group merged.
hipError_t launch_gate_iterate_blocked(grover_ctx *c, uint64_t k);

}  // namespace grover
