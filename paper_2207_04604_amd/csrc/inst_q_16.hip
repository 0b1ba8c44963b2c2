// Kernel instantiations: ring degree 2^16, arithmetic ArithQ.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_q_16()
{
    static const EngineOps ops = Launch<Engine<ArithQ, 16, 3, 12>>::transforms_only();
    return &ops;
}
}
