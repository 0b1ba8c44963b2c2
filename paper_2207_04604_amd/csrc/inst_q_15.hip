// Kernel instantiations: ring degree 2^15, arithmetic ArithQ.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_q_15()
{
    static const EngineOps ops = Launch<Engine<ArithQ, 15, 3, 12>>::transforms_only();
    return &ops;
}
}
