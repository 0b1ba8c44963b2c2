// Kernel instantiations: ring degree 2^13, arithmetic ArithQ.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_q_13()
{
    static const EngineOps ops = Launch<Engine<ArithQ, 13, 3>>::full();
    return &ops;
}
}
