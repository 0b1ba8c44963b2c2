// Kernel instantiations: ring degree 2^11, arithmetic ArithQ.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_q_11()
{
    static const EngineOps ops = Launch<Engine<ArithQ, 11, 3>>::full();
    return &ops;
}
}
