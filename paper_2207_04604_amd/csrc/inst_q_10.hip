// Kernel instantiations: ring degree 2^10, arithmetic ArithQ.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_q_10()
{
    static const EngineOps ops = Launch<Engine<ArithQ, 10, 3>>::full();
    return &ops;
}
}
