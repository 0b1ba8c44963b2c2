// Kernel instantiations: ring degree 2^12, arithmetic ArithQ.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_q_12()
{
    static const EngineOps ops = Launch<Engine<ArithQ, 12, 3>>::full();
    return &ops;
}
}
