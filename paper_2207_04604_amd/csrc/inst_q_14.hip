// Kernel instantiations: ring degree 2^14, arithmetic ArithQ.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_q_14()
{
    static const EngineOps ops = Launch<Engine<ArithQ, 14, 4>, Engine<ArithQ, 14, 3, 13>>::full();
    return &ops;
}
}
