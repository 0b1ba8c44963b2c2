// Kernel instantiations: ring degree 2^10, arithmetic ArithP.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_p_10()
{
    static const EngineOps ops = Launch<Engine<ArithP, 10, 3>>::full();
    return &ops;
}
}
