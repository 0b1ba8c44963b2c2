// Kernel instantiations: ring degree 2^13, arithmetic ArithP.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_p_13()
{
    static const EngineOps ops = Launch<Engine<ArithP, 13, 3>>::full();
    return &ops;
}
}
