// Kernel instantiations: ring degree 2^11, arithmetic ArithP.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_p_11()
{
    static const EngineOps ops = Launch<Engine<ArithP, 11, 3>>::full();
    return &ops;
}
}
