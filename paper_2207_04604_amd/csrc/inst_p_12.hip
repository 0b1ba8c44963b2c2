// Kernel instantiations: ring degree 2^12, arithmetic ArithP.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_p_12()
{
    static const EngineOps ops = Launch<Engine<ArithP, 12, 3>>::full();
    return &ops;
}
}
