// Kernel instantiations: ring degree 2^16, arithmetic ArithP.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_p_16()
{
    static const EngineOps ops = Launch<Engine<ArithP, 16, 3, 12>>::transforms_only();
    return &ops;
}
}
