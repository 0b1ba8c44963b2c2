// Kernel instantiations: ring degree 2^15, arithmetic ArithP.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_p_15()
{
    static const EngineOps ops = Launch<Engine<ArithP, 15, 3, 12>>::transforms_only();
    return &ops;
}
}
