// Kernel instantiations: ring degree 2^14, arithmetic ArithP.
#include "engine_inst.hpp"

namespace d2 {
const EngineOps *ops_p_14()
{
    static const EngineOps ops = Launch<Engine<ArithP, 14, 4>, Engine<ArithP, 14, 3, 13>>::full();
    return &ops;
}
}
