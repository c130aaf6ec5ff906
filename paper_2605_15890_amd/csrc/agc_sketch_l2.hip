// k_sketch for the Euclidean scale.
#include "agc_sketch.h"

namespace agc {

hipError_t launch_sketch(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code, const Workspace& ws,
                         const SketchDev& sk, uint64_t seed, uint64_t step, hipStream_t stream)
{
    const SketchArgs a{ldg, n, k, d, (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32),
                       code.win, code.stream, ws.part_sq, nullptr, sk};
    if (code.band < 0 && !code.win) return hipErrorInvalidValue;  // the window driver reads the records
    switch (code.band) {
        case 1: return launch_sketch_s<1>(G, code, a, stream);
        case 2: return launch_sketch_s<2>(G, code, a, stream);
        case 3: return launch_sketch_s<3>(G, code, a, stream);
        case 4: return launch_sketch_s<4>(G, code, a, stream);
        case 5: return launch_sketch_s<5>(G, code, a, stream);
        case 6: return launch_sketch_s<6>(G, code, a, stream);
        case 7: return launch_sketch_s<7>(G, code, a, stream);
        case 8: return launch_sketch_s<8>(G, code, a, stream);
        case -2: return launch_sketch_s<-2>(G, code, a, stream);
        case -4: return launch_sketch_s<-4>(G, code, a, stream);
        case -8: return launch_sketch_s<-8>(G, code, a, stream);
        default: return code.stream ? launch_sketch_s<kStreamDriver>(G, code, a, stream) : launch_sketch_s<0>(G, code, a, stream);
    }
}

}  // namespace agc
