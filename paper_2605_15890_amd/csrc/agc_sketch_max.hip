// k_sketch_max: one read of G for scales that are the largest magnitude of the vector.
#include "agc_sketch.h"

namespace agc {

hipError_t launch_sketch_max(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code, const Workspace& ws,
                             const SketchDev& sk, const QuantStreams& out, uint64_t seed, uint64_t step, hipStream_t stream)
{
    const SketchArgs a{ldg, n, k, d, (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32),
                       code.win, code.stream, nullptr, ws.part_max, sk};
    if (code.band < 0 && !code.win) return hipErrorInvalidValue;  // the window driver reads the records
    const BitList bits = bit_list(n, out);
    switch (code.band) {
        case 1: return launch_sketch_max_s<1>(G, code, a, bits, stream);
        case 2: return launch_sketch_max_s<2>(G, code, a, bits, stream);
        case 3: return launch_sketch_max_s<3>(G, code, a, bits, stream);
        case 4: return launch_sketch_max_s<4>(G, code, a, bits, stream);
        case 5: return launch_sketch_max_s<5>(G, code, a, bits, stream);
        case 6: return launch_sketch_max_s<6>(G, code, a, bits, stream);
        case 7: return launch_sketch_max_s<7>(G, code, a, bits, stream);
        case 8: return launch_sketch_max_s<8>(G, code, a, bits, stream);
        case -2: return launch_sketch_max_s<-2>(G, code, a, bits, stream);
        case -4: return launch_sketch_max_s<-4>(G, code, a, bits, stream);
        case -8: return launch_sketch_max_s<-8>(G, code, a, bits, stream);
        default: return code.stream ? launch_sketch_max_s<kStreamDriver>(G, code, a, bits, stream) : launch_sketch_max_s<0>(G, code, a, bits, stream);
    }
}

}  // namespace agc
