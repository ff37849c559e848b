// What the softmax backward of one gate reads and writes, shared by the bf16 and the fp32 backward of RetNet and GLA.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace sla {

struct GateGrad {
    const float* g;     // the gate [rows,H]
    const float* part;  // partial planes of its gradient, `plane` floats apart
    int planes;
    size_t plane;
    float* dl;          // gradient of the logits [rows,H]
};

int launch_bwd_logits(const GateGrad& read, const GateGrad& write, size_t rows, int H, const int* cu, int B,
                      hipStream_t stream);

}  // namespace sla
