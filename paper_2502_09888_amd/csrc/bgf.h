// Kernels of the bit-wise gating fusion module (bgf.hip); internal.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace climber {

// fusion attention over the n_blocks rows of every candidate; d_head = 64
hipError_t launch_bgf_attention(const void *qkv, void *o, const int32_t *scen, const float *tau_scen, int n_scen,
                                int64_t m, int nb, int H, float qk_scale, hipStream_t s);
// the fusion layer's QKV projection of fp32 rows e [m * nb][d] and that attention, one launch (bgf_front_bf16.hip), where that is the faster way
bool bgf_front_takes(int64_t m, int nb, int d);
hipError_t launch_bgf_front(const float *e, const void *wqkv, void *o, const int32_t *scen, const float *tau_scen, int n_scen, int64_t m, int nb,
                            int d, float qk_scale, float inv_d, float eps, hipStream_t s);
// Y = G (.) sigmoid(pre), score = <w_head, Y> + b_head
hipError_t launch_bgf_gate_head(const float *g, const void *pre, const float *w_head, float b_head, float *y,
                                float *score, int64_t m, int nd, hipStream_t s);
// the same with both projections of the gate before it (packed weights; gb: bf16 copy of g), where that is the faster way
bool bgf_gate_takes(int64_t m, int nd, int dg, bool with_y);
hipError_t launch_bgf_gate(const void *gb, const float *g, const void *w_down, const void *w_up, const float *w_head, float b_head, float *y,
                           float *score, int64_t m, int nd, int dg, hipStream_t s);
int bgf_max_blocks();

}  // namespace climber
