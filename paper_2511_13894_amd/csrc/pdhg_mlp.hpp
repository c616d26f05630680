// Internal declarations of the fix predictor (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "pdhg.h"

#define MLP_NPARAMS 5313 // w1 (64x16), b1 (64), w2 (64x64), b2 (64), w3 (64), b3 (1)

struct pdhg_mlp {
    hipStream_t stream = nullptr; // of calls that train or take host data, made with the first of them
    float *p = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr; // float32 master values, Adam state
    short *w1b = nullptr, *w2b = nullptr, *w3b = nullptr;           // bfloat16 weight copies
    short *w2tb = nullptr;                                           // W2 transposed (the gradient kernel)
    float *part = nullptr, *lossp = nullptr;                         // per-wave partial gradients and losses
    int max_waves = 0;
    double *loss_acc = nullptr;
    int64_t adam_t = 0;
    int device = -1;
    hipStream_t pass = nullptr; // forward passes of callers who name no stream: one stream for a device's networks
    std::mutex mu;              // held while such a pass is enqueued and while it is decided where they run:
    bool passed = false;        // passes may be in flight on `pass`
    int busy = 0;               // calls that work on `stream`: passes are enqueued there, between a training's steps
    bool beside = false;        // and some have been
    hipEvent_t order[2] = {nullptr, nullptr}; // such a pass after those on `pass`, and the next ones after it
};

namespace pdhg {
hipError_t mlp_sync(pdhg_mlp *net, hipStream_t st); // the bfloat16 copies of the weights
hipError_t mlp_init(pdhg_mlp *net, uint64_t seed);
hipError_t mlp_features_to_bf16(hipStream_t st, const float *src, short *dst, int64_t n_rows);
hipError_t mlp_forward(const pdhg_mlp *net, hipStream_t st, const short *F, int64_t N, float *logits);
hipError_t mlp_grad(pdhg_mlp *net, const short *F, const float *Y, const int *idx, int64_t b0, int bsz, float pw);
// the same minibatch's gradient and Adam step t
hipError_t mlp_train_step(pdhg_mlp *net, const short *F, const float *Y, const int *idx, int64_t b0, int bsz, float pw,
                          float lr, float beta1, float beta2, float eps, int64_t t);
// device address of the no-allocation forward's staging array on the current
// device (looked up once per device)
hipError_t mlp_scratch_setup();
// the network's own stream (net->mu held); take and give back the device's shared pass
// stream; wait for the passes on it (net->mu held)
hipError_t mlp_stream_open(pdhg_mlp *net);
hipError_t mlp_pass_open(pdhg_mlp *net);
void mlp_pass_close(pdhg_mlp *net);
hipError_t mlp_pass_wait(pdhg_mlp *net);
} // namespace pdhg
