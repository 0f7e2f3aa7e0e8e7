// What the kernels of the backward pass share: their parameters, and a chunk of a walk.
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace hgrn2 {

struct BwdGradParams {
    const void* q;
    const void* f;
    const void* v;
    const void* dO;
    const void* ws_s;
    const void* ws_ds;
    void* dq;
    void* df;
    void* dv;
    int BH, N, NC;
    const float* beta;       // [H][dk] lower bounds, or null: the gate tensor holds f itself
    float* beta_partials;    // [B*H*NC][8][dk] per-wave partial sums of the gradient w.r.t. beta
    int H;
    TokenLayout lay;         // (always set: the walks of bwd_walk.hip take strides and offsets from it whatever the layout)
    int dense;               // sequence tensors are [B][H][N][d]: bwd_grad.hip then has compile-time strides
    // Reverse walk (walk_body(), bwd_grad_body<..., FUSED>): the state gradient is carried in registers
    // instead of being read from ws_ds.  Every sequence is cut into R runs of rc chunks, one
    // workgroup each; a run starts from grad_hT (the last one), from bound0[bh] (run 0) or from
    // run_state[bh * seg_tail + r * s_sub - 1] (the state gradient at the end of run r, which a
    // zero-start sweep over the later tokens and its carry have left there); run 0 leaves grad_h0.
    // With light walks (`light`), no boundary states are needed: a workgroup first walks the chunks
    // after its run, from grad_hT, doing nothing but the state-gradient recurrence (a fraction of a
    // chunk's full work), and the runs are cut at bnd[0] = 0 < bnd[1] < ... < bnd[R] = NC so that
    // all workgroups finish together.
    const float* dhT;
    float* dh0;
    const float* bound0;
    const float* run_state;
    int R, rc, s_sub, seg_tail;
    int light;
    int* flag;               // null, or set to 1 when a gate product falls below the floor of the reciprocals
    int beta_spans;          // row sets of partial sums per head (packed batches)
    // What bwd_ends_kernel leaves: per slot a state gradient [dk][dv] and the gate products [dk].  Spans of a
    // packed batch: slot span * H + head, read by the walk over spans (null: every span takes a light walk);
    // runs of segmented sequences: slot = run.
    float* span_add;
    float* span_decay;
    int bnd[kMaxLightRuns + 1];      // (last: whatever is read of the arguments by every walk lies close together)
};

// A chunk of a walk: sequence and chunk within it.
struct ChunkAt { SeqView sv; int bh, n; };

// The reverse walk over runs, or (grouped) over spans of a packed batch (bwd_walk.hip): bf16 storage.
hipError_t launch_bwd_walk(const SeqDims& d, const BwdGradParams& p, bool grouped, hipStream_t stream);
// What a run or a span adds to the state gradient from zero (span_add, span_decay): a workgroup per slot.
hipError_t launch_walk_ends(const SeqDims& d, const BwdGradParams& p, unsigned grid, hipStream_t stream);

}   // namespace hgrn2
