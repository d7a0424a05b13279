// Compiled variants of the stage kernel, by mode: stage_kernels.hip is compiled once per mode
// (ELB_STAGE_MODE) and each compilation gives the two tables of that mode.
#pragma once
#include <hip/hip_runtime.h>

#include "elb_kernels.h"

namespace elb {

// One tile shape of the single-problem stage kernel (k_stage): the tiles of a Q stand in the
// order in which they are considered, and one is taken for at most `cap` blocks.  `launch`
// takes the StageArgs<R> of the mode's storage type.
struct StageKernel {
    int q, S, L, ret, closure, nt, rows, cap;
    void (*launch)(const void *args, int blocks, size_t shm, hipStream_t st);
    int cells() const { return S * L; }
};

// One tile shape of the batched stage kernel (k_stage_batch).  `cap` as above; INT_MAX: the
// large-problem tile and the tuner's alternatives to it.
struct BatchKernel {
    int q, S, L, ret, nt, rows, cap;
    void (*launch)(const BatchStage &bs, int grid, size_t shm, hipStream_t st);
    int cells() const { return S * L; }
};

struct StageTable {
    const StageKernel *stage;
    int stages;
    const BatchKernel *batch;
    int batches;
};

StageTable stage_table_f64();
StageTable stage_table_f32();
StageTable stage_table_mixed();
StageTable stage_table_fixup();

}  // namespace elb
