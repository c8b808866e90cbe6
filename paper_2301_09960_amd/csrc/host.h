// Host-side helpers shared by the single-product and batched C-ABI code.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "residue.h"

namespace mp {
namespace host {

constexpr int kNumFmtH = 4;
extern const int kCompsH[kNumFmtH];

// Options of the calling host thread.
int thread_mode(int fmt);
int layout_for(int fmt);
// The INT8 tile configuration this thread forces (0: chosen by size).
int int8_tile_override();
int split_kernel_override();
int last_slice_option();
int slices_for(int fmt, int mode, int64_t k);
void set_last_slices(int D);
// The slice count of (fmt, mode) is the library's choice on this thread.
bool automatic_slices(int fmt, int mode);

// The shift ceil((S + log2 k) / 2) of Algorithm 1.
int rho_of(int S, int64_t k);

// BLAS-style argument check of one product (0, -position, or MPGEMM_ERR_TOO_LARGE).
int validate(int m, int n, int k, const void *A, int lda, const void *B, int ldb, const void *C, int ldc);

// 0 if the current device is a gfx950, else an MPGEMM_ERR_* code.
int check_device_cached();

int hip_status(hipError_t e);

// What a call takes for residues that need `need` bytes: at most 8 GiB or so many
// quarters of what its slices (digits) take, whichever is more.
size_t residue_room(size_t need, size_t slices, int quarters);

// hipMalloc on the device (the current one); the workspaces kept between calls are
// given back where it fails at first.
bool allocate_device(char **p, size_t bytes, int dev);

// One product as its own call forms it, in a workspace of its own (arguments valid).
template <typename T, int C>
int run_product(int fmt, int mode, int D, bool automatic, int m, int n, int k, const T *A, int lda, const T *B,
                int ldb, T *Cm, int ldc, hipStream_t st);

// Stage-timing hooks (mpgemm_profile_*): events before/after a unit of work.
bool profiling();
void profile_mark3(hipEvent_t (&ev)[3]);
void profile_commit(hipEvent_t (&ev)[3]);

// The residue plan of a FLOAT-form product with the automatic count D; false
// where it goes by slices.
bool float_residue_plan(int fmt, int D, int64_t k, ResiduePlan &p);

}  // namespace host
}  // namespace mp
