// Internal interface of the FP64 symmetric eigensolver.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

#include "host.h"

namespace dfpt2 {

constexpr int kEighMaxN = 16384;

size_t eigh_workspace_bytes(int n);
enum class EighPath {
  kAuto,     // one launch for the reduction where it fits
  kMissed,   // as if a workgroup of that launch never ran: the others give up (after 1 ms), a second attempt follows
  kRefused,  // as if that launch were refused: one launch per column at once
};
// w_out [n] and Z_out [n][n] (column k = eigenvector of w_out[k]); ascending, or
// descending when `descending` is set.  With vec_floor_rel > 0 only eigenvalues
// above vec_floor_rel * max|w| get eigenvectors (the other columns are zero).
// Synchronizes the stream.  Z_out may be A; both are written only when the attempt that
// succeeds ends.
int eigh_run(const double* A, int n, double* w_out, double* Z_out, char* ws, size_t ws_bytes, hipStream_t st,
             int descending, double vec_floor_rel = -1.0, EighPath path = EighPath::kAuto, int* attempts = nullptr);

}  // namespace dfpt2

// dfpt2_eigh_sym by a given path, for the tests of the second attempt; attempts: host out or null
extern "C" int dfpt2_eigh_sym_path(const double* A, int64_t n, double* w, double* Z, void* workspace, size_t ws_bytes,
                                   dfpt2_stream_t stream, int path, int* attempts);
