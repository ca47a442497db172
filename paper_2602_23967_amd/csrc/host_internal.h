// Host-side helpers shared by the single-problem / batched API (host.cpp)
// and the request server (serve.cpp). Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "../../include/pdhcg.h"
#include "prep.h"

namespace pdhcg {

// Streams beside a batch's own (default priority, no events' timing), on which
// kernels of one launch that do not depend on each other run at the same
// time.  Made when a launch first needs them; make() returns false where that
// fails, and then the kernels follow each other on the one stream.
struct SideStreams {
    static constexpr int MAX = 3;
    hipStream_t s[MAX] = {};
    hipEvent_t fork = nullptr, join[MAX] = {};
    bool make(int count);
    void wait();      // for all work on them
    void destroy();
};

// A region of device memory the library does not own (the static workspace of
// qp_batch_solve_static): allocations are carved from it in 256-byte steps
// and never freed; one that does not fit fails with QP_ERR_INVALID_ARG.
struct Arena {
    char* base = nullptr;
    size_t cap = 0, used = 0;
    SideStreams* side = nullptr;   // kept with the region, for one batch at a time
};

// qp_batch_create on a stream lent by the caller (NULL: the batch makes its
// own).  With an arena, every device buffer of the batch comes from it, the
// batch uses `lane` as given (NULL is the null stream) and the arena's side
// streams, and creates no stream or event: nothing is allocated on the device.
int batch_create(hipStream_t lane, int64_t count, const int64_t* var_off, const int64_t* row_off,
                 const int64_t* Qp, const int32_t* Qj, const double* Qv,
                 const int64_t* Ap, const int32_t* Aj, const double* Av,
                 const double* c, const double* b, const char* sense,
                 const double* lb, const double* ub, qp_batch** out, Arena* arena = nullptr);

// asynchronous batched solve: launch on the batch's stream, poll
// (1 finished, 0 running, < 0 error), finish (fetches the outcomes and
// returns the number of OPTIMAL instances)
int batch_launch(qp_batch* bt, const qp_params* params);
int batch_poll(qp_batch* bt);
int batch_finish(qp_batch* bt);
// after batch_finish: outcome of instance i
void batch_info(const qp_batch* bt, int64_t i, qp_info* info);
// after batch_finish: the returned x and y of every instance in one copy each
// (packed like the problem; certificates in place of the iterates, scaled as
// in qp_batch_result)
int batch_results_all(qp_batch* bt, std::vector<double>& x, std::vector<double>& y);

}  // namespace pdhcg

// How many workgroups a solve of this handle runs as one group (coop.hip), 0
// where it takes another path; and at most `cap` of them from now on (0: all).
// With fewer, each has several slices, as when other streams hold the CUs; the
// result is the same.  Not in the header: for the tests of that path.
extern "C" int qp_internal_group(qp_handle* h, int32_t cap);
