// The job server's scheduling on the host, over stand-ins for the HIP calls
// and for the lattices: lane streams that cannot be made.  The job that needs
// the stream ends with PYRO_EDEVICE, its memory comes back, no error is left
// behind, jobs of other lanes run on, and a later job of the lane gets a stream
// when one can be made.  Exit status 0 on success.
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include <hip/hip_runtime.h>

#include "../include/pyro_sw.h"

static int refuse = 0;            // stream creations to refuse
static int streams = 0;           // streams alive
static hipError_t last = hipSuccess;
static int tag;                   // address of a stand-in object

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipGetLastError(void) { const hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned)
{
    if (refuse > 0) {
        --refuse;
        return last = hipErrorOutOfMemory;
    }
    ++streams;
    *st = (hipStream_t)&tag;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { --streams; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)&tag; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }

int pyro_sw_workspace_size(int L, int, size_t *spin, size_t *work)
{
    *spin = (size_t)L * 1024;
    *work = (size_t)L * 4096;
    return PYRO_OK;
}
int pyro_sw_init_ext(pyro_sw **out, int, int, double, double, uint64_t, int, void *stream, void *, size_t, void *, size_t)
{
    *out = (pyro_sw *)&tag;
    return stream ? PYRO_OK : PYRO_EDEVICE;
}
int pyro_sw_moments(pyro_sw *, pyro_sw_record *, int64_t, int64_t *n) { *n = 0; return PYRO_OK; }
int pyro_sw_get_spins(pyro_sw *, void *, size_t) { return PYRO_OK; }
int pyro_sw_destroy(pyro_sw *) { return PYRO_OK; }
int pyro_sw_group_create(pyro_sw_group **out, pyro_sw *const *, int, void *) { *out = (pyro_sw_group *)&tag; return PYRO_OK; }
int pyro_sw_group_set_slices(pyro_sw_group *, int) { return PYRO_OK; }
int pyro_sw_group_sweep(pyro_sw_group *, int64_t, const int64_t *) { return PYRO_OK; }
int pyro_sw_group_destroy(pyro_sw_group *) { return PYRO_OK; }
}
namespace pyro {
int record_error(int status, const char *) { return status; }
}

static int fail(const char *what, long long a, long long b)
{
    fprintf(stderr, "server check failed: %s (%lld, %lld)\n", what, a, b);
    return 1;
}

int main()
{
    pyro_sw_server *s = nullptr;
    if (pyro_sw_server_create(&s, (size_t)1 << 20, 8, 10.0, 0.0)) return fail("create", 0, 0);
    auto submit = [&](int L) {
        pyro_sw_job j{};
        j.model = PYRO_ISING;
        j.L = L;
        j.T = j.J = 1.0;
        j.start = PYRO_START_COLD;
        j.sweeps = 10;
        int64_t id = -1;
        pyro_sw_server_submit(s, &j, &id);
        return id;
    };
    auto error_of = [&](int64_t id) {
        pyro_sw_job_status st{};
        return pyro_sw_server_status(s, id, &st) ? 1 : st.state != PYRO_JOB_DONE ? 2 : st.error;
    };
    auto run = [&]() {
        int q = 1, r = 1, rc = 0;
        for (int k = 0; k < 100 && !rc && (q || r); ++k) rc = pyro_sw_server_step(s, 0.0, &q, &r);
        return rc ? rc : q || r ? 1 : 0;
    };
    // the largest job takes nearly the whole budget (1 MiB): its region has to
    // come back for the second one
    const int big = 200;
    refuse = 1;
    const int64_t a = submit(big);
    if (int rc = run()) return fail("a refused stream ends the run", rc, 0);
    if (error_of(a) != PYRO_EDEVICE) return fail("error of the refused job", error_of(a), PYRO_EDEVICE);
    if (last != hipSuccess) return fail("an error is left behind", last, 0);
    const int64_t b = submit(big);
    if (int rc = run()) return fail("second run", rc, 0);
    if (error_of(b) != PYRO_OK) return fail("the lane's next job", error_of(b), 0);
    // a refusal beside a running lane
    refuse = 1;
    const int64_t c = submit(4), d = submit(big - 20);
    if (int rc = run()) return fail("third run", rc, 0);
    if (error_of(c) != PYRO_EDEVICE || error_of(d) != PYRO_OK) return fail("other lanes run on", error_of(c), error_of(d));
    int64_t n = 0;
    if (pyro_sw_server_take(s, c, nullptr, 0, &n, nullptr, 0) != PYRO_EDEVICE) return fail("take", 0, 0);
    if (pyro_sw_server_destroy(s)) return fail("destroy", 0, 0);
    if (streams != 0) return fail("streams left", streams, 0);
    printf("server ok\n");
    return 0;
}
