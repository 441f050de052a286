// Internal declarations shared by the host and device translation units of
// libplbm (not part of the public ABI).
#pragma once
#include <mutex>

#include "plbm.h"

namespace plbm {
int nq(const plbm_desc *d);
int validate(const plbm_desc *d);

// Records a failed HIP call for plbm_last_hip_error (plbm_kernels.hip).
void note_hip_error(const char *what, int code);

// Device memory for the partial sums of one call that asks for sums (`blocks`
// workgroups, nv doubles each, and nv results).  It is the library's static
// scratch while that is free and the stream belongs to the current device
// (allocating and freeing took 18 us of a 50 us call), else a stream-ordered
// allocation.  walks: the workgroups walk the tiles (see LaneSums), and `blocks` is
// lowered to what the scratch holds partials of, wherever they go in the end.
// Every sums_begin that returned PLBM_OK is followed by sums_end, which
// synchronises the stream before it gives the memory back.
struct SumsArea {
    double *part = nullptr;
    std::mutex *held = nullptr;   // of the scratch in use (null: allocated)
};
int sums_begin(SumsArea &a, int nv, int &blocks, bool walks, void *stream);
// rc: the status of the launches so far; reduces the partials, fetches and
// checks the nv sums.
int sums_end(SumsArea &a, int nv, int blocks, int rc, double *host, void *stream);

// What a call of several steps asks for besides the state.
struct StepCall {
    double *sums = nullptr;   // host: the sums after the last step
    bool keep = false;        // the other buffer ends with the state one step before
    bool noalloc = false;     // sums wait for the library's scratch rather than allocate
    // Of n steps, those that may share launches: not a last one that takes sums
    // or reads the state that is kept.
    int fusable(int n) const { return sums || keep ? n - 1 : n; }
};

// The isothermal three-velocity family (q1d = 3: D1Q3 and its tensor product
// D2Q9), plbm_q3.hip; the public plbm_init / plbm_step / plbm_moments forward
// to these.
int q3_init(const plbm_desc *d, const double *rho, const double *ux, const double *uy, void *f,
            void *stream);
int q3_step(const plbm_desc *d, void *f_a, void *f_b, int nsteps, const StepCall &call, void *stream);
int q3_moments(const plbm_desc *d, const void *f, double *rho, double *ux, double *uy,
               double *theta, double *sums, void *stream);

// General on-lattice velocity sets (plbm_gen.hip): every dim-1/2 descriptor
// with q1d = 3..7 that the symmetric kernels do not take.  The public
// plbm_init / plbm_step / plbm_moments forward here when gen_handles is true.
bool gen_handles(const plbm_desc *d);
int gen_init(const plbm_desc *d, const double *rho, const double *ux, const double *uy,
             const double *theta, void *f, void *stream);
int gen_step(const plbm_desc *d, void *f_a, void *f_b, int nsteps, const StepCall &call, void *stream);
int gen_moments(const plbm_desc *d, const void *f, double *rho, double *ux, double *uy,
                double *theta, double *sums, void *stream);

// The D3Q125 step (plbm_q125.hip); plbm_step forwards dim-3 descriptors here.
int q125_step(const plbm_desc *d, void *f_a, void *f_b, int nsteps, double *sums, void *stream);
} // namespace plbm
