// mc_deposit_op.hip -- the cloud-in-cell charge deposit as a stand-alone
// operation on caller-owned device arrays ("Axisymmetric PIC space charge
// update": bilinear split of each pack's int64 charge onto the four nodes of
// its (r, z) cell, exact per pack).  Two entry points share the deposit kernel
// of the simulation context (k_deposit), which adds straight into the caller's
// grid after a kernel has zeroed it; neither takes scratch memory:
//
//   mc_deposit_cic          waits for the result
//   mc_deposit_cic_noalloc  asynchronous
#include <hip/hip_runtime.h>

#include <cstdint>

#include "mc_kernels.hpp"

using namespace mc;

namespace {

// Nodes of the largest grid the asynchronous entry point takes: a limit of its
// interface, which callers test for (no memory of its own sets it any more).
constexpr int64_t kNoAllocMaxNodes = 1ll << 20;

int32_t check_args(const mc_cic_packs *packs, const mc_grid *grid, const int64_t *q_out) {
    if (!packs || !grid || !q_out) return MC_EINVAL;
    if (grid->nr < 3 || grid->nz < 3 || !(grid->dr > 0.0) || !(grid->dz > 0.0)) return MC_EINVAL;
    if (packs->n < 0) return MC_EINVAL;
    if (packs->n > 0 && (!packs->x || !packs->y || !packs->z || !packs->q || !packs->status)) return MC_EINVAL;
    return MC_OK;
}

int32_t launch_deposit(const mc_cic_packs *packs, const mc_grid *grid, int64_t *q_out, hipStream_t stream) {
    const int64_t nn = (int64_t)grid->nr * grid->nz;
    unsigned long long *q = reinterpret_cast<unsigned long long *>(q_out);
    k_zero_u64<<<(unsigned)((nn + 255) / 256), 256, 0, stream>>>(q, nn);
    if (packs->n > 0) {
        DepositArgs<double> a{};
        a.p.x = const_cast<double *>(packs->x);
        a.p.y = const_cast<double *>(packs->y);
        a.p.z = const_cast<double *>(packs->z);
        a.p.q = const_cast<int64_t *>(packs->q);
        a.p.status = const_cast<int32_t *>(packs->status);
        a.q = q;
        a.n_slots = packs->n;
        a.inv_dr = 1.0 / grid->dr;
        a.inv_dz = 1.0 / grid->dz;
        a.nr = grid->nr;
        a.nz = grid->nz;
        unsigned nb;
        deposit_shape(packs->n, &nb, &a.chunk);
        k_deposit<P64><<<nb, kDepositThreads, 0, stream>>>(a);
    }
    return hipGetLastError() == hipSuccess ? MC_OK : MC_EDEVICE;
}

}  // namespace

extern "C" {

int32_t mc_deposit_cic(const mc_cic_packs *packs, const mc_grid *grid, int64_t *q_out, void *stream) {
    int32_t rc = check_args(packs, grid, q_out);
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    rc = launch_deposit(packs, grid, q_out, s);
    if (hipStreamSynchronize(s) != hipSuccess && !rc) rc = MC_EDEVICE;
    return rc;
}

int32_t mc_deposit_cic_noalloc(const mc_cic_packs *packs, const mc_grid *grid, int64_t *q_out, void *stream) {
    const int32_t rc = check_args(packs, grid, q_out);
    if (rc) return rc;
    if ((int64_t)grid->nr * grid->nz > kNoAllocMaxNodes) return MC_EINVAL;
    return launch_deposit(packs, grid, q_out, static_cast<hipStream_t>(stream));
}

}  // extern "C"
