// mc_io.hpp -- packs, tallies and fields between the device arrays and pinned
// host memory (gfx950).
//
// The kernels here read and write a pinned host buffer directly, in the layout
// of the caller's arrays: the FP32 form's pairs of floats are joined and split
// on the way, and one launch and one wait stand for a copy call per array.  A
// call of a pageable copy costs 16 us whatever its size; 13 of them made up a
// read of 1e4 packs (207 us, 88 us so; its write 195 -> 76 us), eight small
// ones a read of the tallies (188 -> 85 us).
#pragma once
#include "mc_kernels.hpp"
#include "mc_pool.hpp"

namespace mc {

// Pinned staging memory, lent for the length of one call: pieces of two halves
// each.
constexpr size_t kStageHalf = 2u << 20;
struct PinnedPiece {
    static char *make() {
        void *p = nullptr;
        // (coherent: the halves are read after an event, without a wait for the stream)
        const hipError_t e = hipHostMalloc(&p, 2 * kStageHalf, hipHostMallocPortable | hipHostMallocCoherent);
        return e == hipSuccess ? static_cast<char *>(p) : nullptr;
    }
    static void free(char *p) { (void)hipHostFree(p); }
};
inline StagePool<PinnedPiece> &stage_pool() {
    static StagePool<PinnedPiece> pool;
    return pool;
}

// The caller's pack arrays, in the order of mc_packs: nine FP64 fields, id, q,
// tag, status.  A staged pass holds n slots of each array that is asked for,
// one array after the other.
constexpr int kPackArrays = 13, kPackF64 = 9;
inline size_t pack_array_bytes(int k) { return k < kPackF64 + 2 ? 8 : 4; }

struct StagedPacks {
    char *base[kPackArrays];  // host memory that the device reaches; null: not asked for
    int64_t first, n;         // slots [first, first + n)
};

template <class T>
__global__ __launch_bounds__(256) void k_export_packs(PackPtrs<T> p, StagedPacks o) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, s = o.first + k;
    if (k >= o.n) return;
    const T *hi[kPackF64] = {p.x, p.y, p.z, p.vx, p.vy, p.vz, p.e, p.h, nullptr};
    const T *lo[kPackF64] = {p.xl, p.yl, p.zl, nullptr, nullptr, nullptr, p.el, nullptr, nullptr};
#pragma unroll
    for (int a = 0; a < kPackF64 - 1; ++a) {
        if (!o.base[a]) continue;
        double v = hi[a][s];
        if constexpr (sizeof(T) == 4)
            if (a < 3 || a == 6) v += (double)lo[a][s];
        reinterpret_cast<double *>(o.base[a])[k] = v;
    }
    if (o.base[8]) reinterpret_cast<double *>(o.base[8])[k] = p.w[s];
    if (o.base[9]) reinterpret_cast<int64_t *>(o.base[9])[k] = p.id[s];
    if (o.base[10]) reinterpret_cast<int64_t *>(o.base[10])[k] = p.q[s];
    if (o.base[11]) reinterpret_cast<int32_t *>(o.base[11])[k] = p.tag[s];
    if (o.base[12]) reinterpret_cast<int32_t *>(o.base[12])[k] = p.status[s];
}

// A snapshot's packs into their slots: status active, charge from the ion
// charge and the weight.  (q and status of the staged arrays are not read.)
template <class T>
__global__ __launch_bounds__(256) void k_import_packs(PackPtrs<T> p, const int32_t *charge, StagedPacks in) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, s = in.first + k;
    if (k >= in.n) return;
    double v[kPackF64];
#pragma unroll
    for (int a = 0; a < kPackF64; ++a) v[a] = reinterpret_cast<const double *>(in.base[a])[k];
    const int64_t id = reinterpret_cast<const int64_t *>(in.base[9])[k];
    const int32_t tag = reinterpret_cast<const int32_t *>(in.base[11])[k];
    T *hi[kPackF64 - 1] = {p.x, p.y, p.z, p.vx, p.vy, p.vz, p.e, p.h};
    T *lo[kPackF64 - 1] = {p.xl, p.yl, p.zl, nullptr, nullptr, nullptr, p.el, nullptr};
#pragma unroll
    for (int a = 0; a < kPackF64 - 1; ++a) {
        const T h = (T)v[a];
        hi[a][s] = h;
        if constexpr (sizeof(T) == 4)
            if (a < 3 || a == 6) lo[a][s] = (T)(v[a] - (double)h);
    }
    p.w[s] = v[8];
    p.id[s] = id;
    p.tag[s] = tag;
    p.q[s] = fx32((double)charge[tag] * v[8]);
    p.status[s] = ST_ACTIVE;
}

// Up to kGather device arrays of 64-bit words, one after the other.
constexpr int kGather = 8;
struct Gather {
    const unsigned long long *from[kGather];
    int64_t len[kGather];
};
static __global__ __launch_bounds__(256) void k_gather_words(Gather g, unsigned long long *out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int a = 0; a < kGather; ++a) {
        for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < g.len[a]; k += stride)
            out[k] = g.from[a][k];
        out += g.len[a];
    }
}

// The two components of a field, each to an array of its own (null: not asked for).
static __global__ __launch_bounds__(256) void k_export_field(const double2 *e, double *r, double *z, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const double2 v = e[k];
    if (r) r[k] = v.x;
    if (z) z[k] = v.y;
}

}  // namespace mc
