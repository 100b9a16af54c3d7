#include "wreduce_kernels.hpp"

#include <algorithm>

#include "launch.hpp"

namespace canvas {
namespace wreduce {

namespace {

__device__ __forceinline__ unsigned quot(unsigned x, int d, uint32_t magic) { return magic ? __umulhi(x, magic) : x / (unsigned)d; }

// Sum of `segs` ranges of partials for VEC consecutive elements per thread.  A launch of this kernel is bound by the round trips of a
// thread and by the number of workgroups that have to be started (13 000 of them took 20-35 us for 19 MB), not by the bytes: a
// thread loads sixteen partials at once, four elements wide where there are enough of them, and a sum has no more segments than
// that takes (plan).  With one element per thread and 8 segments, 2 below 32 partials: 32 partials of 65 K and of 74 K elements 7.2 us, now 5.5; 8 of
// 262 K and of 295 K 8.4 / 5.6; 256 of 4 K and 228 of 9 K 7.0 / 6.1.
// The padding of the packed layout (whose element order differs from dw: the tap is innermost there) is skipped and the
// small result is written scattered.
// Order of the sum of one element: the partials of a segment in ascending blocks of sixteen and four, then the segments in
// ascending order -- independent of the launch.
template <int VEC>
__device__ __forceinline__ void reduce(const Job& J, float* red) {
    typedef float vec_t __attribute__((ext_vector_type(VEC)));
    const int per_wg = 256 / J.segs;
    const int el = (int)threadIdx.x & (per_wg - 1), seg = (int)threadIdx.x / per_wg;
    const unsigned idx = (blockIdx.x * (unsigned)per_wg + (unsigned)el) * VEC;
    const bool in = idx < J.count;
    vec_t sum = 0.f;
    if (in) {
        const int per = (J.slices + J.segs - 1) / J.segs;
        const int end = min(J.slices, (seg + 1) * per);
        const float* src = J.partial + idx;
        int k = seg * per;
        for (; k + 16 <= end; k += 16) {  // sixteen independent loads in flight (a round trip to memory each), added as a tree (a chain's rounding grows with its length)
            vec_t v[16];
#pragma unroll
            for (int i = 0; i < 16; i++) v[i] = *reinterpret_cast<const vec_t*>(src + (long long)(k + i) * J.count);
#pragma unroll
            for (int w = 1; w < 16; w *= 2)
#pragma unroll
                for (int i = 0; i < 16; i += 2 * w) v[i] += v[i + w];
            sum += v[0];
        }
        for (; k + 4 <= end; k += 4) {
            vec_t v[4];
#pragma unroll
            for (int i = 0; i < 4; i++) v[i] = *reinterpret_cast<const vec_t*>(src + (long long)(k + i) * J.count);
            sum += (v[0] + v[1]) + (v[2] + v[3]);
        }
        for (; k < end; k++) sum += *reinterpret_cast<const vec_t*>(src + (long long)k * J.count);
    }
    if (J.segs > 1) {
        vec_t* part = reinterpret_cast<vec_t*>(red);
        part[threadIdx.x] = sum;
        __syncthreads();
        if (seg == 0)
            for (int i = 1; i < J.segs; i++) sum += part[i * per_wg + el];
    }
    if (seg != 0 || !in) return;
    if (J.kind == 0) {
        *reinterpret_cast<vec_t*>(J.dw + idx) = sum;
        return;
    }
    // (Rp is a multiple of 16: the elements of a thread are rows of one output and tap)
    const unsigned t0 = quot(idx, J.Rp, J.magicRp), rp = idx - t0 * (unsigned)J.Rp;
    const unsigned t1 = quot(t0, J.TV, J.magicTV), tap = t0 - t1 * (unsigned)J.TV;
    const unsigned gmi = quot(t1, J.Omp, J.magicOmp), op = t1 - gmi * (unsigned)J.Omp;
    const unsigned sub = quot(op, J.Og, J.magicOg), o = op - sub * (unsigned)J.Og;
    const unsigned g = gmi * (unsigned)J.gm + sub;
    if ((int)sub >= J.gm || (int)g >= J.G) return;
#pragma unroll
    for (int i = 0; i < VEC; i++) {
        const unsigned subr = quot(rp + i, J.R, J.magicR), row = rp + i - subr * (unsigned)J.R;
        float x;
        if constexpr (VEC == 1) x = sum[0];
        else x = sum[i];
        if (subr == sub) J.dw[(((long long)g * J.Og + o) * J.R + row) * J.TV + tap] = x;
    }
}

// blockIdx.y selects the job.
__global__ __launch_bounds__(256) void k_reduce(Jobs jobs) {
    __shared__ __align__(16) float red[256 * 4];
    const Job& J = jobs.j[blockIdx.y];
    if (blockIdx.x >= J.blocks) return;  // (uniform per workgroup)
    if (J.vec == 4) reduce<4>(J, red);
    else reduce<1>(J, red);
}

}  // namespace

void plan(Job& job) {
    // four elements per thread from 128 K elements on: 16-byte loads and a quarter of the workgroups (one / four per thread, 8 partials of 262 K and 295 K elements 6.9 / 5.6 us; 32 of
    // 65 K and 74 K 5.5 / 6.6, 9 of 83 K 4.1 / 4.8: fewer elements do not fill the chip so)
    job.vec = job.count >= 131072 && job.count % 4 == 0 ? 4 : 1;
    job.segs = 1;
    while (job.segs < 16 && job.slices > 16 * job.segs) job.segs *= 2;
    const unsigned per_wg = 256u / (unsigned)job.segs * (unsigned)job.vec;
    job.blocks = (job.count + per_wg - 1) / per_wg;
    auto magic = [&](int d) { return d > 1 && (uint64_t)job.count * (uint64_t)d < ((uint64_t)1 << 32) ? (uint32_t)((((uint64_t)1 << 32) + (uint64_t)d - 1) / (uint64_t)d) : 0u; };
    if (job.kind != 0) {
        job.magicRp = magic(job.Rp);
        job.magicTV = magic(job.TV);
        job.magicOmp = magic(job.Omp);
        job.magicOg = magic(job.Og);
        job.magicR = magic(job.R);
    }
}

void run(const Jobs& jobs, hipStream_t s) {
    unsigned most = 0;
    for (int k = 0; k < jobs.n; k++) most = std::max(most, jobs.j[k].blocks);
    if (jobs.n > 0 && most > 0) CANVAS_LAUNCH(k_reduce, dim3(most, (unsigned)jobs.n), dim3(256), 0, s, jobs);
}

}  // namespace wreduce
}  // namespace canvas
