// 3-D gamma index (Low et al.; the paper evaluates its plan re-calculations
// with the 3-D gamma computed on the GPU, Sec. II.D): a few lanes per reference
// voxel, a cubic search grid around its centre with trilinear interpolation of
// the evaluated distribution.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>

#include "pmc_unet.h"

namespace pmc {

namespace {

// trilinear interpolation at continuous voxel coordinates (voxel centres at
// integers); the caller keeps the point inside [0, n-1] on every axis
__device__ double trilinear(const double* __restrict__ e, int nx, int ny, int nz, float fx, float fy, float fz)
{
    const int x0 = min((int)fx, nx - 1), y0 = min((int)fy, ny - 1), z0 = min((int)fz, nz - 1);
    const int x1 = min(x0 + 1, nx - 1), y1 = min(y0 + 1, ny - 1), z1 = min(z0 + 1, nz - 1);
    const double tx = fx - x0, ty = fy - y0, tz = fz - z0;
    // the cell's corners as steps from its first one (0 where an axis ends)
    const size_t sx = x1 - x0, sy = (size_t)(y1 - y0) * nx, sz = (size_t)(z1 - z0) * ny * nx;
    const double* c = e + ((size_t)z0 * ny + y0) * nx + x0;
    const double* d = c + sz;
    const double c00 = c[0] * (1 - tx) + c[sx] * tx;
    const double c10 = c[sy] * (1 - tx) + c[sy + sx] * tx;
    const double c01 = d[0] * (1 - tx) + d[sx] * tx;
    const double c11 = d[sy] * (1 - tx) + d[sy + sx] * tx;
    const double c0 = c00 * (1 - ty) + c10 * ty, c1 = c01 * (1 - ty) + c11 * ty;
    return c0 * (1 - tz) + c1 * tz;
}

// Reductions without atomics: a kernel of at most kRedBlocks workgroups
// (kMaxBlocks for the maximum, which the next kernel's workgroups all read) leaves
// one value per workgroup, and the next kernel (or the host) combines them.
// (One atomic per wave on a shared counter serialises at about 12 ns: with
// 16,384 waves and two counters the fallback rule's count took 397 us on
// 160 x 128 x 128 voxels, the maximum 105 us.)
constexpr int kMaxBlocks = 512;
constexpr int kRedBlocks = 2048;

__device__ double block_max(double m, double* sh)
{
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    __syncthreads();
    return m;
}

// partial[b] = the largest value workgroup b sees, at least 0 (NaN ignored)
__global__ void __launch_bounds__(256) max_partials_kernel(const double* __restrict__ a, size_t n,
                                                           double* __restrict__ partial)
{
    __shared__ double sh[4];
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0;
    // four independent loads in flight per lane
    for (; i + 3 * stride < n; i += 4 * stride) {
        const double v0 = a[i], v1 = a[i + stride], v2 = a[i + 2 * stride], v3 = a[i + 3 * stride];
        m0 = fmax(m0, v0);
        m1 = fmax(m1, v1);
        m2 = fmax(m2, v2);
        m3 = fmax(m3, v3);
    }
    for (; i < n; i += stride) m0 = fmax(m0, a[i]);
    const double m = block_max(fmax(fmax(m0, m1), fmax(m2, m3)), sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = m;
}

// the maximum over the workgroups' partials (every lane of the block)
__device__ double max_of_partials(const double* __restrict__ partial, int n, double* sh)
{
    double m = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) m = fmax(m, partial[i]);
    return block_max(m, sh);
}

// the workgroup's two counts to counts[2 b], counts[2 b + 1]
__device__ void block_counts(unsigned long long c0, unsigned long long c1, unsigned long long (*sh)[2],
                             unsigned long long* __restrict__ counts)
{
    for (int o = 32; o > 0; o >>= 1) {
        c0 += __shfl_xor(c0, o);
        c1 += __shfl_xor(c1, o);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6][0] = c0;
        sh[threadIdx.x >> 6][1] = c1;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        counts[2 * blockIdx.x + threadIdx.x] =
            sh[0][threadIdx.x] + sh[1][threadIdx.x] + sh[2][threadIdx.x] + sh[3][threadIdx.x];
}

// The search offsets (i, j, k) with i^2 + j^2 + k^2 <= kNear^2 in order of
// their distance, and how many have a squared distance up to n.
constexpr int kNear = 8;
constexpr int kNearCount = 2109;
struct NearOffsets {
    signed char at[kNearCount][4];
    int upto[kNear * kNear + 1];
};
constexpr NearOffsets near_offsets()
{
    NearOffsets t{};
    int fill[kNear * kNear + 1] = {};
    for (int pass = 0; pass < 2; ++pass) {
        if (pass == 1)
            for (int n = 0, sum = 0; n <= kNear * kNear; ++n) {
                const int c = fill[n];
                fill[n] = sum;
                sum += c;
                t.upto[n] = sum;
            }
        for (int k = -kNear; k <= kNear; ++k)
            for (int j = -kNear; j <= kNear; ++j)
                for (int i = -kNear; i <= kNear; ++i) {
                    const int n = i * i + j * j + k * k;
                    if (n > kNear * kNear) continue;
                    const int e = fill[n]++;
                    if (pass == 0) continue;
                    t.at[e][0] = (signed char)i;
                    t.at[e][1] = (signed char)j;
                    t.at[e][2] = (signed char)k;
                }
    }
    return t;
}
__device__ const NearOffsets kOffsets = near_offsets();
constexpr NearOffsets kOffsetsHost = near_offsets();
static_assert(kOffsetsHost.upto[kNear * kNear] == kNearCount, "offsets within the near sphere");

// Gamma index.  A workgroup takes runs of kGammaRun voxels, lists those at or
// above the cutoff in LDS and hands each to a group of kGroup lanes.  The
// lanes evaluate kGroup offsets at a time, nearest first (staged in LDS with
// their distance terms), and share the smallest value after each round; the
// group stops at the first offset whose distance term alone exceeds it, which
// bounds every farther one too, so the minimum is that of the whole sphere.
// A voxel not settled within the first kFirst offsets (a large gamma: it
// needs most of the sphere) is left to a whole wave.  What bounds it: the
// latency of the eight gathers of a round, about 1.2 us, and of the longest
// voxel's chain of rounds, hence many lanes per voxel.  160 x 128 x 128
// voxels (39,689 above the cutoff), 2%/2 mm, 3 mm search at 0.5 mm: one voxel
// per lane walking all 2,197 offsets of the cube in order 1,426 us, groups of
// eight lanes alone 148 us (one voxel at gamma 2.5 takes 116 rounds), with
// the waves 82 us.  Offsets beyond kNear steps (a search radius of more than 8
// steps) are walked after the near ones by the same wave, a plane of them 64 at
// a time.
//   Runs with half their voxels or more above the cutoff are left to a second
// launch (kDenseRuns), made only where there are any: one voxel per lane, every
// lane of a wave at the same offset until none needs a farther one, half a run
// per workgroup.  What bounds it: the L1's bandwidth for the gathers, which of
// neighbouring voxels fall into the same lines, where those of one voxel's
// offsets scatter.  160 x 128 x 128 voxels, all above the cutoff, 2%/2 mm, the
// evaluated dose 30% off everywhere (every voxel searches the whole sphere):
// 15.5 ms with groups and waves, 8.5 so, with a search of 6 mm 351 and 66 (80 x
// 64 x 64 voxels 61 and 8.4, 9.8 with the whole near sphere in LDS and four
// workgroups a CU).
constexpr int kGammaRun = 512;
constexpr int kGroup = 8;
constexpr int kFirst = 65;   // the zero offset and eight rounds of a group
constexpr int kDense = kGammaRun / 2;
constexpr int kDenseBlocks = 5 * 256;   // as many as are resident
// the near sphere's radius in steps: of a dense run smaller, so that its offsets
// leave LDS for five workgroups a CU
constexpr int near_steps(bool dense) { return dense ? 7 : kNear; }
constexpr unsigned long long kDenseUnit = 1ull << 40;   // a dense run in the count of voxels evaluated
template <bool kDenseRuns>
__global__ void __launch_bounds__(256) gamma_kernel(const double* __restrict__ ref, const double* __restrict__ ev,
                                                    int nx, int ny, int nz, float dx, float dy, float dz,
                                                    const double* __restrict__ partial, int n_partial,
                                                    float dose_frac, float dta, float cutoff, float search,
                                                    float step, int n_near, float* __restrict__ gamma,
                                                    unsigned long long* __restrict__ counts)
{
    constexpr int kSteps = near_steps(kDenseRuns);
    __shared__ double sh[4];
    __shared__ unsigned long long shc[4][2];
    extern __shared__ float4 near[];   // n_near entries: offset in voxels, distance term (negative: not in the sphere)
    __shared__ unsigned short list[kGammaRun], late[kGammaRun];
    __shared__ double late_best[kGammaRun];
    __shared__ int n_list, n_late, n_other;
    __shared__ float far_x[kDenseRuns ? 2 * 64 + 1 : 1];   // offsets along x in voxels (search / step <= 64)
    const int nsteps = (int)floorf(search / step + 1e-4f);
    const bool far = search > step * (kSteps + 0.01f);   // the next shell lies at sqrt(kSteps^2 + 1) steps
    auto dist_term = [&](int i, int j, int k, float& d2) {
        const float ox = i * step, oy = j * step, oz = k * step;
        d2 = ox * ox + oy * oy + oz * oz;
        return d2 / (dta * dta);
    };
    for (int e = threadIdx.x; e < n_near; e += blockDim.x) {
        const int i = kOffsets.at[e][0], j = kOffsets.at[e][1], k = kOffsets.at[e][2];
        float d2;
        const float dist = dist_term(i, j, k, d2);
        const bool in = abs(i) <= nsteps && abs(j) <= nsteps && abs(k) <= nsteps &&
                        !(d2 > search * search * (1.0f + 1e-6f));
        near[e] = make_float4(i * step / dx, j * step / dy, k * step / dz, in ? dist : -1.f);
    }
    if (kDenseRuns && far)
        for (int i = threadIdx.x; i <= 2 * nsteps; i += blockDim.x) far_x[i] = (i - nsteps) * step / dx;
    const double dmax = max_of_partials(partial, n_partial, sh);   // (with its barriers)
    const double crit = dose_frac * dmax;
    // a value that cannot be the smallest needs no division (a bound with a margin
    // far above its roundings, unless crit^2 leaves the range of doubles)
    const double crit2 = crit * crit * (1.0 + 1e-9);
    const bool screen = crit2 > 1e-280 && crit2 < 1e280;
    const size_t nv = (size_t)nx * ny * nz;
    const int lane = threadIdx.x & 63;
    unsigned long long n_eval = 0, n_pass = 0;
    // the offset's gamma^2 at a voxel into best
    auto offer = [&](int x, int y, int z, double r, float fx, float fy, float fz, double dist, double& best) {
        const float px = x + fx, py = y + fy, pz = z + fz;
        // points outside the grid carry no evaluated dose: skipped
        if (px < 0.f || py < 0.f || pz < 0.f || px > nx - 1 || py > ny - 1 || pz > nz - 1) return;
        const double diff = trilinear(ev, nx, ny, nz, px, py, pz) - r;
        if (kDenseRuns && screen && diff * diff > (best - dist) * crit2) return;
        const double dd = diff / crit;
        const double g2 = dist + dd * dd;
        if (g2 < best) best = g2;
    };
    // the smallest value of `width` neighbouring lanes to all of them
    auto share = [&](double& best, int width) {
        for (int o = width / 2; o > 0; o >>= 1) {
            const double other = __shfl_xor(best, o);
            if (other < best) best = other;
        }
    };
    // near offsets e0 .. e_end - 1, `width` lanes at a time; true once every
    // farther offset is too far to matter (the distances of one shell differ
    // in the last bits: the margin keeps a shell open until all of it is)
    auto walk = [&](int e0, int e_end, int sub, int width, int x, int y, int z, double r, double& best) {
        for (; e0 < e_end; e0 += width) {
            const float first = near[e0].w;
            if (first >= 0.f && (double)(first * (1.0f - 2e-6f)) >= best) return true;
            const int e = e0 + sub;
            if (e < e_end) {
                const float4 o = near[e];
                if (o.w >= 0.f && !((double)o.w >= best)) offer(x, y, z, r, o.x, o.y, o.z, (double)o.w, best);
            }
            share(best, width);
        }
        return false;
    };
    // near offsets e0 .. e_end - 1 and, with beyond, the ones past the near sphere,
    // for a voxel per lane
    auto walk_alone = [&](int e0, int e_end, bool beyond, int x, int y, int z, double r, double& best) {
        auto shut = [&](float d) { return (double)(d * (1.0f - 2e-6f)) >= best; };
        for (int e = e0; e < e_end; ++e) {
            const float4 o = near[e];
            if (o.w < 0.f) continue;
            if (__ballot(!shut(o.w)) == 0ull) return;
            if (!((double)o.w >= best)) offer(x, y, z, r, o.x, o.y, o.z, (double)o.w, best);
        }
        if (!beyond) return;
        for (int k = -nsteps; k <= nsteps; ++k)
            for (int j = -nsteps; j <= nsteps; ++j) {
                float d2;
                if (__ballot(!shut(dist_term(0, j, k, d2))) == 0ull || d2 > search * search * (1.0f + 1e-5f)) continue;
                for (int i = -nsteps; i <= nsteps; ++i) {
                    const double dist = dist_term(i, j, k, d2);
                    if (i * i + j * j + k * k <= kSteps * kSteps || d2 > search * search * (1.0f + 1e-6f)) continue;
                    if (!(dist >= best)) offer(x, y, z, r, far_x[i + nsteps], j * step / dy, k * step / dz, dist, best);
                }
            }
    };
    auto locate = [&](size_t v, int& x, int& y, int& z) {
        if (nv <= 0xFFFFFFFFull) {   // 32-bit divisions where they hold the index
            const uint32_t row = (uint32_t)v / (uint32_t)nx;
            x = (int)((uint32_t)v - row * (uint32_t)nx);
            z = (int)(row / (uint32_t)ny);
            y = (int)(row - (uint32_t)z * (uint32_t)ny);
        } else {
            x = (int)(v % nx);
            y = (int)((v / nx) % ny);
            z = (int)(v / ((size_t)nx * ny));
        }
    };
    auto finish = [&](size_t v, double best) {
        const double g = sqrt(best);
        if (gamma) gamma[v] = (float)g;
        ++n_eval;
        n_pass += g <= 1.0;
    };
    const size_t n_work = (nv + kGammaRun - 1) / kGammaRun * (kDenseRuns ? 2 : 1);
    for (size_t u = blockIdx.x; u < n_work; u += gridDim.x) {
        const size_t v0 = (kDenseRuns ? u / 2 : u) * kGammaRun;
        __syncthreads();   // the previous run's lists are no longer read
        if (threadIdx.x == 0) n_list = n_late = n_other = 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kGammaRun / 256; ++q) {
            const size_t v = v0 + q * 256 + threadIdx.x;
            const double r = v < nv ? ref[v] : 0.0;
            const bool take = v < nv && r >= cutoff * dmax && !(dmax <= 0.0);
            const unsigned long long m = __ballot(take);
            if constexpr (kDenseRuns) {
                if (q != (int)(u & 1)) {   // the other half's
                    if (lane == 0 && m) atomicAdd(&n_other, __popcll(m));
                    continue;
                }
            } else {
                if (v < nv && !take && gamma) gamma[v] = -1.f;
            }
            int base = 0;
            if (lane == 0 && m) base = atomicAdd(&n_list, __popcll(m));
            base = __shfl(base, 0);
            if (take) list[base + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)(q * 256 + threadIdx.x);
        }
        __syncthreads();
        const int n = n_list;
        if (((kDenseRuns ? n + n_other : n) >= kDense) != kDenseRuns) {
            if (!kDenseRuns && threadIdx.x == 0) n_eval += kDenseUnit;
            continue;
        }
        const int first_end = min(kFirst, n_near);
        for (int t = threadIdx.x; kDenseRuns && t < n; t += 256) {
            const size_t v = v0 + list[t];
            const double r = ref[v];
            int x, y, z;
            locate(v, x, y, z);
            const double d0 = (ev[v] - r) / crit;
            double best = d0 * d0;
            walk_alone(1, first_end, false, x, y, z, r, best);
            const float next = first_end < n_near ? near[first_end].w : -1.f;
            if (first_end == n_near ? !far : next >= 0.f && (double)(next * (1.0f - 2e-6f)) >= best) {
                finish(v, best);
            } else {
                const int q = atomicAdd(&n_late, 1);
                late[q] = list[t];
                late_best[q] = best;
            }
        }
        for (int t = threadIdx.x / kGroup; !kDenseRuns && t < n; t += 256 / kGroup) {
            const int sub = threadIdx.x & (kGroup - 1);
            const size_t v = v0 + list[t];
            const double r = ref[v];
            int x, y, z;
            locate(v, x, y, z);
            // the zero offset first (interpolation at a voxel centre is exact)
            const double d0 = (ev[v] - r) / crit;
            double best = d0 * d0;
            const bool settled = walk(1, first_end, sub, kGroup, x, y, z, r, best);
            if (sub == 0) {
                if (settled || (first_end == n_near && !far)) {
                    finish(v, best);
                } else {
                    const int q = atomicAdd(&n_late, 1);
                    late[q] = list[t];
                    late_best[q] = best;
                }
            }
        }
        __syncthreads();
        // (of a dense run's many late voxels whole waves)
        const int whole = kDenseRuns && n_late >= kDense / 2 ? n_late & ~63 : 0;
        for (int t = threadIdx.x; kDenseRuns && t < whole; t += 256) {
            const size_t v = v0 + late[t];
            const double r = ref[v];
            double best = late_best[t];
            int x, y, z;
            locate(v, x, y, z);
            walk_alone(first_end, n_near, far, x, y, z, r, best);
            finish(v, best);
        }
        for (int t = whole + (threadIdx.x >> 6); t < n_late; t += 4) {
            const size_t v = v0 + late[t];
            const double r = ref[v];
            double best = late_best[t];
            int x, y, z;
            locate(v, x, y, z);
            if (!walk(first_end, n_near, lane, 64, x, y, z, r, best) && far) {
                const int side = 2 * nsteps + 1;
                for (int k = -nsteps; k <= nsteps; ++k) {
                    for (int j = lane / side - nsteps, i = lane % side - nsteps; j <= nsteps;) {
                        float d2;
                        const double dist = dist_term(i, j, k, d2);
                        if (i * i + j * j + k * k > kSteps * kSteps && !(d2 > search * search * (1.0f + 1e-6f)) && !(dist >= best))
                            offer(x, y, z, r, i * step / dx, j * step / dy, k * step / dz, dist, best);
                        j += 64 / side;
                        i += 64 % side;
                        if (i > nsteps) {
                            i -= side;
                            ++j;
                        }
                    }
                    share(best, 64);
                }
            }
            if (lane == 0) finish(v, best);
        }
    }
    block_counts(n_eval, n_pass, shc, counts);
}

__global__ void __launch_bounds__(256) disagreement_kernel(const float* __restrict__ den,
                                                           const double* __restrict__ mc,
                                                           const double* __restrict__ var, size_t n,
                                                           const double* __restrict__ partial, int n_partial,
                                                           float cutoff, float k,
                                                           unsigned long long* __restrict__ counts)
{
    __shared__ double sh[4];
    __shared__ unsigned long long shc[4][2];
    const double thr = cutoff * max_of_partials(partial, n_partial, sh);
    unsigned long long above = 0, off = 0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const double m = mc[i];
        if (!(m >= thr) || m <= 0.0) continue;
        ++above;
        off += fabs((double)den[i] - m) > k * sqrt(fmax(var[i], 0.0));
    }
    block_counts(above, off, shc, counts);
}

// What the two entry points below keep per device from its first call on
// (nothing is allocated afterwards): the workgroups' maxima on the device and
// their counts in pinned host memory that the kernels write to directly, so
// that a call is two launches and one wait (three and two of pmc_gamma_index
// where it meets dense runs).  The calls are serialised within
// the process, since they share these until the counts have been read.
struct Reduction {
    double* partial = nullptr;
    unsigned long long* counts = nullptr;
};
std::mutex g_reduction_mu;
std::map<int, Reduction> g_reductions;

hipError_t device_reduction(Reduction* out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    auto it = g_reductions.find(dev);
    if (it == g_reductions.end()) {
        Reduction r;
        e = hipMalloc((void**)&r.partial, kMaxBlocks * sizeof(double));
        if (e != hipSuccess) return e;
        e = hipHostMalloc((void**)&r.counts, 2 * kRedBlocks * sizeof(unsigned long long), hipHostMallocDefault);
        if (e != hipSuccess) {
            (void)hipFree(r.partial);
            return e;
        }
        it = g_reductions.emplace(dev, r).first;
    }
    *out = it->second;
    return hipSuccess;
}

unsigned red_blocks(size_t n, size_t per_block, int most)
{
    return (unsigned)std::min<size_t>((n + per_block - 1) / per_block, (size_t)most);
}

// waits for the stream and adds up the workgroups' counts
hipError_t read_counts(const Reduction& r, unsigned blocks, hipStream_t s, unsigned long long* c0,
                       unsigned long long* c1)
{
    const hipError_t e = hipStreamSynchronize(s);
    *c0 = *c1 = 0;
    for (unsigned b = 0; e == hipSuccess && b < blocks; ++b) {
        *c0 += r.counts[2 * b];
        *c1 += r.counts[2 * b + 1];
    }
    return e;
}

}  // namespace

}  // namespace pmc

extern "C" pmc_status pmc_denoise_disagreement(const float* den, const double* mc, const double* var, int64_t n,
                                              float cutoff, float k, double* frac_out, int64_t* n_out, void* stream)
{
    if (!den || !mc || !var || !frac_out || n <= 0 || !(cutoff >= 0) || !(k > 0)) return PMC_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    std::lock_guard<std::mutex> lock(pmc::g_reduction_mu);
    pmc::Reduction red;
    if (pmc::device_reduction(&red) != hipSuccess) return PMC_ERR_NOMEM;
    const unsigned max_blocks = pmc::red_blocks((size_t)n, 256, pmc::kMaxBlocks);
    const unsigned blocks = pmc::red_blocks((size_t)n, 256, pmc::kRedBlocks);
    hipLaunchKernelGGL(pmc::max_partials_kernel, dim3(max_blocks), dim3(256), 0, s, mc, (size_t)n, red.partial);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        hipLaunchKernelGGL(pmc::disagreement_kernel, dim3(blocks), dim3(256), 0, s, den, mc, var, (size_t)n,
                           red.partial, (int)max_blocks, cutoff, k, red.counts);
        e = hipGetLastError();
    }
    unsigned long long above = 0, off = 0;
    if (e == hipSuccess) e = pmc::read_counts(red, blocks, s, &above, &off);
    if (e != hipSuccess) return PMC_ERR_DEVICE;
    *frac_out = above ? (double)off / (double)above : 0.0;
    if (n_out) *n_out = (int64_t)above;
    return PMC_OK;
}

extern "C" pmc_status pmc_gamma_index(const double* ref, const double* ev, int nx, int ny, int nz, float dx,
                                      float dy, float dz, float dose_frac, float dta, float cutoff, float search,
                                      float step, float* gamma, double* pass_rate, int64_t* n_eval, void* stream)
{
    if (!ref || !ev || !pass_rate || nx <= 0 || ny <= 0 || nz <= 0 || !(dx > 0) || !(dy > 0) || !(dz > 0) ||
        !(dose_frac > 0) || !(dta > 0) || !(cutoff >= 0) || !(search >= 0) || !(step > 0) || search / step > 64)
        return PMC_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    std::lock_guard<std::mutex> lock(pmc::g_reduction_mu);
    pmc::Reduction red;
    if (pmc::device_reduction(&red) != hipSuccess) return PMC_ERR_NOMEM;
    const size_t nv = (size_t)nx * ny * nz;
    const unsigned max_blocks = pmc::red_blocks(nv, 256, pmc::kMaxBlocks);
    // the near offsets that can lie in the search sphere
    const double r2 = (double)search / step * ((double)search / step) * 1.001 + 1.0;
    hipLaunchKernelGGL(pmc::max_partials_kernel, dim3(max_blocks), dim3(256), 0, s, ref, nv, red.partial);
    hipError_t e = hipGetLastError();
    unsigned long long evaluated = 0, passed = 0;
    // the runs with few voxels above the cutoff, then, if there are others, these
    // (found by the first launch, so the second waits for its counts)
    for (bool dense : {false, true}) {
        if (dense && evaluated < pmc::kDenseUnit) break;
        evaluated %= pmc::kDenseUnit;
        const int steps = pmc::near_steps(dense);
        const int n_near = pmc::kOffsetsHost.upto[(int)std::min((double)(steps * steps), r2)];
        const unsigned blocks = dense ? pmc::red_blocks(nv, pmc::kGammaRun / 2, pmc::kDenseBlocks)
                                      : pmc::red_blocks(nv, pmc::kGammaRun, pmc::kRedBlocks);
        unsigned long long c0 = 0, c1 = 0;
        if (e == hipSuccess) {
            hipLaunchKernelGGL(dense ? pmc::gamma_kernel<true> : pmc::gamma_kernel<false>, dim3(blocks), dim3(256),
                               n_near * sizeof(float4), s, ref, ev, nx, ny, nz, dx, dy, dz, red.partial, (int)max_blocks, dose_frac,
                               dta, cutoff, search, step, n_near, gamma, red.counts);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = pmc::read_counts(red, blocks, s, &c0, &c1);
        evaluated += c0;
        passed += c1;
    }
    if (e != hipSuccess) return PMC_ERR_DEVICE;
    *pass_rate = evaluated ? (double)passed / (double)evaluated : 1.0;
    if (n_eval) *n_eval = (int64_t)evaluated;
    return PMC_OK;
}
