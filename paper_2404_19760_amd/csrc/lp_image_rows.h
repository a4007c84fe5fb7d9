// Whether a list of rays is made of the pixels of images, row after row, and how long a row is: kernels that take pixels of
// several rows together find it themselves, from the rays.
#pragma once
#include "lp_device.h"

namespace lp {

namespace {

constexpr int kMinRow = 8, kMaxRow = 4096;   // row lengths that are looked for

// Texels between the points of two rays at parameters t0 and t1.
__device__ __forceinline__ double texels_between(const GridDev& g, const RaysDev& rays, long long ray0, double t0, long long ray1, double t1)
{
#pragma clang fp contract(off)
    double sum = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double u[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const long long k = i ? ray1 : ray0;
            double x = (double)rays.origins[3 * k + a] + (i ? t1 : t0) * (double)rays.dirs[3 * k + a];
            if (g.contract > 0.0) {
                const double m = fabs(x), far = 0.5 * ((2.0 - g.contract) * (1.0 - 1.0 / fmax(m, 1.0)) + g.contract);
                x = m <= 1.0 ? 0.5 * g.contract * x : x < 0.0 ? -far : far;
            }
            u[i] = fmin(fmax((x - g.amin[a]) * g.scale[a], 0.0), (double)(g.N[a] - 1));
        }
        sum += (u[1] - u[0]) * (u[1] - u[0]);
    }
    return sqrt(sum);
}

// Length of a row if the list of rays looks like the pixels of images, row after row: the first ray whose end point is
// back near the first ray's, with the ray behind it and the one a row further on where they then have to be; and if neighbouring pixels are at most
// `pixel` texels apart in the middle of their rays (tested where the list is half over, then well inside an image), and consecutive points of a ray `step` texels.  0 otherwise.  All
// threads of the workgroup call it and receive the same value, and so does every workgroup and the other kernel of a pair, of
// which exactly one must find that the work is its own: no contraction of products and sums, which the compiler may choose
// differently in each.  `found`: in LDS, the caller's again when this returns.
__device__ __forceinline__ long long find_row(const GridDev& g, const RaysDev& rays, double pixel, double step, int& found)
{
#pragma clang fp contract(off)
    auto end_point = [&](long long k, float (&p)[3]) {
#pragma clang fp contract(off)
        const float t = rays.far[k];
#pragma unroll
        for (int a = 0; a < 3; ++a) p[a] = rays.origins[3 * k + a] + t * rays.dirs[3 * k + a];
    };
    auto distance2 = [](const float (&a)[3], const float (&b)[3]) {
#pragma clang fp contract(off)
        const float x = a[0] - b[0], y = a[1] - b[1], z = a[2] - b[2];
        return x * x + y * y + z * z;
    };
    float p0[3], p1[3], p2[3];
    const long long last = rays.M - 1;
    end_point(0, p0);
    end_point(min(1LL, last), p1);
    end_point(min(2LL, last), p2);
    const float along = distance2(p0, p1);   // of one pixel, squared
    const float ahead[3] = {p1[0] - p0[0], p1[1] - p0[1], p1[2] - p0[2]};
    // the second pixel's step is the first's
    const float two[3] = {p1[0] + ahead[0], p1[1] + ahead[1], p1[2] + ahead[2]};
    if (!(distance2(two, p2) < 0.25f * along)) return 0;
    // Pixels far apart: no row to look for.  (Two pairs of neighbours, one of which may lie across two rows; in contract
    // coordinates pixels may be nearer each other in the middle of an image than here.  Looking for a row takes 4 us: 2112 rays x 64 points into 86^3 x 16 voxels, 1.4 texels a pixel, are pushed in 111.)
    const long long mid = last / 2;
    const double t_mid = 0.5 * ((double)rays.near[mid] + (double)rays.far[mid]);
    if (!(g.contract > 0.0) && texels_between(g, rays, mid, t_mid, mid + 1, t_mid) > pixel && texels_between(g, rays, mid + 1, t_mid, min(mid + 2, last), t_mid) > pixel) return 0;
    if (threadIdx.x == 0) found = 0x7fffffff;
    __syncthreads();
    const long long limit = min((long long)kMaxRow, last / 2);   // (rays k + 1 and 2 k exist)
    int row = 0x7fffffff;
    for (long long k0 = kMinRow; k0 <= limit; k0 += blockDim.x) {
        const long long k = k0 + threadIdx.x;
        if (k <= limit) {
            float before[3], here[3], next[3], below[3];
            end_point(k - 1, before);
            end_point(k, here);
            end_point(k + 1, next);
            end_point(2 * k, below);
            const float want[3] = {here[0] + ahead[0], here[1] + ahead[1], here[2] + ahead[2]};
            const float want_below[3] = {here[0] + (here[0] - p0[0]), here[1] + (here[1] - p0[1]), here[2] + (here[2] - p0[2])};
            const float back = distance2(here, p0);
            if (back < 16.0f * along && back < 0.25f * distance2(before, p0) && distance2(next, want) < 0.25f * along &&
                distance2(below, want_below) < 0.25f * back)
                atomicMin(&found, (int)k);
        }
        __syncthreads();
        row = found;
        __syncthreads();
        if (row != 0x7fffffff) break;
    }
    if (row == 0x7fffffff) return 0;
    {   // half a row further on the step to the next row is much the same
        float here[3], half[3], half_below[3];
        end_point(row, here);
        end_point(row / 2, half);
        end_point(row + row / 2, half_below);
        const float want[3] = {half[0] + (here[0] - p0[0]), half[1] + (here[1] - p0[1]), half[2] + (here[2] - p0[2])};
        if (!(distance2(half_below, want) < 0.25f * distance2(here, p0))) return 0;
    }
    // a pixel in the middle of a row, well inside an image (the rays of its corners may leave the structure)
    const long long k = min(rays.M / row - 1, (long long)row / 2) * row + row / 2;
    const double t = 0.5 * ((double)rays.near[k] + (double)rays.far[k]);
    const double ahead_t = t + ((double)rays.far[k] - (double)rays.near[k]) / (double)rays.S;
    return texels_between(g, rays, k, t, k + 1, t) <= pixel && texels_between(g, rays, k, t, k, ahead_t) <= step ? row : 0;
}

}  // namespace

}  // namespace lp
