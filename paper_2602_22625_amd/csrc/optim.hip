// Loss gradient and optimiser step (the `mse` loss and Adam optimiser of the paper's
// configuration, Supp. Table S1; here with a flat learning rate). Both are HBM-bound streams.
#include "dbmp_internal.h"
#include "diffbmp.h"

namespace dbmp {

__global__ void __launch_bounds__(256)
k_mse_grad(const float4 *__restrict__ img, const float4 *__restrict__ tgt, long long n4,
           const float *__restrict__ img1, const float *__restrict__ tgt1, long long n,
           float *__restrict__ grad, float scale, float *__restrict__ loss_sum)
{
    float acc = 0.f;
    const long long stride = (long long)gridDim.x * blockDim.x;
    float4 *g4 = (float4 *)grad;
    constexpr int U = 4;  // float4 loads in flight per thread
    for (long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x; i0 < n4;
         i0 += U * stride) {
        float4 a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = i0 + u * stride;
            if (i < n4) { a[u] = img[i]; b[u] = tgt[i]; }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = i0 + u * stride;
            if (i >= n4) continue;
            const float4 d = make_float4(a[u].x - b[u].x, a[u].y - b[u].y, a[u].z - b[u].z,
                                         a[u].w - b[u].w);
            g4[i] = make_float4(scale * d.x, scale * d.y, scale * d.z, scale * d.w);
            acc = fmaf(d.x, d.x, acc); acc = fmaf(d.y, d.y, acc);
            acc = fmaf(d.z, d.z, acc); acc = fmaf(d.w, d.w, acc);
        }
    }
    for (long long i = 4 * n4 + (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += stride) {
        const float d = img1[i] - tgt1[i];
        grad[i] = scale * d;
        acc = fmaf(d, d, acc);
    }
    if (!loss_sum) return;
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    __shared__ float ws[4];
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        // loss_sum[2] accumulates the block sums, loss_sum[1] counts finished blocks; the last
        // block publishes the total in loss_sum[0] and re-arms both for the next call
        unsafeAtomicAdd(loss_sum + 2, ws[0] + ws[1] + ws[2] + ws[3]);
        __threadfence();
        unsigned int *cnt = (unsigned int *)(loss_sum + 1);
        if (atomicAdd(cnt, 1u) == gridDim.x - 1) {
            __threadfence();
            loss_sum[0] = __hip_atomic_load(loss_sum + 2, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
            loss_sum[2] = 0.f;
            *cnt = 0u;
            __threadfence();
        }
    }
}

// At most ADAM_BLOCKS workgroups stride over the parameters: each ends with one atomic on the
// completion counter, and atomics on one address take about 14 ns each, one after the other (with
// a workgroup per 1,024 parameters, 1,919 of them cost 27 of the 33 us that 1.96 million
// parameters took).
constexpr int ADAM_THREADS = 1024;
constexpr int ADAM_BLOCKS = 256;

struct AdamCoef {
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_one(const AdamCoef &a, float &p, float g, float &m, float &v)
{
    m = fmaf(a.b1, m, (1.f - a.b1) * g);
    v = fmaf(a.b2, v, (1.f - a.b2) * g * g);
    const float mhat = m / a.c1, vhat = v / a.c2;
    p = p - a.lr * mhat / (sqrtf(vhat) + a.eps);
}

// n4: leading parameters taken four at a time, 16 bytes per load (0 if a buffer is not aligned)
__global__ void __launch_bounds__(ADAM_THREADS)
k_adam(float *__restrict__ p, float *__restrict__ g, float *__restrict__ m,
       float *__restrict__ v, long long n4, long long n, float lr, float b1, float b2, float eps,
       int *__restrict__ step, unsigned int *__restrict__ done, int zero_grad)
{
    const int t = *step + 1;
    const AdamCoef a{lr, b1, b2, eps, (float)(1.0 - beta_pow((double)b1, t)),
                     (float)(1.0 - beta_pow((double)b2, t))};
    const long long first = (long long)blockIdx.x * ADAM_THREADS + threadIdx.x;
    const long long stride = (long long)gridDim.x * ADAM_THREADS;
    for (long long i = first; i < n4 / 4; i += stride) {
        const float4 gq = reinterpret_cast<const float4 *>(g)[i];
        float4 mq = reinterpret_cast<float4 *>(m)[i], vq = reinterpret_cast<float4 *>(v)[i];
        float4 pq = reinterpret_cast<float4 *>(p)[i];
        if (zero_grad)  // ready for the next accumulating backward
            reinterpret_cast<float4 *>(g)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        adam_one(a, pq.x, gq.x, mq.x, vq.x);
        adam_one(a, pq.y, gq.y, mq.y, vq.y);
        adam_one(a, pq.z, gq.z, mq.z, vq.z);
        adam_one(a, pq.w, gq.w, mq.w, vq.w);
        reinterpret_cast<float4 *>(m)[i] = mq;
        reinterpret_cast<float4 *>(v)[i] = vq;
        reinterpret_cast<float4 *>(p)[i] = pq;
    }
    for (long long i = n4 + first; i < n; i += stride) {
        const float gi = g[i];
        if (zero_grad) g[i] = 0.f;
        float mi = m[i], vi = v[i], pi = p[i];
        adam_one(a, pi, gi, mi, vi);
        m[i] = mi;
        v[i] = vi;
        p[i] = pi;
    }
    // The last block to finish advances the step counter and re-arms the completion counter
    // for the next call. Every block read the step counter (and consumed the value) before its
    // barrier and counts itself done after it, so the last block writes after every read. No
    // fence: nothing else flows between blocks, and on gfx950 a device-scope fence writes back
    // the L2 (once per block it would dominate this kernel).
    __syncthreads();
    if (threadIdx.x == 0 &&
        __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
            gridDim.x - 1) {
        *step = t;
        *done = 0u;
    }
}

}  // namespace dbmp

using namespace dbmp;

extern "C" int dbmp_mse_grad(dbmp_stream stream, const float *image, const float *target,
                             long long n, float *grad, float *loss_sum)
{
    if (n < 0 || (n > 0 && (!image || !target || !grad))) return DBMP_EINVAL;
    if (n == 0) return DBMP_OK;
    hipStream_t st = (hipStream_t)stream;
    const bool aligned = (((uintptr_t)image | (uintptr_t)target | (uintptr_t)grad) & 15) == 0;
    const long long n4 = aligned ? n / 4 : 0;
    long long blocks = (n + 4095) / 4096;
    if (blocks > 256) blocks = 256;
    k_mse_grad<<<(unsigned)blocks, 256, 0, st>>>((const float4 *)image, (const float4 *)target,
                                                 n4, image, target, n, grad, 2.0f / (float)n,
                                                 loss_sum);
    return hipGetLastError() == hipSuccess ? DBMP_OK : DBMP_EHIP;
}

extern "C" int dbmp_adam_step(dbmp_stream stream, float *params, float *grad, float *m,
                              float *v, long long n, float lr, float beta1, float beta2,
                              float eps, int32_t *step, int zero_grad)
{
    if (n < 0 || !step || (n > 0 && (!params || !grad || !m || !v))) return DBMP_EINVAL;
    if (!(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return DBMP_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    const bool aligned =
        (((uintptr_t)params | (uintptr_t)grad | (uintptr_t)m | (uintptr_t)v) & 15) == 0;
    const long long n4 = aligned ? n / 4 * 4 : 0;
    const long long items = n4 > 0 ? (n + 3) / 4 : n;
    const long long blocks = (items + ADAM_THREADS - 1) / ADAM_THREADS;
    k_adam<<<(unsigned)(blocks < 1 ? 1 : blocks > ADAM_BLOCKS ? ADAM_BLOCKS : blocks),
             ADAM_THREADS, 0, st>>>(params, grad, m, v, n4, n, lr, beta1, beta2, eps, step,
                                    (unsigned int *)(step + 1), zero_grad);
    return hipGetLastError() == hipSuccess ? DBMP_OK : DBMP_EHIP;
}
