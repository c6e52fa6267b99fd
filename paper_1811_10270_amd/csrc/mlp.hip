// Multilayer perceptron for the learned GMRES initial guess: nlayers hidden
// layers of nhidden ReLU units and a linear output, FP32, trained with Adam
// on a mean-squared error.  Every step runs in the kernels of this file:
// the GEMMs X W, dZ W^T and X^T dZ on FP32 MFMA with the bias, ReLU and ReLU
// derivative in their epilogues, the bias-gradient column sums, the loss and
// its gradient, and Adam.
//
// Parameter layout (host and device): for each layer l (0 .. nlayers), the
// weights W_l [in_l][out_l] row-major, then the bias b_l [out_l].

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "ehdbim.h"

struct ehd_mlp {
    int device = 0;
    hipStream_t stream = nullptr;
    int nin = 0, nhid = 0, nlay = 0, nout = 0;
    std::vector<int> din, dout;         // per layer
    std::vector<long long> woff, boff;  // offsets into the parameter vector
    long long nparam = 0;
    float *w = nullptr, *g = nullptr, *m1 = nullptr, *m2 = nullptr;
    long long adam_t = 0;
    int cap = 0;                        // batch capacity of the activations
    std::vector<float*> act;            // act[0] = input copy, act[l+1] = output of layer l
    float *dA = nullptr, *dB = nullptr; // backward scratch [cap][max width]
    float* part = nullptr;              // products split over K
    float* red = nullptr;               // loss reduction scratch
    std::string err;
};

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
constexpr int kT = 256;

// C[M][N] = sum_k A(i,k) B(k,j), C row-major, then per element + bias[j],
// ReLU, and times (mask > 0), each where asked for.
struct Epilogue {
    const float* bias;
    const float* mask;
    int relu;
    __device__ __forceinline__ float operator()(float v, long long i, int j, int N) const
    {
        if (bias) v += bias[j];
        if (relu) v = v > 0.0f ? v : 0.0f;
        if (mask) v = mask[i * N + j] > 0.0f ? v : 0.0f;
        return v;
    }
};

// Block: 4 waves, a 64x64 tile in K steps of 32 through LDS (two buffers, the
// next step's loads in flight during the products); wave: 32x32 (2x2 MFMA
// tiles of 16x16).  MFMA f32 16x16x4: lane holds A[lane%16][lane/16] and
// B[lane/16][lane%16]; element r of the result is row 4 (lane/16) + r, column
// lane%16.  KA: A(i,k) = A[i lda + k], else A[k lda + i]; KB: B(k,j) = B[j ldb + k],
// else B[k ldb + j].  An operand contiguous in k keeps rows of 36 in LDS, one
// contiguous in i or j rows of 80: loads are coalesced and the MFMA reads
// free of bank conflicts.  A batch of 128 rows has 16 to 40 tiles only, so the
// grid's z splits K (part[z][M][N], added in order by k_gemm_sum); unsplit the
// epilogue runs here.  Bound by latency and the weights' reads (128 x 4489 x 512:
// one wave per tile reading global memory 203 us, now 17 with the sum).
template <bool KA, bool KB>
__global__ __launch_bounds__(kT) void k_gemm(const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb,
                                             float* __restrict__ C, Epilogue ep, int M, int N, int K, int ksplit)
{
    constexpr int BK = 32, LK = 36, LI = 80, SZ = BK * LI;   // 64 * LK < SZ
    __shared__ float sa[2][SZ], sb[2][SZ];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64, wi = (wv >> 1) * 32, wj = (wv & 1) * 32;
    const int kb = blockIdx.z * ksplit, ke = min(K, kb + ksplit);
    // eight elements of each operand per thread and step (zero outside)
    float ra[8], rb[8];
    auto load = [&](const float* __restrict__ X, int ld, int e0, int E, bool kc, int k0, float* r) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = k0 + (kc ? (tid & 31) : (tid >> 6) + 4 * q), e = e0 + (kc ? (tid >> 5) + 8 * q : (tid & 63));
            const bool on = k < ke && e < E;
            const float v = X[on ? (kc ? (long long)e * ld + k : (long long)k * ld + e) : 0];
            r[q] = on ? v : 0.0f;
        }
    };
    auto store = [&](float* s, bool kc, const float* r) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 8; ++q)
            s[kc ? ((tid >> 5) + 8 * q) * LK + (tid & 31) : ((tid >> 6) + 4 * q) * LI + (tid & 63)] = r[q];
    };
    f4 acc[2][2];
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) acc[a][b] = f4{0, 0, 0, 0};
    const int r16 = lane & 15, k4 = lane >> 4;
    load(A, lda, i0, M, KA, kb, ra);
    load(B, ldb, j0, N, KB, kb, rb);
    int ph = 0;
    for (int k0 = kb; k0 < ke; k0 += BK, ph ^= 1) {
        store(sa[ph], KA, ra);
        store(sb[ph], KB, rb);
        __syncthreads();
        if (k0 + BK < ke) {
            load(A, lda, i0, M, KA, k0 + BK, ra);
            load(B, ldb, j0, N, KB, k0 + BK, rb);
        }
        const float* const ta = sa[ph] + (KA ? (wi + r16) * LK + k4 : k4 * LI + wi + r16);
        const float* const tb = sb[ph] + (KB ? (wj + r16) * LK + k4 : k4 * LI + wj + r16);
#pragma unroll
        for (int k = 0; k < BK; k += 4) {
            float av[2], bv[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                av[a] = ta[KA ? 16 * a * LK + k : k * LI + 16 * a];
                bv[a] = tb[KB ? 16 * a * LK + k : k * LI + 16 * a];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
        }
        // (the other buffer is written next: every wave has read it before the
        // barrier above)
    }
    const bool split = gridDim.z > 1;
    if (split) C += (long long)blockIdx.z * M * N;
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) {
            const int j = j0 + wj + 16 * b + r16;
            if (j >= N) continue;
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + wi + 16 * a + 4 * k4 + r;
                if (i >= M) continue;
                C[(long long)i * N + j] = split ? acc[a][b][r] : ep(acc[a][b][r], i, j, N);
            }
        }
}

// C = epilogue(sum over z of part[z])
__global__ __launch_bounds__(kT) void k_gemm_sum(const float* __restrict__ part, int nz, float* __restrict__ C, Epilogue ep,
                                                 int M, int N)
{
    const long long t = (long long)blockIdx.x * kT + threadIdx.x, n = (long long)M * N;
    if (t >= n) return;
    float v = part[t];
#pragma unroll 8
    for (int z = 1; z < nz; ++z) v += part[(long long)z * n + t];
    const long long i = t / N;
    C[t] = ep(v, i, (int)(t - i * N), N);
}

// db[j] = sum_i dz[i][j] (fixed order): 64 columns per block, four threads each
__global__ __launch_bounds__(kT) void k_colsum(const float* __restrict__ dz, int M, int N, float* __restrict__ db)
{
    __shared__ float sh[4][64];
    const int c = threadIdx.x & 63, q = threadIdx.x >> 6, j = blockIdx.x * 64 + c;
    float s = 0.0f;
    if (j < N)
#pragma unroll 8
        for (int i = q; i < M; i += 4) s += dz[(long long)i * N + j];
    sh[q][c] = s;
    __syncthreads();
    if (q == 0 && j < N) db[j] = (sh[0][c] + sh[1][c]) + (sh[2][c] + sh[3][c]);
}

// dy = 2 (y - t) / n and per-block partial sums of (y - t)^2
__global__ __launch_bounds__(kT) void k_mse(const float* __restrict__ y, const float* __restrict__ t, long long n,
                                            float* __restrict__ dy, float* __restrict__ part)
{
    const long long i = (long long)blockIdx.x * kT + threadIdx.x;
    float e = 0.0f;
    if (i < n) {
        const float d = y[i] - t[i];
        dy[i] = 2.0f * d / (float)n;
        e = d * d;
    }
    __shared__ float sh[kT];
    sh[threadIdx.x] = e;
    __syncthreads();
    for (int o = kT / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m1,
                       float* __restrict__ m2, long long n, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.0f - b1) * gi, b = b2 * m2[i] + (1.0f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    w[i] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

unsigned nb(long long n) { return (unsigned)((n + kT - 1) / kT); }

int fail(ehd_mlp* mlp, int code, const char* msg)
{
    if (mlp) mlp->err = msg;
    return code;
}

#define MLP_HIP(call)                                                                           \
    do {                                                                                        \
        hipError_t _e = (call);                                                                 \
        if (_e != hipSuccess) {                                                                 \
            char _b[256];                                                                       \
            snprintf(_b, sizeof(_b), "%s failed: %s", #call, hipGetErrorString(_e));            \
            return fail(mlp, EHD_E_HIP, _b);                                                    \
        }                                                                                       \
    } while (0)

// Parts of K for an M x N product: a product of fewer than kTiles tiles is cut
// until its grid has that many blocks (1.5 per compute unit) or parts of 64
// terms, so parts x tiles < 2 kTiles, which bounds `part`.
constexpr long long kTiles = 384;
int gemm_parts(const ehd_mlp* mlp, int M, int N, int K)
{
    const long long tiles = (long long)((N + 63) / 64) * ((M + 63) / 64);
    if (!mlp->part || tiles >= kTiles) return 1;
    return (int)std::max<long long>(1, std::min<long long>((kTiles + tiles - 1) / tiles, K / 64));
}

template <bool KA, bool KB>
int gemm(ehd_mlp* mlp, const float* A, int lda, const float* B, int ldb, float* C, Epilogue ep, int M, int N, int K)
{
    const int nz = gemm_parts(mlp, M, N, K), ks = ((K + nz - 1) / nz + 31) / 32 * 32, parts = (K + ks - 1) / ks;
    const dim3 grid((unsigned)((N + 63) / 64), (unsigned)((M + 63) / 64), (unsigned)parts);
    hipLaunchKernelGGL((k_gemm<KA, KB>), grid, dim3(kT), 0, mlp->stream, A, lda, B, ldb, parts > 1 ? mlp->part : C, ep, M, N,
                       K, ks);
    if (parts > 1)
        hipLaunchKernelGGL(k_gemm_sum, dim3(nb((long long)M * N)), dim3(kT), 0, mlp->stream, mlp->part, parts, C, ep, M, N);
    MLP_HIP(hipGetLastError());
    return EHD_OK;
}

int ensure_capacity(ehd_mlp* mlp, int batch)
{
    if (batch <= mlp->cap) return EHD_OK;
    MLP_HIP(hipStreamSynchronize(mlp->stream));   // the old buffers may still be in use
    for (float* a : mlp->act)
        if (a) (void)hipFree(a);
    if (mlp->dA) (void)hipFree(mlp->dA);
    if (mlp->dB) (void)hipFree(mlp->dB);
    if (mlp->part) (void)hipFree(mlp->part);
    mlp->act.assign(mlp->nlay + 2, nullptr);
    mlp->dA = mlp->dB = mlp->part = nullptr;
    mlp->cap = 0;
    int wmax = std::max(mlp->nin, std::max(mlp->nhid, mlp->nout));
    MLP_HIP(hipMalloc(&mlp->act[0], sizeof(float) * (size_t)batch * mlp->nin));
    for (int l = 0; l <= mlp->nlay; ++l)
        MLP_HIP(hipMalloc(&mlp->act[l + 1], sizeof(float) * (size_t)batch * mlp->dout[l]));
    MLP_HIP(hipMalloc(&mlp->dA, sizeof(float) * (size_t)batch * wmax));
    MLP_HIP(hipMalloc(&mlp->dB, sizeof(float) * (size_t)batch * wmax));
    // products split over K; without the memory they run unsplit
    if (hipMalloc(&mlp->part, sizeof(float) * 64 * 64 * 2 * kTiles) != hipSuccess) {
        (void)hipGetLastError();
        mlp->part = nullptr;
    }
    mlp->cap = batch;
    return EHD_OK;
}

uint64_t splitmix(uint64_t& s)
{
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

}  // namespace

extern "C" {

int ehd_mlp_create(ehd_mlp** out, int device, void* stream, int nin, int nhidden, int nlayers, int nout,
                   unsigned long long seed)
{
    if (!out || nin < 1 || nhidden < 1 || nlayers < 0 || nout < 1) return EHD_E_ARG;
    ehd_mlp* mlp = new ehd_mlp;
    *out = nullptr;
    mlp->device = device;
    mlp->stream = (hipStream_t)stream;
    mlp->nin = nin;
    mlp->nhid = nhidden;
    mlp->nlay = nlayers;
    mlp->nout = nout;
    for (int l = 0; l <= nlayers; ++l) {
        mlp->din.push_back(l == 0 ? nin : nhidden);
        mlp->dout.push_back(l == nlayers ? nout : nhidden);
        mlp->woff.push_back(mlp->nparam);
        mlp->nparam += (long long)mlp->din[l] * mlp->dout[l];
        mlp->boff.push_back(mlp->nparam);
        mlp->nparam += mlp->dout[l];
    }
    // He-uniform weights from a counter-based generator, zero biases
    std::vector<float> h((size_t)mlp->nparam, 0.0f);
    uint64_t st = seed;
    for (int l = 0; l <= nlayers; ++l) {
        const double a = std::sqrt(6.0 / mlp->din[l]);
        for (long long i = 0; i < (long long)mlp->din[l] * mlp->dout[l]; ++i) {
            const double u = (double)(splitmix(st) >> 11) * (1.0 / 9007199254740992.0);
            h[(size_t)(mlp->woff[l] + i)] = (float)((2.0 * u - 1.0) * a);
        }
    }
    if (hipSetDevice(device) != hipSuccess || hipMalloc(&mlp->w, sizeof(float) * h.size()) != hipSuccess ||
        hipMalloc(&mlp->g, sizeof(float) * h.size()) != hipSuccess ||
        hipMalloc(&mlp->m1, sizeof(float) * h.size()) != hipSuccess ||
        hipMalloc(&mlp->m2, sizeof(float) * h.size()) != hipSuccess ||
        hipMalloc(&mlp->red, sizeof(float) * 65536) != hipSuccess ||
        hipMemcpy(mlp->w, h.data(), sizeof(float) * h.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemset(mlp->g, 0, sizeof(float) * h.size()) != hipSuccess ||
        hipMemset(mlp->m1, 0, sizeof(float) * h.size()) != hipSuccess ||
        hipMemset(mlp->m2, 0, sizeof(float) * h.size()) != hipSuccess) {
        ehd_mlp_destroy(mlp);
        return EHD_E_HIP;
    }
    *out = mlp;
    return EHD_OK;
}

void ehd_mlp_destroy(ehd_mlp* mlp)
{
    if (!mlp) return;
    (void)hipSetDevice(mlp->device);
    for (float* p : {mlp->w, mlp->g, mlp->m1, mlp->m2, mlp->dA, mlp->dB, mlp->part, mlp->red})
        if (p) (void)hipFree(p);
    for (float* a : mlp->act)
        if (a) (void)hipFree(a);
    delete mlp;
}

const char* ehd_mlp_last_error(const ehd_mlp* mlp) { return mlp ? mlp->err.c_str() : "no network"; }

int ehd_mlp_num_params(const ehd_mlp* mlp, long long* n)
{
    if (!mlp || !n) return EHD_E_ARG;
    *n = mlp->nparam;
    return EHD_OK;
}

int ehd_mlp_get_params(ehd_mlp* mlp, float* host)
{
    if (!mlp || !host) return EHD_E_ARG;
    MLP_HIP(hipSetDevice(mlp->device));
    MLP_HIP(hipStreamSynchronize(mlp->stream));
    MLP_HIP(hipMemcpy(host, mlp->w, sizeof(float) * mlp->nparam, hipMemcpyDeviceToHost));
    return EHD_OK;
}

int ehd_mlp_set_params(ehd_mlp* mlp, const float* host)
{
    if (!mlp || !host) return EHD_E_ARG;
    MLP_HIP(hipSetDevice(mlp->device));
    MLP_HIP(hipStreamSynchronize(mlp->stream));
    MLP_HIP(hipMemcpy(mlp->w, host, sizeof(float) * mlp->nparam, hipMemcpyHostToDevice));
    return EHD_OK;
}

int ehd_mlp_get_grads(ehd_mlp* mlp, float* host)
{
    if (!mlp || !host) return EHD_E_ARG;
    MLP_HIP(hipSetDevice(mlp->device));
    MLP_HIP(hipStreamSynchronize(mlp->stream));
    MLP_HIP(hipMemcpy(host, mlp->g, sizeof(float) * mlp->nparam, hipMemcpyDeviceToHost));
    return EHD_OK;
}

int ehd_mlp_forward(ehd_mlp* mlp, int batch, const float* x_d, float* y_d)
{
    if (!mlp || batch < 1 || !x_d) return fail(mlp, EHD_E_ARG, "invalid forward arguments");
    MLP_HIP(hipSetDevice(mlp->device));
    int rc = ensure_capacity(mlp, batch);
    if (rc) return rc;
    MLP_HIP(hipMemcpyAsync(mlp->act[0], x_d, sizeof(float) * (size_t)batch * mlp->nin, hipMemcpyDeviceToDevice,
                           mlp->stream));
    for (int l = 0; l <= mlp->nlay; ++l) {
        const int K = mlp->din[l], N = mlp->dout[l];
        const bool last = l == mlp->nlay;
        float* const out = last && y_d ? y_d : mlp->act[l + 1];
        if ((rc = gemm<true, false>(mlp, mlp->act[l], K, mlp->w + mlp->woff[l], N, out,
                                    Epilogue{mlp->w + mlp->boff[l], nullptr, last ? 0 : 1}, batch, N, K)))
            return rc;
    }
    return EHD_OK;
}

int ehd_mlp_backward(ehd_mlp* mlp, int batch, const float* dy_d)
{
    if (!mlp || batch < 1 || batch > mlp->cap || !dy_d) return fail(mlp, EHD_E_ARG, "backward needs a forward first");
    MLP_HIP(hipSetDevice(mlp->device));
    int rc;
    const float* dz = dy_d;                                  // dZ of the output layer is dY
    float* next = mlp->dA;
    for (int l = mlp->nlay; l >= 0; --l) {
        const int K = mlp->din[l], N = mlp->dout[l];
        // dW = H_l^T dZ  ([K][N]), db = column sums of dZ
        if ((rc = gemm<false, false>(mlp, mlp->act[l], K, dz, N, mlp->g + mlp->woff[l], Epilogue{}, K, N, batch))) return rc;
        hipLaunchKernelGGL(k_colsum, dim3((N + 63) / 64), dim3(kT), 0, mlp->stream, dz, batch, N, mlp->g + mlp->boff[l]);
        MLP_HIP(hipGetLastError());
        if (l == 0) break;
        // dH_l = dZ W^T ([batch][K]) with the ReLU derivative of layer l-1's output
        if ((rc = gemm<true, true>(mlp, dz, N, mlp->w + mlp->woff[l], N, next, Epilogue{nullptr, mlp->act[l], 0}, batch, K,
                                   N)))
            return rc;
        dz = next;
        next = next == mlp->dA ? mlp->dB : mlp->dA;
    }
    return EHD_OK;
}

int ehd_mlp_mse(ehd_mlp* mlp, int batch, const float* y_d, const float* t_d, float* dy_d, double* loss)
{
    if (!mlp || batch < 1 || !y_d || !t_d || !dy_d) return fail(mlp, EHD_E_ARG, "invalid loss arguments");
    const long long n = (long long)batch * mlp->nout;
    if (nb(n) > 65536) return fail(mlp, EHD_E_ARG, "batch too large for the loss reduction");
    MLP_HIP(hipSetDevice(mlp->device));
    hipLaunchKernelGGL(k_mse, dim3(nb(n)), dim3(kT), 0, mlp->stream, y_d, t_d, n, dy_d, mlp->red);
    MLP_HIP(hipGetLastError());
    if (loss) {
        std::vector<float> part(nb(n));
        MLP_HIP(hipMemcpyAsync(part.data(), mlp->red, sizeof(float) * part.size(), hipMemcpyDeviceToHost, mlp->stream));
        MLP_HIP(hipStreamSynchronize(mlp->stream));
        double s = 0.0;
        for (float v : part) s += v;
        *loss = s / (double)n;
    }
    return EHD_OK;
}

int ehd_mlp_adam(ehd_mlp* mlp, float lr, float beta1, float beta2, float eps)
{
    if (!mlp || !(lr > 0.0f)) return fail(mlp, EHD_E_ARG, "invalid Adam arguments");
    MLP_HIP(hipSetDevice(mlp->device));
    ++mlp->adam_t;
    const float c1 = 1.0f - std::pow(beta1, (float)mlp->adam_t), c2 = 1.0f - std::pow(beta2, (float)mlp->adam_t);
    hipLaunchKernelGGL(k_adam, dim3(nb(mlp->nparam)), dim3(kT), 0, mlp->stream, mlp->w, mlp->g, mlp->m1, mlp->m2,
                       mlp->nparam, lr, beta1, beta2, eps, c1, c2);
    MLP_HIP(hipGetLastError());
    return EHD_OK;
}

}  // extern "C"
