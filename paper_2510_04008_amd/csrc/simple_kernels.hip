// Small kernels outside the passes: the hash tap of the generic family, incremental decoding, the reduction of the
// temperature's partial cotangents, zero fill and the plain copy benchmarks calibrate with.  All arithmetic in fp32 on the
// vector ALUs, any (L, P <= 8, d <= 256), fp32 or bf16 tensors.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace race {
namespace {

// ------------------------------------------------------------------ element access
struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float load_elem(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_elem(const bf16_t *p, size_t i)
{
    return __uint_as_float(static_cast<uint32_t>(p[i].bits) << 16);
}
__device__ __forceinline__ void store_elem(float *p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_elem(bf16_t *p, size_t i, float v)
{
    uint32_t b = __float_as_uint(v);
    if ((b & 0x7fffffffu) > 0x7f800000u) { p[i].bits = 0x7fc0; return; }      // NaN
    b += 0x7fffu + ((b >> 16) & 1u);                                          // nearest even
    p[i].bits = static_cast<uint16_t>(b >> 16);
}

struct Args {
    int H, L, P, R, d, LP;
    int unit;            // 1: rows of Q and K are divided by their Euclidean norms before the projection
    int64_t N;
    float beta;
    const float *W;      // (H, L*P, d)
};

// e = exp(-2 beta |u|), the ratio of the two masses of a bit.  beta = +infinity is the hard hash of Section 3.3:
// e = 0 for u != 0, and for u = 0 (where -inf * 0 is NaN; fmaxf returns its other argument) the bit counts as set, like z >= 0.
__device__ __forceinline__ float mass_ratio(float beta, float u)
{
    return expf(fmaxf(-2.0f * beta * fabsf(u), -1e30f));
}

// Unit-norm option (the setting of Theorem 1's proof, |Q_i| = |K_j| = 1): the factor that turns a row of squared
// length ss into a unit vector; rows shorter than the floor are divided by the floor (a zero row stays zero).
constexpr float kUnitFloor = 1e-12f;
__device__ __forceinline__ float unit_scale(float ss) { return 1.0f / fmaxf(sqrtf(ss), kUnitFloor); }

// Debug tap: hard codes and phi of every (row, table).
template <typename T>
__global__ void simple_hash_tap(Args a, int BH, const T *X, uint8_t *codes, float *phi)
{
    const size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
    const size_t total = static_cast<size_t>(BH) * a.N * a.L;
    if (i >= total) return;
    const size_t row = i / a.L;
    const int l = static_cast<int>(i - row * a.L);
    const int h = static_cast<int>((row / a.N) % a.H);
    const float *Wl = a.W + (static_cast<size_t>(h) * a.LP + l * a.P) * a.d;
    float p[8], q[8];
    unsigned code = 0;
    float inv = 1.f;
    if (a.unit) {
        float ss = 0.f;
        for (int c = 0; c < a.d; ++c) { const float x = load_elem(X, row * a.d + c); ss = fmaf(x, x, ss); }
        inv = unit_scale(ss);
    }
    for (int t = 0; t < a.P; ++t) {
        float z = 0.f;
        for (int c = 0; c < a.d; ++c) z = fmaf(Wl[t * a.d + c], load_elem(X, row * a.d + c), z);
        z *= inv;
        code |= (z >= 0.f ? 1u : 0u) << t;
        const float u = tanhf(z);
        const float e = mass_ratio(a.beta, u);
        const float big = 1.0f / (1.0f + e), small = e / (1.0f + e);
        p[t] = (u >= 0.f) ? big : small;
        q[t] = (u >= 0.f) ? small : big;
    }
    codes[i] = static_cast<uint8_t>(code);
    if (phi) {
        for (int r = 0; r < a.R; ++r) {
            float f = 1.f;
            for (int t = 0; t < a.P; ++t) f *= ((r >> t) & 1) ? p[t] : q[t];
            phi[i * a.R + r] = f;
        }
    }
}

// ------------------------------------------------------------------ incremental decoding
// One decoding step, one workgroup of 1024 threads per (batch, head).  Threads form TF = 1024 / TL slots of
// TL = 64 ceil(d / 64) threads; a slot takes the tables slot, slot + TF, ... one after the other, thread c of a slot
// owning column c: it hashes the new key and query against the table's hyperplanes with its slot-mates (Algorithm 1,
// steps 2-4), adds the key/value to the table's statistics and reads them with the query, column by column
// (Algorithm 2's loop body; coalesced rows of d+1 floats).  The sums over tables and the normalisation follow in the
// same kernel (Algorithm 1, steps 7-8): numerators over the slots in slot order, the normaliser over the wavefronts.
constexpr int kDecodeThreads = 1024;

template <typename T>
__global__ __launch_bounds__(kDecodeThreads) void decode_step_kernel(int H, int L, int P, int d, float beta, int unit, const float *W,
                                                                     const T *q, const T *k, const T *v, float *state,
                                                                     T *o, float *den)
{
    extern __shared__ float lds[];
    const int R = 1 << P, d1 = d + 1;
    const int TL = (d + 63) & ~63, TF = kDecodeThreads / TL, NWV = TL / 64;
    const int tid = threadIdx.x, slot = tid / TL, c = tid % TL, lane = tid & 63, wv = c >> 6;
    const int bh = blockIdx.x, h = bh % H;
    float *zred = lds;                              // [TF][2P+2][NWV] partial projections, then the rows' squared lengths
    float *pq = zred + TF * (2 * P + 2) * NWV;      // [TF][2P][2]   per-bit masses (+1 side, -1 side)
    float *phi = pq + TF * 2 * P * 2;               // [TF][2][R]    assignments of the query (0) and the key (1)
    float *numred = phi + TF * 2 * R;               // [TF][d]       numerators per slot
    float *dred = numred + TF * d;                  // [16]          normaliser per wavefront
    const bool active = slot < TF, colok = active && c < d;
    const float xq = colok ? load_elem(q, static_cast<size_t>(bh) * d + c) : 0.f;
    const float xk = colok ? load_elem(k, static_cast<size_t>(bh) * d + c) : 0.f;
    const float vv = colok ? load_elem(v, static_cast<size_t>(bh) * d + c) : 0.f;
    float num = 0.f, dn = 0.f;
    for (int l0 = 0; l0 < L; l0 += TF) {
        const int l = l0 + slot;
        const bool on = active && l < L;
        const float *Wl = W + (static_cast<size_t>(h) * L + (on ? l : 0)) * P * d;
        for (int t = 0; t <= P; ++t) {              // t = P: the squared lengths |q|^2, |k|^2 instead of a projection
            const float w = (on && c < d) ? (t < P ? Wl[t * d + c] : 1.f) : 0.f;
            float a = w * xq * (t < P ? 1.f : xq), b = w * xk * (t < P ? 1.f : xk);
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) {
                a += __shfl_xor(a, m, 64);
                b += __shfl_xor(b, m, 64);
            }
            if (active && lane == 0) {
                zred[(slot * (2 * P + 2) + 2 * t) * NWV + wv] = a;
                zred[(slot * (2 * P + 2) + 2 * t + 1) * NWV + wv] = b;
            }
        }
        __syncthreads();
        if (on && c < 2 * P) {                      // per-bit masses of the query (c < P) and of the key
            const int side = c / P, t = c % P;
            float z = 0.f, ss = 0.f;
            for (int i = 0; i < NWV; ++i) {
                z += zred[(slot * (2 * P + 2) + 2 * t + side) * NWV + i];
                ss += zred[(slot * (2 * P + 2) + 2 * P + side) * NWV + i];
            }
            if (unit) z *= unit_scale(ss);
            const float u = tanhf(z);
            const float e = mass_ratio(beta, u);
            const float big = 1.0f / (1.0f + e), small = e / (1.0f + e);
            pq[(slot * 2 * P + c) * 2] = (u >= 0.f) ? big : small;          // mass on the +1 side
            pq[(slot * 2 * P + c) * 2 + 1] = (u >= 0.f) ? small : big;
        }
        __syncthreads();
        if (on) {
            for (int r = c; r < 2 * R; r += TL) {
                const int side = r / R, cr = r % R;
                float f = 1.f;
                for (int t = 0; t < P; ++t) f *= pq[(slot * 2 * P + side * P + t) * 2 + (((cr >> t) & 1) ? 0 : 1)];
                phi[(slot * 2 + side) * R + cr] = f;
            }
        }
        __syncthreads();
        if (on) {
            const float *pqv = phi + (slot * 2) * R, *pk = pqv + R;
            float *S = state + (static_cast<size_t>(bh) * L + l) * R * d1;
            if (c < d) {
#pragma unroll 8
                for (int r = 0; r < R; ++r) {
                    const float sv = fmaf(pk[r], vv, S[r * d1 + c]);
                    S[r * d1 + c] = sv;
                    num = fmaf(pqv[r], sv, num);
                }
            }
            for (int r = c; r < R; r += TL) {       // the mass column
                const float sv = S[r * d1 + d] + pk[r];
                S[r * d1 + d] = sv;
                dn = fmaf(pqv[r], sv, dn);
            }
        }
        __syncthreads();
    }
    if (colok) numred[slot * d + c] = num;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dn += __shfl_xor(dn, m, 64);
    if (lane == 0) dred[tid >> 6] = dn;
    __syncthreads();
    if (tid < d) {
        float tot = 0.f, dnt = 0.f;
        for (int sl = 0; sl < TF; ++sl) tot += numred[sl * d + tid];
        for (int i = 0; i < kDecodeThreads / 64; ++i) dnt += dred[i];
        store_elem(o, static_cast<size_t>(bh) * d + tid, dnt > 0.f ? tot / dnt : 0.f);
        if (tid == 0) den[bh] = dnt / static_cast<float>(L);
    }
}

__global__ void zero_kernel(float *dst, size_t n)
{
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = 0.f;
}

// ------------------------------------------------------------------ host side
Args make_args(const Plan &p, const char *ws)
{
    Args a;
    a.H = p.H; a.L = p.L; a.P = p.P; a.R = p.R; a.d = p.d; a.LP = p.LP;
    a.N = p.N; a.beta = p.beta; a.unit = p.unit_qk;
    a.W = reinterpret_cast<const float *>(ws + p.off_W);
    return a;
}

unsigned blocks_for(size_t n, unsigned per) { return static_cast<unsigned>((n + per - 1) / per); }

// One wavefront per (batch, head): every lane takes a fixed share of both sides' partial sums, the lanes are added by a
// butterfly (the order of the sum does not depend on the run).
__global__ __launch_bounds__(64) void dbeta_reduce_kernel(const float *part, int BH, int parts, float *dbeta)
{
    const int bh = blockIdx.x;
    float s = 0.f;
    for (int side = 0; side < 2; ++side) {
        const float *src = part + (static_cast<size_t>(side) * BH + bh) * parts;
        for (int i = threadIdx.x; i < parts; i += 64) s += src[i];
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
    if (threadIdx.x == 0) dbeta[bh] = s;
}

}  // namespace

hipError_t reduce_dbeta(const Plan &p, const float *part, float *dbeta, hipStream_t st)
{
    hipLaunchKernelGGL(dbeta_reduce_kernel, dim3(p.BH), dim3(64), 0, st, part, p.BH, p.dbeta_parts, dbeta);
    return hipGetLastError();
}

// The shapes the generic family takes: one table's statistics and one token's rows within 160 KB.
bool simple_supported(int R, int d, int P)
{
    const size_t floats = static_cast<size_t>(R) * (d + 1) + 2 * d + 2 * (d + 1) + 2 * (5 * P + R + 1) + R + P;
    return floats * sizeof(float) <= 160 * 1024;
}

hipError_t simple_hash(const Plan &p, const void *X, uint8_t *codes, float *phi, char *ws, hipStream_t st)
{
    const Args a = make_args(p, ws);
    const size_t total = static_cast<size_t>(p.BH) * p.N * p.L;
    if (p.dtype == RACE_F32)
        hipLaunchKernelGGL((simple_hash_tap<float>), dim3(blocks_for(total, 128)), dim3(128), 0, st, a, p.BH,
                           (const float *)X, codes, phi);
    else
        hipLaunchKernelGGL((simple_hash_tap<bf16_t>), dim3(blocks_for(total, 128)), dim3(128), 0, st, a, p.BH,
                           (const bf16_t *)X, codes, phi);
    return hipGetLastError();
}

hipError_t zero_floats(float *dst, size_t n, hipStream_t st)
{
    const size_t want = (n + 255) / 256;
    hipLaunchKernelGGL(zero_kernel, dim3(static_cast<unsigned>(want < 4096 ? (want ? want : 1) : 4096)), dim3(256), 0, st,
                       dst, n);
    return hipGetLastError();
}

hipError_t decode_step(const Plan &p, const float *W, const void *q, const void *k, const void *v, float *state,
                       void *o, float *den, hipStream_t st)
{
    const int TL = (p.d + 63) & ~63, TF = kDecodeThreads / TL;
    const size_t lds = (static_cast<size_t>(TF) * (2 * p.P + 2) * (TL / 64) + TF * 4 * p.P + TF * 2 * p.R + TF * p.d + 16) * sizeof(float);
    if (p.dtype == RACE_F32)
        hipLaunchKernelGGL((decode_step_kernel<float>), dim3(p.BH), dim3(kDecodeThreads), lds, st, p.H, p.L, p.P, p.d, p.beta, p.unit_qk, W,
                           (const float *)q, (const float *)k, (const float *)v, state, (float *)o, den);
    else
        hipLaunchKernelGGL((decode_step_kernel<bf16_t>), dim3(p.BH), dim3(kDecodeThreads), lds, st, p.H, p.L, p.P, p.d, p.beta, p.unit_qk, W,
                           (const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v, state, (bf16_t *)o, den);
    return hipGetLastError();
}

// A few tens of KB over PCIe: every thread has one 16-byte read in flight.  (As a stream-ordered copy through the runtime
// the same bytes cost a hand-over to a copy engine and back: 8 us of copy between gaps of 10 and 16 us, 35 us in front of
// every pass, against 3-4 us for this kernel.)
__global__ __launch_bounds__(256) void upload_kernel(uint4 *dst, const uint4 *src, size_t n16)
{
    const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n16) dst[i] = src[i];
}

hipError_t upload(void *dst, const void *src, size_t bytes, hipStream_t st)
{
    const size_t n16 = bytes / 16;
    hipLaunchKernelGGL(upload_kernel, dim3(static_cast<unsigned>((n16 + 255) / 256)), dim3(256), 0, st, static_cast<uint4 *>(dst),
                       static_cast<const uint4 *>(src), n16);
    return hipGetLastError();
}

// One 16-byte load and one 16-byte store per element, grid-stride: every byte is read once and written once.
__global__ void __launch_bounds__(256) calibration_copy_kernel(uint4 *__restrict__ dst, const uint4 *__restrict__ src,
                                                                size_t n16)
{
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

hipError_t calibration_copy(void *dst, const void *src, size_t bytes, hipStream_t st)
{
    const size_t n16 = bytes / 16;
    const size_t want = (n16 + 255) / 256;
    const unsigned blocks = static_cast<unsigned>(want < 16384 ? (want ? want : 1) : 16384);
    hipLaunchKernelGGL(calibration_copy_kernel, dim3(blocks), dim3(256), 0, st, static_cast<uint4 *>(dst),
                       static_cast<const uint4 *>(src), n16);
    return hipGetLastError();
}

}  // namespace race
