// Small kernels outside the passes: incremental decoding, the reduction of the temperature's partial cotangents, zero fill and
// the plain copy benchmarks calibrate with.  All arithmetic in fp32 on the vector ALUs, every shape the generic family takes,
// fp32 or bf16 tensors.
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

// ------------------------------------------------------------------ incremental decoding
// One decoding step.  A workgroup of 256 threads owns up to 32 G bucket rows of one table of one (batch*head): its threads
// form G = 256 / (64 ceil(d / 64)) groups, thread c of group g holding column c of rows g, g + G, ... in registers, and one
// row of the mass column each.  All operands are requested up front, the hyperplanes and the new rows before the statistics
// (loads return in order), so the hashing of the new key and query (Algorithm 1, steps 2-4: 16 threads per dot product) runs
// while the statistics arrive; then update, read-out (Algorithm 2's loop body) and the workgroup's share of numerator and
// normaliser.  The workgroup that finishes last for its (batch*head) adds the shares in order (steps 7-8; bit-reproducible),
// so a step is one launch.  Bound by the latency of that one chain for a few sequences, by the traffic of the states (read
// and written once) for many.  d = 128, L = 8, P = 6, against one workgroup of 1024 threads per (batch*head) that took the
// tables one after the other: B H = 4: 17.5 -> 5.7 us; B H = 256: 36.5 -> 25.3 us (135 MB at 5.4 TB/s; a plain in-place
// update of as many bytes takes 20 us).
//
// The shares cross workgroups (and the XCDs' separate L2s): they are written and read with device-scope accesses, which go
// to the coherence point, and the counter is bumped only when a workgroup's own writes have completed.  The last workgroup
// sets the counter back to zero for the next step; the upload of W clears it in the first place.
constexpr int kDecodeThreads = 256;
constexpr int kDecodeMaxRows = 32;      // bucket rows of a thread

// (a caller's rows need be aligned to their elements only; global memory takes wide loads at any address)
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_of_elements;
typedef __attribute__((ext_vector_type(2), aligned(2))) uint32_t u32x2_of_elements;
__device__ __forceinline__ float4 load_quad(const float *p)
{
    const f32x4_of_elements w = *reinterpret_cast<const f32x4_of_elements *>(p);
    return float4{w.x, w.y, w.z, w.w};
}
__device__ __forceinline__ float4 load_quad(const bf16_t *p)
{
    const u32x2_of_elements w = *reinterpret_cast<const u32x2_of_elements *>(p);
    return float4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                  __uint_as_float(w.y & 0xffff0000u)};
}

// ROWS: bucket rows per thread (R = ROWS G shares-per-table, or R < G and ROWS = 1); NC: 64-column pieces of d.
template <typename T, int ROWS, int NC>
__global__ __launch_bounds__(kDecodeThreads, NC <= 2 && ROWS <= 16 ? 8 : 4) void decode_step_kernel(
    int H, int L, int P, int d, float beta, int unit, const float *W, const T *q, const T *k, const T *v, float *state, float *part,
    unsigned *arrived, T *o, float *den)
{
    __shared__ float zs[18];                        // projections of q (2 t) and k (2 t + 1), then the squared lengths
    __shared__ float2 bits[16];                     // masses (-1 side, +1 side) of bit t of k (t) and q (P + t)
    __shared__ float2 phi[256];                     // assignments (key, query) of the workgroup's rows
    __shared__ float nred[kDecodeThreads], dred[kDecodeThreads / 64];
    __shared__ unsigned last;
    constexpr int TL = 64 * NC, G = kDecodeThreads / TL;
    const int R = 1 << P, d1 = d + 1;
    const int tid = threadIdx.x, g = tid / TL, c = tid - g * TL, l = blockIdx.x, bh = blockIdx.y;
    const int r0 = blockIdx.z * (G * ROWS), nr = R - r0 < G * ROWS ? R - r0 : G * ROWS, shares = L * gridDim.z;
    const bool on = g < G && g < nr && c < d;
    const size_t row = static_cast<size_t>(bh) * d;
    float *S = state + ((static_cast<size_t>(bh) * L + l) * R + r0) * d1;
    const float *Wl = W + (static_cast<size_t>(bh % H) * L + l) * P * d;
    // ---- operands, every lane an in-range address: dot product tid / 16 (the first 16 of them), then the statistics
    const int sub = tid & 15, ndots = 2 * (P + unit), dot0 = tid >> 4 < ndots ? tid >> 4 : 0;
    auto operands = [&](int i, float4 (&w4)[NC], float4 (&x4)[NC]) __attribute__((always_inline)) {
        const T *x = ((i & 1) ? k : q) + row;
        const float *w = Wl + ((i >> 1) < P ? (i >> 1) : 0) * d;
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            const int at = 64 * e + 4 * sub < d ? 64 * e + 4 * sub : 0;
            w4[e] = load_quad(w + at);
            x4[e] = load_quad(x + at);
        }
    };
    float4 w4[NC], x4[NC];
    operands(dot0, w4, x4);
    const float vv = load_elem(v, row + (c < d ? c : 0));
    const uint32_t own = on ? static_cast<uint32_t>(g * d1 + c) : 0u;
    float s[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) s[i] = (S + i * G * d1)[own];
    const float sm = S[static_cast<uint32_t>((tid < nr ? tid : 0) * d1 + d)];
    // ---- hash
    for (int i = dot0; i < ndots; i += kDecodeThreads / 16) {
        if (i != dot0) operands(i, w4, x4);
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            if (64 * e + 4 * sub >= d) continue;
            const float4 x = x4[e], y = (i >> 1) < P ? w4[e] : x;
            a = fmaf(y.x, x.x, fmaf(y.y, x.y, fmaf(y.z, x.z, fmaf(y.w, x.w, a))));
        }
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) a += __shfl_xor(a, m, 64);
        if (sub == 0) zs[i] = a;
    }
    __syncthreads();
    if (tid < 2 * P) {
        const int side = tid < P ? 1 : 0, t = tid < P ? tid : tid - P;
        float z = zs[2 * t + side];
        if (unit) z *= unit_scale(zs[2 * P + side]);
        const float u = tanhf(z);
        const float e = mass_ratio(beta, u);
        const float big = 1.0f / (1.0f + e), small = e / (1.0f + e);
        bits[tid] = u >= 0.f ? float2{small, big} : float2{big, small};
    }
    __syncthreads();
    if (tid < nr) {
        float fk = 1.f, fq = 1.f;
        for (int t = 0; t < P; ++t) {
            const float2 bk = bits[t], bq = bits[P + t];
            const bool set = ((r0 + tid) >> t) & 1;
            fk *= set ? bk.y : bk.x;
            fq *= set ? bq.y : bq.x;
        }
        phi[tid] = float2{fk, fq};
    }
    __syncthreads();
    // ---- update and read-out
    float num = 0.f, dn = 0.f;
    if (on) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const float2 f = phi[g + G * i];
            const float y = fmaf(f.x, vv, s[i]);
            (S + i * G * d1)[own] = y;
            num = fmaf(f.y, y, num);
        }
    }
    if (tid < nr) {                                 // the mass column
        const float2 f = phi[tid];
        const float y = sm + f.x;
        S[static_cast<uint32_t>(tid * d1 + d)] = y;
        dn = f.y * y;
    }
    nred[tid] = num;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dn += __shfl_xor(dn, m, 64);
    if ((tid & 63) == 0) dred[tid >> 6] = dn;
    __syncthreads();
    float *mine = part + (static_cast<size_t>(bh) * shares + l * gridDim.z + blockIdx.z) * d1;
    if (tid < d) {
        float x = nred[tid];
#pragma unroll
        for (int i = 1; i < G; ++i) x += nred[i * TL + tid];
        __hip_atomic_store(mine + tid, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (tid == 0) __hip_atomic_store(mine + d, (dred[0] + dred[1]) + (dred[2] + dred[3]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this thread's share has reached the coherence point
    __syncthreads();
    if (tid == 0) last = __hip_atomic_fetch_add(arrived + bh, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == static_cast<unsigned>(shares - 1);
    __syncthreads();
    if (!last) return;
    if (tid == 0) __hip_atomic_store(arrived + bh, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid < d) {
        const float *all = part + static_cast<size_t>(bh) * shares * d1;
        float tot = 0.f, dnt = 0.f;
        for (int s0 = 0; s0 < shares; s0 += 8) {
            float x[8], y[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int at = s0 + i < shares ? s0 + i : s0;
                x[i] = __hip_atomic_load(all + at * d1 + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                y[i] = __hip_atomic_load(all + at * d1 + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                tot += s0 + i < shares ? x[i] : 0.f;
                dnt += s0 + i < shares ? y[i] : 0.f;
            }
        }
        store_elem(o, row + tid, dnt > 0.f ? tot / dnt : 0.f);
        if (tid == 0) den[bh] = dnt / static_cast<float>(L);
    }
}

__global__ void zero_kernel(float *dst, size_t n)
{
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = 0.f;
}

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

// The shapes the generic family takes: all up to d = 256, tables of 256 bucket rows up to d = 152 (a limit of the interface, from
// the time when a table's statistics had to fit the 160 KB of LDS; these kernels have no such bound).
bool simple_supported(int R, int d) { return R < 256 || d <= 152; }

hipError_t zero_floats(float *dst, size_t n, hipStream_t st)
{
    const size_t want = (n + 255) / 256;
    hipLaunchKernelGGL(zero_kernel, dim3(static_cast<unsigned>(want < 4096 ? (want ? want : 1) : 4096)), dim3(256), 0, st,
                       dst, n);
    return hipGetLastError();
}

namespace {
// bucket rows per thread: all of the table's, at most 32 (8, 16, 32 measured: 31.4, 26.4, 25.3 us at B H = 256)
int decode_rows(const Plan &p)
{
    const int G = kDecodeThreads / ((p.d + 63) & ~63), rows = p.R / G;
    return rows < 1 ? 1 : (rows > kDecodeMaxRows ? kDecodeMaxRows : rows);
}

template <typename T, int ROWS, int NC>
void launch_decode(const Plan &p, const T *q, const T *k, const T *v, float *state, T *o, float *den, char *ws, hipStream_t st)
{
    hipLaunchKernelGGL((decode_step_kernel<T, ROWS, NC>), dim3(p.L, p.BH, decode_shares(p) / p.L), dim3(kDecodeThreads), 0, st, p.H, p.L,
                       p.P, p.d, p.beta, p.unit_qk, reinterpret_cast<const float *>(ws + p.off_W), q, k, v, state,
                       reinterpret_cast<float *>(ws + p.off_part), reinterpret_cast<unsigned *>(ws + p.off_arrived), o, den);
}
template <typename T, int ROWS>
void decode_columns(const Plan &p, const T *q, const T *k, const T *v, float *state, T *o, float *den, char *ws, hipStream_t st)
{
    switch ((p.d + 63) / 64) {
    case 1: return launch_decode<T, ROWS, 1>(p, q, k, v, state, o, den, ws, st);
    case 2: return launch_decode<T, ROWS, 2>(p, q, k, v, state, o, den, ws, st);
    case 3: return launch_decode<T, ROWS, 3>(p, q, k, v, state, o, den, ws, st);
    default: return launch_decode<T, ROWS, 4>(p, q, k, v, state, o, den, ws, st);
    }
}
template <typename T>
void decode_t(const Plan &p, const T *q, const T *k, const T *v, float *state, T *o, float *den, char *ws, hipStream_t st)
{
    switch (decode_rows(p)) {
    case 1: return decode_columns<T, 1>(p, q, k, v, state, o, den, ws, st);
    case 2: return decode_columns<T, 2>(p, q, k, v, state, o, den, ws, st);
    case 4: return decode_columns<T, 4>(p, q, k, v, state, o, den, ws, st);
    case 8: return decode_columns<T, 8>(p, q, k, v, state, o, den, ws, st);
    case 16: return decode_columns<T, 16>(p, q, k, v, state, o, den, ws, st);
    default: return decode_columns<T, 32>(p, q, k, v, state, o, den, ws, st);
    }
}
}  // namespace

int decode_shares(const Plan &p)
{
    const int per = kDecodeThreads / ((p.d + 63) & ~63) * decode_rows(p);
    return p.L * ((p.R + per - 1) / per);
}

hipError_t decode_step(const Plan &p, const void *q, const void *k, const void *v, float *state, void *o, float *den, char *ws,
                       hipStream_t st)
{
    if (p.dtype == RACE_F32) decode_t(p, (const float *)q, (const float *)k, (const float *)v, state, (float *)o, den, ws, st);
    else decode_t(p, (const bf16_t *)q, (const bf16_t *)k, (const bf16_t *)v, state, (bf16_t *)o, den, ws, st);
    return hipGetLastError();
}

// A few tens of KB over PCIe: every thread has one 16-byte read in flight.  (As a stream-ordered copy through the runtime
// the same bytes cost a hand-over to a copy engine and back: 8 us of copy between gaps of 10 and 16 us, 35 us in front of
// every pass, against 3-4 us for this kernel.)
__global__ __launch_bounds__(256) void upload_kernel(uint4 *dst, const uint4 *src, size_t n16, uint4 *clear, size_t c16)
{
    const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n16) dst[i] = src[i];
    if (i < c16) clear[i] = uint4{0u, 0u, 0u, 0u};
}

hipError_t upload(void *dst, const void *src, size_t bytes, void *clear, size_t clear_bytes, hipStream_t st)
{
    const size_t n16 = bytes / 16, c16 = clear_bytes / 16, n = n16 > c16 ? n16 : c16;
    hipLaunchKernelGGL(upload_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, static_cast<uint4 *>(dst),
                       static_cast<const uint4 *>(src), n16, static_cast<uint4 *>(clear), c16);
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
