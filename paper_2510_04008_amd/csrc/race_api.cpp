// Host side of the C ABI: argument validation, planning (segments, workspace layout), the
// seed -> W generator with its host cache, and dispatch to the kernel families.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "internal.h"

namespace race {

bool simple_supported(int R, int d);

namespace {

thread_local std::string g_last_error;

// largest problem the generic kernels are offered, as the bytes of one fp32 gradient row per token and table, three times (a
// limit of the interface: no kernel keeps such rows)
constexpr size_t kGenericPartialLimit = static_cast<size_t>(16) << 30;

constexpr int kMaxHeadTables = 65535;       // B H L
constexpr int64_t kMaxSegments = 65535;     // per (batch, head)

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// ---------------------------------------------------------------- Philox-4x32-10 + Box-Muller
// Counter-based generator of Salmon et al. (SC'11): ten rounds of two 32x32->64 multiplications,
// the key bumped by the Weyl constants between rounds.
struct Philox4 { uint32_t v[4]; };

Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1)
{
    for (int round = 0; round < 10; ++round) {
        if (round) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
        const uint64_t a = 0xD2511F53ull * c0, b = 0xCD9E8D57ull * c2;
        const uint32_t n0 = static_cast<uint32_t>(b >> 32) ^ c1 ^ k0;
        const uint32_t n2 = static_cast<uint32_t>(a >> 32) ^ c3 ^ k1;
        c1 = static_cast<uint32_t>(b);
        c3 = static_cast<uint32_t>(a);
        c0 = n0;
        c2 = n2;
    }
    return Philox4{{c0, c1, c2, c3}};
}

void gaussian_pair(uint32_t x0, uint32_t x1, double *g)
{
    const double u1 = (static_cast<double>(x0) + 0.5) * (1.0 / 4294967296.0);
    const double u2 = (static_cast<double>(x1) + 0.5) * (1.0 / 4294967296.0);
    const double rad = std::sqrt(-2.0 * std::log(u1));
    const double ang = 2.0 * 3.14159265358979323846 * u2;
    g[0] = rad * std::cos(ang);
    g[1] = rad * std::sin(ang);
}

float round_to_bf16(float x)
{
    uint32_t b;
    std::memcpy(&b, &x, 4);
    b += 0x7fffu + ((b >> 16) & 1u);
    b &= 0xffff0000u;
    std::memcpy(&x, &b, 4);
    return x;
}

// ---------------------------------------------------------------- host cache of projection images
struct CacheKey {
    int family, dtype, H, L, P, d;
    std::vector<uint64_t> seeds;
    bool operator<(const CacheKey &o) const
    {
        if (family != o.family) return family < o.family;
        if (dtype != o.dtype) return dtype < o.dtype;
        if (H != o.H) return H < o.H;
        if (L != o.L) return L < o.L;
        if (P != o.P) return P < o.P;
        if (d != o.d) return d < o.d;
        return seeds < o.seeds;
    }
};
struct CacheEntry { void *pinned; const void *device_view; size_t bytes; };
std::mutex g_cache_mutex;
std::map<CacheKey, CacheEntry> g_cache;

}  // namespace

void expand_projection_host(int H, int L, int P, int d, int dtype, const uint64_t *seeds, float *out)
{
    const size_t n = static_cast<size_t>(L) * P * d;
    for (int h = 0; h < H; ++h) {
        const uint32_t k0 = static_cast<uint32_t>(seeds[h]), k1 = static_cast<uint32_t>(seeds[h] >> 32);
        float *w = out + static_cast<size_t>(h) * n;
        for (size_t blk = 0; blk * 4 < n; ++blk) {
            const Philox4 x = philox4x32_10(static_cast<uint32_t>(blk), static_cast<uint32_t>(blk >> 32), 0, 0, k0, k1);
            double g[4];
            gaussian_pair(x.v[0], x.v[1], g);
            gaussian_pair(x.v[2], x.v[3], g + 2);
            for (size_t i = 0; i < 4 && blk * 4 + i < n; ++i) {
                float f = static_cast<float>(g[i]);
                w[blk * 4 + i] = (dtype == RACE_BF16) ? round_to_bf16(f) : f;
            }
        }
    }
}

// An image is never freed or moved once made: an asynchronous copy that was enqueued from it, or a captured graph
// that holds such a copy, may read it at any later time.  The cache is therefore bounded by refusing new keys, not
// by evicting old ones (an image is a few KB to ~100 KB).
const void *projection_image(const Plan &p, const uint64_t *seeds, size_t *bytes, bool may_allocate, const char **why)
{
    CacheKey key{p.family, p.dtype, p.H, p.L, p.P, p.d, std::vector<uint64_t>(seeds, seeds + p.H)};
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    auto it = g_cache.find(key);
    if (it == g_cache.end()) {
        if (!may_allocate) {
            *why = "the projection image of these seeds and this shape has not been prepared by an earlier call";
            return nullptr;
        }
        if (g_cache.size() >= kMaxProjectionImages) {
            *why = "projection image cache full (4096 distinct combinations of seeds and shape in this process)";
            return nullptr;
        }
        std::vector<float> W(static_cast<size_t>(p.H) * p.LP * p.d);
        expand_projection_host(p.H, p.L, p.P, p.d, p.dtype, seeds, W.data());
        CacheEntry e;
        e.bytes = p.bytes_W;
        if (hipHostMalloc(&e.pinned, e.bytes, hipHostMallocDefault) != hipSuccess) {
            *why = "hipHostMalloc(projection image) failed";
            return nullptr;
        }
        void *view = nullptr;
        if (hipHostGetDevicePointer(&view, e.pinned, 0) != hipSuccess) {
            (void)hipHostFree(e.pinned);
            *why = "hipHostGetDevicePointer(projection image) failed";
            return nullptr;
        }
        e.device_view = view;
        if (p.family == kFamilyMfma) mfma_pack_projection(p, W.data(), e.pinned);
        else std::memcpy(e.pinned, W.data(), W.size() * sizeof(float));
        it = g_cache.emplace(std::move(key), e).first;
    }
    *bytes = it->second.bytes;
    return it->second.device_view;
}

hipError_t allow_lds_bytes(const void *kernel, size_t bytes)
{
    if (bytes <= 64 * 1024) return hipSuccess;         // what every kernel may use
    thread_local std::map<std::pair<int, const void *>, size_t> allowed;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    size_t &have = allowed[{dev, kernel}];
    if (bytes <= have) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
    if (e == hipSuccess) have = bytes;
    return e;
}

// ---------------------------------------------------------------- per-kernel timing (benchmark aid)
namespace {
struct ProfileRecord { const char *name; hipEvent_t start, stop; };
thread_local bool g_profile_on = false;
thread_local std::vector<ProfileRecord> g_profile_records;
thread_local std::vector<hipEvent_t> g_profile_pool;

hipEvent_t take_event()
{
    if (!g_profile_pool.empty()) {
        hipEvent_t e = g_profile_pool.back();
        g_profile_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    (void)hipEventCreate(&e);
    return e;
}
}  // namespace

ProfileScope::ProfileScope(const char *name, hipStream_t st) : rec_(nullptr), st_(st)
{
    if (!g_profile_on) return;
    ProfileRecord r{name, take_event(), take_event()};
    if (!r.start || !r.stop) return;
    (void)hipEventRecord(r.start, st);
    g_profile_records.push_back(r);
    rec_ = reinterpret_cast<void *>(g_profile_records.size());      // index + 1
}

ProfileScope::~ProfileScope()
{
    if (!rec_) return;
    const size_t i = reinterpret_cast<size_t>(rec_) - 1;
    if (i < g_profile_records.size()) (void)hipEventRecord(g_profile_records[i].stop, st_);
}

// Segment length the MFMA family chooses, in its 32-token tiles: the k that makes
//     rounds * k * (time of a tile in all passes) + (workgroups) * (time to move a state through passes and scans)
// smallest.  A round is one workgroup per CU (256).  Sequences of medium length come out at one round with as few, long
// segments as fill the chip (two rounds with half the segment take as long and move twice the states; more rounds only
// where B H divides the chip badly), short ones at the balance of the two terms.  Where the second round's states are
// less than a hundredth of the whole (512 bucket rows: from 10^6 tokens at B H = 4), two rounds: segments half as long, so
// that their boundaries stay where callers of race_attn_segment_tokens have had them and a late workgroup delays half as much.
// The two times are fits to sweeps over segment lengths of training steps, us: at 512 bucket rows of 128 columns 22 and 0.31, at 64
// bucket rows 11.5 and 0.04.  They were made with kernels whose tiles took about 7 % longer; the present ones have their
// minimum in the same place (512 bucket rows, B H = 16, N = 1000: 237, 171, 151, 152, 165 us at 11, 6, 4, 3, 2 tiles, the rule's choice
// 151; N = 4096: 294, 406, 430 at 8, 6, 4, the rule's 297; 64 bucket rows, N = 1000: 67, 63, 60, 70 at 4, 3, 2, 1, the rule's 60).  Shapes whose stream kernels fit a CU twice take two workgroups per CU once those
// have a dozen tiles each (64 bucket rows, B H = 64, N = 16384, when the rule was made: 1619 -> 1470 us); before that the gradient kernels, which fit
// once, would run a second, nearly empty round.
static int64_t mfma_segment_tokens(const Plan &p)
{
    const int64_t n = p.N > 0 ? p.N : 1, tiles = (n + 31) / 32;
    const double state_us = static_cast<double>(p.LRc) * (p.d + 1) * 1.2e-6 * 4, tile_us = 10.0 + 12.0 * p.LRc / 512.0;
    const int64_t slots = (mfma_workgroups_per_cu(p) == 2 && tiles * p.BH >= 512 * 12) ? 512 : 256;
    auto cost = [&](int64_t k) {
        const int64_t groups = p.BH * ((tiles + k - 1) / k);
        return static_cast<double>((groups + slots - 1) / slots * k) * tile_us + static_cast<double>(groups) * state_us;
    };
    int64_t best_k = tiles;
    double best = cost(tiles);
    auto consider = [&](int64_t k) {
        if (k < 1 || k > tiles || (tiles + k - 1) / k > kMaxSegments || cost(k) >= best) return;
        best = cost(k);
        best_k = k;
    };
    auto tiles_in_rounds = [&](int64_t rounds) {
        const int64_t nseg = slots * rounds / p.BH;
        return nseg > 0 ? (tiles + nseg - 1) / nseg : 0;
    };
    for (int64_t rounds = 1; rounds <= 4; ++rounds) consider(tiles_in_rounds(rounds));
    const int64_t balance = static_cast<int64_t>(std::sqrt(state_us * static_cast<double>(tiles) * p.BH / tile_us));
    for (int64_t k = balance; k <= balance + 2; ++k) consider(k);
    const int64_t two = tiles_in_rounds(2);
    if (slots == 256 && two >= 1 && two < best_k && cost(two) <= 1.01 * best) best_k = two;
    return best_k * 32;
}

race_status_t make_plan(const race_attn_desc_t *desc, Plan *pl)
{
    if (!desc) return RACE_ERR_INVALID_ARG;
    if (desc->B < 1 || desc->H < 1 || desc->N < 0 || desc->d < 1 || desc->L < 1 || desc->P < 1)
        return RACE_ERR_INVALID_ARG;
    if (!(desc->sharpening > 0.0f)) return RACE_ERR_INVALID_ARG;         // NaN fails too; +infinity = hard hash
    if (desc->causal != 0 && desc->causal != 1) return RACE_ERR_INVALID_ARG;
    if (desc->dtype != RACE_F32 && desc->dtype != RACE_BF16) return RACE_ERR_INVALID_ARG;
    if (desc->chunk < 0) return RACE_ERR_INVALID_ARG;
    if (desc->unit_qk != 0 && desc->unit_qk != 1) return RACE_ERR_INVALID_ARG;
    if (desc->P > 8 || desc->d > 256 || desc->d % 8 != 0) return RACE_ERR_UNSUPPORTED;
    if (desc->L > 4096 || static_cast<int64_t>(desc->B) * desc->H > 65535) return RACE_ERR_UNSUPPORTED;
    if (static_cast<int64_t>(desc->B) * desc->H * desc->L > kMaxHeadTables) return RACE_ERR_UNSUPPORTED;
    if (desc->N > (static_cast<int64_t>(1) << 40)) return RACE_ERR_UNSUPPORTED;

    Plan p{};
    p.B = desc->B; p.H = desc->H; p.BH = desc->B * desc->H; p.d = desc->d; p.L = desc->L; p.P = desc->P;
    p.R = 1 << desc->P; p.LP = p.L * p.P; p.LR = p.L * p.R; p.N = desc->N; p.beta = desc->sharpening;
    p.causal = desc->causal; p.dtype = desc->dtype; p.unit_qk = desc->unit_qk;

    const char *force = std::getenv("RACE_ATTN_FORCE_GENERIC");
    const bool forced = force && force[0] == '1';
    p.Lc = p.L; p.Pc = p.P; p.LRc = p.LR; p.pad = 0;
    if (p.dtype == RACE_BF16 && !forced && mfma_pick(p.d, p.L, p.P, &p.Lc, &p.Pc, &p.pad)) {
        p.family = kFamilyMfma;
        p.LRc = p.Lc * (1 << p.Pc);
    } else if (simple_supported(p.R, p.d)) p.family = kFamilySimple;
    else return RACE_ERR_UNSUPPORTED;

    const int64_t n = p.N > 0 ? p.N : 1;
    if (p.family == kFamilySimple) {
        // (segments as the caller's chunk has them, in eights of tokens: the limit does not follow the kernels' tiles)
        if (desc->chunk > 0 && (n - 1) / ((std::min(desc->chunk, n) + 7) / 8 * 8) + 1 > kMaxSegments) return RACE_ERR_UNSUPPORTED;
        generic_geometry(desc->chunk, &p);
        p.nseg = static_cast<int>((n + p.seg_len - 1) / p.seg_len);
        p.bytes_W = align256(static_cast<size_t>(p.H) * p.LP * p.d * sizeof(float));
        p.bytes_state = align256(static_cast<size_t>(p.BH) * p.nseg * generic_state_floats(p) * sizeof(float));
        p.bytes_mass = align256(static_cast<size_t>(p.BH) * n * p.LP * 2 * sizeof(float));
        p.bytes_part = align256(static_cast<size_t>(p.BH) * n * 2 * sizeof(float));
        // the fp32 path is not a long-context path: problems beyond this size are refused
        const size_t per_table = static_cast<size_t>(p.BH) * p.L * n * sizeof(float);
        const size_t fwd_part = per_table * (p.d + 1), bwd_part = per_table * p.d * 3;
        if (align256(fwd_part > bwd_part ? fwd_part : bwd_part) > kGenericPartialLimit) return RACE_ERR_UNSUPPORTED;
        p.dbeta_parts = p.nseg;
    } else {
        int64_t len = desc->chunk > 0 ? desc->chunk : mfma_segment_tokens(p);
        len = (len + 31) / 32 * 32;
        p.seg_len = len;
        if ((n + len - 1) / len > kMaxSegments) return RACE_ERR_UNSUPPORTED;
        p.nseg = static_cast<int>((n + len - 1) / len);
        p.bytes_W = align256(mfma_projection_bytes(p));
        p.bytes_state = align256(static_cast<size_t>(p.BH) * p.nseg * p.LRc * (p.d + 1) * sizeof(float));
        p.bytes_part = 0;
        p.bytes_mass = align256(mfma_hashed_bytes(p));
        p.bytes_ge = align256(static_cast<size_t>(p.BH) * n * sizeof(float));
        p.dbeta_parts = mfma_dbeta_parts(p);
    }
    p.bytes_dbeta = align256(static_cast<size_t>(2) * p.BH * p.dbeta_parts * sizeof(float));
    // [W | key/value statistics | hashed Q | hashed K | row norms] is what the forward pass leaves behind; [cotangent statistics |
    // extra column of the cotangents | parts of dbeta] follow (the generic family's forward pass may carry statistics in the first
    // of these)
    p.off_W = 0;
    p.off_stateA = p.off_W + p.bytes_W;
    p.off_massQ = p.off_stateA + p.bytes_state;
    p.off_massK = p.off_massQ + p.bytes_mass;
    p.off_part = p.off_massK + p.bytes_mass;
    p.off_stateB = p.off_part + p.bytes_part;
    p.off_ge = p.off_stateB + p.bytes_state;
    p.off_dbeta = p.off_ge + p.bytes_ge;
    p.total = p.off_dbeta + p.bytes_dbeta;
    p.fwd_bytes = (p.family == kFamilySimple && generic_carries(p)) ? p.off_stateB + p.bytes_state : p.off_stateB;
    *pl = p;
    return RACE_OK;
}

namespace {

race_status_t hip_failed(hipError_t e, const char *where)
{
    g_last_error = std::string(where) + ": " + hipGetErrorString(e);
    return RACE_ERR_HIP;
}

race_status_t check_workspace(const Plan &p, const void *ws, size_t bytes, size_t need)
{
    (void)p;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) != 0 || bytes < need) return RACE_ERR_WORKSPACE;
    return RACE_OK;
}

bool any_equal(std::initializer_list<const void *> outs, std::initializer_list<const void *> all)
{
    for (const void *o : outs) {
        int hits = 0;
        for (const void *a : all) hits += (a == o);
        if (hits > 1) return true;
    }
    return false;
}

// Copies the image of W to its place in the workspace (and zeroes `clear_bytes` at `clear` on the way).
race_status_t upload_projection(const Plan &p, const uint64_t *seeds, char *ws, hipStream_t st, bool may_allocate = true,
                                void *clear = nullptr, size_t clear_bytes = 0)
{
    size_t bytes = 0;
    const char *why = "";
    const void *img = projection_image(p, seeds, &bytes, may_allocate, &why);
    if (!img) {
        g_last_error = why;
        return may_allocate ? RACE_ERR_HIP : RACE_ERR_NOT_READY;
    }
    hipError_t e = upload(ws + p.off_W, img, bytes, clear, clear_bytes, st);
    if (e != hipSuccess) return hip_failed(e, "upload of the projection image");
    return RACE_OK;
}

}  // namespace
}  // namespace race

using namespace race;

extern "C" {

size_t race_attn_workspace_bytes(const race_attn_desc_t *desc)
{
    Plan p;
    if (make_plan(desc, &p) != RACE_OK || p.N == 0) return 0;
    return p.total;
}

int race_attn_kernel_family(const race_attn_desc_t *desc)
{
    Plan p;
    if (make_plan(desc, &p) != RACE_OK) return kFamilyNone;
    return p.family;
}

int64_t race_attn_segment_tokens(const race_attn_desc_t *desc)
{
    Plan p;
    if (make_plan(desc, &p) != RACE_OK) return 0;
    return p.seg_len;
}

race_status_t race_attn_fwd(const race_attn_desc_t *desc, const void *Q, const void *K, const void *V,
                            const uint64_t *proj_seeds, void *O, float *den, void *workspace,
                            size_t workspace_bytes, race_stream_t stream)
{
    Plan p;
    race_status_t s = make_plan(desc, &p);
    if (s != RACE_OK) return s;
    if (p.N == 0) return RACE_OK;      // nothing to do, pointers may be null
    if (!Q || !K || !V || !proj_seeds || !O || !den) return RACE_ERR_INVALID_ARG;
    if (any_equal({O, den}, {Q, K, V, O, den})) return RACE_ERR_INVALID_ARG;
    if ((s = check_workspace(p, workspace, workspace_bytes, p.total)) != RACE_OK) return s;
    char *ws = static_cast<char *>(workspace);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if ((s = upload_projection(p, proj_seeds, ws, st)) != RACE_OK) return s;
    hipError_t e = (p.family == kFamilyMfma) ? mfma_fwd(p, Q, K, V, O, den, ws, st)
                                             : simple_fwd(p, Q, K, V, O, den, ws, st);
    return e == hipSuccess ? RACE_OK : hip_failed(e, "race_attn_fwd launch");
}

namespace {
// What the size limit of race_attn_fwd_static counts, with the whole sequence as one segment per (batch, head): W, the
// statistics, and per token and head the hashed rows of Q and K; the generic family is charged two sets of statistics and
// three fp32 rows per token and table.  The limit is part of the interface and does not follow the layout of the workspace;
// the array is half as large again, which covers what that layout adds (rows rounded up to tiles of 32 tokens; the generic
// family's hashed rows and projections, 16 L P bytes against the 12 L d charged, at d = 8 and P > 5).
size_t static_limit_bytes(const Plan &p)
{
    const size_t rows = static_cast<size_t>(p.BH) * p.N, heads = static_cast<size_t>(p.BH);
    if (p.family == kFamilyMfma)
        return p.bytes_W + align256(heads * p.LRc * (p.d + 1) * sizeof(float)) + 2 * align256(rows * p.Lc * p.Pc * sizeof(float));
    return p.bytes_W + 2 * align256(heads * p.LR * (p.d + 1) * sizeof(float)) + align256(3 * rows * p.L * p.d * sizeof(float));
}

race_status_t static_too_large()
{
    g_last_error = "race_attn_fwd_static: the problem needs more than the 32 MiB of built-in scratch; use race_attn_fwd with a workspace";
    return RACE_ERR_WORKSPACE;
}
}  // namespace

// The forward pass on the library's own scratch array: same kernels, same arguments, no allocation of any kind.
race_status_t race_attn_fwd_static(const race_attn_desc_t *desc, const void *Q, const void *K, const void *V,
                                   const uint64_t *proj_seeds, void *O, float *den, race_stream_t stream)
{
    Plan p;
    race_status_t s = make_plan(desc, &p);
    if (s != RACE_OK) return s;
    if (p.N == 0) return RACE_OK;
    if (!Q || !K || !V || !proj_seeds || !O || !den) return RACE_ERR_INVALID_ARG;
    if (any_equal({O, den}, {Q, K, V, O, den})) return RACE_ERR_INVALID_ARG;
    if (static_limit_bytes(p) > kStaticLimitBytes) return static_too_large();
    // Fewer, longer scan segments until the forward's share of the workspace (W, the segment statistics, the hashed rows)
    // fits the array; a caller's own desc->chunk is kept as the smallest segment length tried.
    race_attn_desc_t fit = *desc;
    while (p.fwd_bytes > kStaticScratchBytes) {
        if (p.nseg <= 1) return static_too_large();
        fit.chunk = p.seg_len * 2;
        if ((s = make_plan(&fit, &p)) != RACE_OK) return s;
    }
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    // the image must be there already: making it would allocate pinned host memory
    size_t bytes = 0;
    const char *why = "";
    if (!projection_image(p, proj_seeds, &bytes, false, &why)) {
        g_last_error = std::string("race_attn_fwd_static: ") + why;
        return RACE_ERR_NOT_READY;
    }
    void *scratch = nullptr;
    hipError_t e = static_scratch(&scratch);
    if (e != hipSuccess) return hip_failed(e, "hipGetSymbolAddress(static scratch)");
    char *ws = static_cast<char *>(scratch);
    if ((s = upload_projection(p, proj_seeds, ws, st, false)) != RACE_OK) return s;
    e = (p.family == kFamilyMfma) ? mfma_fwd(p, Q, K, V, O, den, ws, st) : simple_fwd(p, Q, K, V, O, den, ws, st);
    return e == hipSuccess ? RACE_OK : hip_failed(e, "race_attn_fwd_static launch");
}

race_status_t race_attn_bwd(const race_attn_desc_t *desc, const void *Q, const void *K, const void *V,
                            const void *O, const float *den, const void *dO, const uint64_t *proj_seeds,
                            void *dQ, void *dK, void *dV, void *workspace, size_t workspace_bytes,
                            race_stream_t stream)
{
    return race_attn_bwd_beta(desc, Q, K, V, O, den, dO, proj_seeds, dQ, dK, dV, nullptr, workspace, workspace_bytes,
                              stream);
}

namespace {
race_status_t backward(const race_attn_desc_t *desc, const void *Q, const void *K, const void *V, const void *O,
                       const float *den, const void *dO, const uint64_t *proj_seeds, void *dQ, void *dK, void *dV,
                       float *dbeta, void *workspace, size_t workspace_bytes, race_stream_t stream, bool saved);
}

race_status_t race_attn_bwd_beta(const race_attn_desc_t *desc, const void *Q, const void *K, const void *V,
                                 const void *O, const float *den, const void *dO, const uint64_t *proj_seeds,
                                 void *dQ, void *dK, void *dV, float *dbeta, void *workspace,
                                 size_t workspace_bytes, race_stream_t stream)
{
    return backward(desc, Q, K, V, O, den, dO, proj_seeds, dQ, dK, dV, dbeta, workspace, workspace_bytes, stream, false);
}

race_status_t race_attn_bwd_saved(const race_attn_desc_t *desc, const void *Q, const void *K, const void *V,
                                  const void *O, const float *den, const void *dO, const uint64_t *proj_seeds,
                                  void *dQ, void *dK, void *dV, float *dbeta, void *workspace,
                                  size_t workspace_bytes, race_stream_t stream)
{
    return backward(desc, Q, K, V, O, den, dO, proj_seeds, dQ, dK, dV, dbeta, workspace, workspace_bytes, stream, true);
}

namespace {
race_status_t backward(const race_attn_desc_t *desc, const void *Q, const void *K, const void *V, const void *O,
                       const float *den, const void *dO, const uint64_t *proj_seeds, void *dQ, void *dK, void *dV,
                       float *dbeta, void *workspace, size_t workspace_bytes, race_stream_t stream, bool saved)
{
    Plan p;
    race_status_t s = make_plan(desc, &p);
    if (s != RACE_OK) return s;
    if (p.N == 0) return RACE_OK;      // nothing to do, pointers may be null
    if (!Q || !K || !V || !O || !den || !dO || !proj_seeds || !dQ || !dK || !dV) return RACE_ERR_INVALID_ARG;
    if (std::isinf(p.beta)) return RACE_ERR_UNSUPPORTED;      // the hard hash is piecewise constant: inference only
    if (any_equal({dQ, dK, dV}, {Q, K, V, O, den, dO, dQ, dK, dV})) return RACE_ERR_INVALID_ARG;
    if (dbeta && any_equal({dbeta}, {Q, K, V, O, den, dO, dQ, dK, dV, dbeta})) return RACE_ERR_INVALID_ARG;
    if ((s = check_workspace(p, workspace, workspace_bytes, p.total)) != RACE_OK) return s;
    char *ws = static_cast<char *>(workspace);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    // the forward leaves its projection image, hashed rows and segment-start statistics where the backward pass looks for them
    p.fwd_state_kept = saved ? 1 : 0;
    if (!p.fwd_state_kept && (s = upload_projection(p, proj_seeds, ws, st)) != RACE_OK) return s;
    hipError_t e = (p.family == kFamilyMfma) ? mfma_bwd(p, Q, K, V, O, den, dO, dQ, dK, dV, dbeta, ws, st)
                                             : simple_bwd(p, Q, K, V, O, den, dO, dQ, dK, dV, dbeta, ws, st);
    return e == hipSuccess ? RACE_OK : hip_failed(e, "race_attn_bwd launch");
}
}  // namespace

race_status_t race_attn_expand_projection(const race_attn_desc_t *desc, const uint64_t *proj_seeds, float *W_host)
{
    if (!desc || !proj_seeds || !W_host) return RACE_ERR_INVALID_ARG;
    if (desc->H < 1 || desc->L < 1 || desc->P < 1 || desc->d < 1) return RACE_ERR_INVALID_ARG;
    if (desc->dtype != RACE_F32 && desc->dtype != RACE_BF16) return RACE_ERR_INVALID_ARG;
    if (desc->P > 8 || desc->d > 256 || desc->L > 4096) return RACE_ERR_UNSUPPORTED;
    expand_projection_host(desc->H, desc->L, desc->P, desc->d, desc->dtype, proj_seeds, W_host);
    return RACE_OK;
}

race_status_t race_attn_debug_hash(const race_attn_desc_t *desc, const void *X, const uint64_t *proj_seeds,
                                   uint8_t *codes, float *phi, void *workspace, size_t workspace_bytes,
                                   race_stream_t stream)
{
    Plan p;
    race_status_t s = make_plan(desc, &p);
    if (s != RACE_OK) return s;
    if (p.N == 0) return RACE_OK;      // nothing to do, pointers may be null
    if (!X || !proj_seeds || !codes) return RACE_ERR_INVALID_ARG;
    if ((s = check_workspace(p, workspace, workspace_bytes, p.off_W + p.bytes_W)) != RACE_OK) return s;
    char *ws = static_cast<char *>(workspace);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if ((s = upload_projection(p, proj_seeds, ws, st)) != RACE_OK) return s;
    hipError_t e = (p.family == kFamilyMfma) ? mfma_hash(p, X, codes, phi, ws, st)
                                             : simple_hash(p, X, codes, phi, ws, st);
    return e == hipSuccess ? RACE_OK : hip_failed(e, "race_attn_debug_hash launch");
}

race_status_t race_attn_debug_buckets(const race_attn_desc_t *desc, const void *K, const void *V,
                                      const uint64_t *proj_seeds, float *A, float *Bsum, void *workspace,
                                      size_t workspace_bytes, race_stream_t stream)
{
    Plan p;
    race_status_t s = make_plan(desc, &p);
    if (s != RACE_OK) return s;
    if (p.N == 0) return RACE_OK;      // nothing to do, pointers may be null
    if (!K || !V || !proj_seeds || !A || !Bsum) return RACE_ERR_INVALID_ARG;
    if ((s = check_workspace(p, workspace, workspace_bytes, p.total)) != RACE_OK) return s;
    char *ws = static_cast<char *>(workspace);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if ((s = upload_projection(p, proj_seeds, ws, st)) != RACE_OK) return s;
    hipError_t e = (p.family == kFamilyMfma) ? mfma_buckets(p, K, V, A, Bsum, 1, p.d, ws, st)
                                             : simple_buckets(p, K, V, A, Bsum, 1, p.d, ws, st);
    return e == hipSuccess ? RACE_OK : hip_failed(e, "race_attn_debug_buckets launch");
}

size_t race_attn_state_bytes(const race_attn_desc_t *desc)
{
    Plan p;
    race_attn_desc_t one;
    if (!desc) return 0;
    one = *desc;
    one.N = 1;                             // the state does not depend on the context length
    if (one.chunk < 0) one.chunk = 0;
    if (make_plan(&one, &p) != RACE_OK) return 0;
    return static_cast<size_t>(p.BH) * p.LR * (p.d + 1) * sizeof(float);
}

race_status_t race_attn_state_init(const race_attn_desc_t *desc, const void *K, const void *V,
                                   const uint64_t *proj_seeds, float *state, void *workspace,
                                   size_t workspace_bytes, race_stream_t stream)
{
    Plan p;
    race_status_t s = make_plan(desc, &p);
    if (s != RACE_OK) return s;
    if (!state) return RACE_ERR_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (p.N == 0) {                        // empty context
        hipError_t e = zero_floats(state, static_cast<size_t>(p.BH) * p.LR * (p.d + 1), st);
        return e == hipSuccess ? RACE_OK : hip_failed(e, "race_attn_state_init launch");
    }
    if (!K || !V || !proj_seeds) return RACE_ERR_INVALID_ARG;
    if (static_cast<const void *>(state) == K || static_cast<const void *>(state) == V) return RACE_ERR_INVALID_ARG;
    if ((s = check_workspace(p, workspace, workspace_bytes, p.total)) != RACE_OK) return s;
    char *ws = static_cast<char *>(workspace);
    if ((s = upload_projection(p, proj_seeds, ws, st)) != RACE_OK) return s;
    // interleaved layout: per bucket row d sums, then the mass
    hipError_t e = (p.family == kFamilyMfma) ? mfma_buckets(p, K, V, state + p.d, state, p.d + 1, p.d + 1, ws, st)
                                             : simple_buckets(p, K, V, state + p.d, state, p.d + 1, p.d + 1, ws, st);
    return e == hipSuccess ? RACE_OK : hip_failed(e, "race_attn_state_init launch");
}

namespace {
// A decoding step runs on the generic kernels' fp32 image of W whatever family serves the long passes.
race_status_t make_step_plan(const race_attn_desc_t *desc, Plan *pl)
{
    if (!desc) return RACE_ERR_INVALID_ARG;
    race_attn_desc_t one = *desc;
    one.N = 1;
    one.causal = 1;
    one.chunk = 0;
    race_status_t s = make_plan(&one, pl);
    if (s != RACE_OK) return s;
    pl->family = kFamilySimple;
    pl->off_W = 0;
    pl->bytes_W = align256(static_cast<size_t>(pl->H) * pl->LP * pl->d * sizeof(float));
    // [W | arrival counters | shares]: what an earlier step leaves for one without seeds, W and cleared counters, does not depend
    // on B (the counters are those of the largest B H there is)
    pl->off_arrived = pl->bytes_W;
    pl->bytes_arrived = align256(static_cast<size_t>(kMaxHeadTables / pl->L) * sizeof(unsigned));
    pl->off_part = pl->off_arrived + pl->bytes_arrived;
    pl->bytes_part = align256(static_cast<size_t>(pl->BH) * decode_shares(*pl) * (pl->d + 1) * sizeof(float));
    pl->total = pl->off_part + pl->bytes_part;
    return RACE_OK;
}
}  // namespace

size_t race_attn_step_workspace_bytes(const race_attn_desc_t *desc)
{
    Plan p;
    return make_step_plan(desc, &p) == RACE_OK ? p.total : 0;
}

race_status_t race_attn_step(const race_attn_desc_t *desc, const void *q, const void *k, const void *v,
                             const uint64_t *proj_seeds, float *state, void *o, float *den, void *workspace,
                             size_t workspace_bytes, race_stream_t stream)
{
    Plan p;
    race_status_t s = make_step_plan(desc, &p);
    if (s != RACE_OK) return s;
    if (!q || !k || !v || !state || !o || !den) return RACE_ERR_INVALID_ARG;
    if (any_equal({state, o, den}, {q, k, v, state, o, den})) return RACE_ERR_INVALID_ARG;
    if ((s = check_workspace(p, workspace, workspace_bytes, p.total)) != RACE_OK) return s;
    char *ws = static_cast<char *>(workspace);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    // no seeds: the workspace still holds the W and the cleared counters that an earlier step left there
    if (proj_seeds && (s = upload_projection(p, proj_seeds, ws, st, true, ws + p.off_arrived, p.bytes_arrived)) != RACE_OK) return s;
    hipError_t e = decode_step(p, q, k, v, state, o, den, ws, st);
    return e == hipSuccess ? RACE_OK : hip_failed(e, "race_attn_step launch");
}

const char *race_status_string(race_status_t status)
{
    switch (status) {
    case RACE_OK: return "ok";
    case RACE_ERR_INVALID_ARG: return "invalid argument";
    case RACE_ERR_UNSUPPORTED: return "unsupported shape";
    case RACE_ERR_WORKSPACE: return "workspace null, misaligned or too small";
    case RACE_ERR_HIP: return "HIP call failed";
    case RACE_ERR_NOT_READY: return "a call that prepares this one has not been made";
    }
    return "unknown status";
}

const char *race_attn_last_error(void) { return g_last_error.c_str(); }

race_status_t race_attn_calibration_copy(void *dst, const void *src, size_t bytes, race_stream_t stream)
{
    if (bytes == 0) return RACE_OK;
    if (!dst || !src || bytes % 16 != 0) return RACE_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(dst) % 16 != 0 || reinterpret_cast<uintptr_t>(src) % 16 != 0)
        return RACE_ERR_INVALID_ARG;
    const char *a = static_cast<const char *>(src);
    const char *b = static_cast<const char *>(dst);
    if (a < b + bytes && b < a + bytes) return RACE_ERR_INVALID_ARG;
    hipError_t e = calibration_copy(dst, src, bytes, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) {
        g_last_error = std::string("calibration_copy: ") + hipGetErrorString(e);
        return RACE_ERR_HIP;
    }
    return RACE_OK;
}

race_status_t race_attn_calibration_mfma(int workgroups, int iters, int vector_ops, float *sink, race_stream_t stream)
{
    if (!sink || workgroups < 1 || iters < 1 || workgroups > (1 << 20) || iters > (1 << 20)) return RACE_ERR_INVALID_ARG;
    if (vector_ops != 0 && vector_ops != 4 && vector_ops != 8 && vector_ops != 16) return RACE_ERR_INVALID_ARG;
    hipError_t e = calibration_mfma(workgroups, iters, vector_ops, sink, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) {
        g_last_error = std::string("calibration_mfma: ") + hipGetErrorString(e);
        return RACE_ERR_HIP;
    }
    return RACE_OK;
}

void race_attn_profile_enable(int on)
{
    g_profile_on = on != 0;
    if (!on) {
        for (auto &r : g_profile_records) { g_profile_pool.push_back(r.start); g_profile_pool.push_back(r.stop); }
        g_profile_records.clear();
    }
}

int race_attn_profile_read(int max_entries, const char **names, float *total_ms, int *launches)
{
    std::vector<const char *> seen;
    std::vector<float> ms;
    std::vector<int> cnt;
    for (auto &r : g_profile_records) {
        float t = 0.f;
        if (hipEventSynchronize(r.stop) == hipSuccess) (void)hipEventElapsedTime(&t, r.start, r.stop);
        size_t k = 0;
        while (k < seen.size() && std::strcmp(seen[k], r.name) != 0) ++k;
        if (k == seen.size()) { seen.push_back(r.name); ms.push_back(0.f); cnt.push_back(0); }
        ms[k] += t;
        cnt[k] += 1;
        g_profile_pool.push_back(r.start);
        g_profile_pool.push_back(r.stop);
    }
    g_profile_records.clear();
    for (size_t k = 0; k < seen.size() && static_cast<int>(k) < max_entries; ++k) {
        if (names) names[k] = seen[k];
        if (total_ms) total_ms[k] = ms[k];
        if (launches) launches[k] = cnt[k];
    }
    return static_cast<int>(seen.size());
}

}  // extern "C"
