// C-ABI entry points of libsfda: argument validation, then one kernel launch.
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "../../include/sfda.h"
#include "sfda_launch.h"

// Workspace of sfda_chunk_fwd_segmented_noalloc: a file-scope device array, one copy per GPU
// the library runs on, held until the process ends.  In host code its name is only a
// stand-in; the device address comes from hipGetSymbolAddress (per device, with that device
// current) and only that address is handed to kernels.
static __device__ __align__(256) unsigned char scratch[SFDA_NOALLOC_SCRATCH_BYTES];

namespace {

struct Range {
    uintptr_t lo, hi;   // [lo, hi)
};

Range range_of(const void* p, long bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    return Range{a, a + static_cast<uintptr_t>(bytes > 0 ? bytes : 0)};
}

bool overlap(Range a, Range b) {
    return a.lo < a.hi && b.lo < b.hi && a.lo < b.hi && b.lo < a.hi;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

long esize(sfda_dtype_t d) { return d == SFDA_BF16 ? 2 : 4; }

bool dtype_ok(sfda_dtype_t d) { return d == SFDA_F32 || d == SFDA_BF16; }

// the device address of `scratch` on the current device, looked up once per device
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
void* scratch_ptr[MAX_DEVICES];

sfda_status_t scratch_address(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return SFDA_ERR_HIP;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return SFDA_ERR_HIP;
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return SFDA_OK;
}

// compute units of the current device (0 if it cannot be queried), looked up once per device
std::mutex cu_mu;
int cu_count_cache[MAX_DEVICES];

int device_cus()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return 0;
    std::lock_guard<std::mutex> lock(cu_mu);
    if (cu_count_cache[dev] == 0) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        cu_count_cache[dev] = v;
    }
    return cu_count_cache[dev];
}

// sfda_chunk_fwd's value columns per workgroup: all of a head's columns (up to 64), halved
// to 32 while the heads alone would leave more than half of the compute units idle (each
// workgroup scans its head's sequence on one compute unit; the column slices of a head repeat
// its chunk factors but scan in parallel).  Every column's arithmetic is the same for every
// slice, so the results do not depend on it.
int auto_slice(long BH, int n)
{
    int slice = n <= 64 ? ((n + 7) / 8) * 8 : 64;
    const long cus = device_cus();
    if (slice > 32 && cus > 0 && 2 * BH * ((n + slice - 1) / slice) <= cus) slice = 32;
    return slice;
}

// the factored scans run workgroups of 256 threads per head and 8 value columns (bfloat16 operands:
// 512 per 32), in a launch of less than 2^32 threads, and address a 64-token step's rows of v, o and
// dL/do (at most 8 bytes per element) with 32-bit byte offsets
bool factored_fits(long BH, int m, int n, bool in_bf16)
{
    const long threads = sfda::bf16_operands(in_bf16, m) ? 512 * ((n + 31L) / 32) : 256 * ((n + 7L) / 8);
    return (BH + 7) * threads < (1L << 32) && static_cast<long>(64) * n * 8 < 0x80000000L;
}

// most bytes of operand records that the suggested workspace holds at a time (the sequence then
// runs in pieces).  A bound on memory: more is a little faster (us at 64, 128, 256, 512, 1024 MiB:
// decoupled bfloat16 B8 H16 T4096 592, 519, 485, 460, 443; float32 forward 32 heads T 16384 1489, 1284,
// 1202, 1148, 1127; 16 heads T 65536 3235, 3083, 3150, 3129, 3186), less costs launches and state passes.
constexpr size_t FACTORED_CAP = size_t(256) << 20;
// and what the backward's suggested workspace may take past the smaller one where it is more than
// twice that: a training step has to fit beside it
constexpr size_t BWD_EXTRA = size_t(1280) << 20;

// Whether the factored forward is the faster one.
//  * bfloat16 operands (the write-decoupled forward: 256 compute units, m n 64): past 48 tokens, us in
//    place / factored T 48 21/24, T 64 26/24.
//  * float32 operands: by an estimate of both in us, fitted to 5100 measured pairs of 16 .. 6000 heads
//    x 33 .. 1000 tokens (each within 27%, 4 of the rule's picks 3 to 8% behind the other side).  In place:
//    rounds of one workgroup per compute unit, a chain of blocks each.  Factored: a floor of two
//    launches and a chain of blocks, then time per head and block, padding blocks of the last 64-token
//    step among them (preparation: channel blocks; scan: 8-column workgroups), and for every
//    further piece of the sequence its launches and the state's way through memory.  us in place /
//    factored: forward, 4 heads m n 64 T 48 22/23, T 64 28/23; 96 heads m n 64 T 96 41/41;
//    160 heads m 48 n 32 T 80 34/43; 768 heads m 64 n 32 T 160 189/251; 1500 heads m 48 n 64 T 300
//    931/1237; 256 heads m n 64 T 512 265/286, m 16 n 64 257/203; decoupled, 256 heads m 3 n 64 T 80
//    61/80, 1500 heads m 64 n 48 T 160 675/904, m 16 n 8 T 49 215/76.  It takes a workspace, so it has to
//    be 5% ahead.
struct Blocks { long nb, pad, nkb, cols; };    // 16-token blocks, those of whole steps; channel and 8-column blocks
Blocks blocks_of(int T, int m, int n) { return {(T + 15L) / 16, (T + 63L) / 64 * 4, (m + 15) / 16, (n + 7L) / 8}; }
long rounds_of(long workgroups, long cus) { return (workgroups + cus - 1) / cus; }
bool factored_faster(long BH, int T, int m, int n, bool in_bf16, bool dec)
{
    if (T <= (dec && !in_bf16 ? 32 : 48)) return false;
    if (sfda::bf16_operands(in_bf16, m)) return true;
    const long cus = device_cus() > 0 ? device_cus() : 256;
    const Blocks k = blocks_of(T, m, n);
    const int slice = auto_slice(BH, n);
    const double chain = static_cast<double>(rounds_of(BH * ((n + slice - 1) / slice), cus)) * k.nb;
    const double x = static_cast<double>(BH) / cus, wide = static_cast<double>(k.cols * k.nkb);
    const sfda::FactoredPlan p = sfda::factored_plan(BH, T, m, n, in_bf16, dec, sfda::factored_bytes(BH, T, m, n, in_bf16, dec, FACTORED_CAP), cus);
    const double more = p.piece > 0 && !p.beside ? (k.pad / 4 + p.piece - 1) / p.piece - 1 : 0;
    const double in_place = dec ? 5.4 + chain * (8.21 + (slice > 32 ? 3.15 : 0.) + 0.091 * k.nkb)
                                : 5.2 + chain * (5.61 + (slice > 32 ? 2.53 : 0.) + 0.052 * k.nkb);
    const double factored = dec ? 14.5 + 0.468 * k.pad + x * k.pad * (0.610 + 0.841 * k.nkb + 0.831 * k.cols + 0.030 * wide) + more * (21.6 + x * (1.52 * k.cols + 0.096 * wide))
                                : 12.6 + 0.372 * k.pad + x * k.pad * (0.455 + 0.629 * k.nkb + 0.641 * k.cols + 0.013 * wide) + more * (16.7 + x * 1.59 * k.cols);
    return factored < 0.95 * in_place;
}
// The float32 forward over G segments against the one on prepared operands, estimated in us (MI355X):
// the segments' chain costs 8.5 .. 14.5 us a 16-token block with the columns of both sets (past 64
// value columns two launches, 13.5 .. 16), on a G-th of the blocks, and the fold 1.0 .. 2.9 us a
// segment; the prepared operands' chain 0.72 us a block whatever the sizes, and each piece of the
// sequence its launches.  Measured, segments / prepared operands, m n 64: 1 head T 4096 (G 16)
// 268/212, T 16384 (G 64) 410/744, T 65536 (G 256) 967/2886; 8 heads T 16384 (G 32) 618/782; 16
// heads T 65536 (G 16) 3778/3147; 32 heads T 2048 (G 8) 282/153; m n 16: 4 heads T 2048 (G 8)
// 146/113, T 4096 (G 16) 158/203, T 65536 (G 64) 653/2890, 16 heads T 65536 (G 16) 2210/2917;
// m 4 n 16: 1 head T 65536 (G 256) 459/2857, in pieces of one step T 4096 (G 16) 153/516.  A bfloat16
// o takes a third pass in place of the join (another 5.5 .. 8 us a block).
double segments_us(long BH, int T, int m, int n, int G, bool out_bf16, long cus)
{
    const long rounds = (BH * G * ((n + 63L) / 64) + cus - 1) / cus;
    double block = n <= 64 ? 2.6 + 2.95 * ((m + 31) / 32 + (n + 31) / 32) : m <= 32 ? 13.5 : 16.;
    if (out_bf16) block += n <= 32 ? 5.5 : 8.;
    return rounds * block * T / (16. * G) + G * (0.9 + 0.031 * m);
}
double prepared_us(int T, const sfda::FactoredPlan& p)
{
    const long steps = (T + 63L) / 64, pieces = (steps + p.piece - 1) / p.piece;
    return 20. + 0.72 * T / 16 + (pieces - 1) * (p.beside ? 4. : 10.);
}
// and the backward on prepared operands (three launches; two in place).  us in place / factored:
// bfloat16 T 32 30/33, T 48 34/34, T 64 40/34; float32 T 16 34/35, T 32 42/35, 64 heads m n 64 T 32
// 46/53, T 48 56/53, 57 heads m 58 n 32 T 80 64/54, 96 heads m n 64 T 80 83/97, T 96 108/97, 128 heads T 96
// 111/117, T 128 138/119.  With float32 operands, workgroups that fill whole rounds of the chip (the
// padding of the last 64-token step counted in) leave the chain nothing to wait for: 256 heads m n 64
// T 256 511/530, 384 heads T 112 359/396, m 48 768 heads 672/699, 512 heads m 16 T 112 424/361;
// bfloat16 inputs of few channels by their columns alone: 1024 heads m 1 n 64 T 80 607/680, T 96
// 727/683, 768 heads n 96 T 80 769/717.
bool bwd_factored_faster(long BH, int T, int m, int n, bool in_bf16)
{
    if (T <= (in_bf16 ? 48 : 16)) return false;
    if (sfda::bf16_operands(in_bf16, m)) return true;
    const long cus = device_cus() > 0 ? device_cus() : 256;
    const Blocks k = blocks_of(T, m, n);
    const long cols = BH * k.cols;
    const double filled = static_cast<double>(cols) * k.pad / (static_cast<double>(k.nb) * 8 * cus * rounds_of(BH * ((n + 63L) / 64), cus));
    if (in_bf16) return filled < 1.4;
    return T > (cols >= 4 * cus ? 96 : cols >= 3 * cus ? 80 : cols >= 2 * cus ? 32 : 16) && filled * k.nkb / 4 < 0.84;
}

}  // namespace

extern "C" {

const char* sfda_status_string(sfda_status_t s)
{
    switch (s) {
        case SFDA_OK: return "ok";
        case SFDA_ERR_NULL: return "a required pointer is NULL";
        case SFDA_ERR_SHAPE: return "a size is out of range";
        case SFDA_ERR_CHUNK: return "unsupported chunk length (C must be 16, 32, 64 or 128)";
        case SFDA_ERR_DTYPE: return "unsupported dtype";
        case SFDA_ERR_ALIGN: return "a pointer is not 16-byte aligned";
        case SFDA_ERR_ALIAS: return "an output buffer overlaps another buffer";
        case SFDA_ERR_HIP: return "the HIP runtime reported an error";
        case SFDA_ERR_SCRATCH: return "the call needs more workspace than the static scratch holds";
    }
    return "unknown status";
}

int sfda_abi_version(void) { return SFDA_ABI_VERSION; }

// one head's state (m x n complex float32) is addressed with 32-bit byte offsets
static bool state_fits(int m, int n) { return static_cast<long>(m) * n * 8 < 0x80000000L; }
// the float32 path addresses one chunk's rows of v, o and dL/do (C x n complex, at most 8
// bytes per element, C <= 32 in those kernels) with 32-bit byte offsets
static bool chunk_rows_fit(int n) { return static_cast<long>(32) * n * 8 < 0x80000000L; }
// chunk lengths the entry points accept (the kernels' blocking does not change the result,
// Thm 6.1)
static bool chunk_ok(int C) { return C == 16 || C == 32 || C == 64 || C == 128; }

static sfda_status_t chunk_fwd_impl(const void* q, const void* k, const void* v,
                                    const void* alpha, const void* theta, const void* beta,
                                    const float* S0, void* o, float* S_T, int B, int H, int T,
                                    int m, int n, int C, sfda_dtype_t in_dtype,
                                    sfda_dtype_t out_dtype, sfda_stream_t stream, int slice,
                                    void* = nullptr, size_t = 0, bool check_only = false,
                                    const sfda::GateParams* gates = nullptr)
{
    if (!dtype_ok(in_dtype) || !dtype_ok(out_dtype)) return SFDA_ERR_DTYPE;
    if (B < 0 || H < 0 || T < 0 || m < 1 || m > 64 || n < 1 || !state_fits(m, n)) return SFDA_ERR_SHAPE;
    if (!chunk_ok(C)) return SFDA_ERR_CHUNK;
    if (!chunk_rows_fit(n)) return SFDA_ERR_SHAPE;
    if (slice < 8 || slice > 64 || (slice & 7) != 0) return SFDA_ERR_SHAPE;
    const long BH = static_cast<long>(B) * H;
    if (BH * ((n + slice - 1) / slice) > 0x7FFFFFFFL) return SFDA_ERR_SHAPE;
    // bf16 inputs: each head's slice of q, k, v and o is addressed with 32-bit byte offsets
    if (in_dtype == SFDA_BF16 &&
        static_cast<long>(T) * (m > n ? m : n) * 2 * esize(out_dtype) >= 0x80000000L)
        return SFDA_ERR_SHAPE;
    if (BH == 0) return SFDA_OK;
    const bool need_inputs = T > 0;
    if (need_inputs && (!q || !k || !v || !alpha || !theta || !beta || !o)) return SFDA_ERR_NULL;
    const void* ptrs[] = {q, k, v, alpha, theta, beta, S0, o, S_T};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return SFDA_ERR_ALIGN;

    const long ei = esize(in_dtype), eo = esize(out_dtype);
    const long BHT = BH * T;
    const Range rq = range_of(q, BHT * m * 2 * ei), rk = range_of(k, BHT * m * 2 * ei);
    const Range rv = range_of(v, BHT * n * 2 * ei);
    const Range ra = range_of(alpha, BHT * m * ei), rt = range_of(theta, BHT * m * ei);
    const Range rb = range_of(beta, BHT * ei);
    const Range ro = range_of(o, BHT * n * 2 * eo);
    const Range rs0 = range_of(S0, BH * m * n * 2 * 4);
    const Range rst = range_of(S_T, BH * m * n * 2 * 4);
    const Range ins[] = {rq, rk, rv, ra, rt, rb};
    if (need_inputs) {
        for (const Range& r : ins)
            if (overlap(ro, r)) return SFDA_ERR_ALIAS;
        if (overlap(ro, rs0) || overlap(ro, rst)) return SFDA_ERR_ALIAS;
    }
    if (S_T) {
        if (need_inputs)
            for (const Range& r : ins)
                if (overlap(rst, r)) return SFDA_ERR_ALIAS;
        if (S0 && static_cast<const void*>(S0) != static_cast<const void*>(S_T) && overlap(rs0, rst))
            return SFDA_ERR_ALIAS;
    }

    if (check_only) return SFDA_OK;
    sfda::ChunkLaunch L;
    L.q = q; L.k = k; L.v = v; L.alpha = alpha; L.theta = theta; L.beta = beta;
    L.S0 = S0; L.o = o; L.S_T = S_T;
    L.B = B; L.H = H; L.T = T; L.m = m; L.n = n; L.C = C; L.slice = slice;
    L.in_bf16 = in_dtype == SFDA_BF16;
    L.out_bf16 = out_dtype == SFDA_BF16;
    if (gates) {
        L.gated = gates->gated;
        L.alpha_min = gates->alpha_min; L.alpha_max = gates->alpha_max;
        L.theta_max = gates->theta_max; L.eps = gates->eps;
    }
    const hipError_t e = sfda::launch_chunk(L, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
}

sfda_status_t sfda_chunk_fwd(const void* q, const void* k, const void* v, const void* alpha,
                             const void* theta, const void* beta, const float* S0, void* o,
                             float* S_T, int B, int H, int T, int m, int n, int C,
                             sfda_dtype_t in_dtype, sfda_dtype_t out_dtype, sfda_stream_t stream)
{
    const int slice = auto_slice(static_cast<long>(B) * H, n);
    return chunk_fwd_impl(q, k, v, alpha, theta, beta, S0, o, S_T, B, H, T, m, n, C, in_dtype,
                          out_dtype, stream, slice);
}

sfda_status_t sfda_chunk_fwd_sliced(const void* q, const void* k, const void* v,
                                    const void* alpha, const void* theta, const void* beta,
                                    const float* S0, void* o, float* S_T, int B, int H, int T,
                                    int m, int n, int C, int slice, sfda_dtype_t in_dtype,
                                    sfda_dtype_t out_dtype, sfda_stream_t stream)
{
    return chunk_fwd_impl(q, k, v, alpha, theta, beta, S0, o, S_T, B, H, T, m, n, C, in_dtype,
                          out_dtype, stream, slice);
}

sfda_status_t sfda_chunk_fwd_gated(const void* q, const void* k_raw, const void* v,
                                   const void* a, const void* b, const void* c,
                                   const float* S0, void* o, float* S_T, int B, int H, int T,
                                   int m, int n, int C, float alpha_min, float alpha_max,
                                   float theta_max, float eps, sfda_dtype_t in_dtype,
                                   sfda_dtype_t out_dtype, sfda_stream_t stream)
{
    // ALPHA_MIN_GATED <= alpha_min <= alpha_max <= 1: the kernels' 16-token blocks divide by
    // the decay over one block, which stays inside the float range (>= 2^-126) whenever every
    // alpha is at least 2^(-126/16); theta_max and eps finite and >= 0 (NaN fails every
    // comparison)
    constexpr float ALPHA_MIN_GATED = 0.0042719f;     // 2^(-7.875), rounded up
    if (!(alpha_min >= ALPHA_MIN_GATED && alpha_min <= alpha_max && alpha_max <= 1.f)) return SFDA_ERR_SHAPE;
    if (!(theta_max >= 0.f && theta_max < 3.4e38f && eps >= 0.f && eps < 3.4e38f)) return SFDA_ERR_SHAPE;
    const int slice = auto_slice(static_cast<long>(B) * H, n);
    sfda::GateParams gp{true, alpha_min, alpha_max, theta_max, eps};
    return chunk_fwd_impl(q, k_raw, v, a, b, c, S0, o, S_T, B, H, T, m, n, C, in_dtype, out_dtype,
                          stream, slice, nullptr, 0, false, &gp);
}

// the checks of the write-decoupled forward and its launch descriptor (run: false when there is
// nothing to launch)
static sfda_status_t decoupled_prepare(const void* q, const void* k, const void* r, const void* v,
                                       const void* alpha, const void* theta, const void* eta,
                                       const void* beta, const float* S0, void* o, float* S_T,
                                       int B, int H, int T, int m, int n, int C,
                                       sfda_dtype_t in_dtype, sfda_dtype_t out_dtype,
                                       sfda_stream_t stream, sfda::ChunkLaunch& L, bool& run)
{
    run = false;
    const int slice = auto_slice(static_cast<long>(B) * H, n);
    // the shared checks, with the erase strengths in beta's place
    const sfda_status_t st0 = chunk_fwd_impl(q, k, v, alpha, theta, eta, S0, o, S_T, B, H, T, m, n,
                                             C, in_dtype, out_dtype, stream, slice, nullptr, 0,
                                             /*check_only=*/true);
    if (st0 != SFDA_OK) return st0;
    const long BH = static_cast<long>(B) * H;
    if (BH == 0) return SFDA_OK;
    if (T > 0 && (!r || !beta)) return SFDA_ERR_NULL;
    if ((r && !aligned16(r)) || (beta && !aligned16(beta))) return SFDA_ERR_ALIGN;
    const long ei = esize(in_dtype), eo = esize(out_dtype), BHT = BH * T;
    const Range rr = range_of(r, BHT * m * 2 * ei), rb = range_of(beta, BHT * ei);
    if (T > 0 && (overlap(range_of(o, BHT * n * 2 * eo), rr) || overlap(range_of(o, BHT * n * 2 * eo), rb)))
        return SFDA_ERR_ALIAS;
    if (S_T && T > 0 && (overlap(range_of(S_T, BH * m * n * 2 * 4), rr) || overlap(range_of(S_T, BH * m * n * 2 * 4), rb)))
        return SFDA_ERR_ALIAS;
    L.q = q; L.k = k; L.v = v; L.alpha = alpha; L.theta = theta; L.beta = eta;
    L.r = r; L.wbeta = beta;
    L.S0 = S0; L.o = o; L.S_T = S_T;
    L.B = B; L.H = H; L.T = T; L.m = m; L.n = n; L.C = C; L.slice = slice;
    L.in_bf16 = in_dtype == SFDA_BF16;
    L.out_bf16 = out_dtype == SFDA_BF16;
    run = true;
    return SFDA_OK;
}

sfda_status_t sfda_chunk_fwd_decoupled(const void* q, const void* k, const void* r, const void* v,
                                       const void* alpha, const void* theta, const void* eta,
                                       const void* beta, const float* S0, void* o, float* S_T,
                                       int B, int H, int T, int m, int n, int C,
                                       sfda_dtype_t in_dtype, sfda_dtype_t out_dtype,
                                       sfda_stream_t stream)
{
    sfda::ChunkLaunch L;
    bool run;
    const sfda_status_t st0 = decoupled_prepare(q, k, r, v, alpha, theta, eta, beta, S0, o, S_T, B, H, T, m, n, C,
                                                in_dtype, out_dtype, stream, L, run);
    if (st0 != SFDA_OK || !run) return st0;
    const hipError_t e = sfda::launch_chunk_decoupled(L, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
}

size_t sfda_chunk_fwd_factored_workspace_bytes(int B, int H, int T, int m, int n, sfda_dtype_t in_dtype,
                                               int decoupled)
{
    if (B <= 0 || H <= 0 || T <= 0 || m < 1 || m > 64 || n < 1 || !state_fits(m, n) || !chunk_rows_fit(n) ||
        !dtype_ok(in_dtype))
        return 0;
    const long BH = static_cast<long>(B) * H;
    if (!factored_fits(BH, m, n, in_dtype == SFDA_BF16)) return 0;
    return sfda::factored_bytes(BH, T, m, n, in_dtype == SFDA_BF16, decoupled != 0, FACTORED_CAP);
}

int sfda_chunk_fwd_auto_factored(int B, int H, int T, int m, int n, int C, sfda_dtype_t in_dtype, int decoupled)
{
    if (sfda_chunk_fwd_factored_workspace_bytes(B, H, T, m, n, in_dtype, decoupled) == 0) return 0;
    const long BH = static_cast<long>(B) * H;
    // (the workspace holds a step of every head: not past the bound on it)
    if (sfda::factored_bytes(BH, 64, m, n, in_dtype == SFDA_BF16, decoupled != 0, 0) > FACTORED_CAP) return 0;
    if (in_dtype == SFDA_BF16 && !decoupled) {
        // against sfda_chunk_fwd's bfloat16 kernel, whose chain is 0.9 us a block where the scan on
        // prepared operands takes 0.5, and whose segments overtake both on long sequences.  us, in
        // place or in segments / factored, m n 64: 12 heads T 192 20/19, T 256 24/22, T 1536 100/73,
        // T 2560 119/105, T 4096 132/159; 32 heads T 256 24/24, T 1536 100/75; 48 heads T 384 32/35,
        // T 768 55/50, T 3072 193/168; 64 heads T 384 32/34, T 768 55/50, T 1536 101/90, T 2048
        // 130/131; 96 heads T 1024 76/78, T 4096 257/326; 128 heads T 1024 73/100, T 4096 262/372 (records of
        // 495 MB); 256 heads T 4096 351/750; 128 heads T 4096 m 32 n 32 252/301; n 96: 48 heads T 768 56/50, 64 heads T 768 56/50, T 2048 132/136;
        // with half the channels or columns the records are half as many: 64 heads T 2048, T 4096: m 16
        // n 64 130/98, 252/197, m 64 n 16 138/115, 271/249, m 36 n 29 136/107, 267/239
        const long slices = (n + 31L) / 32;
        const bool few = BH <= 32 ? T >= 256 : BH <= 48 ? T >= 640 : BH <= 64 && T >= 640 && (T <= 1536 || (m + 15) / 16 * slices <= 4);
        if (!few || BH * slices > 144) return 0;
        const int G = sfda_chunk_fwd_auto_segments(B, H, T, m, n, C, in_dtype);
        if (G == 1) return 1;
        // (at most four channels, float32 operands: 12 heads n 64 T 2048 356/119; 1 head T 16384 358/734)
        if (!sfda::bf16_operands(true, m)) return T <= 2560;
        // the segments' three passes over a G-th of the blocks and their fold, against the chain, in
        // us, each estimated within 9%: m n 64, 16 heads T 2048 107/88, 12 heads T 4096 132/159; m 8 n 1,
        // 12 heads T 2560 90/109; m 16 n 1, 24 heads T 2048 82/95
        const double cus = static_cast<double>(device_cus()), x = BH / cus, nkb = (m + 15) / 16;
        const double seg = 21.5 + T / (16. * G) * (2.83 + 0.121 * nkb) + G * (0.62 + 0.567 * nkb) + 7.74 * x * ((n + 63) / 64) * G;
        const double fac = 13.6 + 0.532 * T / 16 + x * T / 16 * (0.371 + 0.174 * nkb);
        return fac < 0.96 * seg ? 1 : 0;
    }
    if (!factored_faster(BH, T, m, n, in_dtype == SFDA_BF16, decoupled != 0)) return 0;
    if (!decoupled) {
        const long cus = device_cus();
        const int G = sfda_chunk_fwd_auto_segments(B, H, T, m, n, C, in_dtype);
        if (G > 1 && segments_us(BH, T, m, n, G, false, cus) < prepared_us(T, sfda::factored_plan(BH, T, m, n, false, false,
                sfda_chunk_fwd_factored_workspace_bytes(B, H, T, m, n, in_dtype, 0), cus)))
            return 0;
    }
    return 1;
}

// the checks of both factored entry points past sfda_chunk_fwd's, then the launches
static sfda_status_t factored_impl(const sfda::ChunkLaunch& L, sfda_dtype_t in_dtype, sfda_dtype_t out_dtype,
                                   void* workspace, size_t workspace_bytes, sfda_stream_t stream)
{
    const long BH = static_cast<long>(L.B) * L.H;
    if (!factored_fits(BH, L.m, L.n, L.in_bf16)) return SFDA_ERR_SHAPE;
    const size_t need = sfda_chunk_fwd_factored_workspace_bytes(L.B, L.H, L.T, L.m, L.n, in_dtype, L.r != nullptr);
    if (!workspace) return SFDA_ERR_NULL;
    if (!aligned16(workspace)) return SFDA_ERR_ALIGN;
    if (workspace_bytes < need) return SFDA_ERR_SHAPE;
    const long ei = esize(in_dtype), eo = esize(out_dtype), BHT = BH * L.T, mn = static_cast<long>(L.m) * L.n;
    const Range rw = range_of(workspace, static_cast<long>(need));
    const Range all[] = {range_of(L.q, BHT * L.m * 2 * ei), range_of(L.k, BHT * L.m * 2 * ei),
                         range_of(L.v, BHT * L.n * 2 * ei), range_of(L.alpha, BHT * L.m * ei),
                         range_of(L.theta, BHT * L.m * ei), range_of(L.beta, BHT * ei),
                         range_of(L.o, BHT * L.n * 2 * eo), range_of(L.S0, BH * mn * 8),
                         range_of(L.S_T, BH * mn * 8), range_of(L.r, BHT * L.m * 2 * ei), range_of(L.wbeta, BHT * ei)};
    for (const Range& r : all)
        if (r.lo && overlap(rw, r)) return SFDA_ERR_ALIAS;
    return sfda::launch_factored(L, workspace, need, device_cus(), static_cast<hipStream_t>(stream)) == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
}

sfda_status_t sfda_chunk_fwd_factored(const void* q, const void* k, const void* v, const void* alpha,
                                      const void* theta, const void* beta, const float* S0, void* o,
                                      float* S_T, int B, int H, int T, int m, int n, int C,
                                      sfda_dtype_t in_dtype, sfda_dtype_t out_dtype, void* workspace,
                                      size_t workspace_bytes, sfda_stream_t stream)
{
    const int slice = auto_slice(static_cast<long>(B) * H, n);
    const bool empty = T == 0 || B == 0 || H == 0;      // nothing to factor (T == 0 copies the state)
    const sfda_status_t st0 = chunk_fwd_impl(q, k, v, alpha, theta, beta, S0, o, S_T, B, H, T, m, n, C, in_dtype,
                                             out_dtype, stream, slice, nullptr, 0, /*check_only=*/!empty);
    if (st0 != SFDA_OK || empty) return st0;
    sfda::ChunkLaunch L;
    L.q = q; L.k = k; L.v = v; L.alpha = alpha; L.theta = theta; L.beta = beta;
    L.S0 = S0; L.o = o; L.S_T = S_T;
    L.B = B; L.H = H; L.T = T; L.m = m; L.n = n; L.C = C; L.slice = slice;
    L.in_bf16 = in_dtype == SFDA_BF16;
    L.out_bf16 = out_dtype == SFDA_BF16;
    return factored_impl(L, in_dtype, out_dtype, workspace, workspace_bytes, stream);
}

sfda_status_t sfda_chunk_fwd_decoupled_factored(const void* q, const void* k, const void* r, const void* v,
                                                const void* alpha, const void* theta, const void* eta,
                                                const void* beta, const float* S0, void* o, float* S_T,
                                                int B, int H, int T, int m, int n, int C,
                                                sfda_dtype_t in_dtype, sfda_dtype_t out_dtype,
                                                void* workspace, size_t workspace_bytes, sfda_stream_t stream)
{
    sfda::ChunkLaunch L;
    bool run;
    const sfda_status_t st0 = decoupled_prepare(q, k, r, v, alpha, theta, eta, beta, S0, o, S_T, B, H, T, m, n, C,
                                                in_dtype, out_dtype, stream, L, run);
    if (st0 != SFDA_OK || !run) return st0;
    if (T == 0) {                                       // copies the state
        const hipError_t e = sfda::launch_chunk_decoupled(L, static_cast<hipStream_t>(stream));
        return e == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
    }
    return factored_impl(L, in_dtype, out_dtype, workspace, workspace_bytes, stream);
}

size_t sfda_chunk_fwd_segmented_workspace_bytes(int B, int H, int T, int m, int n, int G,
                                                sfda_dtype_t in_dtype)
{
    if (B <= 0 || H <= 0 || T < 0 || m < 1 || m > 64 || n < 1 || G < 1 || !dtype_ok(in_dtype)) return 0;
    const size_t segs = static_cast<size_t>(B) * H * G, heads = static_cast<size_t>(B) * H;
    // per segment P_g (m x m), B_g and S_in (m x n); with float32 inputs per head and token
    // X_t (m)
    const size_t xt = in_dtype == SFDA_F32 ? heads * static_cast<size_t>(T) * m : 0;
    return (segs * (static_cast<size_t>(m) * m + 2 * static_cast<size_t>(m) * n) + xt) * 8;
}

int sfda_chunk_fwd_auto_segments(int B, int H, int T, int m, int n, int C, sfda_dtype_t in_dtype)
{
    if (B <= 0 || H <= 0 || T <= 0 || m < 1 || m > 64 || n < 1 || !chunk_ok(C) || !dtype_ok(in_dtype))
        return 1;
    const long cus = device_cus();
    if (cus <= 0) return 1;
    const long per = static_cast<long>(B) * H * ((n + 63) / 64);     // workgroups per segment index
    int G = 1;
    while (G < 1024 && per * 2 * G <= cus && T % (2L * G * C) == 0 && T / (2L * G) >= 256) G *= 2;
    // the segmented scan repeats the scan work twice (float32) or three times (bfloat16)
    return G >= (in_dtype == SFDA_F32 ? 4 : 8) ? G : 1;
}

// sfda_chunk_fwd_segmented, and with noalloc the workspace taken from the static scratch
// (its size checked first, its address fetched only after every other argument check)
static sfda_status_t segmented_impl(const void* q, const void* k, const void* v,
                                    const void* alpha, const void* theta, const void* beta,
                                    const float* S0, void* o, float* S_T, int B, int H, int T,
                                    int m, int n, int C, int G, sfda_dtype_t in_dtype,
                                    sfda_dtype_t out_dtype, void* workspace,
                                    size_t workspace_bytes, sfda_stream_t stream, bool noalloc)
{
    if (G < 1) return SFDA_ERR_SHAPE;
    const int slice_n = n <= 64 ? ((n + 7) / 8) * 8 : 64;
    // the shared checks (and the whole call when there is nothing to split)
    if (T == 0 || static_cast<long>(B) * H == 0 || !dtype_ok(in_dtype) || !dtype_ok(out_dtype) ||
        B < 0 || H < 0 || T < 0 || m < 1 || m > 64 || n < 1 || !state_fits(m, n) || !chunk_ok(C))
        return chunk_fwd_impl(q, k, v, alpha, theta, beta, S0, o, S_T, B, H, T, m, n, C, in_dtype,
                              out_dtype, stream, slice_n);
    if (T % (static_cast<long>(G) * C) != 0) return SFDA_ERR_SHAPE;
    const long BH = static_cast<long>(B) * H;
    if (BH * G > 0x7FFFFFFFL) return SFDA_ERR_SHAPE;
    if (noalloc) {
        if (sfda_chunk_fwd_segmented_workspace_bytes(B, H, T, m, n, G, in_dtype) > SFDA_NOALLOC_SCRATCH_BYTES)
            return SFDA_ERR_SCRATCH;
        const sfda_status_t st0 = chunk_fwd_impl(q, k, v, alpha, theta, beta, S0, o, S_T, B, H, T,
                                                 m, n, C, in_dtype, out_dtype, stream, slice_n,
                                                 nullptr, 0, /*check_only=*/true);
        if (st0 != SFDA_OK) return st0;
        const sfda_status_t st1 = scratch_address(&workspace);
        if (st1 != SFDA_OK) return st1;
        workspace_bytes = SFDA_NOALLOC_SCRATCH_BYTES;
    }
    if (!workspace) return SFDA_ERR_NULL;
    if (!aligned16(workspace)) return SFDA_ERR_ALIGN;
    const size_t need = sfda_chunk_fwd_segmented_workspace_bytes(B, H, T, m, n, G, in_dtype);
    if (workspace_bytes < need) return SFDA_ERR_SHAPE;
    // validate the buffers the way sfda_chunk_fwd does (nothing is launched on error)
    {
        const sfda_status_t st0 = chunk_fwd_impl(q, k, v, alpha, theta, beta, S0, o, S_T, B, H, T,
                                                 m, n, C, in_dtype, out_dtype, stream, slice_n,
                                                 nullptr, 0, /*check_only=*/true);
        if (st0 != SFDA_OK) return st0;
    }
    const long ei = esize(in_dtype), eo = esize(out_dtype), BHT = BH * T;
    const Range rw = range_of(workspace, static_cast<long>(need));
    const Range all[] = {range_of(q, BHT * m * 2 * ei), range_of(k, BHT * m * 2 * ei),
                         range_of(v, BHT * n * 2 * ei), range_of(alpha, BHT * m * ei),
                         range_of(theta, BHT * m * ei), range_of(beta, BHT * ei),
                         range_of(o, BHT * n * 2 * eo), range_of(S0, BH * m * n * 2 * 4),
                         range_of(S_T, BH * m * n * 2 * 4)};
    for (const Range& r : all)
        if (overlap(rw, r)) return SFDA_ERR_ALIAS;

    const hipStream_t st = static_cast<hipStream_t>(stream);
    sfda::ChunkLaunch L;
    L.q = q; L.k = k; L.alpha = alpha; L.theta = theta; L.beta = beta;
    L.m = m; L.C = C;
    L.in_bf16 = in_dtype == SFDA_BF16;
    L.out_bf16 = out_dtype == SFDA_BF16;
    if (in_dtype == SFDA_F32) {
        // the workspace holds the operand records of a piece of the sequence: where that is the
        // faster one, the factored forward, which needs no segments
        const long cus = device_cus() > 0 ? device_cus() : 256;
        const sfda::FactoredPlan p = sfda::factored_plan(BH, T, m, n, false, false, need, cus);
        const bool fits = factored_fits(BH, m, n, false) && p.piece > 0;
        if (G == 1 || (fits && prepared_us(T, p) <= segments_us(BH, T, m, n, G, L.out_bf16, cus))) {
            L.v = v; L.B = B; L.H = H; L.T = T; L.n = n; L.S0 = S0; L.S_T = S_T; L.o = o;
            L.slice = auto_slice(BH, n);
            const hipError_t e = fits ? sfda::launch_factored(L, workspace, need, device_cus(), st) : sfda::launch_chunk(L, st);
            return e == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
        }
    }
    const long segs = BH * G;
    float* P = static_cast<float*>(workspace);                      // [segs][m][m]
    float* Bs = P + segs * m * m * 2;                               // [segs][m][n]
    float* Sin = Bs + segs * static_cast<long>(m) * n * 2;          // [segs][m][n]
    float* X = Sin + segs * static_cast<long>(m) * n * 2;           // [segs][T / G][m], float32 inputs
    // [B, H, T, .] with T = G * Ts is [B*H*G, Ts, .]: each segment runs as a head
    const int Ts = T / G;
    // float32 inputs and outputs: the outputs come from the zero-state pass and a join
    // (o0 + S_in^* X), cheaper than a third pass of the latency-bound float32 scan; bfloat16
    // inputs: a third pass of the pipelined kernel from the incoming states (cheaper than
    // writing X in float32 and the join); a bfloat16 o of float32 inputs: a third pass too
    // (the join would round it twice)
    const bool join = in_dtype == SFDA_F32 && !L.out_bf16;
    L.B = static_cast<int>(segs); L.H = 1; L.T = Ts;
    if (in_dtype == SFDA_F32 && n <= 64) {
        // P_g and B_g in one scan per segment (one copy of the chunk factors): the transfer
        // columns from I_m with X_t = P_t^* q_t, the value columns from zero with o0 into o
        L.v = v; L.S0 = nullptr; L.S_T = Bs; L.o = join ? o : nullptr;
        L.n = n; L.slice = slice_n; L.xo = join ? X : nullptr; L.pend = P;
        if (sfda::launch_chunk_segment(L, st) != hipSuccess) return SFDA_ERR_HIP;
    } else {
        // P_g (and with the join X_t = P_t^* q_t, the m-column float32 output): S0 = I,
        // v = 0, in place on the identity
        if (sfda::launch_identity(P, segs, m, st) != hipSuccess) return SFDA_ERR_HIP;
        L.v = nullptr; L.S0 = P; L.S_T = P; L.o = join ? X : nullptr; L.out_bf16 = false;
        L.n = m; L.slice = ((m + 7) / 8) * 8;
        if (sfda::launch_chunk(L, st) != hipSuccess) return SFDA_ERR_HIP;
        // B_g (and with the join the zero-state outputs o0, into o)
        L.v = v; L.S0 = nullptr; L.S_T = Bs; L.o = join ? o : nullptr; L.out_bf16 = out_dtype == SFDA_BF16;
        L.n = n; L.slice = slice_n;
        if (sfda::launch_chunk(L, st) != hipSuccess) return SFDA_ERR_HIP;
    }
    // incoming states and S_T
    if (sfda::launch_fold(P, Bs, Sin, S0, S_T, BH, G, m, n, st) != hipSuccess) return SFDA_ERR_HIP;
    if (join) {
        // o = o0 + S_in^* X (the affine law of each segment, token by token)
        return sfda::launch_join(X, Sin, static_cast<float*>(o), segs, Ts, m, n, st) == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
    }
    // outputs from the exact incoming states
    L.S0 = Sin; L.S_T = nullptr; L.o = o;
    return sfda::launch_chunk(L, st) == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
}

sfda_status_t sfda_chunk_fwd_segmented(const void* q, const void* k, const void* v,
                                       const void* alpha, const void* theta, const void* beta,
                                       const float* S0, void* o, float* S_T, int B, int H, int T,
                                       int m, int n, int C, int G, sfda_dtype_t in_dtype,
                                       sfda_dtype_t out_dtype, void* workspace,
                                       size_t workspace_bytes, sfda_stream_t stream)
{
    return segmented_impl(q, k, v, alpha, theta, beta, S0, o, S_T, B, H, T, m, n, C, G, in_dtype,
                          out_dtype, workspace, workspace_bytes, stream, false);
}

sfda_status_t sfda_chunk_fwd_segmented_noalloc(const void* q, const void* k, const void* v,
                                               const void* alpha, const void* theta,
                                               const void* beta, const float* S0, void* o,
                                               float* S_T, int B, int H, int T, int m, int n,
                                               int C, int G, sfda_dtype_t in_dtype,
                                               sfda_dtype_t out_dtype, sfda_stream_t stream)
{
    return segmented_impl(q, k, v, alpha, theta, beta, S0, o, S_T, B, H, T, m, n, C, G, in_dtype,
                          out_dtype, nullptr, 0, stream, true);
}

// The backward runs 16-token chunks whatever C is (the gradients do not depend on the
// chunk length, to rounding): 1 / g of a 16-token chunk stays finite while the chunk's
// decay is at least 2^-126, the forward's range, and measured on MI355X it is as fast as
// 32-token chunks (the scans' steps are shorter, the gradient pass has twice the
// workgroups).
static int bwd_chunk(int) { return 16; }

size_t sfda_chunk_bwd_workspace_bytes(int B, int H, int T, int m, int n, int C)
{
    if (B <= 0 || H <= 0 || T < 0 || m < 1 || m > 64 || n < 1) return 0;
    if (!chunk_ok(C)) return 0;
    C = bwd_chunk(C);
    const size_t chunks = static_cast<size_t>(B) * H * ((static_cast<size_t>(T) + C - 1) / C);
    // per chunk: S entering and dL/dS leaving (m x n each), Delta and G_F (C x n each)
    return chunks * (2 * static_cast<size_t>(m) * n + 2 * static_cast<size_t>(C) * n) * 8;
}

// the workspace of the backward on prepared operands, 0 where the call never takes it
static size_t bwd_factored_need(int B, int H, int T, int m, int n, int C, sfda_dtype_t in_dtype)
{
    const size_t need = sfda_chunk_bwd_workspace_bytes(B, H, T, m, n, C);
    const long BH = static_cast<long>(B) * H;
    if (need == 0 || !dtype_ok(in_dtype) || !sfda::bwd_factored_fits(BH, T, n) ||
        !bwd_factored_faster(BH, T, m, n, in_dtype == SFDA_BF16))
        return 0;
    // (with few value columns the operand records are many times the states: m 64 in float32, 1.6
    // times the smaller workspace at n 64, 6.7 times at n 8, 53 times at n 1)
    const size_t bytes = sfda::bwd_factored_bytes(BH, T, m, n, in_dtype == SFDA_BF16);
    return bytes <= std::max(2 * need, need + BWD_EXTRA) ? std::max(need, bytes) : 0;
}

size_t sfda_chunk_bwd_auto_workspace_bytes(int B, int H, int T, int m, int n, int C, sfda_dtype_t in_dtype)
{
    const size_t factored = bwd_factored_need(B, H, T, m, n, C, in_dtype);
    return factored ? factored : sfda_chunk_bwd_workspace_bytes(B, H, T, m, n, C);
}

sfda_status_t sfda_chunk_bwd(const void* q, const void* k, const void* v, const void* alpha,
                             const void* theta, const void* beta, const float* S0,
                             const void* dO, const float* dS_T, void* dq, void* dk, void* dv,
                             void* dalpha, void* dtheta, void* dbeta, float* dS0, int B, int H,
                             int T, int m, int n, int C, sfda_dtype_t in_dtype,
                             sfda_dtype_t out_dtype, void* workspace, size_t workspace_bytes,
                             sfda_stream_t stream)
{
    if (!dtype_ok(in_dtype) || !dtype_ok(out_dtype)) return SFDA_ERR_DTYPE;
    if (B < 0 || H < 0 || T < 0 || m < 1 || m > 64 || n < 1 || !state_fits(m, n)) return SFDA_ERR_SHAPE;
    if (!chunk_ok(C)) return SFDA_ERR_CHUNK;
    if (!chunk_rows_fit(n)) return SFDA_ERR_SHAPE;
    const size_t need = sfda_chunk_bwd_workspace_bytes(B, H, T, m, n, C);
    const int requested_C = C;
    C = bwd_chunk(C);
    const long BH = static_cast<long>(B) * H;
    const int slice = n <= 64 ? ((n + 7) / 8) * 8 : 64;
    const long nchunks = (static_cast<long>(T) + C - 1) / C;
    if (BH * ((n + slice - 1) / slice) > 0x7FFFFFFFL || BH * nchunks > 0x7FFFFFFFL) return SFDA_ERR_SHAPE;
    if (BH == 0) return SFDA_OK;
    const bool need_inputs = T > 0;
    if (need_inputs && (!q || !k || !v || !alpha || !theta || !beta || !dO || !dq || !dk || !dv ||
                        !dalpha || !dtheta || !dbeta))
        return SFDA_ERR_NULL;
    if (need > 0 && !workspace) return SFDA_ERR_NULL;
    const void* ptrs[] = {q, k, v, alpha, theta, beta, S0, dO, dS_T, dq, dk, dv, dalpha, dtheta,
                          dbeta, dS0, workspace};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return SFDA_ERR_ALIGN;
    if (workspace_bytes < need) return SFDA_ERR_SHAPE;

    const long ei = esize(in_dtype), eo = esize(out_dtype), BHT = BH * T;
    const Range ins[] = {range_of(q, BHT * m * 2 * ei), range_of(k, BHT * m * 2 * ei),
                         range_of(v, BHT * n * 2 * ei), range_of(alpha, BHT * m * ei),
                         range_of(theta, BHT * m * ei), range_of(beta, BHT * ei),
                         range_of(S0, BH * m * n * 2 * 4), range_of(dO, BHT * n * 2 * eo),
                         range_of(dS_T, BH * m * n * 2 * 4)};
    const Range outs[] = {range_of(dq, BHT * m * 2 * ei), range_of(dk, BHT * m * 2 * ei),
                          range_of(dv, BHT * n * 2 * ei), range_of(dalpha, BHT * m * ei),
                          range_of(dtheta, BHT * m * ei), range_of(dbeta, BHT * ei),
                          range_of(dS0, BH * m * n * 2 * 4),
                          range_of(workspace, static_cast<long>(need))};
    for (int a = 0; a < 8; ++a) {
        for (const Range& r : ins)
            if (overlap(outs[a], r)) return SFDA_ERR_ALIAS;
        for (int b = a + 1; b < 8; ++b)
            if (overlap(outs[a], outs[b])) return SFDA_ERR_ALIAS;
    }
    // the factored scans, where the workspace has room for the operand records (a caller's
    // tensors past the needed bytes, inside workspace_bytes, are none of its own: scans in place)
    const size_t facs = bwd_factored_need(B, H, T, m, n, requested_C, in_dtype);
    bool factored = facs > 0 && workspace_bytes >= facs;
    const Range whole = range_of(workspace, static_cast<long>(facs));
    if (factored) {
        for (const Range& r : ins) factored = factored && !overlap(whole, r);
        for (int a = 0; a < 7; ++a) factored = factored && !overlap(whole, outs[a]);
    }

    const hipStream_t st = static_cast<hipStream_t>(stream);
    float* S_rec = static_cast<float*>(workspace);
    float* G_rec = S_rec + BH * nchunks * m * n * 2;
    float* D_rows = G_rec + BH * nchunks * m * n * 2;
    float* F_rows = D_rows + BH * nchunks * C * n * 2;
    sfda::ChunkLaunch L;
    L.q = q; L.k = k; L.v = v; L.alpha = alpha; L.theta = theta; L.beta = beta;
    L.B = B; L.H = H; L.T = T; L.m = m; L.n = n; L.C = C; L.slice = slice;
    L.in_bf16 = in_dtype == SFDA_BF16;
    L.out_bf16 = out_dtype == SFDA_BF16;
    L.o = nullptr;
    // forward scan (the state entering every chunk and Delta) and reverse scan (dL/dS leaving
    // every chunk, G_F, dv and dS0; with T == 0 only dS0 = dS_T), in one launch
    sfda::ChunkLaunch F = L;
    F.S0 = S0; F.S_T = nullptr; F.ck_state = S_rec; F.ck_rows = D_rows;
    L.S0 = dS_T; L.S_T = dS0; L.ck_state = G_rec; L.ck_rows = F_rows; L.dO = dO; L.dv = dv;
    sfda::GradLaunch Gl;
    Gl.q = q; Gl.k = k; Gl.v = v; Gl.alpha = alpha; Gl.theta = theta; Gl.beta = beta; Gl.dO = dO;
    Gl.S_rec = S_rec; Gl.G_rec = G_rec; Gl.D_rows = D_rows; Gl.F_rows = F_rows;
    Gl.dq = dq; Gl.dk = dk; Gl.dalpha = dalpha; Gl.dtheta = dtheta; Gl.dbeta = dbeta;
    Gl.B = B; Gl.H = H; Gl.T = T; Gl.m = m; Gl.n = n; Gl.C = C;
    Gl.in_bf16 = L.in_bf16; Gl.out_bf16 = L.out_bf16;
    if (factored) return sfda::launch_bwd_factored(F, L, Gl, workspace, st) == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
    if (sfda::launch_bwd_scans(F, L, st) != hipSuccess) return SFDA_ERR_HIP;
    if (!need_inputs) return SFDA_OK;
    return sfda::launch_chunk_grad(Gl, st) == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
}

sfda_status_t sfda_chunk_solve_monitor(const void* k, const void* alpha, const void* theta,
                                       const void* beta, float* residual, float* lnorm, int B,
                                       int H, int T, int m, sfda_dtype_t in_dtype,
                                       sfda_stream_t stream)
{
    if (!dtype_ok(in_dtype)) return SFDA_ERR_DTYPE;
    if (B < 0 || H < 0 || T < 0 || m < 1 || m > 64) return SFDA_ERR_SHAPE;
    const long BH = static_cast<long>(B) * H, nb = (static_cast<long>(T) + 15) / 16;
    if (BH * nb > 0x7FFFFFFFL) return SFDA_ERR_SHAPE;
    if (BH == 0 || T == 0) return SFDA_OK;
    if (!k || !alpha || !theta || !beta || (!residual && !lnorm)) return SFDA_ERR_NULL;
    const void* ptrs[] = {k, alpha, theta, beta, residual, lnorm};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return SFDA_ERR_ALIGN;
    const long ei = esize(in_dtype), BHT = BH * T;
    const Range ins[] = {range_of(k, BHT * m * 2 * ei), range_of(alpha, BHT * m * ei),
                         range_of(theta, BHT * m * ei), range_of(beta, BHT * ei)};
    const Range outs[] = {range_of(residual, BH * nb * 4), range_of(lnorm, BH * nb * 4)};
    for (const Range& o : outs)
        for (const Range& r : ins)
            if (overlap(o, r)) return SFDA_ERR_ALIAS;
    if (overlap(outs[0], outs[1])) return SFDA_ERR_ALIAS;
    sfda::ChunkLaunch L;
    L.q = k; L.k = k; L.v = nullptr; L.alpha = alpha; L.theta = theta; L.beta = beta;
    L.S0 = nullptr; L.o = nullptr; L.S_T = nullptr;
    L.B = B; L.H = H; L.T = T; L.m = m; L.n = 8; L.C = 16; L.slice = 8;
    L.in_bf16 = in_dtype == SFDA_BF16;
    L.out_bf16 = false;
    if (sfda::launch_solve_monitor(L, residual, lnorm, static_cast<hipStream_t>(stream)) != hipSuccess)
        return SFDA_ERR_HIP;
    return SFDA_OK;
}

sfda_status_t sfda_step(const void* q, const void* k, const void* v, const void* alpha,
                        const void* theta, const void* beta, float* S, void* o, int B, int H,
                        int m, int n, sfda_dtype_t in_dtype, sfda_dtype_t out_dtype,
                        sfda_stream_t stream)
{
    if (!dtype_ok(in_dtype) || !dtype_ok(out_dtype)) return SFDA_ERR_DTYPE;
    if (B < 0 || H < 0 || m < 1 || m > 64 || n < 1 || !state_fits(m, n)) return SFDA_ERR_SHAPE;
    if (n >= (1 << 22)) return SFDA_ERR_SHAPE;   // state rows addressed with 32-bit offsets
    const long BH = static_cast<long>(B) * H;
    int np = 1;
    while (np < n && np < 64) np <<= 1;
    if (BH * ((n + np - 1) / np) > 0x7FFFFFFFL) return SFDA_ERR_SHAPE;
    if (BH == 0) return SFDA_OK;
    if (!q || !k || !v || !alpha || !theta || !beta || !S || !o) return SFDA_ERR_NULL;
    const void* ptrs[] = {q, k, v, alpha, theta, beta, S, o};
    for (const void* p : ptrs)
        if (!aligned16(p)) return SFDA_ERR_ALIGN;
    const long ei = esize(in_dtype), eo = esize(out_dtype);
    const Range ins[] = {range_of(q, BH * m * 2 * ei), range_of(k, BH * m * 2 * ei),
                         range_of(v, BH * n * 2 * ei), range_of(alpha, BH * m * ei),
                         range_of(theta, BH * m * ei), range_of(beta, BH * ei)};
    const Range rs = range_of(S, BH * m * n * 2 * 4);
    const Range ro = range_of(o, BH * n * 2 * eo);
    if (overlap(ro, rs)) return SFDA_ERR_ALIAS;
    for (const Range& r : ins)
        if (overlap(ro, r) || overlap(rs, r)) return SFDA_ERR_ALIAS;

    sfda::StepLaunch L;
    L.q = q; L.k = k; L.v = v; L.alpha = alpha; L.theta = theta; L.beta = beta;
    L.S = S; L.o = o; L.B = B; L.H = H; L.m = m; L.n = n;
    L.in_bf16 = in_dtype == SFDA_BF16;
    L.out_bf16 = out_dtype == SFDA_BF16;
    const hipError_t e = sfda::launch_step(L, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? SFDA_OK : SFDA_ERR_HIP;
}

}  // extern "C"
