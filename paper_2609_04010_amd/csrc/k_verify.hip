// Speculative verification of drafted blocks (Alg. 1, linear sampler).
//
// For sequence s the target logits p_1..p_B and the draft logits q_1..q_{B-1} are rows of two
// [rows][ld] matrices, the drafted tokens x_1..x_{B-1} a [S][B-1] array.  With acceptance uniforms
// u_i (word (STREAM_VERIFY, step, row0 + s, i)):
//   n = first i with u_i > min(1, p_i(x_i) / q_i(x_i)), else B
//   z ~ Norm([p_n - q_n]_+) if n < B, else z ~ p_B     (p_n itself if the residual has no mass)
// Rows whose logits give no valid draw (NaN, +inf, no finite logit) set DD_DEVERR_LOGITS and
// emit z = 0.
// z is drawn with the two-level Gumbel-max of the posterior kernel (groups of DD_GUMBEL_GROUP
// classes, no mask group): the draw is invariant to the normaliser, so group masses and class
// scores use the unnormalised residual.
//
// Kernel 1 (one workgroup per position of a sequence, rows p_i and q_i, or per row): row log-sum-exps
// in fp32.
// Kernel 2 (one workgroup per sequence): n from the B - 1 acceptance tests, then one pass over the
// chosen row pair for the group masses and the two-level draw.
//
// Only the rows up to the first rejection matter.  With many sequences kernel 1 therefore also makes
// its position's acceptance test and lowers n_out[s] to a rejected position; workgroups are dispatched
// position by position, and one that starts after an earlier position of its sequence was rejected
// leaves at once.  That is a hint only: kernel 2 makes the tests again from the log-sum-exps (those of
// positions below n are always there), so a hint that arrives late costs time and nothing else.
#include <math.h>

#include <mutex>
#include <type_traits>

#include "elem.h"
#include "kernels.h"
#include "rng.h"

namespace dd {

namespace {

// Threads per workgroup of kernel 1 and of kernel 2; 256 in both on short rows (SHORT_CHUNKS chunks of
// 16 bytes), where more only idle: S 250, B 3, V 5000 15.8 against 20.5 us, S 200, B 16, V 2000 27.6
// against 30.6; S 3, B 16, V 20000 20.9 against 16.1 the other way.
constexpr int VT_LONG = 512, VT2_LONG = 1024, VT_SHORT = 256, SHORT_CHUNKS = 2048;

DD_DEV uint32_t verify_word(const VerifyArgs& a, int s, uint32_t stream, int idx, int explicit_off) {
    if (a.noise) return a.noise[(int64_t)s * a.nu + explicit_off + idx];
    return counter_word(a.seed, stream, a.step, a.row0 + (uint32_t)s, (uint32_t)idx);
}

DD_DEV float word_uniform_f(uint32_t w) { return ((float)w + 0.5f) * 0x1p-32f; }

// Draft position i of sequence s is rejected: u_i > min(1, p_i(x_i) / q_i(x_i)), from the rows and
// their log-sum-exps.  An id outside [0, V) is clamped (kernel 2 reports those it needed).
template <typename T>
DD_DEV bool rejected(const VerifyArgs& a, int s, int i, float lse_p, float lse_q) {
    const int x = min(max(a.draft[(int64_t)s * (a.B - 1) + i], 0), a.V - 1);
    const char* pr = (const char*)a.p + ((size_t)s * a.B + i) * a.ld * sizeof(T);
    const char* qr = (const char*)a.q + ((size_t)s * (a.B - 1) + i) * a.ld * sizeof(T);
    const float lp = Elem<T>::load1(pr, x) - lse_p, lq = Elem<T>::load1(qr, x) - lse_q;
    const float ratio = fminf(1.f, __builtin_amdgcn_exp2f((lp - lq) * LOG2E));
    return word_uniform_f(verify_word(a, s, STREAM_VERIFY, i, 0)) > ratio;
}

// One pass over the rows: each thread keeps a running maximum m and the sum of exp(l - m), rescaled
// when m rises; the workgroup then combines the (m, sum) pairs.  The result is that of the two-pass
// definition: NaN if a logit is NaN, else +inf if one is +inf, else -inf if none is finite.
// The hot loop spends four full-rate operations and one exp2 per logit: a thread takes VU chunks of
// both rows at a time (loaded together, the next VU loaded while these are reduced), takes a row's
// maximum with fmax (which passes over NaN), rescales its sum when the maximum rises, and adds
// exp2(l log2 e - m log2 e).  A NaN or +inf logit makes that sum NaN (exp2 of NaN, or of inf - inf),
// so such rows are told apart afterwards by a second scan that only they take.  Bound by HBM; S 256,
// B 16, V 50257 with 4.8 positions kept on average: 131 us over every row, 81 us with the hint (two
// chunks per row in flight; with four the kernel needs 148 registers, one workgroup per CU, 115 us).
template <typename T, int VT, int VU>
__global__ __launch_bounds__(VT, 4) void row_lse_kernel(VerifyArgs a, float* lse, int hint) {
    __shared__ float sh_m[2][VT / 64], sh_s[2][VT / 64];
    __shared__ int sh_f[VT / 64], sh_skip;
    constexpr int E = Elem<T>::E, NW = VT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // with the hint a workgroup takes a position, position by position; without it one row (target
    // rows first)
    const int np = a.S * a.B, r0 = (int)blockIdx.x;
    const int i = hint ? r0 / a.S : 0, s = hint ? r0 - i * a.S : 0;
    const int V = a.V, nchunk = (V + E - 1) / E;
    if (hint) {
        if (tid == 0) sh_skip = __hip_atomic_load(a.n_out + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= i;
        __syncthreads();
        if (sh_skip) return;
    }
    const bool pair = hint && i < a.B - 1;
    const char* rows[2] = {hint ? (const char*)a.p + ((size_t)s * a.B + i) * a.ld * sizeof(T)
                           : r0 < np ? (const char*)a.p + (size_t)r0 * a.ld * sizeof(T)
                                     : (const char*)a.q + (size_t)(r0 - np) * a.ld * sizeof(T),
                           pair ? (const char*)a.q + ((size_t)s * (a.B - 1) + i) * a.ld * sizeof(T) : nullptr};
    float m[2] = {-INFINITY, -INFINITY}, sum[2] = {0.f, 0.f};
    constexpr int TS = VU * VT;   // chunks per tile
    // chunks c0 + u VT + tid, u < VU; chunks past the row read as -inf, and so does the part of the
    // last chunk past V
    auto load = [&](uint4 (&x)[VU], const char* rowp, int c0) {
        if ((c0 + TS) * E <= V) {   // every element of the tile is in the row
#pragma unroll
            for (int u = 0; u < VU; ++u) x[u] = *(const uint4*)(rowp + (size_t)(c0 + u * VT + tid) * 16);
        } else {
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                const int c = c0 + u * VT + tid;
                const uint4 y = *(const uint4*)(rowp + (size_t)min(c, nchunk - 1) * 16);
                x[u] = c < nchunk ? y : Elem<T>::NEG_INF4;
            }
            if (V % E != 0) {
#pragma unroll
                for (int u = 0; u < VU; ++u)
                    if (c0 + u * VT + tid == nchunk - 1) Elem<T>::clip(x[u], V % E);
            }
        }
    };
    auto absorb = [&](const uint4 (&x)[VU], float& m, float& sum) {
        float cm = -INFINITY;
#pragma unroll
        for (int u = 0; u < VU; ++u)
#pragma unroll
            for (int e = 0; e < E; ++e) cm = fmaxf(cm, Elem<T>::get(x[u], e));
        if (cm > m) {
            sum *= __builtin_amdgcn_exp2f((m - cm) * LOG2E);   // m = -inf: sum is 0 already
            m = cm;
        }
        const float moff = m == -INFINITY ? 0.f : -m * LOG2E;
#pragma unroll
        for (int u = 0; u < VU; ++u)
#pragma unroll
            for (int e = 0; e < E; ++e) sum += __builtin_amdgcn_exp2f(fmaf(Elem<T>::get(x[u], e), LOG2E, moff));
    };
    auto scan = [&](auto pair_c) {
        constexpr int R = decltype(pair_c)::value ? 2 : 1;
        uint4 xa[R][VU], xb[R][VU];
#pragma unroll
        for (int r = 0; r < R; ++r) load(xa[r], rows[r], 0);
        for (int c0 = 0; c0 < nchunk; c0 += 2 * TS) {
            const bool more = c0 + TS < nchunk;
            if (more) {
#pragma unroll
                for (int r = 0; r < R; ++r) load(xb[r], rows[r], c0 + TS);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) absorb(xa[r], m[r], sum[r]);
            if (!more) break;
            if (c0 + 2 * TS < nchunk) {
#pragma unroll
                for (int r = 0; r < R; ++r) load(xa[r], rows[r], c0 + 2 * TS);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) absorb(xb[r], m[r], sum[r]);
        }
    };
    if (pair) scan(std::true_type{});
    else scan(std::false_type{});
    // workgroup: maximum, then the sums rescaled to it
    float M[2], Mref[2], S[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (r == 1 && !pair) break;
        M[r] = wave_max(m[r]);
        if (lane == 0) sh_m[r][wave] = M[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (r == 1 && !pair) break;
        M[r] = sh_m[r][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) M[r] = fmaxf(M[r], sh_m[r][w]);
        Mref[r] = M[r] == -INFINITY ? 0.f : M[r];
        // a thread that met no finite logit has sum 0, or NaN if it met a NaN: kept as it is
        const float part = wave_sum(m[r] == -INFINITY ? sum[r] : sum[r] * __builtin_amdgcn_exp2f((m[r] - Mref[r]) * LOG2E));
        if (lane == 0) sh_s[r][wave] = part;
    }
    __syncthreads();
    float out[2] = {0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (r == 1 && !pair) break;
        S[r] = sh_s[r][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) S[r] += sh_s[r][w];
        out[r] = Mref[r] + logf(S[r]);
        if (!(S[r] == S[r]) || M[r] == INFINITY) {
            // a NaN or +inf logit (the sum is NaN): NaN if any logit is NaN, else +inf
            int fl = 0;
            for (int c = tid; c < nchunk; c += VT) {
                uint4 x = *(const uint4*)(rows[r] + (size_t)c * 16);
                if (V % E != 0 && c == nchunk - 1) Elem<T>::clip(x, V % E);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const float t = Elem<T>::get(x, e);
                    fl |= (t != t) ? 1 : (t == INFINITY ? 2 : 0);
                }
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) fl |= __shfl_xor(fl, o, 64);
            __syncthreads();          // the other row's flags have been read
            if (lane == 0) sh_f[wave] = fl;
            __syncthreads();
            fl = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) fl |= sh_f[w];
            out[r] = (fl & 1) ? __int_as_float(0x7FC00000) : INFINITY;
        }
    }
    if (tid == 0) {
        lse[hint ? (size_t)s * a.B + i : (size_t)r0] = out[0];
        if (pair) {
            lse[np + (size_t)s * (a.B - 1) + i] = out[1];
            if (rejected<T>(a, s, i, out[0], out[1])) atomicMin(a.n_out + s, i + 1);
        }
    }
}

// n_out[s] = B: the hint of kernel 1 starts without a rejection
__global__ void verify_start_kernel(int32_t* n_out, int S, int B) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s < S) n_out[s] = B;
}

// The pass over the row pair is one CU's work per sequence, so what bounds it is how much that CU has
// in flight: 1024 threads, VU chunks of both rows each.  The tests of the drafted positions run one
// per lane, and the draw takes one Philox block per four words (S 4, B 16, V 50257: 32.7 us with 256
// threads, one chunk each, the tests one after the other by one thread and a block per word).
template <typename T, int VT2, int VU>
__global__ __launch_bounds__(VT2) void verify_kernel(VerifyArgs a, const float* lse) {
    extern __shared__ float s_mass[];   // one mass per group
    __shared__ int sh_n;
    __shared__ float sh_tot[VT2 / 64];
    constexpr int E = Elem<T>::E, NW = VT2 / 64;
    constexpr int LPG = DD_GUMBEL_GROUP / E;   // chunks (lanes) per group
    const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int B = a.B, V = a.V;
    const int ngroups = (V + DD_GUMBEL_GROUP - 1) / DD_GUMBEL_GROUP;
    const float* lse_p = lse + (size_t)s * B;
    const float* lse_q = lse + (size_t)a.S * B + (size_t)s * (B - 1);

    // ---- acceptance: the first rejected draft position (1-based), or B ----
    if (tid < 64) {
        int n = B;
        for (int i0 = 0; i0 < B - 1; i0 += 64) {
            const int i = i0 + lane;
            const bool in = i < B - 1;
            const uint64_t rej = __ballot(in && rejected<T>(a, s, in ? i : 0, in ? lse_p[i] : 0.f, in ? lse_q[i] : 0.f));
            const int first = rej ? (int)__builtin_ctzll(rej) : 64;
            if (in && lane <= first && a.err) {   // the tests up to the first rejection count
                const int x = a.draft[(int64_t)s * (B - 1) + i];
                if (x < 0 || x >= V) atomicOr(a.err, DD_DEVERR_TOKEN);
            }
            if (rej) {
                n = i0 + first + 1;
                break;
            }
        }
        if (lane == 0) sh_n = n;
    }
    __syncthreads();
    const int n = sh_n;
    const bool resid = n < B;
    const char* pr = (const char*)a.p + ((size_t)s * B + n - 1) * a.ld * sizeof(T);
    const char* qr = resid ? (const char*)a.q + ((size_t)s * (B - 1) + n - 1) * a.ld * sizeof(T) : nullptr;
    const float lp0 = lse_p[n - 1], lq0 = resid ? lse_q[n - 1] : 0.f;

    // unnormalised class mass: [p - q]_+ for a rejection, p for the bonus (use_p: residual empty)
    auto cls_mass = [&](float lpv, float lqv, bool use_p) -> float {
        const float ep = __builtin_amdgcn_exp2f((lpv - lp0) * LOG2E);
        if (!resid || use_p) return ep;
        return fmaxf(ep - __builtin_amdgcn_exp2f((lqv - lq0) * LOG2E), 0.f);
    };

    // ---- group masses: lanes of a group hold consecutive chunks; reduce over LPG lanes ----
    const int nchunk = (V + E - 1) / E;
    auto masses = [&](bool use_p) -> float {
        float tot = 0.f;
        for (int c0 = 0; c0 < nchunk; c0 += VU * VT2) {
            uint4 xp[VU], xq[VU];
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                const int c = min(c0 + u * VT2 + tid, nchunk - 1);
                xp[u] = *(const uint4*)(pr + (size_t)c * 16);
                if (resid && !use_p) xq[u] = *(const uint4*)(qr + (size_t)c * 16);
                else xq[u] = Elem<T>::NEG_INF4;
            }
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                const int c = c0 + u * VT2 + tid;
                float sum = 0.f;
                if (c < nchunk) {
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        if (c * E + e < V) sum += cls_mass(Elem<T>::get(xp[u], e), Elem<T>::get(xq[u], e), use_p);
                }
#pragma unroll
                for (int o = 1; o < LPG; o <<= 1) sum += __shfl_xor(sum, o, 64);
                if ((lane & (LPG - 1)) == 0 && c < nchunk) {
                    s_mass[c / LPG] = sum;
                    tot += sum;
                }
            }
        }
        tot = wave_sum(tot);
        if (lane == 0) sh_tot[tid >> 6] = tot;
        __syncthreads();
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += sh_tot[w];
        __syncthreads();
        return t;
    };
    bool use_p = false;
    if (!(masses(false) > 0.f)) {   // empty residual: draw from p_n
        use_p = true;
        masses(true);
    }

    // ---- two-level draw (one wavefront): four consecutive words per lane and Philox block ----
    if (tid >= 64) return;
    const int ntop = ngroups;
    auto words = [&](uint32_t stream, int base, int count, int explicit_off, uint32_t (&wd)[4]) {
        if (a.noise) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                wd[k] = base + k < count ? a.noise[(int64_t)s * a.nu + explicit_off + base + k] : 0u;
        } else {
            const Words4 W = philox4x32_10((uint32_t)(base >> 2), a.row0 + (uint32_t)s, a.step, stream,
                                           (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
#pragma unroll
            for (int k = 0; k < 4; ++k) wd[k] = W.w[k];
        }
    };
    auto argmax = [&](float best, int bi) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float s2 = __shfl_xor(best, o, 64);
            const int i2 = __shfl_xor(bi, o, 64);
            const bool take = s2 > best || (s2 == best && i2 < bi);
            best = take ? s2 : best;
            bi = take ? i2 : bi;
        }
        return bi;
    };
    float best = -INFINITY;
    int bi = 0x7FFFFFFF;
    for (int g0 = 4 * lane; g0 < ngroups; g0 += 256) {
        uint32_t wd[4];
        words(STREAM_TOP, g0, ngroups, B - 1, wd);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (g0 + k >= ngroups) continue;
            const float sc = logf(s_mass[g0 + k]) + word_gumbel_f(wd[k]);
            const bool take = sc > best || (sc == best && g0 + k < bi);
            best = take ? sc : best;
            bi = take ? g0 + k : bi;
        }
    }
    const int gstar = argmax(best, bi);
    // no group with a valid score (NaN or +inf logits): report, emit token 0, index nothing
    const bool bad = gstar >= ngroups || !isfinite(lp0) || (resid && !use_p && !isfinite(lq0));
    best = -INFINITY;
    bi = 0x7FFFFFFF;
    const int j0 = bad ? V : gstar * DD_GUMBEL_GROUP + 4 * lane;
    if (j0 < V) {
        uint32_t wd[4];
        words(STREAM_CLASS, j0, V, B - 1 + ntop, wd);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = j0 + k;
            if (j >= V) continue;
            const float lpv = Elem<T>::load1(pr, j);
            const float lqv = (resid && !use_p) ? Elem<T>::load1(qr, j) : 0.f;
            const float sc = logf(cls_mass(lpv, lqv, use_p)) + word_gumbel_f(wd[k]);
            const bool take = sc > best || (sc == best && j < bi);
            best = take ? sc : best;
            bi = take ? j : bi;
        }
    }
    bi = argmax(best, bi);
    const bool bad_z = bad || bi >= V;
    if (lane == 0) {
        if (bad_z && a.err) atomicOr(a.err, DD_DEVERR_LOGITS);
        a.n_out[s] = n;
        a.z_out[s] = bad_z ? 0 : bi;
    }
}

}  // namespace

// Row log-sum-exps of dd_spec_verify_noalloc: a file-scope device array instead of a caller
// workspace, one copy per device, held until the process ends.  In host code `scratch` names a
// host-side stand-in, not device memory: the host takes each device's address from
// hipGetSymbolAddress (once per device, with that device current) and passes that address on.
static __device__ __align__(256) float scratch[DD_SPEC_VERIFY_NOALLOC_ROWS];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static float* g_scratch_dev[kMaxDevices] = {};

dd_status verify_noalloc_scratch(float** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_error("spec_verify_noalloc: hipGetDevice: %s", hipGetErrorString(e));
        return DD_E_HIP;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        set_error("spec_verify_noalloc: device %d beyond the %d this library tracks", dev, kMaxDevices);
        return DD_E_UNSUPPORTED;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_error("spec_verify_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
            return DD_E_HIP;
        }
        g_scratch_dev[dev] = (float*)p;
    }
    *out = g_scratch_dev[dev];
    return DD_OK;
}

dd_status launch_verify(const VerifyArgs& a, int logits_dtype, float* lse, hipStream_t s) {
    if (a.S == 0) return DD_OK;
    const int ngroups = (a.V + DD_GUMBEL_GROUP - 1) / DD_GUMBEL_GROUP;
    const size_t shmem = (size_t)ngroups * sizeof(float);
    // Up to about 1024 positions everything starts at once and the hint never comes in time (and a
    // short row is no loss): its launch is left out, and a workgroup takes one row instead of two (S 4,
    // B 16: 7 against 10 us).
    const int chunk = logits_dtype == DD_BF16 ? 8 : 4;
    const bool is_short = a.V <= SHORT_CHUNKS * chunk;
    const int hint = !is_short && a.B > 2 && (int64_t)a.S * a.B > 1024;
    if (hint) launch_k(verify_start_kernel, dim3((a.S + 255) / 256), dim3(256), 0, s, a.n_out, a.S, a.B);
    const dim3 grid((unsigned)(hint ? a.S * a.B : a.S * (2 * a.B - 1)));
    auto run = [&](auto lse_k, auto draw_k, int vt, int vt2) {
        launch_k(lse_k, grid, dim3(vt), 0, s, a, lse, hint);
        launch_k(draw_k, dim3(a.S), dim3(vt2), shmem, s, a, (const float*)lse);
    };
    // chunks in flight per thread and row: two where 256 threads cover the row with that
    const bool two = a.V <= 2 * VT_SHORT * chunk;
    auto pick = [&](auto t) {
        using T = decltype(t);
        if (two) run(row_lse_kernel<T, VT_SHORT, 2>, verify_kernel<T, VT_SHORT, 2>, VT_SHORT, VT_SHORT);
        else if (is_short) run(row_lse_kernel<T, VT_SHORT, 4>, verify_kernel<T, VT_SHORT, 4>, VT_SHORT, VT_SHORT);
        else run(row_lse_kernel<T, VT_LONG, 2>, verify_kernel<T, VT2_LONG, 4>, VT_LONG, VT2_LONG);
    };
    if (logits_dtype == DD_BF16) pick(bf16_t{});
    else pick(float{});
    return launch_status("spec_verify");
}

}  // namespace dd
