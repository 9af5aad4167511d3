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

constexpr int SHORT_CHUNKS = 2048;   // 16-byte chunks of a short row

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
// HINT is a template parameter because the pair's registers (bf16: 128 instead of 80 at four chunks) cost
// the one-row form its occupancy: S 256, B 16, V 5000 24.3 -> 17.8 us without them.
template <typename T, int VT, int VU, bool HINT>
__global__ __launch_bounds__(VT, HINT ? 4 : 1) void row_lse_kernel(VerifyArgs a, float* lse) {
    constexpr int E = Elem<T>::E, NW = VT / 64, NR = HINT ? 2 : 1;   // NR: rows of a workgroup
    __shared__ float sh_m[NR][NW], sh_s[NR][NW];
    __shared__ int sh_f[NW], sh_skip;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // with the hint a workgroup takes a position, position by position; without it one row (target
    // rows first)
    const int np = a.S * a.B, r0 = (int)blockIdx.x;
    const int i = HINT ? r0 / a.S : 0, s = HINT ? r0 - i * a.S : 0;
    const int V = a.V, nchunk = (V + E - 1) / E;
    if constexpr (HINT) {
        if (tid == 0) sh_skip = __hip_atomic_load(a.n_out + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= i;
        __syncthreads();
        if (sh_skip) return;
    }
    const bool pair = HINT && i < a.B - 1;
    const char* rows[NR];
    if constexpr (HINT) {
        rows[0] = (const char*)a.p + ((size_t)s * a.B + i) * a.ld * sizeof(T);
        rows[1] = pair ? (const char*)a.q + ((size_t)s * (a.B - 1) + i) * a.ld * sizeof(T) : nullptr;
    } else {
        rows[0] = r0 < np ? (const char*)a.p + (size_t)r0 * a.ld * sizeof(T)
                          : (const char*)a.q + (size_t)(r0 - np) * a.ld * sizeof(T);
    }
    float m[NR], sum[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        m[r] = -INFINITY;
        sum[r] = 0.f;
    }
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
    if constexpr (HINT) {
        if (pair) scan(std::true_type{});
        else scan(std::false_type{});
    } else {
        scan(std::false_type{});
    }
    // workgroup: maximum, then the sums rescaled to it
    float M[NR], Mref[NR], S[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if (r == 1 && !pair) break;
        M[r] = wave_max(m[r]);
        if (lane == 0) sh_m[r][wave] = M[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) {
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
    float out[NR] = {};
#pragma unroll
    for (int r = 0; r < NR; ++r) {
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
        lse[HINT ? (size_t)s * a.B + i : (size_t)r0] = out[0];
        if constexpr (HINT) {
            if (pair) {
                lse[np + (size_t)s * (a.B - 1) + i] = out[1];
                if (rejected<T>(a, s, i, out[0], out[1])) atomicMin(a.n_out + s, i + 1);
            }
        }
    }
}

// n_out[s] = B: the hint of kernel 1 starts without a rejection
__global__ void verify_start_kernel(int32_t* n_out, int S, int B) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s < S) n_out[s] = B;
}

// The pass over the row pair is one CU's work per sequence, so what bounds it is how much that CU has
// in flight: VT2 threads (the launcher has the lines), VU chunks of both rows each.  The tests of the
// drafted positions run one per lane, and the draw takes one Philox block per four words, or where 64
// lanes cover the candidates one each, since four scores one after the other cost more than the
// blocks (V 64 7.5 -> 5.2 us).  S 4, B 16, V 50257: 32.7 -> 14.5 us against 256 threads, one chunk each,
// the tests by one thread and a block per word.
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
                if (c0 + u * VT2 >= nchunk) break;   // the same for the whole workgroup
                const int c = min(c0 + u * VT2 + tid, nchunk - 1);
                xp[u] = *(const uint4*)(pr + (size_t)c * 16);
                if (resid && !use_p) xq[u] = *(const uint4*)(qr + (size_t)c * 16);
                else xq[u] = Elem<T>::NEG_INF4;
            }
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                if (c0 + u * VT2 >= nchunk) break;
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

    // ---- two-level draw (one wavefront): one candidate per lane up to 64, beyond that four
    // consecutive words per lane and Philox block ----
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
    // score of class (or group) j with mass `mass` and word w against the best so far
    float best = -INFINITY;
    int bi = 0x7FFFFFFF;
    auto consider = [&](int j, float mass, uint32_t w, bool in) {
        const float sc = logf(mass) + word_gumbel_f(w);
        const bool take = in && (sc > best || (sc == best && j < bi));
        best = take ? sc : best;
        bi = take ? j : bi;
    };
    if (ngroups <= 64) {
        if (lane < ngroups) consider(lane, s_mass[lane], verify_word(a, s, STREAM_TOP, lane, B - 1), true);
    } else {
        for (int g0 = 4 * lane; g0 < ngroups; g0 += 256) {
            uint32_t wd[4];
            words(STREAM_TOP, g0, ngroups, B - 1, wd);
#pragma unroll
            for (int k = 0; k < 4; ++k) consider(g0 + k, s_mass[min(g0 + k, ngroups - 1)], wd[k], g0 + k < ngroups);
        }
    }
    const int gstar = argmax(best, bi);
    // no group with a valid score (NaN or +inf logits): report, emit token 0, index nothing
    const bool bad = gstar >= ngroups || !isfinite(lp0) || (resid && !use_p && !isfinite(lq0));
    best = -INFINITY;
    bi = 0x7FFFFFFF;
    if (!bad) {
        const int base = gstar * DD_GUMBEL_GROUP, n2 = min(V - base, DD_GUMBEL_GROUP);
        const bool with_q = resid && !use_p;
        if (n2 <= 64) {
            const int j = base + lane;
            if (lane < n2)
                consider(j, cls_mass(Elem<T>::load1(pr, j), with_q ? Elem<T>::load1(qr, j) : 0.f, use_p),
                         verify_word(a, s, STREAM_CLASS, j, B - 1 + ntop), true);
        } else if (4 * lane < n2) {
            const int j0 = base + 4 * lane;
            // the four classes' loads go out together (those past V read the last class and are not taken)
            float lpv[4], lqv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = min(j0 + k, V - 1);
                lpv[k] = Elem<T>::load1(pr, j);
                lqv[k] = with_q ? Elem<T>::load1(qr, j) : 0.f;
            }
            uint32_t wd[4];
            words(STREAM_CLASS, j0, V, B - 1 + ntop, wd);
#pragma unroll
            for (int k = 0; k < 4; ++k) consider(j0 + k, cls_mass(lpv[k], lqv[k], use_p), wd[k], j0 + k < V);
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
    const int chunk = logits_dtype == DD_BF16 ? 8 : 4, nchunk = (a.V + chunk - 1) / chunk;
    // Up to about 1024 positions everything starts at once and the hint never comes in time (and a
    // short row is no loss): its launch is left out, and a workgroup takes one row instead of two (S 4,
    // B 16: 7 against 10 us).
    const bool is_short = nchunk <= SHORT_CHUNKS;
    const bool hint = !is_short && a.B > 2 && (int64_t)a.S * a.B > 1024;
    if (hint) launch_k(verify_start_kernel, dim3((a.S + 255) / 256), dim3(256), 0, s, a.n_out, a.S, a.B);
    const int rows = a.S * (hint ? a.B : 2 * a.B - 1);
    auto lse_run = [&](auto kernel, int vt) { launch_k(kernel, dim3(rows), dim3(vt), 0, s, a, lse); };
    auto draw_run = [&](auto kernel, int vt) { launch_k(kernel, dim3(a.S), dim3(vt), shmem, s, a, (const float*)lse); };
    auto pick = [&](auto t) {
        using T = decltype(t);
        // Threads and chunks in flight per thread of a row, bf16 us with 256 x 2 / 256 x 4 / 512 x 2: two
        // where 256 threads then cover the row (S 1000, B 2, V 2000 6.4 / 8.3 / 10.8), four up to 2048
        // chunks (S 256, B 16, V 5000 19.2 / 17.8 / 24.4), 512 threads on longer rows (S 1, B 2, V 50257
        // 6.5 / 6.0 / 5.6; S 3000 151 / 151 / 149).  By the row's length alone: its sum does not depend on
        // how many rows the call has.
        if (hint) lse_run(row_lse_kernel<T, 512, 2, true>, 512);
        else if (nchunk <= 2 * 256) lse_run(row_lse_kernel<T, 256, 2, false>, 256);
        else if (is_short) lse_run(row_lse_kernel<T, 256, 4, false>, 256);
        else lse_run(row_lse_kernel<T, 512, 2, false>, 512);
        // Threads of a sequence's draw: as many as fit where every sequence has a CU to itself, fewer the
        // more of them share one (bf16, B 2 or 3, us with 256 / 512 / 1024 threads: V 50257 S 256 28.8 /
        // 19.0 / 15.9, S 700 32.9 / 27.5 / 34.1, S 3000 87 / 88 / 123; V 5000 10.6 / 9.7 / 9.4, 11.0 / 10.3 /
        // 14.3, 22.2 / 27.2 / 41.1); 256 where those cover the row
        if (nchunk <= 2 * 256 || a.S > 768) draw_run(verify_kernel<T, 256, 2>, 256);
        else if (a.S > 256) draw_run(verify_kernel<T, 512, 2>, 512);
        else draw_run(verify_kernel<T, 1024, 2>, 1024);
    };
    if (logits_dtype == DD_BF16) pick(bf16_t{});
    else pick(float{});
    return launch_status("spec_verify");
}

}  // namespace dd
