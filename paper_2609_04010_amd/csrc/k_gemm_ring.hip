// Dense layers on few rows, or with K not a multiple of 128: C = A W^T (+ epilogue), bf16 operands,
// the operand layouts of k_gemm.hip.
//
// The 256-row tiles of k_gemm.hip leave most CUs idle when M is small (M = 1024, N = 768: 16 tiles
// for 256 CUs), and each tile then walks its whole K loop alone.  Here the tiles are 128 x 128 to
// 64 x 64, so the same product makes 48 to 192 of them, and the residual layers (attention output,
// MLP down) also split K over workgroups: split 0 adds its part and the bias to the residual row in
// place, the others write fp32 partials into slabs of free workspace, which the normalisation that
// reads the row next adds first (in slab order, so results do not depend on timing).
//
// With so little work per CU the K loop is bound by the latency of its loads, not by the matrix
// cores: operand K-tiles of 64 go global -> LDS (global_load_lds_dwordx4, XOR-swizzled 128-byte rows
// as in k_gemm.hip) through a ring of NST stages, so NST - 1 K-tiles are in flight while one is
// computed; each K-tile waits for its own loads by count and costs one barrier.
//
// Measured (MI355X, weights of 12 layers in turn; 256-row tiles -> ring): M 1024, d 768: QKV 20.3 ->
// 11.1 us, attention output 22.5 -> 7.6, MLP up 21.0 -> 11.6, MLP down 57.6 -> 13.6; M 64: 19.7 -> 6.4,
// 19.5 -> 4.5, 19.5 -> 6.4, 53.4 -> 7.5.  What bounds it now: at M 64 the K loop, 0.21 us per K-tile
// (fragment reads, loads into LDS and four dependent MFMAs); at M 1024 the operand stream through
// L2, 16 TB/s.  Against the register-staged 128 x 128 tiles this kernel replaced for K % 128 != 0:
// M 1320, N 3072, K 832 24.0 -> 13.3 us, M 16384 143.5 -> 134.4.
//
// fp32 (the validation build) takes the same kernel with v_mfma_f32_32x32x2_f32 and the smallest of the
// 32 x 32, 32 x 64 and 64 x 64 tiles that fits the CUs once, not split over workgroups, bound by the matrix
// cores: 12 layers d 768 on 256 rows 15.3 -> 1.45 ms per forward pass against the VALU kernel it
// replaced (with the attention of k_attn.hip), error against float64 1.2e-6 -> 0.55e-6.
//
// Between the two (about 1300 to 3000 rows) 128 x 192 tiles take one round of the CUs: M 2000, K 768, N
// 2304 / 3072 15.6 / 16.6 us against 18.3 / 20.2 with 64 x 64 tiles and 20.4 / 20.9 with 256-row ones.
// Their two sets of fragments would not leave room for the sums: they read after the barrier (with
// two sets 17.9 / 18.9).
//
// Where even 32 x 32 tiles do not fill the CUs, four wavefronts share such a tile's K-tiles (each with
// stages of its own) and their sums meet in LDS: the adapter down-projection of 1320 rows to rank 64,
// K 3072 15.1 -> 7.7 us, K 768 6.0 -> 4.8; M 32, N 2304, K 768 6.2 -> 4.9; fp32, M 128, N 1024, K 256
// 9.8 -> 6.4.
//
// K needs only K % 8 == 0: the chunks of the last K-tile past K are loaded from the row's first chunk
// (in bounds) and their fragments are replaced by zeros.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "gemm_common.h"
#include "kernels.h"

namespace dd {

constexpr int ROWB = 128;   // bytes of an operand row in a K-tile: 64 bf16 or 32 fp32

// The operand types: a K-tile is KT deep, a 16-byte chunk holds CH elements, and the two lane halves
// of a fragment read hold neighbouring chunks.
template <typename T> struct RingOp;
template <> struct RingOp<bf16_t> {
    static constexpr int KT = 64, CH = 8;
    typedef bf16x8 frag;
    DD_DEV static f32x16 mfma(frag w, frag a, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, a, c, 0, 0, 0); }
};
template <> struct RingOp<float> {
    static constexpr int KT = 32, CH = 4;
    typedef f32x4 frag;
    // element e of the lanes 0..31 and of the lanes 32..63 are the two k of one 32x32x2 product
    DD_DEV static f32x16 mfma(frag w, frag a, f32x16 c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(w[e], a[e], c, 0, 0, 0);
        return c;
    }
};
DD_DEV float ring_bias(const bf16_t* b, int i) { return bf16_to_f32(b[i]); }
DD_DEV float ring_bias(const float* b, int i) { return b[i]; }

// BM x BN x one K-tile tiles over WGM x WGN wavefronts of MB x NB 32x32 MFMA blocks, NST stages; with
// KG > 1, KG such sets of wavefronts and stages share a tile's K-tiles and their sums meet in LDS
template <int BM_, int BN_, int WGM_, int WGN_, int NST_, int KG_ = 1, bool AHEAD_ = true> struct RingShape {
    static constexpr bool AHEAD = AHEAD_;   // fragments are read one K-tile ahead (two sets)
    static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, NST = NST_, KG = KG_;
    static constexpr int NW = WGM * WGN, THREADS = 64 * NW * KG;   // NW: wavefronts per K group
    static constexpr int WM = BM / WGM, WN = BN / WGN, MB = WM / 32, NB = WN / 32;
    static constexpr int NA = BM / 8 / NW, NWL = BN / 8 / NW, NL = NA + NWL;   // 1 KB loads per wave and K-tile
    static constexpr int STAGE = (BM + BN) * ROWB;   // bytes
    static constexpr size_t LDS = (size_t)KG * NST * STAGE;
    static constexpr int WG_PER_CU = LDS * 2 <= 160 * 1024 ? 2 : 1;
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && WM % 32 == 0 && WN % 32 == 0, "split");
    static_assert(LDS <= 160 * 1024 && NST >= 2 && (NST - 2) * NL < 64, "stages; the wait counts the loads");
    static_assert((size_t)NW * 32 * 32 * 4 <= LDS, "epilogue staging");
};

// s_waitcnt vmcnt(N) alone
template <int N> DD_DEV void wait_vm() { __builtin_amdgcn_s_waitcnt(0x3F70 | (N & 15) | ((N >> 4) << 14)); }

template <typename T, int EPI, class S>
__global__ __launch_bounds__(S::THREADS, S::WG_PER_CU * S::NW * S::KG >= 8 ? S::WG_PER_CU * S::NW * S::KG / 4 : 1) void gemm_ring_kernel(GemmArgs g, int tiles_m, int tiles_n) {
    constexpr int MB = S::MB, NB = S::NB, NA = S::NA, NWL = S::NWL, NST = S::NST;
    constexpr int AROWS = S::BM / S::NW, WROWS = S::BN / S::NW;
    using Op = RingOp<T>;
    constexpr int KT = Op::KT, CH = Op::CH, ES = sizeof(T);
    extern __shared__ __attribute__((aligned(1024))) char ring_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    constexpr int KG = S::KG;
    const int kg = KG == 1 ? 0 : (tid >> 6) / S::NW, wave = KG == 1 ? tid >> 6 : (tid >> 6) % S::NW;
    char* smem = ring_smem + kg * (NST * S::STAGE);
    const int wm = wave / S::WGN, wn = wave % S::WGN;
    int M = g.M;
    if (g.m_count) {
        M = *g.m_count;
        tiles_m = (M + S::BM - 1) / S::BM;
        if (g.m_gate > 0 && ((M > g.m_gate) == (g.m_side != 0))) return;   // the other launch's rows
    }
    // splits outermost: an XCD's run of work indices then covers one K range of neighbouring tiles
    const int tiles = tiles_m * tiles_n, nsplit = g.splits > 1 ? g.splits : 1, work = tiles * nsplit;
    if ((int)blockIdx.x >= work) return;
    const int id = xcd_linear(blockIdx.x, work);
    const int split = id / tiles;
    int tm, tn;
    {
        const int t = id - split * tiles, in_group = 8 * tiles_n, grp = t / in_group, first = grp * 8;
        const int gsz = min(tiles_m - first, 8), r = t - grp * in_group;
        tm = first + r % gsz;
        tn = r / gsz;
    }
    const int m0 = tm * S::BM, n0 = tn * S::BN;
    const int nkt = (g.K + KT - 1) / KT, klast = g.K - (nkt - 1) * KT;   // valid k of the last K-tile
    const int nkb = g.k_base > 0 ? (g.k_base + KT - 1) / KT : nkt;   // K-tiles that are cut evenly
    const int ks0 = split * nkb / nsplit, ks1 = split + 1 == nsplit ? nkt : (split + 1) * nkb / nsplit;
    // K group kg takes nt K-tiles from kt0; the last groups may have fewer (`mine`): they load the
    // split's last K-tile again and leave it out, so that every wavefront meets the same barriers
    const int nt = (ks1 - ks0 + KG - 1) / KG, kt0 = ks0 + kg * nt;
    const int mine = KG == 1 ? nt : max(0, min(nt, ks1 - kt0));

    // This lane's 16-byte slot of row r holds K-chunk (lane % 8) ^ ((r >> 1) & 7).  Byte offsets from
    // the tile's first row (under 256 rows, so 32 bits), and the chunk's first k in the K-tile.
    const char* Ab = (const char*)g.A + (int64_t)m0 * g.lda * ES;
    const char* Wb = (const char*)g.W + (int64_t)n0 * g.ldw * ES;
    uint32_t offA[NA], offW[NWL];
    int chA[NA], chW[NWL];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int rl = AROWS * wave + 8 * i + (lane >> 3);
        chA[i] = ((lane & 7) ^ ((rl >> 1) & 7)) * CH;
        offA[i] = (uint32_t)(min(rl, M - 1 - m0) * (int)g.lda + chA[i]) * (uint32_t)ES;
    }
#pragma unroll
    for (int i = 0; i < NWL; ++i) {
        const int rl = WROWS * wave + 8 * i + (lane >> 3);
        chW[i] = ((lane & 7) ^ ((rl >> 1) & 7)) * CH;
        offW[i] = (uint32_t)(min(rl, g.N - 1 - n0) * (int)g.ldw + chW[i]) * (uint32_t)ES;
    }
    auto load = [&](int t, int stage, auto whole_c) {
        if (KG > 1) t = min(t, ks1 - 1);
        char* st = smem + stage * S::STAGE;
        const char* ap = Ab + (int64_t)t * ROWB;
        const char* wp = Wb + (int64_t)t * ROWB;
        if (!decltype(whole_c)::value && t == nkt - 1 && klast < KT) {
#pragma unroll
            for (int i = 0; i < NA; ++i)
                __builtin_amdgcn_global_load_lds((gbl_void*)(ap + (offA[i] - (chA[i] < klast ? 0 : chA[i] * ES))),
                                                 (lds_void*)(st + (AROWS * wave + 8 * i) * ROWB), 16, 0, 0);
#pragma unroll
            for (int i = 0; i < NWL; ++i)
                __builtin_amdgcn_global_load_lds((gbl_void*)(wp + (offW[i] - (chW[i] < klast ? 0 : chW[i] * ES))),
                                                 (lds_void*)(st + (S::BM + WROWS * wave + 8 * i) * ROWB), 16, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < NA; ++i)
                __builtin_amdgcn_global_load_lds((gbl_void*)(ap + offA[i]),
                                                 (lds_void*)(st + (AROWS * wave + 8 * i) * ROWB), 16, 0, 0);
#pragma unroll
            for (int i = 0; i < NWL; ++i)
                __builtin_amdgcn_global_load_lds((gbl_void*)(wp + offW[i]),
                                                 (lds_void*)(st + (S::BM + WROWS * wave + 8 * i) * ROWB), 16, 0, 0);
        }
    };

    f32x16 acc[NB][MB];
    if constexpr (EPI == EPI_BIAS_RESID) {
        // split 0 starts from the residual row: h is C itself, or the rows of c_in that c_rows lists
        const float* C = g.c_in ? g.c_in : (const float*)g.C;
        int64_t hrow[MB];
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            hrow[j] = min(m0 + wm * S::WM + j * 32 + (lane & 31), M - 1);
            if (g.c_in && g.c_rows) hrow[j] = g.c_rows[hrow[j]];
        }
        // rows past M and columns past N (N % 4 == 0) read a neighbour inside the matrix and are not
        // stored: no test between the loads, so that all are in flight together
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int j4 = 0; j4 < 4; ++j4) {
                    const int n = min(n0 + wn * S::WN + i * 32 + 8 * j4 + 4 * (lane >> 5), g.N - 4);
                    float4 h = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (split == 0 && kg == 0) h = *(const float4*)(C + hrow[j] * g.ldc + n);
                    acc[i][j][4 * j4] = h.x;
                    acc[i][j][4 * j4 + 1] = h.y;
                    acc[i][j][4 * j4 + 2] = h.z;
                    acc[i][j][4 * j4 + 3] = h.w;
                }
    } else {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    }

    // Two sets of fragments: a K-tile's are read while the MFMAs of the one before run (one set, read
    // after the barrier, left the LDS reads, the LDS writes of the loads and the MFMAs one after the
    // other: the wavefronts of a workgroup pass the barrier together).
    constexpr int KS = ROWB / 32;   // fragment steps of a K-tile: two chunks each
    typedef typename Op::frag frag;
    struct Frags {
        frag a[KS][MB], w[KS][NB];
    };
    const int frow = lane & 31, fsw = (lane >> 1) & 7, fhalf = lane >> 5;
    auto read = [&](Frags& f, int stage) {
        const char* sA = smem + stage * S::STAGE + (wm * S::WM + frow) * ROWB;
        const char* sW = smem + stage * S::STAGE + (S::BM + wn * S::WN + frow) * ROWB;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const int slot = ((2 * kk + fhalf) ^ fsw) * 16;
#pragma unroll
            for (int i = 0; i < MB; ++i) f.a[kk][i] = *(const frag*)&sA[32 * i * ROWB + slot];
#pragma unroll
            for (int i = 0; i < NB; ++i) f.w[kk][i] = *(const frag*)&sW[32 * i * ROWB + slot];
        }
    };
    auto mfmas = [&](const Frags& f) {
        if constexpr (ES == 4) {
            // Each K-tile's 32 products are summed from zero and added to the running sum by the VALU
            // (16 adds beside 1024 MFMA cycles): with the running sum inside the MFMAs the logits of
            // a 12-layer d 768 model are 2.7e-6 off the float64 result.
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    f32x16 part = {};
#pragma unroll
                    for (int kk = 0; kk < KS; ++kk) part = Op::mfma(f.w[kk][nb], f.a[kk][mb], part);
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[nb][mb][e] += part[e];
                }
            return;
        }
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    acc[nb][mb] = Op::mfma(f.w[kk][nb], f.a[kk][mb], acc[nb][mb]);
    };
    auto clear_past = [&](Frags& f) {   // the last K-tile's fragments past K
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const bool past = (2 * kk + fhalf) * CH >= klast;
            const frag z = {};
#pragma unroll
            for (int i = 0; i < MB; ++i) f.a[kk][i] = past ? z : f.a[kk][i];
#pragma unroll
            for (int i = 0; i < NB; ++i) f.w[kk][i] = past ? z : f.w[kk][i];
        }
    };
    // this lane's loads of K-tile t landed (`ahead` K-tiles after it may be in flight), then everyone's
    auto publish = [&](int ahead) {
        if (ahead >= NST - 2) wait_vm<(NST - 2) * S::NL>();
        else if (NST > 3 && ahead == NST - 3) wait_vm<(NST > 3 ? NST - 3 : 0) * S::NL>();
        else if (NST > 4 && ahead == NST - 4) wait_vm<(NST > 4 ? NST - 4 : 0) * S::NL>();
        else if (NST > 5 && ahead == NST - 5) wait_vm<(NST > 5 ? NST - 5 : 0) * S::NL>();
        else wait_vm<0>();
        asm volatile("s_barrier" ::: "memory");
    };

#pragma unroll
    for (int p = 0; p < NST - 1; ++p)
        if (p < nt) load(kt0 + p, p, std::false_type{});
    if constexpr (!S::AHEAD) {
        // one set: a K-tile's fragments are read after the barrier that publishes it
        static_assert(KG == 1, "K groups read ahead");
        Frags f;
        int cur = 0, ld = NST - 1;
        for (int t = 0; t < nt; ++t) {
            publish(min(nt - 1 - t, NST - 2));
            if (t + NST - 1 < nt) load(kt0 + t + NST - 1, ld, std::false_type{});
            read(f, cur);
            if (kt0 + t == nkt - 1 && klast < KT) clear_past(f);
            mfmas(f);
            // the next barrier lets the other wavefronts load over this stage: the reads are waited for
            // by the products that use them, which must not sink below it (scalar instructions may: with
            // the loop counter held behind the products the tile takes 1.5 % longer)
            __builtin_amdgcn_sched_barrier(0x4);
            cur = cur + 1 == NST ? 0 : cur + 1;
            ld = ld + 1 == NST ? 0 : ld + 1;
        }
    } else {
        Frags f0, f1;
        publish(min(nt - 1, NST - 2));
        read(f0, 0);
        int rd = 1, ld = NST - 1;   // stages of K-tile t + 1 and of K-tile t + NST - 1
        // K-tile t from `cur`; K-tile t + 1 is read into `nxt` and K-tile t + NST - 1 loaded into the
        // stage of K-tile t - 1, whose fragments every wavefront had waited for before this barrier.
        // `steady`: both exist, and nothing branches, so that the compiler's waits before the MFMAs count
        // the reads of `nxt` as still in flight.
        auto step = [&](int t, Frags& cur, Frags& nxt, auto steady_c) {
            constexpr bool steady = decltype(steady_c)::value;
            if (steady || t + 1 < nt) {
                if constexpr (steady) {
                    wait_vm<(NST - 3) * S::NL>();
                    asm volatile("s_barrier" ::: "memory");
                } else {
                    publish(min(nt - 2 - t, NST - 3));
                }
                read(nxt, rd);
                if (steady || t + NST - 1 < nt) load(kt0 + t + NST - 1, ld, steady_c);
                rd = rd + 1 == NST ? 0 : rd + 1;
                ld = ld + 1 == NST ? 0 : ld + 1;
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (!steady) {
                if (kt0 + t == nkt - 1 && klast < KT) clear_past(cur);
                if (KG > 1 && t >= mine) return;
            }
            mfmas(cur);
            __builtin_amdgcn_sched_barrier(0);
        };
        int t = 0;
        // (the last K-tile, which may be ragged, is loaded below; all groups leave this loop together)
        const int nsteady = KG == 1 ? nt : ks1 - ks0 - (KG - 1) * nt;
        for (; t + NST + 1 < nsteady; t += 2) {
            step(t, f0, f1, std::true_type{});
            step(t + 1, f1, f0, std::true_type{});
        }
        for (; t < nt; t += 2) {
            step(t, f0, f1, std::false_type{});
            if (t + 1 < nt) step(t + 1, f1, f0, std::false_type{});
        }
    }
    __syncthreads();   // the stages become the epilogue's staging area
    smem = ring_smem;
    if constexpr (KG > 1) {
        float4* part = (float4*)ring_smem;   // [KG - 1][NW][4 MB NB][64]
        constexpr int PV = 4 * MB * NB;
        static_assert((size_t)(KG - 1) * S::NW * PV * 64 * 16 <= S::LDS, "partial sums");
        if (kg > 0) {
#pragma unroll
            for (int i = 0; i < PV; ++i) {
                const f32x16& c = acc[i / 4 / MB][i / 4 % MB];
                part[(((kg - 1) * S::NW + wave) * PV + i) * 64 + lane] =
                    make_float4(c[4 * (i & 3)], c[4 * (i & 3) + 1], c[4 * (i & 3) + 2], c[4 * (i & 3) + 3]);
            }
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int w = 0; w < KG - 1; ++w)
#pragma unroll
                for (int i = 0; i < PV; ++i) {
                    const float4 p = part[((w * S::NW + wave) * PV + i) * 64 + lane];
                    f32x16& c = acc[i / 4 / MB][i / 4 % MB];
                    c[4 * (i & 3)] += p.x; c[4 * (i & 3) + 1] += p.y; c[4 * (i & 3) + 2] += p.z; c[4 * (i & 3) + 3] += p.w;
                }
        }
        __syncthreads();
        if (kg > 0) return;
    }

    if constexpr (EPI == EPI_BIAS_RESID || ES == 4) {
        // fp32 rows: one 32 x 32 block at a time through this wavefront's 4 KB, chunk-swizzled by row,
        // so that eight lanes write one 128-byte row segment
        float* cst = (float*)smem + wave * (32 * 32);
        float* C = split == 0 ? (float*)g.C : g.slab[split - 1];
        const T* bias = (const T*)g.bias;
        const int rr = lane >> 3, c4 = (lane & 7) * 4;
        constexpr bool BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RESID;
        float bv[NB][4];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                bv[nb][e] = BIAS && split == 0 ? ring_bias(bias, min(n0 + wn * S::WN + nb * 32 + c4 + e, g.N - 1)) : 0.f;
#pragma unroll
        for (int b = 0; b < MB * NB; ++b) {
            const int mb = b % MB, nb = b / MB;
            const int wr = lane & 31;
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4) {
                const int slot = (2 * j4 + (lane >> 5)) ^ ((wr >> 1) & 7);
                *(float4*)&cst[wr * 32 + slot * 4] = make_float4(acc[nb][mb][4 * j4], acc[nb][mb][4 * j4 + 1],
                                                                 acc[nb][mb][4 * j4 + 2], acc[nb][mb][4 * j4 + 3]);
            }
            const int n = n0 + wn * S::WN + nb * 32 + c4;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int r = rr + 8 * it;
                const float4 v = *(const float4*)&cst[r * 32 + (((c4 >> 2) ^ ((r >> 1) & 7)) * 4)];
                const int m = m0 + wm * S::WM + mb * 32 + r;
                if (m >= M || n >= g.N) continue;
                float o[4] = {v.x + bv[nb][0], v.y + bv[nb][1], v.z + bv[nb][2], v.w + bv[nb][3]};
                if constexpr (EPI == EPI_BIAS_GELU)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = gelu_tanh_f32(o[e]);
                if constexpr (EPI == EPI_GATE) {
                    const float rs = gate_row_scale(g, m);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] *= rs;
                }
                float* dst = C + (int64_t)m * g.ldc + n;
                if (EPI == EPI_BIAS_RESID || n + 3 < g.N) {
                    *(f32x4*)dst = f32x4{o[0], o[1], o[2], o[3]};
                } else {
                    for (int e = 0; n + e < g.N; ++e) dst[e] = o[e];
                }
            }
        }
    } else {
        // one 32 x 32 block at a time through this wavefront's staging rows (80 bytes), then 16-byte
        // pieces of 64-byte row segments
        constexpr int CSTR = 40;
        bf16_t* cst = (bf16_t*)smem + wave * (32 * CSTR);
        bf16_t* C = (bf16_t*)g.C;
        const bf16_t* bias = (const bf16_t*)g.bias;
        float b4[EPI == EPI_BIAS || EPI == EPI_BIAS_GELU ? NB : 1][16];
        if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    b4[nb][e] = bf16_to_f32(bias[min(n0 + wn * S::WN + nb * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3), g.N - 1)]);
        }
#pragma unroll
        for (int b = 0; b < MB * NB; ++b) {
            const int mb = b % MB, nb = b / MB;
            float rs = 1.f;
            if constexpr (EPI == EPI_GATE) rs = gate_row_scale(g, m0 + wm * S::WM + mb * 32 + (lane & 31));
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4) {
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float x = acc[nb][mb][4 * j4 + e];
                    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU) x += b4[nb][4 * j4 + e];
                    if constexpr (EPI == EPI_BIAS_GELU) x = gelu_tanh(x);
                    if constexpr (EPI == EPI_GATE) x *= rs;
                    o[e] = x;
                }
                uint2 pk;
                pk.x = pack_bf16x2(o[0], o[1]);
                pk.y = pack_bf16x2(o[2], o[3]);
                *(uint2*)&cst[(lane & 31) * CSTR + 8 * j4 + 4 * (lane >> 5)] = pk;
            }
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int r = 16 * it + (lane >> 2), c = (lane & 3) * 8;
                const uint4 v = *(const uint4*)&cst[r * CSTR + c];
                const int m = m0 + wm * S::WM + mb * 32 + r, n = n0 + wn * S::WN + nb * 32 + c;
                if (m >= M || n >= g.N) continue;
                bf16_t* dst = C + (int64_t)m * g.ldc + n;
                if (n + 7 < g.N) {
                    *(u32x4*)dst = u32x4{v.x, v.y, v.z, v.w};
                } else {
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
                    for (int e = 0; n + e < g.N; ++e) dst[e] = (bf16_t)((w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
                }
            }
        }
    }
}


template <typename T, int EPI, class S>
static void launch_shape(const GemmArgs& g, hipStream_t s) {
    const int tm = ((g.m_rows > 0 ? g.m_rows : g.M) + S::BM - 1) / S::BM, tn = (g.N + S::BN - 1) / S::BN;
    static std::once_flag once;   // opt-in to more than 64 KB of LDS per workgroup
    std::call_once(once, [] {
        (void)hipFuncSetAttribute((const void*)gemm_ring_kernel<T, EPI, S>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)S::LDS);
    });
    launch_k((gemm_ring_kernel<T, EPI, S>), dim3(tm * tn * std::max(g.splits, 1)), dim3(S::THREADS), S::LDS, s, g, tm, tn);
}

template <int EPI>
static void launch_epi(int dtype, RingTile tile, const GemmArgs& g, hipStream_t s) {
    if (dtype == DD_FP32) {
        switch (tile) {
            case RING_32K: launch_shape<float, EPI, RingShape<32, 32, 1, 1, 4, 4>>(g, s); break;
            case RING_32X64: launch_shape<float, EPI, RingShape<32, 64, 1, 2, 3, 2>>(g, s); break;
            default: launch_shape<float, EPI, RingShape<64, 64, 2, 2, 4>>(g, s); break;
        }
        return;
    }
    switch (tile) {
        case RING_128: launch_shape<bf16_t, EPI, RingShape<128, 128, 4, 2, 4>>(g, s); break;
        case RING_64_DEEP: launch_shape<bf16_t, EPI, RingShape<64, 64, 2, 2, 4>>(g, s); break;
        case RING_32K: launch_shape<bf16_t, EPI, RingShape<32, 32, 1, 1, 4, 4>>(g, s); break;
        case RING_128X192: launch_shape<bf16_t, EPI, RingShape<128, 192, 4, 2, 3, 1, false>>(g, s); break;
        default: launch_shape<bf16_t, EPI, RingShape<64, 64, 2, 2, 3>>(g, s); break;
    }
}

void launch_gemm_ring(int dtype, RingTile tile, int epi, const GemmArgs& g, hipStream_t s) {
    switch (epi) {
        case EPI_BIAS: launch_epi<EPI_BIAS>(dtype, tile, g, s); break;
        case EPI_BIAS_GELU: launch_epi<EPI_BIAS_GELU>(dtype, tile, g, s); break;
        case EPI_BIAS_RESID: launch_epi<EPI_BIAS_RESID>(dtype, tile, g, s); break;
        case EPI_GATE: launch_epi<EPI_GATE>(dtype, tile, g, s); break;
        default: launch_epi<EPI_PLAIN>(dtype, tile, g, s); break;
    }
}

// Estimated time (us) of C [M][N] = A W^T over K on a ring tile.  Rounds of up to P workgroups per CU,
// each a fixed part and per K-tile the larger of its own latency and the share of the CU that its
// co-residents leave it.  Fitted to 17 products (N 64..4096, K 256..4096) at 16 row counts from 64 to
// 16384, 1 to 4 splits, the weights rotating as the layers of a model do: 9 to 13 % rms.
double gemm_ring_us(RingTile tile, int64_t M, int64_t N, int64_t K, int splits, int cus) {
    struct Fit {
        int bm, bn, P;
        double t0, tw, lat, share;
    };
    static const Fit fits[] = {{128, 128, 1, 0.0, 6.3, 0.49, 0.49},
                               {64, 64, 2, 1.3, 2.9, 0.21, 0.214},
                               {64, 64, 3, 0.5, 3.3, 0.41, 0.241},
                               {128, 192, 1, 1.8, 2.2, 1.0, 1.0}};
    const Fit& f = fits[tile == RING_128 ? 0 : tile == RING_64_DEEP ? 1 : tile == RING_64 ? 2 : 3];
    const int64_t wg = ((M + f.bm - 1) / f.bm) * ((N + f.bn - 1) / f.bn) * splits;
    const int64_t kt = ((K + BK - 1) / BK + splits - 1) / splits;
    const int64_t full = wg / ((int64_t)cus * f.P), rest = wg - full * cus * f.P;
    double t = f.t0 + (double)full * (f.tw + (double)kt * std::max(f.lat, f.P * f.share));
    if (rest > 0) t += f.tw + (double)kt * std::max(f.lat, (double)((rest + cus - 1) / cus) * f.share);
    return t;
}

}  // namespace dd
