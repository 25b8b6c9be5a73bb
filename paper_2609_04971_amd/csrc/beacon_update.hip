// (a1) Beacon maintenance for gfx950.
//
// Beacons stand for clusters of pre-RoPE queries under cosine similarity
// (Section 3.2 "Beacon queries"; Section 4.2; the nearest-representative
// similarity of Appendix D.1, Algorithm 1).  Online rule: each new query
// fills the lowest empty slot if there is one; otherwise it joins the slot
// of largest cosine similarity (ties -> lowest slot, cosine 0 when a norm is
// 0) and that slot moves to the running mean of its members.
//
// Heads of up to 16 slots take one wave (a 64-thread workgroup) each: the
// queries of a head are taken strictly in order, each seeing the previous
// update, so a head's work is one sequential chain, and small workgroups let
// many heads' chains run side by side on a compute unit (a layer-stacked
// call has thousands of heads).  Lanes 4c .. 4c+3 each take a quarter of
// slot c's dot product and a quad sum completes it.  Heads of more slots
// take four waves: all four bring the beacons in and compute their norms in
// one pass, the first takes the queries with one lane per slot, and the
// others wait for it at the barrier before the write-back.  The head's
// beacons live in LDS (rows padded to D + 4 floats) together with their
// squared norms, which are kept up to date as slots change; every 16-byte
// beacon load of a chunk is issued before the first wait.  Per query an
// argmax over the lanes (DPP, no LDS round trip) picks the slot and the
// lanes update that slot's D coordinates and its norm in parallel.  Finally
// the changed slots are written back (at most T*G of the C rows; the others
// still hold what was read).  The LDS is sized by C.
//
// Calls that bring many queries per head (prompts) take beacon_batch_kernel
// instead, which forms the cosines of 16 queries with every slot and with
// each other on the matrix cores and keeps only the assignments serial; its
// results are the same, bit for bit (see there for the rule and why).
#include <math.h>

#include "device_common.h"
#include "internal.h"

namespace bkv {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Query elements are loaded raw and widened only where they are used, so
// that a prefetch is not waited on right after it is issued.
__device__ __forceinline__ float widen(uint16_t v) { return dev::bf16_to_f32(v); }
__device__ __forceinline__ float widen(float v) { return v; }

// Dot product of two LEN-float rows in LDS (16-byte aligned), with four
// independent partial sums so that the FMAs do not wait on each other.
template <int LEN>
__device__ __forceinline__ float row_dot(const float* a, const float* b) {
    const float4* ar = reinterpret_cast<const float4*>(a);
    const float4* br = reinterpret_cast<const float4*>(b);
    float p0 = 0.f, p1 = 0.f, p2 = 0.f, p3 = 0.f;
#pragma unroll 8
    for (int d4 = 0; d4 < LEN / 4; ++d4) {
        const float4 u = ar[d4], v = br[d4];
        p0 = fmaf(u.x, v.x, p0);
        p1 = fmaf(u.y, v.y, p1);
        p2 = fmaf(u.z, v.z, p2);
        p3 = fmaf(u.w, v.w, p3);
    }
    return (p0 + p1) + (p2 + p3);
}

// Orders the wave's LDS accesses for the compiler: one lane's write before
// the fence is seen by another lane's read after it.  A wave's LDS
// instructions execute in order, so a wavefront-scope fence needs no wait
// instruction; in particular it does not wait for the next query's global
// loads in flight (a workgroup-scope fence or barrier would).
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

__device__ __forceinline__ float cosine(float dot, float xn, float bn) {
    return (xn == 0.f || bn == 0.f) ? 0.f : dot * __builtin_amdgcn_rsqf(xn) * __builtin_amdgcn_rsqf(bn);
}

// The slot of largest cosine with the query xs (squared norm xn), ties ->
// lowest slot: the smallest inverted order key of the cosine over the wave,
// then the lowest lane that holds it.  The cosine takes hardware reciprocal
// square roots (about 1 ulp each), so the choice can differ from exact
// arithmetic only where the two best cosines lie within a few 1e-7 of each
// other.  bl [C][D + 4], xs [D] and the slots' squared norms bn2 in LDS.
// QUAD (C <= 16): lanes 4c .. 4c+3 each take a quarter of slot c; else lane
// c takes slot c, quarter by quarter (the sums are the same).
template <int D, bool QUAD>
__device__ __forceinline__ int nearest_slot(const float* bl, const float* xs, const float* bn2, float xn, int C,
                                            int lane) {
    constexpr int LD = D + 4, QD = D / 4;
    unsigned key = ~0u;
    bool holds;  // this lane speaks for a slot
    if constexpr (QUAD) {
        const int c = lane >> 2, part = lane & 3;
        const float dot = dev::quad_sum(c < C ? row_dot<QD>(&bl[c * LD + part * QD], &xs[part * QD]) : 0.f);
        holds = c < C && part == 0;
        if (holds) key = ~dev::ord_key(cosine(dot, xn, bn2[c]));
    } else {
        float dot = 0.f;
        if (lane < C) {
            const f32x4* b = reinterpret_cast<const f32x4*>(&bl[lane * LD]);
            const f32x4* x = reinterpret_cast<const f32x4*>(xs);
            float part[4];
#pragma unroll
            for (int k = 0; k < 4; k += 2) {  // two quarters side by side: four would cost half the occupancy
                f32x4 p[2];
#pragma unroll
                for (int i = 0; i < QD / 4; ++i)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const f32x4 u = b[(k + c) * (QD / 4) + i], v = x[(k + c) * (QD / 4) + i];
#pragma unroll
                        for (int e = 0; e < 4; ++e) p[c][e] = fmaf(u[e], v[e], i ? p[c][e] : 0.f);
                    }
#pragma unroll
                for (int c = 0; c < 2; ++c) part[k + c] = (p[c][0] + p[c][1]) + (p[c][2] + p[c][3]);
            }
            dot = (part[0] + part[1]) + (part[2] + part[3]);
        }
        holds = lane < C;
        if (holds) key = ~dev::ord_key(cosine(dot, xn, bn2[lane]));
    }
    const unsigned kmin = dev::wave_min_u32(key);
    return (__ffsll(__ballot(holds && key == kmin)) - 1) >> (QUAD ? 2 : 0);
}

// Every squared norm is summed in one order, whoever forms it, so that equal
// rows have equal norms and tie exactly: D / 64 neighbouring coordinates one
// after the other, then their sums pairwise, as dev::wave_sum adds those of
// 64 lanes.  sumsq_quarter is the part of one quarter (v(e) its coordinate
// e), whose four results (a + b) + (c + d) makes the norm.
template <int D, typename V>
__device__ __forceinline__ float sumsq_quarter(V&& v) {
    constexpr int PER = D / 64;
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float l[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            l[j] = 0.f;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const float x = v((4 * i + j) * PER + k);
                l[j] = fmaf(x, x, l[j]);
            }
        }
        s[i] = (l[0] + l[1]) + (l[2] + l[3]);
    }
    return (s[0] + s[1]) + (s[2] + s[3]);
}

// (a + b) + (c + d) of the wave's four rows of 16 lanes, lane by lane.
__device__ __forceinline__ float rows_sum(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Squared norm of a row in LDS, a quarter of it to each of four lanes.
template <int D>
__device__ __forceinline__ float quarter_norm(const float* quarter, bool live) {
    float p = 0.f;
    if (live) {
        f32x4 u[D / 16];
#pragma unroll
        for (int i = 0; i < D / 16; ++i) u[i] = reinterpret_cast<const f32x4*>(quarter)[i];
        p = sumsq_quarter<D>([&](int e) { return u[e / 4][e % 4]; });
    }
    return dev::quad_sum(p);
}

constexpr int kMaxSlots = 64;   // the boundary rejects C > 64: one bit per slot in a 64-bit mask
constexpr int kLoadChunk = 8;   // 16-byte beacon loads in flight per thread
constexpr int kQuadSlots = 16;  // C up to this: one wave per head, four lanes per slot's dot product
static_assert(kMaxSlots <= 64, "one lane of the query wave per slot holds its count and its dirty bit");

// LDS bytes of one head: C padded beacon rows, the current query, C norms,
// C counts, the mask of changed slots.
template <int D>
constexpr size_t smem_bytes(int C) {
    return ((size_t)C * (D + 4) + D + C) * sizeof(float) + (size_t)C * sizeof(int) + sizeof(unsigned long long);
}

// NW waves per workgroup: 1 for C <= kQuadSlots (the query wave alone, four
// lanes per slot's dot product), 4 for more slots (all four waves load the
// beacons and compute their norms in one pass, the first wave takes the
// queries with one lane per slot, the others wait at the barrier before the
// write-back).
template <typename T, int D, int NW>
__global__ __launch_bounds__(64 * NW) void beacon_update_kernel(const T* __restrict__ q_new, int T_steps,
                                                                float* beacons, int32_t* counts, int32_t* assign,
                                                                int Hq, int Hkv, int C) {
    constexpr int NT = 64 * NW;    // threads
    constexpr int LD = D + 4;      // padded row
    constexpr int PER = D / 64;    // coordinates per lane in lane-parallel loops, neighbours
    constexpr int QD = D / 4;      // coordinates per lane of a slot's dot product (four lanes per slot)
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* bl = smem;                            // [C][LD]
    float* xs = bl + C * LD;                     // [D], 16-byte aligned: C * LD and D are multiples of 4
    float* bn2 = xs + D;                         // [C] squared norm of each slot
    int* cnt = reinterpret_cast<int*>(bn2 + C);  // [C]
    unsigned long long* dirty_out = reinterpret_cast<unsigned long long*>(cnt + C);  // 8-byte aligned
    auto sync = [] {
        if constexpr (NW > 1)
            __syncthreads();
        else
            wave_lds_fence();
    };
    const int tid = threadIdx.x, lane = tid & 63;
    const int h = blockIdx.x, b = h / Hkv, kh = h % Hkv;
    const int G = Hq / Hkv;
    float* bh = beacons + (size_t)h * C * D;
    const int nq = T_steps * G;
    auto query_ptr = [&](int qq) {
        const int t = qq / G, g = qq - t * G;
        return q_new + (((size_t)b * Hq + (size_t)kh * G + g) * T_steps + t) * D;
    };
    // The first query, the counts and a chunk of beacon vectors are loaded
    // unconditionally (threads past the end re-read the last element) and
    // pinned by an empty asm before the first store uses them, so the
    // compiler neither sinks a load into the guarded store nor waits
    // between loads: a chunk's loads all issue before the first wait (the
    // beacons of 16 slots, or of 64 with four waves, are one chunk).
    T xnext[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) xnext[k] = query_ptr(0)[PER * lane + k];
    int cv = counts[(size_t)h * C + min(tid, C - 1)];
    asm volatile("" : "+v"(cv));
    const int n4 = C * D / 4;
    for (int base = 0; base < n4; base += NT * kLoadChunk) {
        dev::u32x4 v[kLoadChunk];
#pragma unroll
        for (int k = 0; k < kLoadChunk; ++k)
            v[k] = reinterpret_cast<const dev::u32x4*>(bh)[min(base + tid + NT * k, n4 - 1)];
#pragma unroll
        for (int k = 0; k < kLoadChunk; ++k) asm volatile("" : "+v"(v[k]));
#pragma unroll
        for (int k = 0; k < kLoadChunk; ++k) {
            const int i = base + tid + NT * k;
            if (i < n4) *reinterpret_cast<dev::u32x4*>(&bl[(4 * i) / D * LD + (4 * i) % D]) = v[k];
        }
    }
    if (tid < C) cnt[tid] = cv;
    sync();
    // squared norms: four threads per slot
    for (int c0 = 0; c0 < C; c0 += NT / 4) {
        const int c = c0 + (tid >> 2), part = tid & 3;
        const float p = quarter_norm<D>(&bl[c * LD + part * QD], c < C);
        if (c < C && part == 0) bn2[c] = p;
    }
    sync();

    if (tid < 64) {
        unsigned long long dirty = 0;  // slots changed (wave-uniform)
        for (int q = 0; q < nq; ++q) {
            float xn = 0.f;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const float x = widen(xnext[k]);
                xs[PER * lane + k] = x;
                xn = fmaf(x, x, xn);
            }
            // the next query (the last one again at the end: no branch to
            // join, so nothing waits for it before its use)
#pragma unroll
            for (int k = 0; k < PER; ++k) xnext[k] = query_ptr(min(q + 1, nq - 1))[PER * lane + k];
            xn = dev::wave_sum(xn);
            wave_lds_fence();
            // lowest empty slot, if any
            const unsigned long long empty = __ballot(lane < C && cnt[lane] == 0);
            int chosen;
            if (empty) {
                chosen = __ffsll(empty) - 1;
#pragma unroll
                for (int k = 0; k < PER; ++k) bl[chosen * LD + PER * lane + k] = xs[PER * lane + k];
                if (lane == 0) {
                    cnt[chosen] = 1;
                    bn2[chosen] = xn;
                }
            } else {
                chosen = nearest_slot<D, NW == 1>(bl, xs, bn2, xn, C, lane);
                const int n = cnt[chosen] + 1;
                const float inv = 1.0f / (float)n;
                float p = 0.f;
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const int d = PER * lane + k;
                    const float bv = bl[chosen * LD + d];
                    const float nv = bv + (xs[d] - bv) * inv;
                    bl[chosen * LD + d] = nv;
                    p = fmaf(nv, nv, p);
                }
                p = dev::wave_sum(p);
                if (lane == 0) {
                    cnt[chosen] = n;
                    bn2[chosen] = p;
                }
            }
            dirty |= 1ull << chosen;
            if (assign && lane == 0) assign[(size_t)h * T_steps * G + q] = chosen;
            wave_lds_fence();
        }
        if (lane == 0) *dirty_out = dirty;
    }
    sync();
    // write back the changed slots only: the others still hold what was read
    const unsigned long long dirty = *dirty_out;
    for (int i = tid; i < n4; i += NT) {
        const int c = (4 * i) / D, d = (4 * i) % D;
        if ((dirty >> c) & 1ull) reinterpret_cast<float4*>(bh)[i] = *reinterpret_cast<const float4*>(&bl[c * LD + d]);
    }
    if (tid < C && ((dirty >> tid) & 1ull)) counts[(size_t)h * C + tid] = cnt[tid];
}

// ---- many queries per head ---------------------------------------------------
//
// A prompt's queries are one chain per head, and the kernel above spends
// 0.5 to 1.3 us on each: a dot product with every slot, an argmax and the
// update of a row, all dependent.  Here 16 queries are taken at a time.  Their
// dot products with every slot (the beacons stay in registers) and with each other come
// from MFMA, and the chain then works on those numbers only: one wave, lane
// = slot, picks the slot and applies the update to the slot's remaining dot
// products and its squared norm,
//     <x', b + (x - b)/n> = <x', b> + (<x', x> - <x', b>)/n,
//     |b + (x - b)/n|^2 = (1 - 1/n)^2 |b|^2 + |x|^2/n^2 + 2 (1 - 1/n)/n <x, b>,
// after which the waves apply the batch's updates to the beacons themselves,
// query by query with the same arithmetic as above, and take the norms
// afresh.  The numbers of a batch carry a few more roundings than direct
// ones (a few 1e-7 of a cosine).  So where a query's two best cosines lie
// within kNearTie (about one in 10^4) the chain ends before it, and the rest
// of the batch is taken one by one with the arithmetic above; where an update
// cancels most of a beacon the batch ends, so that the next one starts from
// the beacons again: the choices are those of the kernel above, and so are
// the results; batches with a norm or count out of the chain's reach (zero
// queries among them) go one by one as well.  Equal beacons (repeated tokens) make ties of many queries:
// with ties in every batch 128 heads of 2048 queries take 1858 us (64 slots;
// the kernel above 2395) and 1572 (16 slots; 1587), 8 heads of 16 queries 12
// (12); only many heads of a single batch lose by it (4608 of 16 slots 55
// against 42, 1024 of 64 slots 130 against 91; without ties 38 against 44
// and 76 against 94).
//
// Bound by the chain, about 100 instructions a query on one wave, and by the
// batch's phases around it.  128 heads of 2048 queries: 64 slots 948 us
// (2395 with the kernel above), 16 slots 1019 (1584); 4608 heads of 256
// queries, 64 slots: 860 (1850).
constexpr int kBatchQ = 16;   // queries per batch: one MFMA tile
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

template <int D, int NW>
struct alignas(16) BatchLds {
    static constexpr int QP = D / 4 + 4;  // a quarter of a query, padded
    float xs[2][kBatchQ][4 * QP];         // this batch's queries and the next one's
    float dot[kBatchQ][16 * NW + 4];      // <query, slot>
    float gram[kBatchQ][kBatchQ + 4];     // <query, query>
    float margin[kBatchQ];                // near-tie margin of each query's products
    float bn2[16 * NW];                   // squared norm of each slot
    struct {
        int slot;   // the slot a query joined; + kFill: it filled an empty one
        float inv;  // 1/n of the update
    } joined[kBatchQ];
    int done;                             // queries of the batch that the chain took; + kFill: empty slots are left
    int alone;                            // the ones behind them to take one at a time
    int cnt[64];                          // counts of the slots, for those
    unsigned long long best[2][NW];       // each wave's nearest slot: inverted order key of the cosine, slot
    unsigned long long dirty;
};
constexpr int kFill = 256;
constexpr float kNearTie = 4e-6f;  // cosines this close are settled by the arithmetic of one query at a time
constexpr float kNormMin = 1e-18f, kNormMax = 1e18f;  // squared norms that the chain takes
constexpr int kCountMax = (1 << 21) - kBatchQ;        // counts that it takes
constexpr int kBatchMin = 16;  // queries per head from which the batches are taken

// Maximum over the wave, the same in every lane.
template <int CTRL>
__device__ __forceinline__ int dpp_max_i32(int v) {
    const int w = __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
    return w > v ? w : v;
}
__device__ __forceinline__ int wave_max_i32(int v) {
    v = dpp_max_i32<0x140>(dpp_max_i32<0x141>(dpp_max_i32<0x4e>(dpp_max_i32<0xb1>(v))));
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// NW = ceil(C / 16) waves; wave w holds slots 16 w .. 16 w + 15, lane (g =
// lane / 16, c = lane % 16) elements g D/4 .. (g + 1) D/4 - 1 of slot 16 w + c.
template <typename T, int D, int NW>
__global__ __launch_bounds__(64 * NW) void beacon_batch_kernel(const T* __restrict__ q_new, int T_steps, float* beacons,
                                                              int32_t* counts, int32_t* assign, int Hq, int Hkv, int C) {
    constexpr int NT = 64 * NW, Q = D / 4, EV = 16 / (int)sizeof(T), CPR = D / EV;  // 16-byte chunks per query
    constexpr int NL = (kBatchQ * CPR + NT - 1) / NT;                                // chunks per thread of a batch
    using L = BatchLds<D, NW>;
    __shared__ L sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c16 = lane & 15;
    const int h = blockIdx.x, b = h / Hkv, kh = h % Hkv, G = Hq / Hkv;
    const int nq = T_steps * G;
    float* bh = beacons + (size_t)h * C * D;
    const int slot = wave * 16 + c16;

    dev::u32x4 xr[NL];
    auto load_queries = [&](int base) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int id = tid + NT * i, qq = base + id / CPR;
            xr[i] = dev::u32x4{0u, 0u, 0u, 0u};
            if (id < kBatchQ * CPR && qq < nq) {
                const int t = qq / G, gq = qq - t * G;
                xr[i] = *reinterpret_cast<const dev::u32x4*>(
                    q_new + (((size_t)b * Hq + (size_t)kh * G + gq) * T_steps + t) * D + id % CPR * EV);
            }
        }
    };
    auto stage_queries = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int id = tid + NT * i;
            if (id < kBatchQ * CPR) {
                const int e0 = id % CPR * EV;  // EV divides a quarter
                float* o = &sh.xs[buf][id / CPR][e0 / Q * L::QP + e0 % Q];
#pragma unroll
                for (int w = 0; w < EV; w += 4) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (sizeof(T) == 2) {
                            const unsigned u = xr[i][(w + e) / 2];
                            v[e] = __uint_as_float(e & 1 ? u & 0xffff0000u : u << 16);
                        } else {
                            v[e] = __uint_as_float(xr[i][e]);
                        }
                    }
                    *reinterpret_cast<f32x4*>(o + w) = v;
                }
            }
        }
    };
    load_queries(0);
    f32x4 beta[Q / 4];
#pragma unroll
    for (int i = 0; i < Q / 4; ++i)
        beta[i] = slot < C ? reinterpret_cast<const f32x4*>(bh + (size_t)slot * D + g * Q)[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    int cnt = (wave == 0 && lane < C) ? counts[(size_t)h * C + lane] : 1;  // wave 0: lane = slot
    bool touched = false;  // wave 0: this lane's slot changed
    auto store_norms = [&] {
        const float p = rows_sum(sumsq_quarter<D>([&](int e) { return beta[e / 4][e % 4]; }));
        if (g == 0) sh.bn2[slot] = p;
    };
    // Query qq (coordinates at xq, squared norm xn) with the arithmetic of
    // beacon_update_kernel, bit for bit.
    auto take_one = [&](const float* xq, float xn, int qq, int odd) {
        wave_lds_fence();  // the norms stored before
        f32x4 x[Q / 4], p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < Q / 4; ++i) x[i] = *reinterpret_cast<const f32x4*>(xq + g * L::QP + 4 * i);
#pragma unroll
        for (int i = 0; i < Q / 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = fmaf(beta[i][e], x[i][e], p[e]);
        const float dot = rows_sum((p[0] + p[1]) + (p[2] + p[3]));
        const bool holds = slot < C && g == 0;  // this lane speaks for its slot
        const unsigned key = holds ? ~dev::ord_key(cosine(dot, xn, sh.bn2[slot])) : ~0u;
        const unsigned kmin = dev::wave_min_u32(key);
        int chosen = wave * 16 + ((__ffsll(__ballot(holds && key == kmin)) - 1) & 15);
        if constexpr (NW > 1) {
            if (lane == 0) sh.best[odd][wave] = ((unsigned long long)kmin << 32) | (unsigned)chosen;
            __syncthreads();
            unsigned long long b = sh.best[odd][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) b = min(b, sh.best[odd][w]);
            chosen = (int)(unsigned)b;
        }
        chosen = __builtin_amdgcn_readfirstlane(chosen);
        if (lane == chosen) {
            ++cnt;
            touched = true;
        }
        const float inv = 1.0f / (float)__builtin_amdgcn_readlane(cnt, chosen);
        if (wave == chosen >> 4) {
            if (slot == chosen) {
#pragma unroll
                for (int i = 0; i < Q / 4; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) beta[i][e] = beta[i][e] + (x[i][e] - beta[i][e]) * inv;
            }
            store_norms();
        }
        if (assign && tid == 0) assign[(size_t)h * nq + qq] = chosen;
    };
    store_norms();
    stage_queries(0);
    if (wave == 0) {
        const bool left = __ballot(lane < C && cnt == 0) != 0;
        if (lane == 0) sh.done = left ? kFill : 0;
    }
    __syncthreads();

    int buf = 0;
    bool filling = (__builtin_amdgcn_readfirstlane(sh.done) & kFill) != 0;
    for (int base = 0; base < nq;) {
        load_queries(base + kBatchQ);  // the next batch, unless this one ends early
        // dot products with the wave's slots; wave 0: with each other too
        // (queries that fill empty slots need neither)
        if (!filling) {
            f32x4 x[Q / 4];
#pragma unroll
            for (int i = 0; i < Q / 4; ++i) x[i] = *reinterpret_cast<const f32x4*>(&sh.xs[buf][c16][g * L::QP + 4 * i]);
            f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
#pragma unroll
            for (int i = 0; i < Q / 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(beta[i][e], x[i][e], a0, 0, 0, 0);
                    a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(beta[i][e + 1], x[i][e + 1], a1, 0, 0, 0);
                }
            // rows 4 g + v: slots, column c16: the query
            *reinterpret_cast<f32x4*>(&sh.dot[c16][wave * 16 + 4 * g]) = a0 + a1;
            if (wave == 0) {
                f32x4 r = {0.f, 0.f, 0.f, 0.f};
                if constexpr (sizeof(T) == 2) {  // the queries are bf16 values: exact in bf16
#pragma unroll
                    for (int i = 0; i < Q / 4; i += 2) {
                        dev::u32x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const f32x4& y = x[i + (e >> 1)];
                            o[e] = (__float_as_uint(y[2 * (e & 1)]) >> 16) | __float_as_uint(y[2 * (e & 1) + 1]);
                        }
                        const bf16x8_t f = __builtin_bit_cast(bf16x8_t, o);
                        r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, f, r, 0, 0, 0);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < Q / 4; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) r = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][e], x[i][e], r, 0, 0, 0);
                }
                *reinterpret_cast<f32x4*>(&sh.gram[c16][4 * g]) = r;  // symmetric
            }
        }
        __syncthreads();
        if (wave == 0) {  // the chain
            int done = min(kBatchQ, nq - base), alone = 0;
            if (filling) {
                // while slots are empty each query fills the lowest one; the
                // batch ends with the last
                const unsigned long long empty = __ballot(lane < C && cnt == 0);
                done = min(done, (int)__popcll(empty));
                const int q = __popcll(empty & ((1ull << lane) - 1));
                if (((empty >> lane) & 1ull) && q < done) {
                    cnt = 1;
                    sh.joined[q] = {lane | kFill, 0.f};
                    touched = true;
                }
            } else {
                // lanes past C never hold the largest product
                const int ls = min(lane, C - 1);
                const bool mine = lane < C;
                const int all = done;
                bool tie = false;
                float d[kBatchQ];
#pragma unroll
                for (int q = 0; q < kBatchQ; ++q) d[q] = mine ? sh.dot[q][ls] : -INFINITY;
                float bn = mine ? sh.bn2[ls] : 1.f;
                // far from the ends of the float range only (a norm or a
                // product under- or overflows at another place there), and
                // with counts whose reciprocal below is exact; else one by one
                const float xs2 = lane < all ? sh.gram[lane][lane] : 1.f;
                if (__ballot((bn != 0.f && !(bn >= kNormMin && bn <= kNormMax)) ||
                             !(xs2 >= kNormMin && xs2 <= kNormMax) || cnt >= kCountMax)) {
                    done = 0;
                    tie = true;
                }
                // 1/|b| (0 for a zero beacon), 1/n of the slot's next update
                auto inv_root = [](float x) { return x == 0.f ? 0.f : __builtin_amdgcn_rsqf(x); };
                auto inv_count = [](int n) {  // one Newton step past the 1-ulp reciprocal: 1/n to the last bit below 2.7 million
                    const float f = (float)n, r = __builtin_amdgcn_rcpf(f);
                    return fmaf(fmaf(-f, r, 1.f), r, r);
                };
                float rb = inv_root(bn), inv = inv_count(cnt + 1);
                // the near-tie margin of each query, beside its products
                if (lane < kBatchQ) sh.margin[lane] = kNearTie * sqrtf(sh.gram[lane][lane]);
                wave_lds_fence();
                f32x4 gr[2][4];  // <query q, the others> and its margin, read one query ahead
                float margin[2];
                auto fetch = [&](auto q) {
#pragma unroll
                    for (int o = q / 4; o < 4; ++o) gr[q & 1][o] = *reinterpret_cast<const f32x4*>(&sh.gram[q][4 * o]);
                    margin[q & 1] = sh.margin[q];
                };
                fetch(std::integral_constant<int, 0>{});
                dev::static_for<kBatchQ>([&](auto q) {
                    if constexpr (q + 1 < kBatchQ) fetch(std::integral_constant<int, q + 1>{});
                    if (q >= done) return;  // uniform
                    const f32x4* gq = gr[q & 1];
                    const float xn = gq[q / 4][q % 4];
                    // the cosines but for the common factor 1/|x|, which moves
                    // no argmax, as integers of the same order (-0 as +0)
                    int key = __float_as_int(fmaf(d[q], rb, 0.f));
                    key ^= (key >> 31) & 0x7fffffff;
                    const int top = wave_max_i32(key);
                    const unsigned long long at = __ballot(key == top);
                    const int chosen = __ffsll(at) - 1;
                    // another cosine within rounding of the largest: the chain
                    // ends before this query
                    const int tb = top ^ ((top >> 31) & 0x7fffffff);
                    const unsigned long long near = __ballot(d[q] * rb >= __int_as_float(tb) - margin[q & 1]);
                    if (near & (near - 1)) {
                        done = q;
                        tie = true;
                        return;
                    }
                    const float keep = 1.f - inv;
                    const float parts = fmaf(keep * keep, bn, inv * inv * xn);
                    const float nbn = fmaf(2.f * inv * keep, d[q], parts);
                    // most of the beacon cancels: start over from the updated beacons
                    const unsigned long long cancels = __ballot(!(nbn >= 0.25f * parts));
                    if ((cancels >> chosen) & 1ull) done = q + 1;
                    if (lane == chosen) {
                        sh.joined[q] = {lane, inv};
                        touched = true;
                        ++cnt;
                        bn = nbn;
#pragma unroll
                        for (int o = q + 1; o < kBatchQ; ++o) d[o] = fmaf(gq[o / 4][o % 4] - d[o], inv, d[o]);
                    }
                    rb = inv_root(bn);
                    inv = inv_count(cnt + 1);
                });
                if (tie) alone = all - done;
            }
            if (lane >= done && lane < kBatchQ) sh.joined[lane] = {-1, 0.f};
            sh.cnt[lane] = cnt;
            const bool left = __ballot(lane < C && cnt == 0) != 0;
            if (lane == 0) {
                sh.done = done | (left ? kFill : 0);
                sh.alone = alone;
            }
        }
        __syncthreads();
        int done = __builtin_amdgcn_readfirstlane(sh.done);
        filling = (done & kFill) != 0;
        done &= kFill - 1;
        const int alone = __builtin_amdgcn_readfirstlane(sh.alone);
        if (assign && tid < done) assign[(size_t)h * nq + base + tid] = sh.joined[tid].slot & (kFill - 1);
        // the batch's updates, every slot's in order (its queries all fill, or
        // all join)
        const bool fills = __builtin_amdgcn_readfirstlane(sh.joined[0].slot & kFill) != 0;
        unsigned todo = 0;
#pragma unroll
        for (int q = 0; q < kBatchQ; ++q) {
            const int at = sh.joined[q].slot;  // -1: not taken
            todo |= (at == slot || at == (slot | kFill)) ? 1u << q : 0u;
        }
        while (__ballot(todo != 0)) {
            if (todo) {
                const int q = __ffs(todo) - 1;
                todo &= todo - 1;
                const float inv = sh.joined[q].inv;
#pragma unroll
                for (int i = 0; i < Q / 4; ++i) {
                    const f32x4 x = *reinterpret_cast<const f32x4*>(&sh.xs[buf][q][g * L::QP + 4 * i]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) beta[i][e] = fills ? x[e] : beta[i][e] + (x[e] - beta[i][e]) * inv;
                }
            }
        }
        store_norms();
        if (alone > 0) {
            cnt = sh.cnt[lane];  // every wave follows the counts here
            f32x4 x[Q / 4];
#pragma unroll
            for (int i = 0; i < Q / 4; ++i) x[i] = *reinterpret_cast<const f32x4*>(&sh.xs[buf][c16][g * L::QP + 4 * i]);
            const float xn = rows_sum(sumsq_quarter<D>([&](int e) { return x[e / 4][e % 4]; }));  // of query c16
            for (int i = 0; i < alone; ++i)
                take_one(&sh.xs[buf][done + i][0],
                         __int_as_float(__builtin_amdgcn_readlane(__float_as_int(xn), done + i)), base + done + i, i & 1);
            done += alone;
        }
        base += done;
        if (done < kBatchQ && base < nq) load_queries(base);
        stage_queries(buf ^ 1);
        buf ^= 1;
        __syncthreads();
    }
    if (wave == 0) {
        const unsigned long long m = __ballot(touched);
        if (lane == 0) sh.dirty = m;
    }
    __syncthreads();
    const unsigned long long changed = sh.dirty;
    if (slot < C && ((changed >> slot) & 1ull)) {
#pragma unroll
        for (int i = 0; i < Q / 4; ++i) reinterpret_cast<f32x4*>(bh + (size_t)slot * D + g * Q)[i] = beta[i];
    }
    if (wave == 0 && lane < C && ((changed >> lane) & 1ull)) counts[(size_t)h * C + lane] = cnt;
}

template <typename T, int D>
void launch_batch(const bkv_dims& d, const T* q_new, int T_steps, float* beacons, int32_t* counts, int32_t* assign,
                  hipStream_t s) {
    const dim3 grid(d.B * d.Hkv);
    switch ((d.C + 15) / 16) {
        case 1: hipLaunchKernelGGL((beacon_batch_kernel<T, D, 1>), grid, dim3(64), 0, s, q_new, T_steps, beacons, counts, assign, d.Hq, d.Hkv, d.C); break;
        case 2: hipLaunchKernelGGL((beacon_batch_kernel<T, D, 2>), grid, dim3(128), 0, s, q_new, T_steps, beacons, counts, assign, d.Hq, d.Hkv, d.C); break;
        case 3: hipLaunchKernelGGL((beacon_batch_kernel<T, D, 3>), grid, dim3(192), 0, s, q_new, T_steps, beacons, counts, assign, d.Hq, d.Hkv, d.C); break;
        default: hipLaunchKernelGGL((beacon_batch_kernel<T, D, 4>), grid, dim3(256), 0, s, q_new, T_steps, beacons, counts, assign, d.Hq, d.Hkv, d.C); break;
    }
}

}  // namespace

hipError_t launch_beacon_update(const bkv_dims& d, const void* q_new, int T, float* beacons, int32_t* counts,
                                int32_t* assign, hipStream_t s) {
    const int P = d.B * d.Hkv;
    if (P == 0 || T == 0) return hipSuccess;
    const bool bf = d.dtype == BKV_BF16;
    // 16 queries or more per head (a batch), readable 16 bytes at a time: from
    // there on the batches are ahead on every shape measured (16 queries: 8
    // heads of 16 slots 7 us against 12, 4608 heads of 16 slots 38 against
    // 44, 1024 heads of 64 slots 76 against 94; 8 queries would leave half of
    // every batch empty)
    if ((long long)T * (d.Hq / d.Hkv) >= kBatchMin && (reinterpret_cast<uintptr_t>(q_new) & 15) == 0) {
        if (bf && d.D == 128)
            launch_batch<uint16_t, 128>(d, static_cast<const uint16_t*>(q_new), T, beacons, counts, assign, s);
        else if (bf)
            launch_batch<uint16_t, 64>(d, static_cast<const uint16_t*>(q_new), T, beacons, counts, assign, s);
        else if (d.D == 128)
            launch_batch<float, 128>(d, static_cast<const float*>(q_new), T, beacons, counts, assign, s);
        else
            launch_batch<float, 64>(d, static_cast<const float*>(q_new), T, beacons, counts, assign, s);
        return hipGetLastError();
    }
#define BKV_LAUNCH_BU(TY, DD)                                                                                   \
    if (d.C <= kQuadSlots)                                                                                  \
        hipLaunchKernelGGL((beacon_update_kernel<TY, DD, 1>), dim3(P), dim3(64), smem_bytes<DD>(d.C), s,            \
                           static_cast<const TY*>(q_new), T, beacons, counts, assign, d.Hq, d.Hkv, d.C);           \
    else                                                                                                    \
        hipLaunchKernelGGL((beacon_update_kernel<TY, DD, 4>), dim3(P), dim3(256), smem_bytes<DD>(d.C), s,           \
                           static_cast<const TY*>(q_new), T, beacons, counts, assign, d.Hq, d.Hkv, d.C)
    if (bf && d.D == 128) {
        BKV_LAUNCH_BU(uint16_t, 128);
    } else if (bf) {
        BKV_LAUNCH_BU(uint16_t, 64);
    } else if (d.D == 128) {
        BKV_LAUNCH_BU(float, 128);
    } else {
        BKV_LAUNCH_BU(float, 64);
    }
#undef BKV_LAUNCH_BU
    return hipGetLastError();
}

}  // namespace bkv
